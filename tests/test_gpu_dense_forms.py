"""Dense attention at the ends of its range: more key blocks than an entry of the sparse key list can
number."""
import math

import numpy as np
import pytest

import paper_2609_37001_amd as psa

import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_more_blocks_than_a_list_entry_numbers(d, block):
    """8192 blocks of 128 and 200 tokens more.  Only the last 200 keys have a score above zero and a
    value: a block number cut to 13 bits (or to 12) would read an early block in their place."""
    t = gu.torch()
    extra, n = 200, 8192 * 128 + 200
    q = t.ones((1, 1, n, d), device="cuda", dtype=t.bfloat16)
    k, v = t.zeros_like(q), t.zeros_like(q)
    k[:, :, -extra:] = 64.0 / d
    v[:, :, -extra:] = 1.0
    scale = 0.25                       # scores 16 and 0: the last keys hold all but 0.06 % of the weight
    o, lse = psa.dense_fwd(q, k, v, block, scale, return_lse=True)
    # the score of the last keys on the kernel's operand (q scaled and rounded once), in powers of two
    s = 64.0 * float(gu.kernel_q(np.ones(1), scale)[0])
    want = math.log(n - extra + extra * 2.0 ** s)
    assert float((lse - want).abs().max()) <= gu.LSE_ABS_TOL
    assert float((o.float() - 1.0).abs().max()) <= 2.0 ** -8
