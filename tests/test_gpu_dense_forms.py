"""Dense attention at the ends of its range: more key blocks than an entry of the sparse key list can
number, more heads than one launch can take."""
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


@pytest.mark.parametrize("d", [64, 128])
def test_more_heads_than_one_launch_takes(d):
    """One workgroup per item (no workspace) and 2^24 + 3 heads of one token: of 256 threads each they
    are more than the 2^32 - 1 threads of a launch.  The only key has weight 1, so o = v and the
    normaliser is the score."""
    t = gu.torch()
    heads = 2 ** 24 + 3
    q = t.full((1, heads, 1, d), 0.5, device="cuda", dtype=t.bfloat16)
    v = t.randn(q.shape, device="cuda", dtype=t.bfloat16, generator=t.Generator(device="cuda").manual_seed(2))
    o, lse = psa.dense_fwd(q, q, v, 64, 0.125, return_lse=True, balanced=False, out=t.full_like(v, float("nan")))
    assert t.equal(o, v)
    s = 0.5 * d * float(gu.kernel_q(np.full(1, 0.5), 0.125)[0]) * math.log(2.0)
    assert float((lse - s).abs().max()) <= 1e-5
