"""Dense attention at the ends of its range: more key blocks than an entry of the sparse key list can
number, more heads than one launch can take; and at the sizes where the shape of its kernel changes."""
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


# heads, tokens.  More query blocks than the split engine takes: 64-row pairs up to 512 tokens (one
# block, two, an odd number, a last block of one row), then 128-row pairs -- at head dim 64 up to 256 of
# them, 64-row pairs again beyond -- with a last 128-row block of at most 64 rows.
SHAPES = [(530, 1), (530, 64), (530, 65), (270, 129), (180, 320), (130, 512), (110, 513), (64, 769), (64, 1024),
          (65, 1025), (90, 831)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("d,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_shapes(d, block, shape):
    """Fixed grid and armed queues (a workspace used twice) give the same bits; every row of some heads
    is compared with the oracle, and every row's normaliser with a plain fp32 product."""
    t = gu.torch()
    heads, n = shape
    assert heads * -(-n // block) > 256 * (128 // block)
    rng = np.random.default_rng([21, d, block, n])
    gen = t.Generator(device="cuda").manual_seed(n)
    q, k, v = (t.randn((1, heads, n, d), generator=gen, device="cuda", dtype=t.bfloat16) for _ in range(3))
    o, lse = psa.dense_fwd(q, k, v, block, 0.1, return_lse=True, balanced=False)
    ws = t.empty(psa.dense_workspace_size(), dtype=t.uint8, device="cuda")
    for _ in range(2):
        o2, lse2 = psa.dense_fwd(q, k, v, block, 0.1, return_lse=True, workspace=ws, out=t.full_like(q, float("nan")))
        assert t.equal(o, o2) and t.equal(lse, lse2)
    pick = sorted({0, heads - 1, int(rng.integers(heads))})
    nb = -(-n // block)
    host = lambda x: x[:, pick].float().cpu().numpy()
    gu.compare_all(host(q), host(k), host(v), np.ones((len(pick), nb, nb), np.uint8), block, 0.1, host(o),
                   lse[:, pick].cpu().numpy()).check("d=%d block=%d heads=%d n=%d:" % (d, block, heads, n))
    ref = t.logsumexp(0.1 * t.matmul(q[0].float(), k[0].float().transpose(1, 2)), -1)
    # scores of up to 60 with the kernel's q off by Q_ROUND of each element: as in lse_plain_bound
    bound = gu.LSE_ABS_TOL + gu.Q_ROUND * 0.1 * t.matmul(q[0].float().abs(), k[0].float().abs().transpose(1, 2)).amax(-1)
    assert bool(((lse[0] - ref).abs() <= bound).all())
