"""Every query row of a plan is computed over its own keys, at the sizes where the plan changes its
kernels: 128 | 129 blocks (one kernel per head | several), 64 | 65 heads (one block of parameters | two),
16384 | 16640 items at block 64 and 2048 | 2080 at block 128 (listed longest first | by heads), 255 | 256
heads of four or five items (spread over the queues | whole), fewer items than queues, the largest number
of blocks, all-equal and all-different rows, batch 2.

With q = 0 every kept key has the same weight, so the normaliser is the logarithm of the number of kept
keys and o is the mean of v, which is +1 or -1 by (batch, head, key block, channel): a block too many, too
few, or of another head changes it.  Outputs start as NaN."""
import numpy as np
import pytest

import oracle
import paper_2609_37001_amd as psa

import gpu_util as gu

pytestmark = pytest.mark.gpu
INF = 0x7FFFFFFF


def stripes(heads, f, sp, seed):
    rng = np.random.default_rng([13, seed])
    out = [(f, 0, INF, sp, 0, INF), (1, 0, INF, 1, 0, INF), (1, f + 3, INF, 1, 0, INF)]   # all, diagonal, none
    while len(out) < heads:
        out.append((int(rng.integers(1, f + 1)), int(rng.integers(-2, 3)), int(rng.choice([1, 2, 3, INF])),
                    int(rng.integers(1, sp + 1)), int(rng.integers(-1, 2)), int(rng.choice([1, 3, 5, 6, INF]))))
    return out[:heads]


# batch, heads, (F, H, W, text), block, head_dim.  The first lines are the sizes at which a call changes
# between the split engine (up to 256 query blocks, 512 unless every head keeps every block; twice as
# many at block 64, and at block 128 only with one or more than eight blocks per head beyond 256) and
# the pair engine.
CASES = [(1, 4, (4, 8, 256, 0), 128, 128), (1, 4, (4, 8, 256, 1), 128, 128), (1, 4, (8, 8, 256, 0), 128, 64),
         (1, 4, (8, 8, 256, 1), 128, 64), (2, 4, (4, 8, 128, 0), 64, 64), (2, 4, (4, 8, 128, 2), 64, 128),
         (2, 4, (8, 8, 128, 0), 64, 128), (2, 4, (8, 8, 128, 3), 64, 64), (1, 1, (64, 8, 128, 0), 64, 64),
         (1, 1, (64, 8, 128, 0), 128, 128),
         (1, 64, (1, 8, 128, 0), 128, 128), (1, 56, (1, 8, 144, 0), 128, 128), (1, 200, (1, 8, 32, 0), 128, 64),
         (1, 1, (1, 1, 7, 0), 64, 64), (2, 3, (1, 8, 16, 0), 128, 128), (1, 3, (2, 8, 16, 5), 128, 64),
         (1, 4, (16, 8, 128, 0), 128, 128), (1, 4, (16, 8, 128, 1), 128, 128), (2, 4, (16, 8, 64, 0), 64, 128),
         (1, 64, (3, 8, 24, 3), 64, 64), (2, 65, (3, 8, 24, 3), 64, 64), (1, 65, (3, 4, 11, 0), 128, 128),
         (1, 256, (1, 8, 64, 0), 64, 128), (2, 130, (1, 8, 80, 9), 64, 64), (1, 257, (1, 5, 77, 0), 128, 128), (1, 255, (1, 8, 64, 0), 64, 64),
         (1, 2, (62, 64, 128, 0), 64, 64), (1, 2, (62, 64, 128, 0), 64, 128), (1, 2, (62, 128, 128, 0), 128, 64),
         (1, 64, (64, 8, 64, 0), 64, 64), (1, 65, (64, 8, 64, 0), 64, 64),
         (2, 32, (8, 8, 128, 0), 128, 64), (2, 33, (8, 8, 128, 0), 128, 64), (1, 16, (32, 8, 128, 0), 128, 128)]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_every_row_over_its_own_keys(case):
    batch, heads, grid, block, d = case
    f, h, w, nt = grid
    t = gu.torch()
    n = f * h * w + nt
    params = stripes(heads, f, -(-(h * w) // block), heads)
    gen = t.Generator(device="cuda").manual_seed(5)
    k = t.randn((batch, heads, n, d), generator=gen, device="cuda", dtype=t.bfloat16)
    signs = t.randint(0, 2, (batch, heads, -(-n // block), d), generator=gen, device="cuda") * 2.0 - 1.0
    v = signs.repeat_interleave(block, 2)[:, :, :n].to(k).contiguous()
    q = t.zeros_like(k)
    o = t.full_like(k, float("nan"))
    o, lse, kept = psa.attention_fwd(q, k, v, grid, block, params, out=o, return_lse=True, return_kept_per_row=True)
    t.cuda.synchronize()
    keep = oracle.blockmap(params, f, h, w, nt, block).astype(bool)
    assert np.array_equal(kept.cpu().numpy(), keep.sum(2))
    size = np.minimum(block, n - block * np.arange(keep.shape[1]))
    keys = np.repeat(keep @ size, size, axis=1)                          # [heads, n]
    with np.errstate(divide="ignore"):
        want = np.log(keys)
    got = lse.cpu().numpy()
    # sums of up to 2^24 ones are exact in fp32; ln 2 x log2 in fp32 is within 2^-21 of ln here
    assert np.array_equal(np.isneginf(got), np.broadcast_to(keys == 0, got.shape))
    fin = np.broadcast_to(keys > 0, got.shape)
    assert np.abs(got[fin] - np.broadcast_to(want, got.shape)[fin]).max() <= 2e-5
    # o: exact fp32 sums of the weights of one size, one division and one rounding to bf16
    mean = t.matmul((t.from_numpy(keep).cuda() * t.from_numpy(size).cuda()).float(), signs)
    mean = (mean / t.from_numpy(keep @ size).cuda().clamp(min=1)[None, :, :, None]).repeat_interleave(block, 2)[:, :, :n]
    assert bool(((o.float() - mean).abs() <= mean.abs() * 2.0 ** -8 + 1e-6).all())


@pytest.mark.parametrize("grid,heads", [((4, 8, 256, 0), 4), ((4, 8, 256, 0), 6), ((4, 8, 256, 9), 8), ((2, 3, 5, 2), 300)])
@pytest.mark.parametrize("d,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_full_density_same_bits_as_dense(d, block, grid, heads):
    """At full density the sparse path (both calls of it, and a run whose density only the device knows)
    returns the dense path's bits, on either engine; with one head thinned it does not depend on the
    call either."""
    t = gu.torch()
    f, h, w, nt = grid
    n = f * h * w + nt
    gen = t.Generator(device="cuda").manual_seed(9)
    q, k, v = (t.randn((1, heads, n, d), generator=gen, device="cuda", dtype=t.bfloat16) for _ in range(3))
    full = [(f, 0, INF, -(-(h * w) // block), 0, INF) if i % 2 else (1, 3, 1, 2, -1, 2) for i in range(heads)]
    dense, dense_lse = psa.dense_fwd(q, k, v, block, return_lse=True)
    for params in (full, full[:-1] + [(1, 0, INF, 1, 0, INF)]):
        o, lse = psa.attention_fwd(q, k, v, grid, block, params, return_lse=True)
        ws = psa.plan(params, grid, block)
        for _ in range(2):
            o2, lse2 = psa.run(q, k, v, grid, block, ws, return_lse=True, out=t.full_like(q, float("nan")))
            assert t.equal(o, o2) and t.equal(lse, lse2)
        if params is full:
            assert t.equal(o, dense) and t.equal(lse, dense_lse)


@pytest.mark.parametrize("grid,stripe,heads", [((1, 30, 52, 226), (1, 0, INF, 12, 0, INF), 24),
                                               ((1, 10, 20, 100), (1, 0, INF, 1, 0, INF), 100),
                                               ((1, 3, 43, 1), (1, 0, INF, 1, 0, INF), 150),
                                               ((2, 10, 20, 30), (1, 0, 2, 2, 0, INF), 70)])
@pytest.mark.parametrize("d", [64, 128])
def test_full_by_text_same_bits_as_dense(d, grid, stripe, heads):
    """Maps that are full only because the text has taken the video's last slot or frame, between the
    sizes at which the density chooses the engine (257 to 512 blocks of 128); the last is not full."""
    t = gu.torch()
    f, h, w, nt = grid
    n = f * h * w + nt
    keep = oracle.blockmap([stripe], f, h, w, nt, 128)
    assert bool(keep.all()) == (f == 1) and 256 < heads * keep.shape[1] <= 512
    gen = t.Generator(device="cuda").manual_seed(3)
    q, k, v = (t.randn((1, heads, n, d), generator=gen, device="cuda", dtype=t.bfloat16) for _ in range(3))
    o, lse = psa.attention_fwd(q, k, v, grid, 128, [stripe] * heads, return_lse=True)
    o2, lse2 = psa.run(q, k, v, grid, 128, psa.plan([stripe] * heads, grid, 128), return_lse=True)
    assert t.equal(o, o2) and t.equal(lse, lse2)
    dense, dense_lse = psa.dense_fwd(q, k, v, 128, return_lse=True)
    if f == 1:
        assert t.equal(o, dense) and t.equal(lse, dense_lse)
    else:
        assert not t.equal(lse, dense_lse)


def halves_word(ws, heads, nb):
    """The word of a plan's queue area that names the shape of head dim 64 at block 128."""
    up = lambda x: (x + 255) // 256 * 256
    at = up(256 + 24 * heads) + up(8 * nb) + 2 * up(4 * heads * nb)         # header, stripes, coordinates, counts, order
    return ws.tensor[at + 4 * 17:at + 4 * 18].view(gu.torch().int32)


@pytest.mark.parametrize("pb", [None, (2, 8, 8), (1, 8, 32)])
@pytest.mark.parametrize("nt,text_rows", [(0, False), (65, False), (130, True)])
def test_both_shapes_of_head_dim_64_give_the_same_bits(pb, nt, text_rows):
    """At head dim 64 and block 128 the plan chooses between one item and two per pair; a run does what
    the plan says, on either layout, with the same bits, and some heads are compared with the oracle.
    The long rows of text at low density choose one item, full rows two."""
    t = gu.torch()
    f, h, w, d, heads = 5, 14, 45, 64, 40
    n, grid = f * h * w + nt, (f, h, w, nt)
    rng = np.random.default_rng([23, nt, 0 if pb is None else pb[0]])
    tp, sp = (f, -(-(h * w) // 128)) if pb is None else (-(-f // pb[0]), -(-h // pb[1]) * -(-w // pb[2]))
    if text_rows:
        params = [(1, 0, INF, 1, 0, INF)] * heads
    else:
        params = [(tp, 0, INF, sp, 0, INF) if i % 4 else (int(rng.integers(1, tp + 1)), int(rng.integers(-1, 2)), 3,
                                                         int(rng.integers(1, sp + 1)), 0, 5) for i in range(heads)]
    gen = t.Generator(device="cuda").manual_seed(nt + 1)
    q, k, v = (t.randn((1, heads, n, d), generator=gen, device="cuda", dtype=t.bfloat16) for _ in range(3))
    if pb is None:
        ws = psa.plan(params, grid, 128)
        go = lambda: psa.run(q, k, v, grid, 128, ws, 0.1, return_lse=True, out=t.full_like(q, float("nan")))
    else:
        ws = psa.plan_3d(params, grid, pb, 128)
        qb, kb, vb = (psa.to_blocks(x, grid, pb) for x in (q, k, v))

        def go():
            o, lse = psa.run_3d(qb, kb, vb, grid, pb, 128, ws, 0.1, return_lse=True, out=t.full_like(qb, float("nan")))
            lse = t.stack([t.from_numpy(oracle.from_blocks(lse[0, i].cpu().numpy()[:, None], f, h, w, nt, pb)[:, 0])
                           for i in range(heads)])[None]
            return psa.from_blocks(o, grid, pb), lse
    word = halves_word(ws, heads, -(-(n if pb is None else psa.blocked_tokens(grid, pb)) // 128))
    assert int(word) == (0 if text_rows else 1)
    o, lse = go()
    word.fill_(1 - int(word))
    o2, lse2 = go()
    assert t.equal(o, o2) and t.equal(lse, lse2)
    pick = [0, 1, heads - 1]
    host = lambda x: x[:, pick].float().cpu().numpy()
    if pb is None:
        keep, groups = oracle.blockmap(params, f, h, w, nt, 128), None
    else:
        keep, groups = oracle.psablock_map(params, f, h, w, nt, pb), oracle.token_groups(f, h, w, nt, pb)
    gu.compare_all(host(q), host(k), host(v), keep[pick], 128, 0.1, host(o), lse[:, pick].cpu().numpy(),
                   groups=groups).check("pb %s, %d text:" % (pb, nt))


@pytest.mark.parametrize("block,magic", [(64, 0x50534131), (128, 0x50534132)])
@pytest.mark.parametrize("grid", [(4, 8, 128, 0), (16, 8, 128, 0)])
@pytest.mark.parametrize("d", [64, 128])
def test_plan_of_another_format_is_left_alone(d, grid, block, magic):
    """A header that names the right sizes but another kind of plan: nothing is written."""
    t = gu.torch()
    n = grid[0] * grid[1] * grid[2]
    params = [(2, 0, INF, 3, 0, INF)] * 8
    q = t.ones((1, 8, n, d), device="cuda", dtype=t.bfloat16)
    ws = psa.plan(params, grid, block)
    head = ws.tensor.view(t.uint8)[:4]
    good = head.clone()
    for want, word in ((0, magic), (n * 8 * d, None)):
        head.copy_(good if word is None else t.tensor(list(word.to_bytes(4, "little")), dtype=t.uint8))
        o = psa.run(q, q, q, grid, block, ws, out=t.full_like(q, float("nan")))
        assert int((~o.isnan()).sum()) == want
