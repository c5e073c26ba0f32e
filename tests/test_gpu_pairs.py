"""The pair engine against the oracle, on random q, k and v and partial stripes, above the sizes that
the split engine takes: every instantiation (head dim, block, one-dimensional blocks and PSABlocks), both
listings of the items, whole heads on one queue, ragged ends, text, batch 2."""
import numpy as np
import pytest

import oracle
import paper_2609_37001_amd as psa

import gpu_util as gu

pytestmark = pytest.mark.gpu
INF = 0x7FFFFFFF
SHAPES = [(64, 64), (64, 128), (128, 64), (128, 128)]


def random_params(rng, n, tmax, smax):
    """Stripes of the paper's ranges, two of them with leftover query blocks in either pairing order, one
    that keeps nothing but text and one that keeps everything."""
    out = [(min(tmax, 3), 0, INF, 1, 0, 3), (1, 0, INF, min(smax, 2), 0, INF), (1, tmax + 1, INF, 1, 0, INF),
           (tmax, 0, INF, smax, 0, INF)]
    while len(out) < n:
        out.append((int(rng.integers(1, tmax + 1)), int(rng.choice([0, 1, -1, 2, -2])), int(rng.choice([1, 2, 3, INF])),
                    int(rng.integers(1, smax + 1)), int(rng.choice([0, 1, -1])), int(rng.choice([1, 3, 5, 6, INF]))))
    return out[:n]


def inputs(batch, heads, n, d, seed):
    t = gu.torch()
    gen = t.Generator(device="cuda").manual_seed(seed)
    return [t.randn((batch, heads, n, d), generator=gen, device="cuda", dtype=t.bfloat16) for _ in range(3)]


def pick(heads, rng, some=8):
    return list(range(heads)) if heads <= some else sorted({0, 1, 2, 3, heads - 1, *map(int, rng.integers(0, heads, some))})


# batch, heads, (F, H, W, text): five to nineteen blocks a head; whole heads on one queue; more items than
# are listed longest first at block 128, and at block 64.
GRIDS = [(2, 60, (3, 7, 23, 37)), (1, 70, (4, 10, 30, 0)), (2, 150, (3, 7, 23, 37)), (1, 700, (3, 7, 23, 1)),
         (2, 512, (3, 16, 44, 0))]


@pytest.mark.parametrize("case", GRIDS, ids=str)
@pytest.mark.parametrize("d,block", SHAPES)
def test_one_dimensional_blocks(d, block, case):
    batch, heads, grid = case
    f, h, w, nt = grid
    n = f * h * w + nt
    rng = np.random.default_rng([31, d, block, heads])
    params = random_params(rng, heads, f, -(-(h * w) // block))
    q, k, v = inputs(batch, heads, n, d, heads)
    nb = -(-n // block)
    assert gu.engine(batch * heads, nb, block) == "pairs"
    if batch * heads == 1024:
        assert gu.listed_by_heads(batch * heads, nb, block)
    out = gu.torch().full_like(q, float("nan"))
    o, lse, kept = psa.attention_fwd(q, k, v, grid, block, params, 0.11, out=out, return_lse=True, return_kept_per_row=True)
    ws = psa.plan(params, grid, block, batch=batch)
    for _ in range(2):
        o2, lse2 = psa.run(q, k, v, grid, block, ws, 0.11, return_lse=True)
        assert gu.torch().equal(o, o2) and gu.torch().equal(lse, lse2)
    keep = oracle.blockmap(params, f, h, w, nt, block)
    assert np.array_equal(kept.cpu().numpy(), oracle.kept_per_row(keep))
    assert bool(gu.torch().isfinite(o).all())
    p = pick(heads, rng)
    host = lambda x: x[:, p].float().cpu().numpy()
    gu.compare_all(host(q), host(k), host(v), keep[p], block, 0.11, host(o), lse[:, p].cpu().numpy()).check(
        "d=%d block=%d %s:" % (d, block, case))


# batch, heads, grid, PSABlock: tiles partly of padding on every axis, tiles of nothing else, text.
GRIDS_3D = [(2, 60, (3, 6, 20, 40), (2, 4, 16)), (1, 130, (5, 9, 17, 0), (1, 8, 16)), (2, 150, (2, 10, 20, 70), (4, 4, 8)),
            (1, 700, (3, 5, 30, 3), (2, 2, 64))]


@pytest.mark.parametrize("case", GRIDS_3D, ids=str)
@pytest.mark.parametrize("d,tile", SHAPES)
def test_psablocks(d, tile, case):
    batch, heads, grid, pb = case
    f, h, w, nt = grid
    n = f * h * w + nt
    (tp, hp, wp), _ = oracle.psablock_grid(f, h, w, pb)
    rng = np.random.default_rng([37, d, tile, heads])
    params = random_params(rng, heads, tp, hp * wp)
    q, k, v = inputs(batch, heads, n, d, heads + 1)
    tiles = -(-psa.blocked_tokens(grid, pb) // tile)
    copies = gu.copies_for(batch * heads, tiles, tile)
    assert copies == 1, "raise the heads to %d" % (copies * heads)
    qb, kb, vb = (psa.to_blocks(x, grid, pb) for x in (q, k, v))
    ob, lseb = psa.attention_fwd_3d(qb, kb, vb, grid, pb, params, tile, 0.11, return_lse=True)
    o = psa.from_blocks(ob, grid, pb)
    assert bool(gu.torch().isfinite(o).all())
    p = pick(heads, rng)
    host = lambda x: x[:, p].float().cpu().numpy()
    lse = np.stack([np.stack([oracle.from_blocks(lseb[b, i].cpu().numpy()[:, None], f, h, w, nt, pb)[:, 0] for i in p])
                    for b in range(batch)])
    keep, groups = oracle.psablock_map(params, f, h, w, nt, pb), oracle.token_groups(f, h, w, nt, pb)
    gu.compare_all(host(q), host(k), host(v), keep[p], tile, 0.11, host(o), lse, groups=groups).check(
        "d=%d tile=%d %s:" % (d, tile, case))
