"""Forms of the block map kernel, against the oracle: axes shorter and longer than its tables (4096
positions), rows of any length modulo the four entries of a store, one head's map at any byte offset,
blocks larger than a frame, strides and widths at the ends of their range; and its division by
multiplication for every distance that can occur."""
import numpy as np
import pytest

import oracle
import paper_2609_37001_amd as psa

INF = 0x7FFFFFFF
PARAMS = [(1, 0, 1, 1, 0, 1), (2, -3, 5, 3, 1, 7), (1, 2 ** 24, 2, 1, -2 ** 24, 3), (INF, 0, INF, 2, 0, 2 ** 30),
          (1, -1, INF, 5, 1, 6), (3, 1, 2, 1, 0, INF), (1, 0, 4097, 4096, 0, 4097)]


@pytest.mark.gpu
@pytest.mark.parametrize("grid,block", [((5, 3, 7, 0), 1), ((5, 3, 7, 2), 1), ((7, 2, 5, 3), 16), ((1, 1, 5000, 0), 1),
                                        ((4098, 1, 1, 1), 1), ((4096, 1, 1, 0), 1), ((9, 4, 4, 0), 64),
                                        ((3, 16, 17, 9), 8)])
def test_map_forms(grid, block):
    f, h, w, nt = grid
    ref = oracle.blockmap(PARAMS, f, h, w, nt, block)
    bm, pr, ph = psa.build_blockmap(PARAMS, grid, block)
    assert np.array_equal(bm.cpu().numpy(), ref)
    assert np.array_equal(pr.cpu().numpy(), oracle.kept_per_row(ref))
    assert np.array_equal(ph.cpu().numpy(), oracle.kept_per_head(ref))
    _, pr2, ph2 = psa.build_blockmap(PARAMS, grid, block, blockmap=False)
    assert np.array_equal(pr2.cpu().numpy(), pr.cpu().numpy()) and np.array_equal(ph2.cpu().numpy(), ph.cpu().numpy())


@pytest.mark.parametrize("stride", [2, 3, 4, 5, 6, 7, 63, 64, 65, 1000, 4097, 2 ** 24 - 1, 2 ** 25 + 1, 2 ** 30, INF])
def test_reciprocal_is_exact(stride):
    """The reciprocal of AxisTest, in Python integers: exact at every multiple of the stride up to
    2^31, the points at which a wrong quotient would show, and the entries before and after."""
    l = (stride - 1).bit_length()
    mul = -(-(1 << (31 + l)) // stride)
    assert mul < 1 << 32
    k = np.unique(np.concatenate([np.arange(0, 2000), np.linspace(0, (2 ** 31 - 1) // stride, 20001).astype(np.int64)]))
    x = (k[:, None] * stride + np.array([-1, 0, 1])).ravel()
    x = x[(x >= 0) & (x < 2 ** 31)]
    q = np.array([(int(v) * mul >> 32) >> (l - 1) for v in x])
    assert np.array_equal(q, x // stride)
