"""The base that the softmax weights are taken from, against the oracle: scores that rise or fall by
tens along the sequence (the base moves many times, or the first keys outweigh all later ones),
scores that are all far below zero or above it, at sequence ends that leave the second half of the
last 128-key block partly filled or empty.  On the split engine (its halves of a block) and, with the
heads repeated, on the pair engine (steps of 64 keys)."""
import numpy as np
import pytest

import oracle
import paper_2609_37001_amd as psa
from workloads.inputs import bf16_round

import gpu_util as gu

pytestmark = pytest.mark.gpu
INF = 0x7FFFFFFF
PARAMS = [(4, 0, INF, 9, 0, INF), (2, 0, INF, 2, 0, INF), (1, 1, 2, 3, -1, 3)]


def dev(x):
    t = gu.torch()
    return t.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to("cuda:0").bfloat16()


# Score offset of the key at position x in [0, 1] of the sequence, in natural-log units.
SHAPES = {"rising": lambda x: 90 * x, "falling": lambda x: -90 * x, "low": lambda x: 0 * x - 150,
          "high": lambda x: 0 * x + 150, "steps": lambda x: 40 * np.floor(5 * x)}


@pytest.mark.parametrize("engine", ["split", "pairs"])
@pytest.mark.parametrize("nt", [0, 1, 65])
@pytest.mark.parametrize("d,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_scores_far_from_zero(shape, d, block, nt, engine):
    f, hh, ww = 4, 8, 40                     # 1280 video tokens: ten blocks of 128
    n = f * hh * ww + nt
    rng = np.random.default_rng([11, d, block, nt])
    q, k, v = (rng.standard_normal((1, len(PARAMS), n, d)).astype(np.float32) for _ in range(3))
    # channel 0 of q is 8 / scale-free: its product with channel 0 of k is the offset alone
    scale = 0.125
    q[..., 0] = 8.0
    k[..., 0] = SHAPES[shape](np.arange(n) / n)
    q, k, v = (bf16_round(x) for x in (q, k, v))
    grid = (f, hh, ww, nt)
    keep = oracle.blockmap(PARAMS, f, hh, ww, nt, block)
    r = gu.copies_for(len(PARAMS), keep.shape[1], block) if engine == "pairs" else 1
    assert gu.engine(r * len(PARAMS), keep.shape[1], block) == engine
    o, lse = psa.attention_fwd(*(dev(x).repeat(1, r, 1, 1) for x in (q, k, v)), grid, block, PARAMS * r, scale,
                               return_lse=True)
    gu.torch().cuda.synchronize()
    o, lse = o[:, -len(PARAMS):], lse[:, -len(PARAMS):]
    par = gu.compare_all(q, k, v, keep, block, scale, o.float().cpu().numpy(), lse.cpu().numpy())
    # Where few keys carry the weight P's rounding does not average out: a row is off by up to
    # 2^-8 (P) + 2^-9 (O) of its values' size, which may partly cancel in O; the normaliser's bound
    # is relative and does not depend on the base, plus fp32 rounding of scores of up to 220
    # (2^-24 x 220 x log2 e per score, below 1e-4).
    print(par.summary())
    assert par.rel <= gu.REL_L2_TOL and par.max_row <= gu.ROW_REL_TOL, par.summary()
    assert par.max_lse <= gu.LSE_ABS_TOL + 1e-4, par.summary()
