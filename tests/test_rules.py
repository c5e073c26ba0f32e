"""The host rules of the library that need no GPU, compiled from the library's header and compared with
the oracle: which plans count as full (every head keeps every key block)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from paper_2609_37001_amd import build

import gpu_util as gu

INF = 0x7FFFFFFF
MAIN = r"""
#include <stdio.h>
#include "psa_launch.h"
int main(int argc, char**) {
  int f, h, w, text, block, n_bh, nb, full;
  while (argc > 1 && scanf("%d %d %d %d", &n_bh, &nb, &block, &full) == 4)
    printf("%d\n", (int)psa::split_plan(n_bh, nb, block, full));
  psa_stripe_t m;
  while (scanf("%d %d %d %d %d %d %d %d %d %d %d", &f, &h, &w, &text, &block, &m.t_w, &m.t_o, &m.t_s, &m.s_w, &m.s_o,
               &m.s_s) == 11) {
    psa::Geometry g{};
    g.hw = h * w;
    g.n_video = g.hw * f;
    g.n = g.n_video + text;
    g.n_text = text;
    g.block = block;
    g.nb = (g.n + block - 1) / block;
    g.frames = f;
    printf("%d\n", (int)psa::plan_full(g, &m, 1));
  }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "main.cc", d / "main"
    src.write_text(MAIN)
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", build.INCLUDE,
                    "-I", build.CSRC, str(src), "-o", str(exe)], check=True)

    def ask(cases, *args):
        text = "\n".join(" ".join(str(x) for x in c) for c in cases)
        out = subprocess.run([str(exe), *args], input=text, capture_output=True, text=True, check=True).stdout.split()
        return [int(x) for x in out]

    return ask


def draw(rng, n):
    """Grids around the sizes at which a frame, a block and the text meet, masks around full."""
    out = []
    while len(out) < n:
        block = int(rng.choice([4, 8, 16]))
        f, h, w = int(rng.integers(1, 5)), int(rng.integers(1, 6)), int(rng.integers(1, 14))
        text = int(rng.choice([0, 1, int(rng.integers(1, 3 * block))]))
        sp = -(-(h * w) // block)
        m = [int(rng.integers(1, f + 2)), int(rng.integers(-2, 3)), int(rng.choice([1, 2, 3, 5, INF])),
             int(rng.integers(max(1, sp - 2), sp + 2)), int(rng.integers(-1, 2)), int(rng.choice([1, 2, 4, sp + 1, INF]))]
        out.append((f, h, w, text, block, *m))
    return out


def test_full_plans_are_those_that_keep_every_block(rules):
    cases = draw(np.random.default_rng(17), 6000)
    # text that takes the last slot or frame of the video from the map
    cases += [(1, 30, 52, 226, 128, 1, 0, INF, 12, 0, INF), (1, 10, 20, 100, 128, 1, 0, INF, 1, 0, INF),
              (1, 3, 43, 1, 128, 1, 0, INF, 1, 0, INF), (2, 3, 43, 1, 128, 1, 0, 2, 1, 0, 1),
              (1, 2, 3, 40, 8, 1, 9, INF, 1, 9, INF)]
    seen = {0: 0, 1: 0}
    for c, got in zip(cases, rules(cases)):
        f, h, w, text, block, m = *c[:5], c[5:]
        full = bool(oracle.blockmap([m], f, h, w, text, block).all())
        if block > h * w:
            assert got == 1, c                  # counts as full whatever it keeps
        else:
            assert got == full, c
            seen[got] += 1
    assert min(seen.values()) > 500


def test_split_engine_lines(rules):
    rng = np.random.default_rng(19)
    cases = [(int(rng.integers(1, 1025)), int(np.exp(rng.uniform(0, 7))), block, full)
             for block in (64, 128) for full in (0, 1) for _ in range(2000)]
    cases += [(n, nb, block, full) for block in (64, 128) for full in (0, 1) for nb in (1, 2, 8, 9, 64)
              for lim in (256, 512) for n in (lim * 128 // block // nb, lim * 128 // block // nb + 1)]
    got = ["split" if x else "pairs" for x in rules(cases, "split")]
    assert got == [gu.engine(*c) for c in cases]
    assert min(got.count("split"), got.count("pairs")) > 500
