"""The calls that users of paper_2609_37001_amd make, as cases for timing and comparing them.

A case is a dict of plain values.  Its "kind" names the entry point:

* ``fwd``       attention_fwd: plan and sparse attention in one call (a layer whose stripes change,
                or a program that keeps no plan);
* ``run``       run over a plan made in advance (a layer at every denoising step);
* ``run_3d``    the PSABlock layout: to_blocks of q, k, v, run_3d over a plan, from_blocks of o;
* ``dense``     dense_fwd: the denoising steps that stay dense, and the search's reference;
* ``blockmap``  build_blockmap: the map of every head with its counts (inspecting masks);
* ``search``    search.score: the losses of a few candidate masks of every head.

The sizes are a video DiT's attention layers: ``frames x height x width`` latent tokens, and
``text`` tokens behind them.  Stripe parameters are drawn from the candidate sets of the paper's
search, each head's close to a target density; they belong to the layer (to the case), q, k and v
to the seed.
"""
import math
import random

import numpy as np
import torch

import paper_2609_37001_amd as psa
from paper_2609_37001_amd import search

T_OFFSETS, T_STRIDES = (0, 1, -1, 2, -2), (1, 2, 3, psa.STRIDE_INF)
S_OFFSETS, S_STRIDES = (0, 1, -1), (1, 3, 5, 6, psa.STRIDE_INF)


def _case(name, kind, batch, heads, grid, dim, block, **more):
    c = {"kind": kind, "batch": batch, "heads": heads, "frames": grid[0], "height": grid[1],
         "width": grid[2], "text": grid[3], "dim": dim, "block": block, "low": 0.1, "high": 0.4,
         "stripes": 1, "lse": False}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call, a 16x16 latent of four frames with two heads, planned on the spot:
        # launches and latency are all there is.
        _case("tiny fwd b64 d64", "fwd", 1, 2, (4, 16, 16, 0), 64, 64, low=0.3, high=0.8),
        # A short low-resolution preview clip: about one work item per compute unit.
        _case("preview fwd b128 d128", "fwd", 1, 12, (5, 30, 52, 0), 128, 128, low=0.15),
        # A small-model clip with text and a ragged end, two prompts, narrow heads, fine blocks,
        # with the softmax normaliser (merged with another attention afterwards).
        _case("clip fwd b64 d64 text", "fwd", 2, 16, (13, 30, 45, 226), 64, 64, lse=True),
        # The same range of models with coarse blocks.
        _case("clip run b128 d64 text", "run", 2, 30, (13, 30, 45, 226), 64, 128),
        # Wan 2.1 1.3B, 480p: an ordinary layer, planned on the spot.
        _case("wan1.3b fwd b128 d128", "fwd", 1, 12, (21, 30, 52, 0), 128, 128, low=0.15),
        # The same layer with masks at twice the resolution.
        _case("wan1.3b fwd b64 d128", "fwd", 1, 12, (21, 30, 52, 0), 128, 64, low=0.15),
        # Wan 2.1 14B, 720p, at a sparse denoising step (the headline layer).
        _case("wan14b run b128 d128", "run", 1, 40, (21, 45, 80, 0), 128, 128),
        # The same layer in the paper's own PSABlock layout, converted on the way in and out.
        _case("wan14b run_3d b128 d128", "run_3d", 1, 40, (21, 45, 80, 0), 128, 128,
              pt=3, ph=8, pw=16),
        # The same layer's dense steps (the first 20 % of the denoising): the largest case.
        _case("wan14b dense b128 d128", "dense", 1, 40, (21, 45, 80, 0), 128, 128),
        # HunyuanVideo, 720p, joint attention with text tokens at a sparse denoising step.
        _case("hunyuan run b128 d128", "run", 1, 24, (33, 45, 80, 256), 128, 128, high=0.35),
        # Every head's map of the Wan 2.1 14B layer.
        _case("wan14b blockmap", "blockmap", 1, 40, (21, 45, 80, 0), 128, 128),
        # Three candidates for every head of the Wan 2.1 1.3B layer.
        _case("wan1.3b search b128", "search", 1, 12, (21, 30, 52, 0), 128, 128, candidates=3,
              low=0.1, high=0.9),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, its sizes spread over the range of the listed ones."""
    kind = rng.choice(["fwd", "fwd", "run", "run", "run_3d", "dense", "blockmap", "search"])
    while True:
        dim, block = rng.choice([(128, 128), (128, 128), (64, 64), (128, 64), (64, 128)])
        batch, heads = rng.choice([1, 1, 1, 2, 3]), _log(rng, 2, 40)
        frames, height, width = rng.randint(1, 33), rng.randint(12, 48), rng.randint(12, 80)
        text = rng.choice([0, 0, 0, 77, 226, 256, 512])
        n = frames * height * width + text
        if 700 <= n <= 119056 and 4.0 * n * n * dim * batch * heads <= 2.5e13:
            break
    low = rng.uniform(0.05, 0.4)
    more = {"low": round(low, 3), "high": round(low + rng.uniform(0.02, 0.5), 3),
            "stripes": rng.randrange(1 << 30), "lse": rng.random() < 0.3}
    if kind == "run_3d":
        more["pt"], more["ph"], more["pw"] = rng.choice([(1, 8, 16), (3, 8, 16), (2, 8, 8), (4, 8, 4)])
    if kind == "search":
        more["candidates"] = rng.randint(2, 4)
    return _case(None, kind, batch, heads, (frames, height, width, text), dim, block, **more)


# ------------------------------------------------------------------------------------------------
# Stripes and block geometry, from their definitions.
# ------------------------------------------------------------------------------------------------

def _grid(case):
    return case["frames"], case["height"], case["width"], case["text"]


def _tokens(case):
    f, h, w, text = _grid(case)
    return f * h * w + text


def _extent(case):
    """Temporal and spatial extent in the units of the stripes."""
    f, h, w, _ = _grid(case)
    if case["kind"] == "run_3d":
        return -(-f // case["pt"]), -(-h // case["ph"]) * -(-w // case["pw"])
    return f, -(-h * w // case["block"])


def _axis(extent, w, o, s):
    """[extent, extent] float: whether a query at row i keeps a key at column j on one axis."""
    i = np.arange(extent)
    return (np.abs(i[None, :] - i[:, None] - o) % s < w).astype(np.float64)


def _stripes(case, count=1):
    """`count` masks for every head: of 150 random candidates the one whose density (on a full
    grid) is nearest to a target drawn from the case's band."""
    tp, sp = _extent(case)
    rng = random.Random(case["stripes"])
    out = []
    for _ in range(case["heads"]):
        cands = [(rng.randint(1, tp), rng.choice(T_OFFSETS), rng.choice(T_STRIDES),
                  rng.randint(1, sp), rng.choice(S_OFFSETS), rng.choice(S_STRIDES)) for _ in range(150)]
        d = np.array([_near(tp, *c[:3]) * _near(sp, *c[3:]) for c in cands])
        out.append([cands[int(np.argmin(np.abs(d - rng.uniform(case["low"], case["high"]))))]
                    for _ in range(count)])
    return out


def _near(extent, w, o, s):
    """Share of the pairs of one axis that are kept."""
    d = np.arange(-(extent - 1), extent)
    return float(((np.abs(d - o) % s < w) * (extent - np.abs(d))).sum()) / extent ** 2


def _coords(case):
    """(frame, slot, tokens) of every mask unit of the sequence; frame -1 is a global unit.
    Units are runs of `block` tokens, or PSABlocks (run_3d) of the tokens _unit_of() names."""
    f, h, w, text = _grid(case)
    n, hw = _tokens(case), h * w
    if case["kind"] == "run_3d":
        tp, sp = _extent(case)
        size = np.bincount(_unit_of(case), minlength=tp * sp + (text > 0))
        t = np.arange(tp * sp) // sp
        s = np.arange(tp * sp) % sp
        if text:
            t, s = np.append(t, -1), np.append(s, 0)
        return t, s, size
    b = case["block"]
    i0 = np.arange(-(-n // b)) * b
    size = np.minimum(b, n - i0)
    t, s = i0 // hw, i0 % hw // b
    glob = (i0 + size > f * hw) if text else np.zeros(len(i0), bool)
    return np.where(glob, -1, t), np.where(glob, 0, s), size


def _unit_of(case):
    """Mask unit of every token."""
    f, h, w, text = _grid(case)
    if case["kind"] != "run_3d":
        return np.arange(_tokens(case)) // case["block"]
    hp, wp = -(-h // case["ph"]), -(-w // case["pw"])
    i = np.arange(f * h * w)
    t, y, x = i // (h * w), i % (h * w) // w, i % w
    u = (t // case["pt"] * hp + y // case["ph"]) * wp + x // case["pw"]
    return np.append(u, np.full(text, -(-f // case["pt"]) * hp * wp))


def _map(case, m):
    """[units, units] bool: the units that a mask keeps (Algorithm 1 of the paper)."""
    t, s, _ = _coords(case)
    tp, sp = _extent(case)
    tv, sv = np.maximum(t, 0), np.minimum(s, sp - 1)
    keep = (_axis(tp, *m[:3]) > 0)[tv][:, tv] & (_axis(sp, *m[3:]) > 0)[sv][:, sv]
    return keep | (t < 0)[:, None] | (t < 0)[None, :]


def _kept_pairs(case, m):
    """Query-key pairs of tokens that a mask keeps."""
    t, s, size = _coords(case)
    tp, sp = _extent(case)
    video = t >= 0
    tokens = np.zeros((tp, sp))
    np.add.at(tokens, (t[video], s[video]), size[video])
    pairs = ((tokens @ _axis(sp, *m[3:])) * (_axis(tp, *m[:3]) @ tokens)).sum()
    return float(pairs) + float(size.sum()) ** 2 - float(size[video].sum()) ** 2


# ------------------------------------------------------------------------------------------------
# The calls.
# ------------------------------------------------------------------------------------------------

def _qkv(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    shape = (case["batch"], case["heads"], _tokens(case), case["dim"])
    return [torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3)]


def prepare(case, seed):
    kind, grid, block = case["kind"], _grid(case), case["block"]
    st = {"case": case, "grid": grid, "block": block}
    if kind == "blockmap":
        # another seed is another layer: its masks are the inputs
        st["params"] = [m[0] for m in _stripes(dict(case, stripes=case["stripes"] + 1000003 * seed))]
        return st
    st["q"], st["k"], st["v"] = _qkv(case, seed)
    if kind == "search":
        st["candidates"] = _stripes(case, case["candidates"])
    elif kind != "dense":
        st["params"] = [m[0] for m in _stripes(case)]
    if kind == "run":
        st["plan"] = psa.plan(st["params"], grid, block, batch=case["batch"])
    elif kind == "run_3d":
        st["pb"] = (case["pt"], case["ph"], case["pw"])
        st["plan"] = psa.plan_3d(st["params"], grid, st["pb"], block, batch=case["batch"])
    return st


def run(st):
    case, grid, block = st["case"], st["grid"], st["block"]
    kind = case["kind"]
    if kind == "blockmap":
        return psa.build_blockmap(st["params"], grid, block)
    q, k, v = st["q"], st["k"], st["v"]
    if kind == "fwd":
        return psa.attention_fwd(q, k, v, grid, block, st["params"], return_lse=case["lse"])
    if kind == "run":
        return psa.run(q, k, v, grid, block, st["plan"], return_lse=case["lse"])
    if kind == "dense":
        return psa.dense_fwd(q, k, v, block, return_lse=case["lse"])
    if kind == "run_3d":
        qb, kb, vb = (psa.to_blocks(x, grid, st["pb"]) for x in (q, k, v))
        return psa.from_blocks(psa.run_3d(qb, kb, vb, grid, st["pb"], block, st["plan"]), grid, st["pb"])
    res = search.score(q, k, v, grid, block, st["candidates"])
    return res.loss, res.sparsity


def work(case):
    n, bh, d = _tokens(case), case["batch"] * case["heads"], case["dim"]
    kind = case["kind"]
    if kind == "blockmap":
        nb = -(-n // case["block"])
        return {"bytes": float(case["heads"]) * (nb * nb + 4 * nb + 8), "flops": 0.0}
    tensor = 2.0 * bh * n * d
    pairs = {"dense": lambda: case["heads"] * float(n) * n,
             "search": lambda: case["heads"] * float(n) * n
             + sum(_kept_pairs(case, m) for h in _stripes(case, case["candidates"]) for m in h)}.get(
                 kind, lambda: sum(_kept_pairs(case, m[0]) for m in _stripes(case)))()
    flops = 4.0 * d * case["batch"] * pairs
    if kind == "search":
        return {"bytes": 3 * tensor + 16.0 * case["heads"] * case["candidates"], "flops": flops}
    lse = 4.0 * bh * n if case["lse"] and kind != "run_3d" else 0.0
    return {"bytes": 4 * tensor + lse, "flops": flops}


def tolerance(case):
    # The outputs of attention are bf16 over bf16 weights: measured 2.9e-3 from the exact values.
    # The losses of a search are norms of differences of such outputs, where the roundings average
    # out: measured 1.5e-5 (the smallest calls average over 1000 times fewer values).
    return {"blockmap": "exact", "search": {"rel": 2e-4}}.get(case["kind"], {"rel": 1e-2})


# ------------------------------------------------------------------------------------------------
# The same in 64 bits.
# ------------------------------------------------------------------------------------------------

def _attend(case, q, k, v, m):
    """(o, lse) in float64 of one head [N, d], restricted to the units that m keeps (all: None)."""
    n, d = q.shape
    q, k, v = q.double() * d ** -0.5, k.double(), v.double()
    o, lse = torch.zeros_like(q), torch.full((n,), -math.inf, dtype=torch.float64, device=q.device)
    if m is None:
        jobs = [(torch.arange(i, min(i + 2048, n), device=q.device), slice(None)) for i in range(0, n, 2048)]
    else:
        # query units that keep the same key units are taken together
        unit = _unit_of(case)
        rows, group = np.unique(_map(case, m), axis=0, return_inverse=True)
        group = group.reshape(-1)[unit]
        jobs = []
        for g in range(len(rows)):
            keys = torch.from_numpy(np.nonzero(rows[g][unit])[0]).to(q.device)
            mine = torch.from_numpy(np.nonzero(group == g)[0]).to(q.device)
            if len(keys):
                jobs += [(part, keys) for part in mine.split(4096)]
    for rows_i, keys in jobs:
        s = q[rows_i] @ k[keys].T
        lse[rows_i] = torch.logsumexp(s, 1)
        o[rows_i] = torch.softmax(s, 1) @ v[keys]
    return o, lse


def exact(case, seed):
    kind = case["kind"]
    if kind == "blockmap":
        st = _stripes(dict(case, stripes=case["stripes"] + 1000003 * seed))
        maps = torch.from_numpy(np.stack([_map(case, m[0]) for m in st])).cuda()
        return maps.to(torch.uint8), maps.sum(2).int(), maps.sum((1, 2))
    n, d, b, h = _tokens(case), case["dim"], case["batch"], case["heads"]
    if work(case)["flops"] > 4e13:
        return None
    q, k, v = _qkv(case, seed)
    if kind == "search":
        cands = _stripes(case, case["candidates"])
        loss, sparsity = np.zeros((h, len(cands[0]))), np.zeros((h, len(cands[0])))
        for j in range(h):
            full = [_attend(case, q[i, j], k[i, j], v[i, j], None)[0] for i in range(b)]
            ref = sum(float((f * f).sum()) for f in full)
            for c, m in enumerate(cands[j]):
                part = [_attend(case, q[i, j], k[i, j], v[i, j], m)[0] for i in range(b)]
                err = sum(float(((p - f) ** 2).sum()) for p, f in zip(part, full))
                loss[j, c], sparsity[j, c] = math.sqrt(err / ref), 1.0 - _map(case, m).mean()
        return loss, sparsity
    masks = [None] * h if kind == "dense" else [m[0] for m in _stripes(case)]
    o = torch.empty((b, h, n, d), dtype=torch.float64, device="cuda")
    lse = torch.empty((b, h, n), dtype=torch.float64, device="cuda")
    for i in range(b):
        for j in range(h):
            o[i, j], lse[i, j] = _attend(case, q[i, j], k[i, j], v[i, j], masks[j])
    return (o, lse) if case["lse"] and kind != "run_3d" else o
