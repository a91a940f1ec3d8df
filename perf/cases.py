"""The work a user of this framework has it do, as a list of measurable cases.

Every case goes through the public binding (``paper_2411_12229_amd.qg``): searching an index (single queries,
batches, per-query settings, the learned stop), building an index from a graph, building the graph itself
(Algorithm 2) and rotating vectors.  Inputs are drawn on the device from a seed.  Their distributions follow the
synthetic workloads of this repository: integer-valued SIFT-shaped data at D = 128, a non-negative factor model at
D = 960, unit-norm embeddings with a low local dimension at D = 96 and 768.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2411_12229_amd import qg

SHAPES = ((96, 32), (96, 64), (128, 32), (128, 64), (768, 32), (768, 64), (960, 32), (960, 64))  # built (D, R)


def listed():
    return [
        # one query at a time: an online service's smallest call, all latency and launches
        dict(name="search_1", kind="search", n=300_000, d=128, r=32, nq=1, k=10, ef=48),
        # a handful of wide queries: a re-ranker's or a crawler's small call
        dict(name="search_small_wide", kind="search", n=60_000, d=960, r=64, nq=37, k=10, ef=128),
        # the benchmark's shape: 1M x 128, 10,000 queries, k = 10 at recall 0.95's beam
        dict(name="search_bench", kind="search", n=1_000_000, d=128, r=32, nq=10_000, k=10, ef=48),
        # a large offline batch at a higher recall
        dict(name="search_large", kind="search", n=1_000_000, d=128, r=32, nq=60_000, k=10, ef=96),
        # text or image embeddings, D = 768
        dict(name="search_embed", kind="search", n=200_000, d=768, r=32, nq=10_000, k=10, ef=48),
        # high recall at k = 100 on wide vectors: the beam outgrows the registers
        dict(name="search_wide_k100", kind="search", n=60_000, d=960, r=64, nq=1_000, k=100, ef=384),
        # what the serving loop launches: requests with their own k and beam in one ragged batch
        dict(name="mixed_serving", kind="mixed", n=300_000, d=96, r=32, nq=3_001, k=100, ef=192),
        # learned early stop on a batch
        dict(name="stop_batch", kind="stop", n=300_000, d=128, r=32, nq=10_000, k=10, ef=64),
        # encoding an index from a finished graph
        dict(name="encode_index", kind="index", n=100_000, d=128, r=32),
        # Algorithm 2, SIFT-shaped, with the refinement and the connectivity repair
        dict(name="build_graph", kind="graph", n=50_000, d=128, r=32, ef=200, iters=2),
        # Algorithm 2 on few wide vectors at R = 64
        dict(name="build_graph_wide", kind="graph", n=6_001, d=960, r=64, ef=150, iters=1),
        # rotating a batch of vectors (the first step of searching and of encoding)
        dict(name="rotate_wide", kind="rotate", n=4_000, d=960, r=64, nq=20_011),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("search", "search", "search", "mixed", "stop", "index", "graph", "rotate"))
    d, r = rng.choice(SHAPES)
    wide = d > 256
    if kind in ("search", "mixed", "stop"):
        n = _log_int(rng, 30_000, 60_000 if wide else 300_000)
        k = rng.choice((1, 10, 10, 20, 64, 65, 100))
        ef = _log_int(rng, 16, 384)
        nq = _log_int(rng, 1, 5_000 if wide else 30_000)
        return dict(kind=kind, n=n, d=d, r=r, nq=nq, k=k, ef=ef)
    if kind == "index":
        return dict(kind=kind, n=_log_int(rng, 2_000, 15_000 if wide else 90_000), d=d, r=r)
    if kind == "graph":
        return dict(kind=kind, n=_log_int(rng, 1_000, 5_000 if wide else 30_000), d=d, r=r,
                    ef=_log_int(rng, 64, 150 if wide else 200), iters=rng.choice((1, 2)))
    return dict(kind=kind, n=4_000, d=d, r=r, nq=_log_int(rng, 1, 20_000))


# ------------------------------------------------------------------ inputs

def _generator(seed, stream, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(1_000_003 * int(seed) + stream)
    return g


def _vectors(d, n, seed, what):
    """n vectors from the distribution of `seed`; `what` (an int) picks independent draws from it."""
    shared, g = _generator(seed, 1), _generator(seed, 10 + what)

    def normal(gen, *shape):
        return torch.randn(shape, generator=gen, device="cuda")

    if d == 960:  # non-negative factor model
        w = normal(shared, d, 64).abs_().div_(8.0)
        out = torch.empty((n, d), device="cuda")
        for s in range(0, n, 1 << 16):
            m = min(n, s + (1 << 16)) - s
            out[s:s + m] = (normal(g, m, 64).abs_() @ w.T + 0.05 * normal(g, m, d)).clamp_(min=0.0)
        return out
    # blobs overlapping in a low-dimensional latent space, with a few directions of each blob's own and a floor
    latent, blobs, own = (12, 1000, 4) if d == 128 else (16, 2048, 4)
    w = normal(shared, d, latent) / math.sqrt(latent)
    centre = normal(shared, blobs, latent)
    dirs = normal(shared, blobs, own, d) * (0.3 / math.sqrt(own))
    label = torch.randint(blobs, (n,), generator=g, device="cuda")
    out = torch.empty((n, d), device="cuda")
    for s in range(0, n, 1 << 16):
        lab = label[s:s + (1 << 16)]
        m = lab.numel()
        v = (centre[lab] + (0.6 if d == 128 else 1.0) * normal(g, m, latent)) @ w.T
        c = normal(g, m, own)
        for j in range(own):
            v += c[:, j:j + 1] * dirs[lab, j]
        v += 0.11 * normal(g, m, d)
        if d == 128:
            out[s:s + m] = (64.0 + 26.0 * v).clamp_(0.0, 255.0).round_()
        else:
            out[s:s + m] = v / v.norm(dim=1, keepdim=True)
    return out


def _rotation(d, seed):
    a = np.random.Generator(np.random.PCG64(1_000_003 * int(seed) + 7)).standard_normal((d, d))
    q, t = np.linalg.qr(a)
    m = np.round((q * np.sign(np.diag(t))).T * 2.0 ** 24) / 2.0 ** 24
    return torch.from_numpy(np.ascontiguousarray(m, dtype=np.float32)).cuda()


def _random_ids(n, r, seed, stream):
    """r distinct ids other than its own for every vertex."""
    gap = torch.randint(1, (n - 1) // r + 1, (n, r), generator=_generator(seed, stream), device="cuda")
    own = torch.arange(n, device="cuda")[:, None]
    return ((own + gap.cumsum(1)) % n).to(torch.int32)


def _entry(x):
    return int((x - x.mean(0)).square_().sum(1).argmin().item())


def _index(case, seed):
    """A navigable index for the search cases: Algorithm 2 with a small beam (a search works without the repair)."""
    n, d, r = case["n"], case["d"], case["r"]
    x, m = _vectors(d, n, seed, 0), _rotation(d, seed)
    entry = _entry(x)
    graph, _ = qg.qg_build_graph(x, r, 48, 2, m, entry, _random_ids(n, r, seed, 2), _random_ids(n, r, seed, 3),
                                 refine=True, repair=False)
    return qg.qg_build_index(x, graph, m, entry)


def _stop_model(seed):
    """A stop model of the library's layout: stop once the nearest neighbours have not changed for some expansions
    (input 3), with small random weights everywhere else."""
    g = np.random.Generator(np.random.PCG64(1_000_003 * int(seed) + 8))
    w1, b1 = 0.02 * g.standard_normal((64, 16)), np.zeros(64)
    w2, b2 = 0.02 * g.standard_normal((64, 64)), np.zeros(64)
    w3, b3 = 0.02 * g.standard_normal(64), np.array([-2.0])
    w1[0, 3], w2[0, 0], w3[0] = 1.0, 1.0, 2.5
    p = torch.from_numpy(np.concatenate([w1.ravel(), b1, w2.ravel(), b2, w3, b3])).to(torch.bfloat16)
    return p.view(torch.int16).cuda()


def prepare(case, seed):
    kind, d, r = case["kind"], case["d"], case["r"]
    state = dict(case=case)
    if kind in ("search", "mixed", "stop"):
        state["index"] = _index(case, seed)
        state["queries"] = _vectors(d, case["nq"], seed, 1)
    if kind == "mixed":
        nq, k, ef = case["nq"], case["k"], case["ef"]
        g = _generator(seed, 4)
        ks = torch.tensor([1, max(1, k // 10), k], dtype=torch.int32, device="cuda")
        efs = torch.tensor([max(1, ef // 8), max(1, ef // 4), ef], dtype=torch.int32, device="cuda")
        state["ks"] = ks[torch.randint(3, (nq,), generator=g, device="cuda")]
        state["efs"] = efs[torch.randint(3, (nq,), generator=g, device="cuda")]
    elif kind == "stop":
        state["mlp"] = _stop_model(seed)
    elif kind in ("index", "graph"):
        n = case["n"]
        state["x"], state["rot"] = _vectors(d, n, seed, 0), _rotation(d, seed)
        state["entry"] = _entry(state["x"])
        state["graph"] = _random_ids(n, r, seed, 2)
        if kind == "graph":
            state["fill"] = _random_ids(n, r, seed, 3)
        else:
            state["graph"][:: 97, r - 3:] = -1  # some vertices short of neighbours
    elif kind == "rotate":
        n = case["n"]
        state["rot"] = _rotation(d, seed)
        state["index"] = qg.qg_build_index(_vectors(d, n, seed, 0), _random_ids(n, r, seed, 2), state["rot"], 0)
        state["queries"] = _vectors(d, case["nq"], seed, 1)
    torch.cuda.synchronize()
    return state


# --------------------------------------------------------------------- run

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "search":
        return state["index"].search(state["queries"], case["k"], case["ef"])
    if kind == "mixed":
        return state["index"].search_mixed(state["queries"], state["ks"], state["efs"], k_max=case["k"],
                                           ef_max=case["ef"])
    if kind == "stop":
        ids, dists, _, _ = state["index"].search_stop(state["queries"], case["k"], case["ef"], state["mlp"],
                                                      theta=0.0, t_min=8, t_every=4)
        return ids, dists
    if kind == "index":
        return qg.qg_build_index(state["x"], state["graph"], state["rot"], state["entry"]).blocks()
    if kind == "graph":
        graph, _ = qg.qg_build_graph(state["x"], case["r"], case["ef"], case["iters"], state["rot"], state["entry"],
                                     state["graph"], state["fill"], refine=True, repair=True)
        return graph
    return state["index"].rotate(state["queries"])


def _block_bytes(d, r):
    return (4 * d + r * (d // 8) + 12 * r + 127) // 128 * 128


def work(case):
    """Bytes and operations one pass cannot do without."""
    kind, d, r = case["kind"], case["d"], case["r"]
    block = _block_bytes(d, r)

    def searches(nq, k, ef):
        # expansions per query: 0.6 to 0.8 times the beam and about ten to reach the neighbourhood
        e = 10 + 0.65 * ef
        # a block holds the raw vector (3 operations a dimension) and r codes (one add for four dimensions)
        return (min(nq * e, case["n"]) * block + nq * (4 * d + 8 * k),
                nq * (2 * d * d + e * (3 * d + r * d / 4)))

    if kind in ("search", "mixed", "stop"):
        nq, k, ef = case["nq"], case["k"], case["ef"]
        if kind == "mixed":
            parts = [searches(nq / 3, k, e) for e in (max(1, ef // 8), max(1, ef // 4), ef)]
            b, f = min(sum(p[0] for p in parts), case["n"] * block + nq * (4 * d + 8 * k)), sum(p[1] for p in parts)
        else:
            b, f = searches(nq, k, ef)
        return {"bytes": int(b + 4 * d * d), "flops": int(f)}
    n = case["n"]
    if kind == "rotate":
        return {"bytes": 8 * case["nq"] * d + 4 * d * d, "flops": 2 * case["nq"] * d * d}
    enc_b = 4 * n * (d + r) + 4 * d * d + n * block
    enc_f = 2 * n * d * d + 6 * n * r * d
    if kind == "index":
        return {"bytes": enc_b, "flops": enc_f}
    ef, it = case["ef"], case["iters"]
    c = ef + r
    sb, sf = searches(n, ef, ef)
    prune = n * 3 * d * (c + r * c / 2)  # distances to the vertex, tests against the kept ones
    refine = n * 5 * d * c * c / 4       # cosines of the pruned candidates to the closer ones
    return {"bytes": int(it * (enc_b + n * block) + 4 * n * (d + 3 * r)),
            "flops": int(it * (enc_f + sf + prune) + refine)}


# ------------------------------------------------------------------- exact

def exact(case, seed):
    """The outputs in 64 bits.  Only the rotation has such values: a search's distances belong to the ids that the
    beam search reaches, and ids, graphs and encoded blocks are whole numbers and bytes."""
    if case["kind"] != "rotate":
        return None
    d = case["d"]
    return _vectors(d, case["nq"], seed, 1).double().cpu() @ _rotation(d, seed).double().cpu().T
