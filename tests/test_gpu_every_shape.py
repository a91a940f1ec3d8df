"""Every built (D, R) against the oracle: the estimator at the ends of the query's
range, searches through the kernels of batches above 64 queries (binaries of
their own, beside those of smaller batches) with every beam storage, plain, with
settings per query, with the learned stop and captured; and the widest pruning.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2411_12229_amd import qg  # noqa: E402

DEV = torch.device("cuda:0")
SHAPES = [(D, R) for D in (96, 128, 768, 960) for R in (32, 64)]
# a beam for each number of beam registers (1 .. 4, 6, 8) and one in LDS, with k in and beyond the result registers
SETTINGS = [(10, 48), (65, 128), (130, 192), (193, 256), (384, 384), (513, 512), (20, 520)]


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.fixture(scope="module")
def made():
    cache = {}

    def get(D, R, n=1200, nq=26):
        if (D, R) not in cache:
            g = np.random.Generator(np.random.PCG64(7 * D + R))
            c = g.standard_normal((12, D))
            X = (c[g.integers(0, 12, n)] + 0.5 * g.standard_normal((n, D))).astype(np.float32)
            Q = (c[g.integers(0, 12, nq)] + 0.5 * g.standard_normal((nq, D))).astype(np.float32)
            M, G, e = synth.rotation(D, 3), synth.knn_graph(X, R, 4), synth.medoid(X)
            G[::7, R - 1] = -1
            cache[D, R] = (qg.qg_build_index(T(X), T(G), T(M), e), oracle.encode(X, G, M), M, e, Q)
        return cache[D, R]

    return get


@pytest.mark.parametrize("D,R", SHAPES)
def test_estimates(made, D, R):
    idx, blocks, M, e, Q = made(D, R)
    g = np.random.Generator(np.random.PCG64(D))
    signs = np.where(g.random((4, D)) < 0.5, -1.0, 1.0)
    signs[0], signs[1] = 1.0, -1.0
    flat = signs @ M.astype(np.float64)  # rotated: about +-1 in every dimension, so +-127 or next to it
    spike = np.zeros((3, D))
    spike[0, 0], spike[1, D - 1], spike[2, D // 2] = 1.0, -1.0, 1.0
    spike = spike @ M.astype(np.float64)  # rotated: one dimension +-127, the others about 0
    q = np.concatenate([np.zeros((1, D)), flat, 1e-3 * flat, spike, Q]).astype(np.float32)
    v = g.integers(0, len(blocks), len(q)).astype(np.int32)
    print(f"estimate D={D} R={R}", flush=True)
    S, est, dist = (x.cpu().numpy() for x in idx.estimate(T(q), T(v)))
    qrot = oracle.rotate(M, q)
    for i in range(len(q)):
        oS, oe, od = oracle.estimate(blocks, D, R, q[i], qrot[i], int(v[i]))
        assert np.array_equal(S[i], oS) and np.array_equal(est[i], oe) and dist[i] == np.float32(od)


@pytest.mark.parametrize("D,R", SHAPES)
@pytest.mark.parametrize("k,ef", SETTINGS)
def test_plain(made, D, R, k, ef):
    idx, blocks, M, e, Q = made(D, R)
    pick = np.arange(130) % len(Q)
    oi, od, os_ = oracle.search(blocks, D, R, e, M, Q, k, ef, with_stats=True)
    layouts = (1, 0, 3, 2) if (D, R) == (128, 32) else (1,)  # the one shape with a table in LDS
    try:
        for lut in layouts:
            idx.set_launch(4, 3, 0, 1, lut)
            for nq in (130, len(Q)):
                print(f"plain D={D} R={R} k={k} ef={ef} nq={nq} lut={lut}", flush=True)
                ids, dists, st = idx.search(T(Q[pick[:nq]]), k, ef, stats=True)
                assert np.array_equal(ids.cpu().numpy(), oi[pick[:nq]])
                assert np.array_equal(dists.cpu().numpy(), od[pick[:nq]])
                assert np.array_equal(st.cpu().numpy()[:, :3], os_[pick[:nq], :3])
    finally:
        idx.set_launch(4, 3, 0, 1, 1)


@pytest.mark.parametrize("D,R", [(96, 32), (128, 32), (128, 64)])
def test_large_narrow_batch(made, D, R):
    """Beams above 256 entries move to LDS above 3,072 queries."""
    idx, blocks, M, e, Q = made(D, R)
    k, ef = 10, 300
    oi, od = oracle.search(blocks, D, R, e, M, Q, k, ef)
    for nq in (3072, 3073):
        pick = np.arange(nq) % len(Q)
        print(f"D={D} R={R} nq={nq}", flush=True)
        ids, dists = idx.search(T(Q[pick]), k, ef)
        assert np.array_equal(ids.cpu().numpy(), oi[pick]) and np.array_equal(dists.cpu().numpy(), od[pick])


@pytest.mark.parametrize("D,R", SHAPES)
@pytest.mark.parametrize("k,ef", SETTINGS)
def test_mixed(made, D, R, k, ef):
    idx, blocks, M, e, Q = made(D, R)
    own = [(1, 1), (min(10, k), ef // 3), (k, ef)]
    layouts = (1, 3) if (D, R) == (128, 32) else (1,)
    want = [oracle.search(blocks, D, R, e, M, Q, a, b) for a, b in own]
    try:
        for lut in layouts:
            idx.set_launch(4, 3, 0, 1, lut)
            for nq in (130, len(Q)):
                row, which = np.arange(nq) % len(Q), np.arange(nq) % 3
                print(f"mixed D={D} R={R} k={k} ef={ef} nq={nq} lut={lut}", flush=True)
                ids, dists = idx.search_mixed(T(Q[row]), T(np.array([o[0] for o in own], np.int32)[which]),
                                              T(np.array([o[1] for o in own], np.int32)[which]), k_max=k, ef_max=ef)
                ids, dists = ids.cpu().numpy(), dists.cpu().numpy()
                for j, (a, _) in enumerate(own):
                    s = which == j
                    assert np.array_equal(ids[s, :a], want[j][0][row[s]])
                    assert np.array_equal(dists[s, :a], want[j][1][row[s]])
                    assert (ids[s, a:] == -1).all() and np.isinf(dists[s, a:]).all()
    finally:
        idx.set_launch(4, 3, 0, 1, 1)


@pytest.mark.parametrize("D,R", SHAPES)
@pytest.mark.parametrize("k,ef", SETTINGS)
def test_stop(made, D, R, k, ef):
    idx, blocks, M, e, Q = made(D, R)
    g = np.random.Generator(np.random.PCG64(5))
    w = [0.05 * g.standard_normal(n) for n in (64 * 16, 64, 64 * 64, 64, 64)] + [np.array([-1.0])]
    w[0][3], w[2][0], w[4][0] = 1.0, 1.0, 1.5  # mostly: expansions since the results changed
    bits = torch.from_numpy(np.concatenate(w)).to(torch.bfloat16).view(torch.int16)
    stop = dict(theta=0.0, t_min=4, t_every=3)
    print(f"stop D={D} R={R} k={k} ef={ef}", flush=True)
    oi, od, _, _ = oracle.search_ls(blocks, D, R, e, M, Q, k, ef, w=bits.numpy().view(np.uint16), **stop)
    pick = np.arange(130) % len(Q)
    ids, dists, _, _ = idx.search_stop(T(Q[pick]), k, ef, bits.to(DEV), **stop)
    assert np.array_equal(ids.cpu().numpy(), oi[pick]) and np.array_equal(dists.cpu().numpy(), od[pick])
    ks, efs = (torch.full((len(pick),), x, dtype=torch.int32, device=DEV) for x in (k, ef))
    ids, dists = idx.search_mixed_stop(T(Q[pick]), ks, efs, bits.to(DEV), k_max=k, ef_max=ef, **stop)
    assert np.array_equal(ids.cpu().numpy(), oi[pick]) and np.array_equal(dists.cpu().numpy(), od[pick])


@pytest.mark.parametrize("D,R,k,ef", [(128, 32, 10, 48), (128, 64, 100, 200), (768, 32, 10, 96), (960, 64, 100, 384)])
@pytest.mark.parametrize("nq", [20, 90])
def test_captured(made, D, R, k, ef, nq):
    """Recorded searches, replayed between eager ones; some queries outgrow the on-chip visited set."""
    idx, blocks, M, e, Q = made(D, R)
    q = T(Q[np.arange(nq) % len(Q)])
    flags = qg.QG_SEARCH_SMALL_HASH
    oi, od = (x[np.arange(nq) % len(Q)] for x in oracle.search(blocks, D, R, e, M, Q, k, ef))
    idx.search(q, k, ef, flags=flags)
    torch.cuda.synchronize()
    ids = torch.empty((nq, k), dtype=torch.int32, device=DEV)
    dists = torch.empty((nq, k), dtype=torch.float32, device=DEV)
    g = torch.cuda.CUDAGraph()
    try:
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            idx.set_stream(torch.cuda.current_stream())
            qg.qg_search_ex(idx, q, nq, k, ef, flags, ids, dists)
        idx.set_stream(None)
        for rep in range(4):
            print(f"replay {rep} D={D} R={R} nq={nq}", flush=True)
            ids.fill_(-7)
            dists.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(ids.cpu().numpy(), oi) and np.array_equal(dists.cpu().numpy(), od)
            again = idx.search(q, k, ef, flags=flags)
            torch.cuda.synchronize()
            assert np.array_equal(again[0].cpu().numpy(), oi)
    finally:
        idx.set_stream(None)


@pytest.mark.parametrize("refine", [True, False])
def test_wide_prune_in_two_passes(refine):
    """Algorithm 2 at the largest dimension with lists of up to 452 candidates (two passes over the dimensions)."""
    n, D, R, EF = 470, 960, 64, 388
    g = np.random.Generator(np.random.PCG64(9))
    X = (g.standard_normal((12, D))[g.integers(0, 12, n)] + 0.4 * g.standard_normal((n, D))).astype(np.float32)
    M, e = synth.rotation(D, 5), synth.medoid(X)
    G0, fill = synth.random_graph(n, R, 1), synth.random_graph(n, R, 2)
    print(f"prune D={D} EF={EF} refine={refine}", flush=True)
    G, _ = qg.qg_build_graph(T(X), R, EF, 1, T(M), e, T(G0), T(fill), refine=refine, repair=True)
    assert np.array_equal(G.cpu().numpy(), oracle.build_graph(X, R, EF, 1, M, e, G0, fill, refine=refine))
