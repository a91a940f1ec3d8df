"""Searches at the edges of the beam's and the result list's register counts
(64 entries a register), against the oracle, through the C ABI."""
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


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.fixture(scope="module")
def made():
    cache = {}

    def get(D, R, n=1500, nq=40):
        if (D, R) not in cache:
            g = np.random.Generator(np.random.PCG64(D + R))
            c = g.standard_normal((12, D))
            X = (c[g.integers(0, 12, n)] + 0.5 * g.standard_normal((n, D))).astype(np.float32)
            Q = (c[g.integers(0, 12, nq)] + 0.5 * g.standard_normal((nq, D))).astype(np.float32)
            M, G, e = synth.rotation(D, 3), synth.knn_graph(X, R, 4), synth.medoid(X)
            idx = qg.qg_build_index(T(X), T(G), T(M), e)
            cache[D, R] = (idx, oracle.encode(X, G, M), M, e, Q)
        return cache[D, R]

    return get


@pytest.mark.parametrize("D,R", [(96, 32), (128, 64), (960, 64)])
@pytest.mark.parametrize("k,ef", [
    (10, 64), (10, 65), (65, 128), (128, 129), (129, 192), (192, 193), (193, 256), (256, 256), (257, 256),
    (300, 193), (10, 257), (64, 130), (1, 255), (384, 384), (385, 384), (10, 385), (100, 512), (513, 512), (10, 513),
])
def test_equals_oracle(made, D, R, k, ef):
    idx, blocks, M, e, Q = made(D, R)
    print(f"D={D} R={R} k={k} ef={ef}", flush=True)
    oi, od, os_ = oracle.search(blocks, D, R, e, M, Q, k, ef, with_stats=True)
    for flags in (0, qg.QG_SEARCH_SMALL_HASH, qg.QG_SEARCH_LDS_BEAM):
        ids, dists, st = idx.search(T(Q), k, ef, flags=flags, stats=True)
        assert np.array_equal(ids.cpu().numpy(), oi) and np.array_equal(dists.cpu().numpy(), od)
        assert np.array_equal(st.cpu().numpy()[:, :3], os_[:, :3])


@pytest.mark.parametrize("D,R", [(96, 32), (960, 64)])
@pytest.mark.parametrize("k_max,ef_max", [(300, 200), (100, 192), (260, 256), (400, 300), (100, 500)])
def test_mixed_rows_equal_oracle(made, D, R, k_max, ef_max):
    """Per-query settings over the whole range of one launch, output rows wider than the registers hold."""
    idx, blocks, M, e, Q = made(D, R)
    ks = np.array([1, 10, 64, 65, min(129, k_max), k_max], np.int32)[np.arange(len(Q)) % 6]
    efs = np.array([1, 64, 65, 130, ef_max], np.int32)[np.arange(len(Q)) % 5]
    print(f"mixed D={D} R={R} k_max={k_max} ef_max={ef_max}", flush=True)
    ids, dists = idx.search_mixed(T(Q), T(ks), T(efs), k_max=k_max, ef_max=ef_max)
    ids, dists = ids.cpu().numpy(), dists.cpu().numpy()
    for i in range(len(Q)):
        k = int(ks[i])
        oi, od = oracle.search(blocks, D, R, e, M, Q[i:i + 1], k, int(efs[i]))
        assert np.array_equal(ids[i, :k], oi[0]) and np.array_equal(dists[i, :k], od[0])
        assert (ids[i, k:] == -1).all() and np.isinf(dists[i, k:]).all()


@pytest.mark.parametrize("D,R", [(96, 32), (128, 64), (960, 64)])
@pytest.mark.parametrize("nq", [1, 7, 40, 64, 65, 130])
@pytest.mark.parametrize("k,ef", [(10, 48), (100, 200), (70, 600)])
def test_overflowing_queries(made, D, R, nq, k, ef):
    """Queries that outgrow the on-chip visited set, in one launch (at most 64 queries) and in the overflow pass."""
    idx, blocks, M, e, Q = made(D, R)
    q = np.concatenate([Q] * 4)[:nq]
    ids, dists, st = idx.search(T(q), k, ef, flags=qg.QG_SEARCH_SMALL_HASH, stats=True)
    oi, od, os_ = oracle.search(blocks, D, R, e, M, Q, k, ef, with_stats=True)
    oi, od, os_ = (np.concatenate([x] * 4)[:nq] for x in (oi, od, os_))
    print(f"D={D} R={R} nq={nq} k={k} ef={ef}: {int((st[:, 3] == 1).sum())} overflowed", flush=True)
    assert (ef == 48 or (st[:, 3] == 1).any())
    assert np.array_equal(ids.cpu().numpy(), oi) and np.array_equal(dists.cpu().numpy(), od)
    assert np.array_equal(st.cpu().numpy()[:, :3], os_[:, :3])
    ks, efs = np.full(nq, k, np.int32), np.full(nq, ef, np.int32)
    ids, dists = idx.search_mixed(T(q), T(ks), T(efs), k_max=k, ef_max=ef, flags=qg.QG_SEARCH_SMALL_HASH)
    assert np.array_equal(ids.cpu().numpy(), oi) and np.array_equal(dists.cpu().numpy(), od)


@pytest.mark.parametrize("D,R", [(96, 32), (128, 64), (768, 32)])
@pytest.mark.parametrize("k,ef", [(10, 65), (10, 128), (70, 130), (100, 193), (10, 256), (200, 300), (10, 512)])
def test_stop_equals_oracle(made, D, R, k, ef):
    """The learned stop with every beam storage: a model that stops some queries early."""
    idx, blocks, M, e, Q = made(D, R)
    g = np.random.Generator(np.random.PCG64(5))
    w = [0.05 * g.standard_normal(n) for n in (64 * 16, 64, 64 * 64, 64, 64)] + [np.array([-1.0])]
    w[0][3], w[2][0], w[4][0] = 1.0, 1.0, 1.5  # mostly: expansions since the results changed
    bits = torch.from_numpy(np.concatenate(w)).to(torch.bfloat16).view(torch.int16)
    print(f"stop D={D} R={R} k={k} ef={ef}", flush=True)
    oi, od, os_, _ = oracle.search_ls(blocks, D, R, e, M, Q, k, ef, w=bits.numpy().view(np.uint16), theta=0.0, t_min=4,
                                      t_every=3)
    for flags in (0, qg.QG_SEARCH_LDS_BEAM):
        ids, dists, st, _ = idx.search_stop(T(Q), k, ef, bits.to(DEV), theta=0.0, t_min=4, t_every=3, flags=flags,
                                            stats=True)
        assert np.array_equal(ids.cpu().numpy(), oi) and np.array_equal(dists.cpu().numpy(), od)
        assert np.array_equal(st.cpu().numpy()[:, :3], os_[:, :3])


@pytest.mark.parametrize("nq", [1, 40, 90])
def test_captured_searches_replay(made, nq):
    """Small batches (one search launch) and larger ones (with the overflow pass) recorded into a graph, replayed
    between eager calls; some queries outgrow the on-chip visited set."""
    idx, blocks, M, e, Q = made(96, 32)
    q = T(np.concatenate([Q] * 3)[:nq])
    flags = qg.QG_SEARCH_SMALL_HASH
    want = idx.search(q, 10, 130, flags=flags)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    ids = torch.empty((nq, 10), dtype=torch.int32, device=DEV)
    dists = torch.empty((nq, 10), dtype=torch.float32, device=DEV)
    g = torch.cuda.CUDAGraph()
    try:
        with torch.cuda.graph(g, stream=s):
            idx.set_stream(torch.cuda.current_stream())
            qg.qg_search_ex(idx, q, nq, 10, 130, flags, ids, dists)
        idx.set_stream(None)
        for _ in range(4):
            ids.fill_(-7)
            dists.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(ids, want[0]) and torch.equal(dists, want[1])
            again = idx.search(q, 10, 130, flags=flags)
            torch.cuda.synchronize()
            assert torch.equal(again[0], want[0])
    finally:
        idx.set_stream(None)


@pytest.mark.parametrize("mode", ["plain", "mixed", "stop", "mixed stop"])
def test_batch_sizes_agree(made, mode):
    """The workgroup's size follows the batch's: around each change (with 256 compute units) every row is the
    oracle's."""
    D, R, k, ef = 96, 32, 10, 40
    idx, blocks, M, e, Q = made(D, R)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.Generator(np.random.PCG64(5))
    mlp = torch.from_numpy(0.1 * rng.standard_normal(qg.QG_STOP_MLP_PARAMS)).to(torch.bfloat16).view(torch.int16)
    stop = dict(theta=0.0, t_min=4, t_every=3)
    if "stop" in mode:
        o = oracle.search_ls(blocks, D, R, e, M, Q, k, ef, w=mlp.numpy().view(np.uint16), **stop)
    else:
        o = oracle.search(blocks, D, R, e, M, Q, k, ef)
    for nq in (7, 8, cus, 2 * cus, 2 * cus + 1, 4 * cus, 4 * cus + 1, 8 * cus, 8 * cus + 1):
        pick = np.arange(nq) % len(Q)
        q = T(Q[pick])
        ks, efs = (torch.full((nq,), v, dtype=torch.int32, device=DEV) for v in (k, ef))
        print(f"{mode} nq={nq}", flush=True)
        if mode == "plain":
            got = idx.search(q, k, ef)
        elif mode == "mixed":
            got = idx.search_mixed(q, ks, efs, k_max=k, ef_max=ef)
        elif mode == "stop":
            got = idx.search_stop(q, k, ef, mlp.to(DEV), **stop)
        else:
            got = idx.search_mixed_stop(q, ks, efs, mlp.to(DEV), k_max=k, ef_max=ef, **stop)
        assert np.array_equal(got[0].cpu().numpy(), o[0][pick]) and np.array_equal(got[1].cpu().numpy(), o[1][pick])
