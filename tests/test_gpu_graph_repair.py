"""Reachability and connectivity repair of Algorithm 2 on given graphs (no
iterations), against the oracle: deep graphs (more breadth-first levels than one
run of launches), many vertices linked from one, full rows, several rounds."""
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


def _graph(kind, n, R, g):
    G = np.full((n, R), -1, np.int32)
    if kind == "path":  # n - 1 levels
        G[:-1, 0] = np.arange(1, n)
    elif kind == "path and islands":  # the islands' only way in are links from the path
        m = n // 2
        G[: m - 1, 3] = np.arange(1, m)
    elif kind == "full hub":  # every reachable row is full: links replace edges
        m = R + 1
        for u in range(m):
            G[u] = [v for v in range(m) if v != u][:R]
    elif kind == "two cliques":  # rows full on both sides
        h = n // 2
        for u in range(n):
            o = g.permutation(h - 1)[:R]
            base = 0 if u < h else h
            G[u] = base + (u - base + 1 + o) % h
    return G


@pytest.mark.parametrize("kind,n", [("path", 150), ("path", 17), ("path and islands", 300), ("full hub", 400),
                                    ("two cliques", 500)])
@pytest.mark.parametrize("R", [32, 64])
def test_repair_equals_oracle(kind, n, R):
    if kind == "two cliques":
        n = max(n, 4 * R)
    g = np.random.Generator(np.random.PCG64(n + R))
    X = g.standard_normal((n, 128)).astype(np.float32)
    X[5] = X[4]  # a tie of distances
    M = synth.rotation(128, 3)
    G0 = _graph(kind, n, R, g)
    print(f"repair {kind} n={n} R={R}", flush=True)
    G, st = qg.qg_build_graph(T(X), R, 64, 0, T(M), 0, T(G0), None, refine=False, repair=True)
    Go = oracle.build_graph(X, R, 64, 0, M, 0, G0, G0, refine=False)
    assert np.array_equal(G.cpu().numpy(), Go)
    assert st["reach_after_repair"] == n and st["reach_before_repair"] == synth.reachable(G0, 0)
    assert st["repairs"] == 0 or st["reach_before_repair"] < n
