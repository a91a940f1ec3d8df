"""The encoder at the edges of its work split (workgroups of four vertices,
edges by four) and its check of the graph, through the C ABI."""
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


def _inputs(n, D, R):
    g = np.random.Generator(np.random.PCG64(n + D + R))
    X = g.standard_normal((n, D)).astype(np.float32)
    return X, synth.rotation(D, 3), synth.random_graph(n, R, 4)


@pytest.mark.parametrize("D", [96, 128, 768, 960])
@pytest.mark.parametrize("R", [32, 64])
@pytest.mark.parametrize("n", [65, 67, 301])
def test_blocks_equal_oracle(n, D, R):
    X, M, G = _inputs(n, D, R)
    X[7] = X[3]  # a degenerate edge: the two vectors coincide
    G[3, 0] = 7 if 7 not in G[3] else G[3, 0]
    G[0, :] = -1  # no neighbours
    G[1, R - 1] = -1
    G[2, ::2] = -1
    G[n - 1, 5] = n - 1  # a self edge
    print(f"encode n={n} D={D} R={R}", flush=True)
    got = qg.qg_build_index(T(X), T(G), T(M), 0).blocks().cpu().numpy()
    assert np.array_equal(got, oracle.encode(X, G, M))


@pytest.mark.parametrize("D,R", [(96, 32), (960, 64)])
@pytest.mark.parametrize("u,j,what", [
    (0, 0, "high"), (66, 0, "negative"), (66, -1, "high"), (33, 5, "negative"),
    (0, -1, "repeat"), (66, 1, "repeat"), (31, 17, "repeat"),
])
def test_bad_graphs_are_refused(D, R, u, j, what):
    X, M, G = _inputs(67, D, R)
    j %= R
    G[u, j] = {"high": 67, "negative": -2, "repeat": G[u, 0 if j else 1]}[what]
    with pytest.raises(qg.QGError) as e:
        qg.qg_build_index(T(X), T(G), T(M), 0)
    assert e.value.code == qg.QG_EINVAL
    assert ("repeats" if what == "repeat" else "out of range") in str(e.value)
    _, _, G = _inputs(67, D, R)  # the next call is not affected
    assert qg.qg_build_index(T(X), T(G), T(M), 0).n == 67
