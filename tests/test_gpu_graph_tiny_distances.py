"""Pruning of Algorithm 2 where candidates' distances at one vertex lie more
than 31 decades apart, against the oracle: the unit vectors' scales and the
limits that the products are compared with leave the range of fp32 there, and
every such pair has to be decided by the fp64 sums."""
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


def _data(kind, n, D, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    X = g.standard_normal((n, D))
    tiny = np.arange(n) % 4 == 0
    m = int(tiny.sum())
    if kind == "ray":  # multiples of one direction around 1e-33: cosines of exactly 1 beside candidates at 1
        X[tiny] = X[0] * g.integers(1, 40, (m, 1)) * 1e-34
    elif kind == "ball":
        X[tiny] *= 1e-33
    else:  # every scale on both sides of where fp32 ends
        X[tiny] *= 10.0 ** g.uniform(-36, -27, (m, 1))
    return X.astype(np.float32)


@pytest.mark.parametrize("kind", ["ray", "ball", "decades"])
@pytest.mark.parametrize("D,R,EF", [(128, 32, 150), (96, 64, 300), (960, 32, 120)])
@pytest.mark.parametrize("refine", [True, False])
def test_prune_equals_oracle(kind, D, R, EF, refine):
    n = 360
    X = _data(kind, n, D, D + EF)
    M = synth.rotation(D, 5)
    e = synth.medoid(X)
    G0, fill = synth.random_graph(n, R, 1), synth.random_graph(n, R, 2)
    print(f"{kind} D={D} R={R} EF={EF} refine={refine}", flush=True)
    G, _ = qg.qg_build_graph(T(X), R, EF, 1, T(M), e, T(G0), T(fill), refine=refine, repair=True)
    G = G.cpu().numpy()
    Go = oracle.build_graph(X, R, EF, 1, M, e, G0, fill, refine=refine)
    bad = np.nonzero((G != Go).any(axis=1))[0]
    assert bad.size == 0, f"{bad.size} rows differ, e.g. {bad[:5].tolist()}: {G[bad[0]]} vs {Go[bad[0]]}"
