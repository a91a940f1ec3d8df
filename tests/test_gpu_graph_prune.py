"""Pruning and refinement of Algorithm 2 at the edges of their kernel's tiling, against the oracle.

Every pair of candidates is decided from an approximate cosine or, near a
decision, from the fp64 sums the rules state, so the graph must equal the
oracle's id for id whatever the list length (tiles of 32 candidates, one or
several passes over the dimensions, chunks of 32 or 16 dimensions) and also
where many comparisons are ties: duplicated vectors, coinciding directions,
small-integer coordinates.
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


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _data(kind, n, D, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    if kind == "blobs":
        X = g.standard_normal((20, D))[g.integers(0, 20, n)] + 0.4 * g.standard_normal((n, D))
    elif kind == "duplicates":  # every fourth vector is a copy of another
        X = g.standard_normal((n, D))
        X[::4] = X[1::4][: len(X[::4])]
    elif kind == "rays":  # few directions at many radii: cosines of exactly or nearly 1
        X = g.standard_normal((12, D))[g.integers(0, 12, n)] * g.integers(1, 9, (n, 1))
    elif kind == "integers":  # -1, 0, 1: most distances are tied
        X = g.integers(-1, 2, (n, D)).astype(np.float64)
    elif kind == "scales":  # nearest neighbours at distances from 1e-12 to 1e6
        X = g.standard_normal((n, D)) * 10.0 ** g.uniform(-12, 6, (n, 1))
    return X.astype(np.float32)


@pytest.mark.parametrize("kind,n,D,R,EF", [
    ("blobs", 1500, 128, 32, 1),      # 33 candidates: one past a tile
    ("blobs", 1500, 96, 32, 32),      # 64: whole tiles
    ("blobs", 40, 128, 32, 100),      # lists of at most 39
    ("blobs", 1200, 128, 32, 224),    # 256: the last of the five-tile kernel
    ("blobs", 1200, 768, 32, 225),    # 257: the first of the ten-tile kernel
    ("blobs", 900, 128, 64, 388),     # 452: two passes
    ("blobs", 1150, 96, 64, 1024),    # 1088: the longest lists, chunks of 16 dimensions
    ("duplicates", 1000, 128, 32, 150),
    ("rays", 600, 96, 32, 120),
    ("integers", 800, 96, 64, 200),
    ("scales", 800, 128, 32, 150),
])
@pytest.mark.parametrize("refine", [True, False])
def test_prune_equals_oracle(kind, n, D, R, EF, refine):
    X = _data(kind, n, D, 11 + EF)
    M = synth.rotation(D, 5)
    e = synth.medoid(X)
    G0, fill = synth.random_graph(n, R, 1), synth.random_graph(n, R, 2)
    print(f"{kind} n={n} D={D} R={R} EF={EF} refine={refine}", flush=True)
    G, _ = qg.qg_build_graph(T(X), R, EF, 1, T(M), e, T(G0), T(fill), refine=refine, repair=True)
    G = G.cpu().numpy()
    Go = oracle.build_graph(X, R, EF, 1, M, e, G0, fill, refine=refine)
    bad = np.nonzero((G != Go).any(axis=1))[0]
    assert bad.size == 0, f"{bad.size} rows differ, e.g. {bad[:5].tolist()}: {G[bad[0]]} vs {Go[bad[0]]}"
