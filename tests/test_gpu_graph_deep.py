"""Reachability of deep graphs in Algorithm 2's repair: the result on graphs with
more breadth-first levels than the device runs by itself, and the time."""
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


def _layers(n, width, R, g):
    """Levels of `width` vertices each, with ids in any order; every vertex has R random neighbours in the next."""
    order = g.permutation(n).astype(np.int32)
    G = np.full((n, R), -1, np.int32)
    for s in range(0, n - width, width):
        nxt = order[s + width:s + 2 * width]
        for i, u in enumerate(order[s:s + width]):
            pick = np.unique(np.append(g.integers(0, len(nxt), R - 1), i % len(nxt)))
            G[u, :len(pick)] = nxt[pick]
    return G, order


@pytest.mark.parametrize("width,islands", [(1, False), (1, True), (7, True), (100, True), (500, True), (500, False)])
def test_deep_graphs_equal_oracle(width, islands):
    n, D, R = 9000, 96, 32  # two looks of 16 levels each on the device
    g = np.random.Generator(np.random.PCG64(width))
    X = g.standard_normal((n, D)).astype(np.float32)
    M = synth.rotation(D, 3)
    G0, order = _layers(n, width, R, g)
    entry = int(order[0])
    if islands:  # the last third loses its ways in
        inner = np.isin(G0, order[2 * n // 3:]) & np.isin(np.arange(n), order[:2 * n // 3])[:, None]
        G0[inner] = -1
    G0[order[:width], R - 1] = np.roll(order[:width], 1) if width > 1 else -1  # the first level reaches itself
    print(f"width={width} islands={islands}", flush=True)
    G, st = qg.qg_build_graph(T(X), R, 64, 0, T(M), entry, T(G0), None, refine=False, repair=True)
    assert st["reach_before_repair"] == synth.reachable(G0, entry) and st["reach_after_repair"] == n
    assert np.array_equal(G.cpu().numpy(), oracle.build_graph(X, R, 64, 0, M, entry, G0, G0, refine=False))


def test_a_path_does_not_cost_a_launch_per_vertex():
    """200,000 levels of one vertex each.  A host walk takes some 20 ms; a launch per level takes over a second."""
    D, R = 96, 32
    M = T(synth.rotation(D, 3))
    took = {}
    for n in (64, 200_000):  # the small one loads the kernels
        G0 = np.full((n, R), -1, np.int32)
        G0[:-1, 0] = np.arange(1, n)
        G, st = qg.qg_build_graph(torch.zeros((n, D), device=DEV), R, 16, 0, M, 0, T(G0), None, refine=False,
                                  repair=True)
        assert st["reach_before_repair"] == n and st["repairs"] == 0 and torch.equal(G, T(G0))
        took[n] = st["microseconds"]
    print(took, flush=True)
    assert took[200_000] < 400_000
