"""Large batches with the learned stop, whose workgroups are of four or eight wavefronts by what the LDS holds,
against the oracle on both sides of the rule's lines (with 256 compute units)."""
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


@pytest.mark.parametrize("D,R,ef,waves", [(128, 32, 300, 12), (96, 64, 384, 12), (128, 32, 256, 12), (128, 64, 193, 12),
                                          (768, 32, 700, 8), (960, 64, 2000, 8)])
def test_stop_equals_oracle(D, R, ef, waves):
    g = np.random.Generator(np.random.PCG64(D + R))
    c = g.standard_normal((12, D))
    X = (c[g.integers(0, 12, 900)] + 0.5 * g.standard_normal((900, D))).astype(np.float32)
    Q = (c[g.integers(0, 12, 20)] + 0.5 * g.standard_normal((20, D))).astype(np.float32)
    M, G, e = synth.rotation(D, 3), synth.knn_graph(X, R, 4), synth.medoid(X)
    idx, blocks = qg.qg_build_index(T(X), T(G), T(M), e), oracle.encode(X, G, M)
    w = [0.05 * g.standard_normal(n) for n in (64 * 16, 64, 64 * 64, 64, 64)] + [np.array([-1.0])]
    w[0][3], w[2][0], w[4][0] = 1.0, 1.0, 1.5  # mostly: expansions since the results changed
    bits = torch.from_numpy(np.concatenate(w)).to(torch.bfloat16).view(torch.int16)
    stop = dict(theta=0.0, t_min=4, t_every=3)
    oi, od, _, _ = oracle.search_ls(blocks, D, R, e, M, Q, 10, ef, w=bits.numpy().view(np.uint16), **stop)
    line = waves * torch.cuda.get_device_properties(0).multi_processor_count
    for nq in (line, line + 1):
        pick = np.arange(nq) % len(Q)
        print(f"stop D={D} R={R} ef={ef} nq={nq}", flush=True)
        ks, efs = (torch.full((nq,), x, dtype=torch.int32, device=DEV) for x in (10, ef))
        for got in (idx.search_stop(T(Q[pick]), 10, ef, bits.to(DEV), **stop),
                    idx.search_mixed_stop(T(Q[pick]), ks, efs, bits.to(DEV), k_max=10, ef_max=ef, **stop)):
            assert np.array_equal(got[0].cpu().numpy(), oi[pick]) and np.array_equal(got[1].cpu().numpy(), od[pick])
