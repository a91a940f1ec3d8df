"""Rotation on both sides of the line between single tiles and blocks of 2 x 2 for wide rows, against the oracle."""
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


@pytest.mark.parametrize("D,n", [(768, 1792), (768, 1793), (768, 2048), (768, 2049), (960, 1424), (960, 1425),
                                 (960, 1632), (960, 1633)])
@pytest.mark.parametrize("offset", [0, 1])
def test_rotation_equals_oracle(D, n, offset):
    g = np.random.Generator(np.random.PCG64(D))
    M = synth.rotation(D, 2)
    X = torch.from_numpy(g.standard_normal((40, D)).astype(np.float32)).to(DEV)
    G = torch.from_numpy(synth.random_graph(40, 32, 1)).to(DEV)
    idx = qg.qg_build_index(X, G, torch.from_numpy(M).to(DEV), 0)
    x = g.standard_normal((n, D)).astype(np.float32)
    buf = torch.zeros(n * D + 4, dtype=torch.float32, device=DEV)
    buf[offset: offset + n * D] = torch.from_numpy(x).to(DEV).reshape(-1)
    print(f"rotate D={D} n={n} offset={offset}", flush=True)
    out = idx.rotate(buf[offset: offset + n * D].view(n, D)).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(40), np.arange(n - 70, n), g.integers(0, n, 150)]))
    assert np.array_equal(out[rows], oracle.rotate(M, x[rows]))
