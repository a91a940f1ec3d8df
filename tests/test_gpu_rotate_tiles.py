"""The rotation at the edges of its tilings (one 16 x 16 tile a wavefront or a
block of 2 x 2, chunks of 32 or 64 columns), bit for bit against the oracle."""
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


@pytest.fixture(scope="module")
def index():
    cache = {}

    def get(D):
        if D not in cache:
            g = np.random.Generator(np.random.PCG64(D))
            X = torch.from_numpy(g.standard_normal((40, D)).astype(np.float32)).to(DEV)
            G = torch.from_numpy(synth.random_graph(40, 32, 1)).to(DEV)
            M = synth.rotation(D, 2)
            cache[D] = (qg.qg_build_index(X, G, torch.from_numpy(M).to(DEV), 0), M)
        return cache[D]

    return get


@pytest.mark.parametrize("D", [96, 128, 768, 960])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 257, 1000, 2729, 8193, 10921])
@pytest.mark.parametrize("offset", [0, 1])
def test_rotation_equals_oracle(index, D, n, offset):
    """offset 1: rows that start 4 bytes past a 16-byte boundary (one column per lane)."""
    if offset and n > 1000:
        n = 1000 + n % 16
    idx, M = index(D)
    g = np.random.Generator(np.random.PCG64(n))
    x = g.standard_normal((n, D)).astype(np.float32)
    buf = torch.zeros(n * D + 4, dtype=torch.float32, device=DEV)
    buf[offset: offset + n * D] = torch.from_numpy(x).to(DEV).reshape(-1)
    v = buf[offset: offset + n * D].view(n, D)
    assert v.data_ptr() % 16 == 4 * offset
    out = idx.rotate(v).cpu().numpy()
    rows = np.arange(n) if n <= 1000 else np.unique(np.concatenate([np.arange(40), np.arange(n - 70, n),
                                                                    g.integers(0, n, 200)]))
    assert np.array_equal(out[rows], oracle.rotate(M, x[rows]))
