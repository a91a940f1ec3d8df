"""The tuner times the beam in LDS for beams of at most 128 entries only; the storage of larger ones is 1."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2411_12229_amd import qg  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("D,R", [(96, 32), (128, 32)])
@pytest.mark.parametrize("mixed", [False, True])
def test_settings_timed(D, R, mixed):
    g = np.random.Generator(np.random.PCG64(D))
    X = g.standard_normal((500, D)).astype(np.float32)
    idx = qg.qg_build_index(*(torch.from_numpy(a).to(DEV) for a in (X, synth.knn_graph(X, R, 4), synth.rotation(D, 3))),
                            synth.medoid(X))
    q = torch.from_numpy(X[:130].copy()).to(DEV)
    launches = {}
    for ef in (128, 129, 300):
        idx.timing(True)
        if mixed:
            ks, efs = (torch.full((130,), v, dtype=torch.int32, device=DEV) for v in (10, ef))
            beam = idx.autotune_mixed(q, ks, efs, 10, ef)[4]
        else:
            beam = idx.autotune(q, 10, ef)[4]
        idx.timing(False)
        launches[ef] = idx.timing_read(1)[0]
        assert ef == 128 or beam == 1
    print(f"D={D} R={R} mixed={mixed}: search launches {launches}", flush=True)
    assert launches[128] == launches[129] + 8 and launches[129] == launches[300]  # eight calls a setting
