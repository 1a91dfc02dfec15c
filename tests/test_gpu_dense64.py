"""FP64 linewidths on the matrix cores (the dense crystal kernel) against the oracle.

Tolerance: both sides sum the same terms in FP64, each |V|^2 from dot products
of at most a few thousand terms, so they agree to about 1e-12 of the largest
linewidth; 1e-10 is the bound of the FP64 form everywhere.
"""
import numpy as np
import pytest

from oracle import linewidths as olw
from oracle import phonons as oph
from synthetic import configs, models

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2602_23728_amd import kaldo as K  # noqa: E402


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


def run(m, mesh, b, subset=None):
    om, ev, ve = oph.phonons(m, mesh)
    c = K.Crystal.from_model(m)
    sub = None if subset is None else dev(np.asarray(subset, np.int32))
    g = K.linewidths(c, mesh, dev(om), dev(ev), dev(ve), 300.0, b, K.FP64, subset=sub)
    c.device_status()
    return g.cpu().numpy(), olw.crystal_linewidths(m, mesh, om, ev, ve, 300.0, b)


# (atoms, mesh): 1 and 2 atoms by request only (fewer than 9 branches), 3 to 5 by
# default; the random cells' atom pairs have more than four blocks (padded steps and
# several groups of branches), the perovskite's at most four; a unit axis, meshes with
# and without points q1 = q2
@pytest.mark.parametrize("atoms,mesh", [(1, (3, 3, 4)), (2, (4, 3, 2)), (3, (2, 3, 4)), (4, (3, 1, 3)),
                                        (5, (2, 2, 3)), ("perovskite", (5, 3, 2))])
@pytest.mark.parametrize("shape,adaptive", [(configs.GAUSS, True), (configs.LORENTZ, False)])
def test_dense_fp64_matches_oracle(atoms, mesh, shape, adaptive, monkeypatch):
    m = configs.build_model(atoms) if atoms == "perovskite" else models.random_cell(20 + atoms, atoms)
    monkeypatch.setenv("KALDO_CRYSTAL_PATH", "mfma")
    g, go = run(m, mesh, configs.Broadening(shape=shape, adaptive=adaptive, sigma_thz=0.3))
    assert np.max(np.abs(g - go)) <= 1e-10 * go.max()


def test_dense_fp64_subset_and_unpaired_tensor():
    """Only the listed modes are written, and a Phi3 that is not symmetric in its last two
    slots is swept over every ordered pair."""
    m = configs.build_model("perovskite")
    b = configs.Broadening(adaptive=True)
    sub = [0, 17, 44, 61, 90, 91, 119]
    g, go = run(m, (2, 2, 2), b, sub)
    keep = np.zeros(go.size, bool)
    keep[sub] = True
    assert np.max(np.abs(g.reshape(-1) - go.reshape(-1))[keep]) <= 1e-10 * go.max()
    assert np.all(g.reshape(-1)[~keep] == 0.0)
    val = m.fc3_val.copy()
    val[np.flatnonzero(m.fc3_j < m.fc3_k)[::7]] *= 1.25
    m2 = models.Model(**{**m.__dict__, "fc3_val": val})
    g, go = run(m2, (3, 2, 2), b)
    assert np.max(np.abs(g - go)) <= 1e-10 * go.max()
