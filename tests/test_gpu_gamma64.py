"""Gamma-point linewidths in FP64 on the matrix cores, and every form's tiling at its edges.

Tolerance in FP64: both sides sum the same terms, each V an inner product of 3N terms, so they
agree to about 1e-12 of the largest linewidth; 1e-10 is the bound of the FP64 form everywhere.
FP32: products rounded to 6e-8, times the cancellation in V (up to a few hundred on these small
clusters), 1e-4 on modes above 1e-3 of the largest linewidth.
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


def inputs(name):
    if name == "supercell":
        return models.supercell_gamma(configs.build_model("diamond"), (3, 3, 3))
    return models.random_cluster_glass(seed=31 + name, n_atoms=name, box=6.0 * (name / 8.0) ** (1 / 3))


# 3 N below, at and past a strip of 16, a W block of 64, a tile of 128 and two tiles
@pytest.mark.parametrize("name", [2, 5, 16, 21, 22, 43, 86, "supercell"])
@pytest.mark.parametrize("shape", [configs.GAUSS, configs.LORENTZ])
def test_gamma_point_fp64(name, shape):
    m = inputs(name)
    om, E = oph.phonons_gamma_real(m)
    b = configs.Broadening(shape=shape, adaptive=False, sigma_thz=0.3)
    c = K.Crystal.from_model(m)
    g = K.linewidths_gamma(c, dev(om), dev(E), 300.0, b, K.FP64).cpu().numpy()
    c.device_status()
    go = olw.gamma_point_linewidths(m, om, E, 300.0, b)
    assert np.max(np.abs(g - go)) <= 1e-10 * go.max()


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 1e-4)])
def test_gamma_point_unpaired_tensor(prec, tol):
    """A Phi3 that is not symmetric in its last two slots: every tile, each in its own order."""
    m = inputs(50)
    val = m.fc3_val.copy()
    val[np.flatnonzero(m.fc3_j < m.fc3_k)[::5]] *= 1.3
    m = models.Model(**{**m.__dict__, "fc3_val": val})
    om, E = oph.phonons_gamma_real(m)
    b = configs.Broadening(adaptive=False, sigma_thz=0.3)
    P = K.FP64 if prec == "fp64" else K.FP32
    g = K.linewidths_gamma(K.Crystal.from_model(m), dev(om), dev(E), 300.0, b, P).cpu().numpy()
    go = olw.gamma_point_linewidths(m, om, E, 300.0, b)
    big = go > 1e-3 * go.max()
    assert np.max(np.abs(g - go)[big]) <= tol * go.max() if prec == "fp64" else \
        np.max(np.abs(g - go)[big] / go[big]) <= tol


def test_gamma_point_fp64_batches():
    """Modes on both sides of the batch limits of a cell of several batches."""
    m = models.glass(3, ncell=3)
    om, E = oph.phonons_gamma_real(m)
    b = configs.Broadening(adaptive=False)
    pick = [230, 254, 255, 256, 257, 400, 510, 511, 512, 513, 647]
    g = K.linewidths_gamma(K.Crystal.from_model(m), dev(om), dev(E), 300.0, b, K.FP64,
                           subset=dev(np.array(pick, np.int32))).cpu().numpy()
    go = olw.gamma_point_linewidths(m, om, E, 300.0, b, modes=pick)
    assert np.max(np.abs(g[pick] - go[pick])) <= 1e-10 * go[pick].max()
    rest = np.ones(len(g), bool)
    rest[pick] = False
    assert np.all(g[rest] == 0.0)
