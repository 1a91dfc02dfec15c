"""FP64 linewidths of a Gamma-point solid of more than 4,096 branches, whose modes go 64 a batch,
on eigenvectors that are any orthonormal basis.

Tolerance: both sides sum the same terms in FP64, each V an inner product of 5,184 terms: 1e-10 of
the largest linewidth as in the smaller cells.
"""
import numpy as np
import pytest

from oracle import linewidths as olw
from synthetic import configs, models

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2602_23728_amd import kaldo as K  # noqa: E402


def test_modes_on_both_sides_of_a_batch():
    m = models.glass(3, ncell=6)
    n = 3 * m.n_basis
    assert n > 4096
    rng = np.random.default_rng(11)
    om = np.sort(rng.uniform(2 * np.pi, 2 * np.pi * 16.0, n))
    E = np.linalg.qr(rng.normal(size=(n, n)))[0]
    b = configs.Broadening(adaptive=False, sigma_thz=0.1)
    pick = [0, 63, 64, 4095, 4096, n - 1]
    c = K.Crystal.from_model(m)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()  # noqa: E731
    g = K.linewidths_gamma(c, dev(om), dev(E), 300.0, b, K.FP64, subset=dev(np.array(pick, np.int32))).cpu().numpy()
    c.device_status()
    c.close()
    go = olw.gamma_point_linewidths(m, om, E, 300.0, b, modes=pick)
    assert np.max(np.abs(g[pick] - go[pick])) <= 1e-10 * go[pick].max()
