"""The isotope sum where its words of 64 live tiles begin and end: a branch of 64 tiles of
partners, of 65, of 129; tiles wider than 64 points, on one atom and on five.

Tolerance: the sum's terms are those of the oracle in FP64, in another order: 1e-11 of each
linewidth as in the tests of the larger meshes.
"""
import numpy as np
import pytest

from oracle import isotope as oiso
from synthetic import configs, models

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2602_23728_amd import kaldo as K  # noqa: E402


@pytest.mark.parametrize("atoms,mesh", [(2, (16, 16, 16)), (3, (13, 16, 20)), (1, (1, 127, 65)),
                                        (5, (20, 22, 20)), (1, (31, 42, 50))])
@pytest.mark.parametrize("sigma", [0.02, 0.5])
def test_isotope_tiles_by_words(atoms, mesh, sigma):
    m = models.random_cell(70 + atoms, atoms)
    g = np.linspace(2e-4, 4e-4, atoms)
    b = configs.Broadening(adaptive=False, sigma_thz=sigma)
    c = K.Crystal.from_model(m)
    om, ev, ve = K.phonons(c, mesh)
    got = K.isotope_linewidths(c, mesh, om, ev, ve, list(g), b).cpu().numpy()
    c.device_status()
    evh = (ev if ev.is_complex() else torch.view_as_complex(ev)).cpu().numpy()
    nq = int(np.prod(mesh))
    qs = np.unique(np.r_[0, np.random.default_rng(nq).integers(nq, size=3), nq - 1])
    want = oiso.isotope_linewidths(m, mesh, om.cpu().numpy(), evh, ve.cpu().numpy(), g, b, q_list=qs)[qs]
    np.testing.assert_allclose(got[qs], want, rtol=1e-11, atol=1e-13 * max(want.max(), 1e-300))
    c.close()
