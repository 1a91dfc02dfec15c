"""The scattering matrix's rows against the oracle at the edges of their rounds and queues:
fewer partners than a wave, one round exactly, one more, wide cuts that pass nearly every
pair (queues that fill within one (s', s'')), one and two atoms, each smearing.

Tolerance: both sides sum the same FP64 terms: 1e-10 of the largest element, as in the tests
of the whole matrix.
"""
import numpy as np
import pytest

from oracle import bte as obte
from oracle import phonons as oph
from synthetic import configs, models

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2602_23728_amd import kaldo as K  # noqa: E402

ADAPT = configs.Broadening(adaptive=True)
WIDE = configs.Broadening(adaptive=False, sigma_thz=3.0)
LORENTZ = configs.Broadening(shape=configs.LORENTZ, adaptive=False, sigma_thz=0.3)


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("atoms,mesh,b", [(1, (2, 3, 2), ADAPT), (1, (4, 4, 4), WIDE), (1, (1, 5, 13), LORENTZ),
                                          (2, (1, 1, 3), WIDE), (2, (2, 4, 8), ADAPT), (2, (3, 4, 6), WIDE),
                                          (2, (5, 3, 3), LORENTZ)])
def test_rows_match_oracle(atoms, mesh, b):
    m = models.random_cell(60 + atoms, atoms)
    om, ev, ve = oph.phonons(m, mesh)
    g0, g1 = obte.scattering_matrix(m, mesh, om, ev, ve, 300.0, b)
    want = g1 + np.diag(g0)
    act = obte.active_modes(om, g0, b.nu_min_thz)
    want[~act, :] = 0.0
    want[:, ~act] = 0.0
    want[np.flatnonzero(~act), np.flatnonzero(~act)] = 1.0
    c = K.Crystal.from_model(m)
    mat, g = K.scattering_matrix(c, mesh, dev(om), dev(ev), dev(ve), 300.0, b)
    c.device_status()
    np.testing.assert_allclose(g.cpu().numpy().ravel(), g0.ravel(), rtol=1e-10, atol=1e-12 * g0.max())
    assert np.max(np.abs(mat.cpu().numpy() - want)) <= 1e-10 * np.abs(want).max()
    again, _ = K.scattering_matrix(c, mesh, dev(om), dev(ev), dev(ve), 300.0, b)
    assert torch.equal(again, mat)
    c.close()
