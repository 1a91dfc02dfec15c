"""Sweeps over temperatures in a workspace for eight of them: the same batches but the first.

Tolerance: each temperature sums the same entries in FP64; the order depends on the batch it is
in, 1e-12 of the largest linewidth.
"""
import numpy as np
import pytest

from oracle import phonons as oph
from synthetic import configs, models

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2602_23728_amd import kaldo as K  # noqa: E402


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n_temps", [1, 8, 9, 16, 31])
def test_workspace_for_eight_temperatures(n_temps):
    m = models.diamond()
    mesh = (4, 4, 4)
    om, ev, ve = (dev(x) for x in oph.phonons(m, mesh))
    b = configs.Broadening(adaptive=True)
    c = K.Crystal.from_model(m)
    cache = K.tcache_build(c, mesh, om, ev, ve, b, K.FP64)
    temps = np.linspace(20.0, 2000.0, n_temps)
    want = K.tcache_gamma(c, cache, om, b.nu_min_thz, temps).cpu().numpy()
    eight = 8 * 8 * om.numel()
    assert eight < K.tcache_gamma_workspace(c, mesh)
    for fill in (0x00, 0xFF):
        ws = torch.full((eight,), fill, dtype=torch.uint8, device="cuda")
        got = K.tcache_gamma(c, cache, om, b.nu_min_thz, temps, workspace=ws).cpu().numpy()
        assert np.max(np.abs(got - want)) <= 1e-12 * want.max()
    with pytest.raises(K.KaldoError):
        K.tcache_gamma(c, cache, om, b.nu_min_thz, temps,
                       workspace=torch.empty(eight - 8, dtype=torch.uint8, device="cuda"))
    c.close()
