"""A branch whose input is not finite does not reach the linewidths of modes that never meet it."""
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


# the dense kernel: atom pairs of at most four blocks, and of more (padded to a multiple of four)
@pytest.mark.parametrize("atoms,cutoff", [(4, 2.4), (3, 3.6)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_dense_branch_stays_clean_beside_one_that_is_not(atoms, cutoff, prec, monkeypatch):
    monkeypatch.setenv("KALDO_CRYSTAL_PATH", "mfma")
    m = models.random_cell(40 + atoms, atoms, cutoff=cutoff)
    mesh, q0 = (4, 4, 4), 27  # several branches a workgroup
    om, ev, ve = oph.phonons(m, mesh)
    b = configs.Broadening(adaptive=False, sigma_thz=0.05)
    nb3 = om.shape[1]
    n = np.array(np.unravel_index(q0, mesh))
    q2 = int(np.ravel_multi_index((-2 * n) % mesh, mesh))  # q0 + q0 + q2 = G
    wide = 2 * 2 * np.pi * b.sigma_thz * 1.01
    c = K.Crystal.from_model(m)
    P = getattr(K, prec.upper())

    def run(e, mode):
        return K.linewidths(c, mesh, dev(om), dev(e), dev(ve), 300.0, b, P,
                            subset=dev(np.array([mode], np.int32))).cpu().numpy().reshape(-1)[mode]
    tested = 0
    for bad in range(1, nb3):
        w, w1, w2 = om[q0, bad - 1], om[q0, bad], om[q2]
        if min(np.abs(w + w1 - w2).min(), np.abs(w - w1 - w2).min(), np.abs(w + w2 - w1).min()) < wide:
            continue  # the bad mode is a partner of the one before it
        ev1 = ev.copy()
        ev1[q0, :, bad] = np.nan
        clean = run(ev, q0 * nb3 + bad - 1)
        c.device_status()
        assert run(ev1, q0 * nb3 + bad - 1) == clean, bad
        with pytest.raises(K.KaldoError):
            c.device_status()
        tested += 1
    assert tested >= 3
    c.close()
