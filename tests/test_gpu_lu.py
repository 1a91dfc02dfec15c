"""The blocked LU behind the direct inversion against numpy, at its edges: one block, blocks
and panels (eight blocks) with and without a remainder, odd leading dimensions, with
scattered modes left out.

Tolerance: the matrices are diagonally dominant (condition number below 10), so the solution
of n <= 1200 equations is good to about 10 n 2^-53 ~ 1e-12 of its largest entry; 1e-11.
"""
import numpy as np
import pytest

from synthetic import models

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2602_23728_amd import kaldo as K  # noqa: E402


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("mesh,n", [((1, 1, 1), 3), ((1, 1, 1), 1), ((2, 1, 11), 63), ((2, 1, 11), 64),
                                    ((2, 1, 11), 65), ((5, 5, 3), 225), ((6, 6, 5), 511), ((6, 6, 5), 512),
                                    ((6, 6, 5), 513), ((7, 5, 5), 525), ((7, 7, 5), 577), ((7, 7, 5), 735),
                                    ((7, 8, 7), 1024), ((7, 8, 7), 1101)])
def test_lu_matches_numpy(mesh, n):
    n_all = 3 * int(np.prod(mesh))
    rng = np.random.default_rng(n_all + n)
    act = np.zeros(n_all, bool)
    act[np.sort(rng.choice(n_all, n, replace=False))] = True
    a = rng.uniform(-1.0, 1.0, (n_all, n_all)) / n_all
    a[np.arange(n_all), np.arange(n_all)] = rng.uniform(1.0, 2.0, n_all)
    v = rng.uniform(-1.0, 1.0, (n_all, 3))
    om = np.where(act, 10.0, 0.01)  # rad/ps: the others lie below the floor
    c = K.Crystal.from_model(models.random_cell(41, 1))
    mat = dev(a)
    lam, _ = K.bte_solve(c, mesh, dev(om.reshape(-1, 3)), dev(v.reshape(-1, 3, 3)),
                         dev(np.ones(n_all).reshape(-1, 3)), 300.0, 0.1, mat)
    c.device_status()
    want = np.zeros((n_all, 3))
    want[act] = np.linalg.solve(a[np.ix_(act, act)], v[act])
    assert np.max(np.abs(lam.cpu().numpy() - want)) <= 1e-11 * np.abs(want).max()
    c.close()


def test_singular_matrix_is_reported():
    mesh = (2, 1, 11)
    a = np.diag(np.r_[np.ones(40), 0.0, np.ones(25)])
    c = K.Crystal.from_model(models.random_cell(41, 1))
    K.bte_solve(c, mesh, dev(np.full((22, 3), 10.0)), dev(np.ones((22, 3, 3))), dev(np.ones((22, 3))), 300.0,
                0.1, dev(a))
    with pytest.raises(Exception):
        c.device_status()
    c.close()
