"""Gamma-point linewidths by the kernels without matrix cores, by themselves and on request.

Tolerance in FP64: both sides sum the same terms, each V an inner product of 3N terms, 1e-10 of
the largest linewidth; FP32: products rounded to 6e-8, times the cancellation in V (up to a few
hundred on these small clusters), 1e-4 on modes above 1e-3 of the largest linewidth.
"""
import contextlib
import ctypes

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


@contextlib.contextmanager
def kernels(names):
    """Adds to `names` the kernels launched inside, and how often."""
    K.lib().kaldo_profile_begin()
    yield
    rec, n = (K.KernelTime * 64)(), ctypes.c_int32()
    K._check(K.lib().kaldo_profile_end(rec, 64, ctypes.byref(n)))
    names.update({rec[i].name.decode(): rec[i].launches for i in range(n.value)})


def cluster(n):
    return models.random_cluster_glass(seed=31 + n, n_atoms=n, box=6.0 * (n / 8.0) ** (1 / 3))


def run(m, b, P):
    """Linewidths and the names of the kernels that made them."""
    om, E = oph.phonons_gamma_real(m)
    c = K.Crystal.from_model(m)
    names = {}
    with kernels(names):
        g = K.linewidths_gamma(c, dev(om), dev(E), 300.0, b, P).cpu().numpy()
    c.device_status()
    c.close()
    return g, names, om, E


# at most one tile of 64 branches, and past it
@pytest.mark.parametrize("name,kernel", [(5, "gp_gemm"), (21, "gp_gemm"), (22, "gm_gemm_fp64")])
def test_fp64_small_cells_run_without_matrix_cores(name, kernel):
    m = cluster(name)
    b = configs.Broadening(adaptive=False, sigma_thz=0.3)
    g, names, om, E = run(m, b, K.FP64)
    assert kernel in names and len(set(names) & {"gp_gemm", "gm_gemm_fp64"}) == 1
    go = olw.gamma_point_linewidths(m, om, E, 300.0, b)
    assert np.max(np.abs(g - go)) <= 1e-10 * go.max()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_cell_without_third_order_constants(prec):
    m = cluster(2)
    none = {f: getattr(m, f)[:0] for f in ("fc3_i", "fc3_j", "fc3_k", "fc3_val")}
    g, *_ = run(models.Model(**{**m.__dict__, **none}), configs.Broadening(adaptive=False), getattr(K, prec.upper()))
    assert np.all(g == 0.0)


@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
def test_launches_of_the_smallest_cells(prec):
    """Their time is launches: eleven of them."""
    _, names, *_ = run(cluster(2), configs.Broadening(adaptive=False, sigma_thz=0.3), getattr(K, prec.upper()))
    assert sum(names.values()) <= 11, names


def close(got, want, prec):
    if prec == "fp64":
        assert np.max(np.abs(got - want)) <= 1e-10 * want.max()
    else:
        big = want > 1e-3 * want.max()
        assert np.max(np.abs(got - want)[big] / want[big]) <= 1e-4


# 150 branches: tiles of 64 and a ragged one
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [configs.GAUSS, configs.LORENTZ])
@pytest.mark.parametrize("paired", [True, False])
def test_kernels_without_matrix_cores(prec, shape, paired, monkeypatch):
    m = cluster(50)
    if not paired:
        val = m.fc3_val.copy()
        val[np.flatnonzero(m.fc3_j < m.fc3_k)[::5]] *= 1.3
        m = models.Model(**{**m.__dict__, "fc3_val": val})
    b = configs.Broadening(shape=shape, adaptive=False, sigma_thz=0.3)
    monkeypatch.setenv("KALDO_FORCE_GENERIC", "1")
    g, names, om, E = run(m, b, getattr(K, prec.upper()))
    assert "gp_gemm" in names and not any(k.startswith("gm_") for k in names)
    close(g, olw.gamma_point_linewidths(m, om, E, 300.0, b), prec)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_every_atom_bound_to_every_other(prec):
    """372 columns to a tile of rows, more than the matrix-core form stages."""
    m = models.random_cluster_glass(seed=1, n_atoms=124, box=14.0, cutoff=20.0)
    b = configs.Broadening(adaptive=False, sigma_thz=0.5)
    g, names, om, E = run(m, b, getattr(K, prec.upper()))
    assert "gp_gemm" in names and not any(k.startswith("gm_") for k in names)
    pick = [0, 3, 4, 63, 64, 150, 255, 256, 300, 371]
    close(g[pick], olw.gamma_point_linewidths(m, om, E, 300.0, b, modes=pick)[pick], prec)


@pytest.mark.parametrize("name", [21, 22, 50])
def test_fp64_workspace_contents_do_not_matter(name):
    """Filled with 0x00, 0xff and 0x7f, twice each: bitwise the same linewidths."""
    m = cluster(name)
    om, E = oph.phonons_gamma_real(m)
    b = configs.Broadening(adaptive=False, sigma_thz=0.3)
    c = K.Crystal.from_model(m)
    size = int(K.lib().kaldo_linewidths_gamma_workspace(c.handle, K.FP64))
    ref = None
    for fill in (0x00, 0xFF, 0x7F):
        ws = torch.full((size,), fill, dtype=torch.uint8, device="cuda")
        for _ in range(2):
            g = K.linewidths_gamma(c, dev(om), dev(E), 300.0, b, K.FP64, workspace=ws).cpu().numpy()
            ref = g if ref is None else ref
            assert np.array_equal(g, ref), fill
    c.close()
