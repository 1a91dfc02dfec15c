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
