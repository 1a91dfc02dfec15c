"""Which kernel serves a crystal request on both sides of the rules that choose it, and the
linewidths of each against the oracle.

Tolerance: FP64 sums the same terms on both sides, each |V|^2 from at most a thousand products:
1e-10 of the largest linewidth.
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


MAIN = {"lw_fused", "lw_rounds", "lw_crystal", "lw_mfma_fp64"}


# three and four atoms whose pruned tables fit, on both sides of 80 points; the perovskite's do not
@pytest.mark.parametrize("atoms,cutoff,mesh,kernel", [
    (3, 2.2, (4, 5, 4), "lw_mfma_fp64"), (3, 2.2, (3, 3, 9), "lw_rounds"), (3, 2.2, (4, 6, 4), "lw_rounds"),
    (4, 2.4, (4, 5, 4), "lw_mfma_fp64"), (4, 2.4, (4, 6, 4), "lw_rounds"), ("perovskite", 0, (4, 6, 4), "lw_mfma_fp64")])
def test_fp64_route(atoms, cutoff, mesh, kernel):
    m = configs.build_model(atoms) if atoms == "perovskite" else models.random_cell(40 + atoms, atoms, cutoff=cutoff)
    b = configs.Broadening(adaptive=True)
    om, ev, ve = oph.phonons(m, mesh)
    c = K.Crystal.from_model(m)
    names = {}
    with kernels(names):
        g = K.linewidths(c, mesh, dev(om), dev(ev), dev(ve), 300.0, b, K.FP64).cpu().numpy()
    c.device_status()
    assert MAIN & set(names) == {kernel}
    sub = [k for k in range(0, om.shape[0], 7)]
    go = olw.crystal_linewidths(m, mesh, om, ev, ve, 300.0, b, q_list=sub)
    assert np.max(np.abs(g - go)[sub]) <= 1e-10 * go[sub].max()
    c.close()


# one- and two-atom cells: by boxes, but long thin meshes and, in FP32, a few q of a small mesh
# in rounds; meshes of one chunk per q, and (from 4^3 on) of several
@pytest.mark.parametrize("mesh,prec,modes,kernel", [
    ((2, 2, 2), "fp64", None, "lw_fused"), ((3, 3, 3), "fp32", None, "lw_fused"), ((4, 4, 4), "fp32", None, "lw_fused"),
    ((4, 4, 1), "fp64", None, "lw_fused"), ((5, 5, 1), "fp64", None, "lw_rounds"), ((1, 2, 9), "fp32", None, "lw_rounds"),
    ((6, 6, 6), "fp64", None, "lw_fused"), ((6, 6, 6), "fp32", None, "lw_fused"), ((9, 9, 9), "fp64", None, "lw_fused"),
    ((6, 6, 6), "fp64", 48, "lw_fused"), ((6, 6, 6), "fp32", 48, "lw_rounds"), ((8, 8, 8), "fp32", 1200, "lw_fused"),
    ((12, 12, 12), "fp64", 60, "lw_fused")])
def test_boxes_or_rounds(mesh, prec, modes, kernel):
    m = models.diamond()
    b = configs.Broadening(adaptive=True)
    P = getattr(K, prec.upper())
    om, ev, ve = oph.phonons(m, mesh)
    c = K.Crystal.from_model(m)
    n = om.size
    pick = np.arange(n) if modes is None else np.arange(n // 3, n // 3 + modes)
    sub = None if modes is None else dev(pick.astype(np.int32))
    q = np.unique(pick // 6)
    q = q[:: max(1, len(q) // 20)]
    go = olw.crystal_linewidths(m, mesh, om, ev, ve, 300.0, b, q_list=[int(x) for x in q])
    names = {}
    with kernels(names):
        g = K.linewidths(c, mesh, dev(om), dev(ev), dev(ve), 300.0, b, P, subset=sub).cpu().numpy()
    c.device_status()
    assert MAIN & set(names) == {kernel}
    keep = np.zeros(n, bool)
    keep[pick] = True
    keep = keep.reshape(om.shape) & ~np.isnan(go)
    tol = 1e-10 if prec == "fp64" else 1e-5
    assert np.max(np.abs(g - go)[keep]) <= tol * np.nanmax(go)
    # the temperature cache's passes go the same way and place every chunk's entries
    names = {}
    with kernels(names):
        tc = K.tcache_build(c, mesh, dev(om), dev(ev), dev(ve), b, P, subset=sub)
    assert MAIN & set(names) == {kernel}
    gt = K.tcache_gamma(c, tc, dev(om), b.nu_min_thz, [300.0]).cpu().numpy()[0]
    c.device_status()
    assert np.max(np.abs(gt - go)[keep]) <= tol * np.nanmax(go)
    c.close()
