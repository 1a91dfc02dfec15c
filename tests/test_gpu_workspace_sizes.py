"""Workspaces smaller than the queries return that the calls have always taken: the linewidths
are those of a workspace of the query's size, and what is too small is refused.

Tolerance: other batches of modes and the same kernel, the same bits; another kernel, the same
FP64 terms in another order, 1e-10 of the largest linewidth (FP32: 1e-5).
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


def buffer(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda")


def total(*sizes):
    """Bytes of buffers that each start on a multiple of 256."""
    return sum((int(s) + 255) // 256 * 256 for s in sizes)


def gamma_point_sizes(m, prec):
    """The smallest workspace of a Gamma-point cell: in FP64 of the kernels without matrix cores,
    otherwise 512 modes a batch without the lists of the 16 x 16 blocks."""
    n = 3 * m.n_basis
    bc = np.unique(np.stack([m.fc3_j, m.fc3_k]), axis=1)
    masks = (8 * n, n, n)
    if prec == K.FP64:
        nt = -(-n // 64)
        return total(*masks, 8 * n * n, 8 * 64 * bc.shape[1], 8 * 64 * n * n, 8 * n * nt * nt)
    npad = -(-n // 128) * 128
    nt = npad // 128
    tri = nt * (nt + 1) // 2
    split = (4 * npad * npad,) if prec == K.BF16X3 else ()
    return total(*masks, 4 * npad * npad, 4 * n * n, *split, 4 * 512 * npad * np.bincount(bc[0]).max(),
                 4 * 512 * npad * npad, 8 * n * tri, 16 * nt, 512 * nt, 4 * (-(-n // 512)) * (512 * tri + 1))


# 3 N past one tile, of several tiles, and (glass) of several batches
@pytest.mark.parametrize("name", [22, 43, 130, "glass"])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_gamma_point_smaller_workspace(name, prec):
    m = models.glass(3, ncell=3) if name == "glass" else \
        models.random_cluster_glass(seed=31 + name, n_atoms=name, box=6.0 * (name / 8.0) ** (1 / 3))
    om, E = (dev(x) for x in K.phonons_gamma(m.n_basis, m.mass, m.fc2))
    b = configs.Broadening(adaptive=False, sigma_thz=0.3)
    P = getattr(K, prec.upper())
    c = K.Crystal.from_model(m)
    want = K.linewidths_gamma(c, om, E, 300.0, b, P).cpu().numpy()
    size = gamma_point_sizes(m, P)
    assert size <= int(K.lib().kaldo_linewidths_gamma_workspace(c.handle, P))
    got = K.linewidths_gamma(c, om, E, 300.0, b, P, workspace=buffer(size)).cpu().numpy()
    c.device_status()
    if prec == "fp64":
        assert np.max(np.abs(got - want)) <= 1e-10 * want.max()
    else:
        assert np.array_equal(got, want)
    if prec == "fp64":
        with pytest.raises(K.KaldoError):
            K.linewidths_gamma(c, om, E, 300.0, b, P, workspace=buffer(size - 256))
    c.close()


def test_gamma_point_batches_are_the_same_to_the_bit():
    """FP64 in workspaces for 256, 64 and a few dozen modes a batch."""
    m = models.random_cluster_glass(seed=161, n_atoms=130, box=6.0 * (130 / 8.0) ** (1 / 3))
    om, E = (dev(x) for x in K.phonons_gamma(m.n_basis, m.mass, m.fc2))
    b = configs.Broadening(adaptive=False, sigma_thz=0.3)
    c = K.Crystal.from_model(m)
    full = int(K.lib().kaldo_linewidths_gamma_workspace(c.handle, K.FP64))
    ref = K.linewidths_gamma(c, om, E, 300.0, b, K.FP64).cpu().numpy()
    for size in (full - 256, full // 2, full // 4, full // 6):
        got = K.linewidths_gamma(c, om, E, 300.0, b, K.FP64, workspace=buffer(size)).cpu().numpy()
        assert np.array_equal(got, ref), size
    c.close()


def crystal_sizes(c, mesh, prec, n_d):
    """The workspace of the kernel that sweeps in rounds."""
    nq, nb3 = int(np.prod(mesh)), c.nb3
    cs = 16 if prec == K.FP64 else 8
    return total(8 * nq * nb3, nq * nb3, nq * nb3, 16 * nq * nb3, cs * nq * nb3 * nb3, cs * nq * n_d,
                 4 * (2 * nq + 1), 8 * nq * 16 * nb3, 48 * nq * nb3)


def differences(m):
    rep, nb = np.asarray(m.rep), m.n_basis
    return len({tuple(d) for d in rep[m.fc3_j // 3 // nb] - rep[m.fc3_k // 3 // nb]})


# small meshes, whose tables for the sweep by boxes take more
@pytest.mark.parametrize("mesh", [(1, 1, 1), (3, 3, 3), (5, 4, 7)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_crystal_smaller_workspace(mesh, prec):
    m = models.diamond()
    P = getattr(K, prec.upper())
    om, ev, ve = (dev(x) for x in oph.phonons(m, mesh))
    b = configs.Broadening(adaptive=True)
    c = K.Crystal.from_model(m)
    want = K.linewidths(c, mesh, om, ev, ve, 300.0, b, P).cpu().numpy()
    size = crystal_sizes(c, mesh, P, differences(m))
    got = K.linewidths(c, mesh, om, ev, ve, 300.0, b, P, workspace=buffer(size)).cpu().numpy()
    assert np.max(np.abs(got - want)) <= (1e-10 if prec == "fp64" else 1e-5) * want.max()
    with pytest.raises(K.KaldoError):
        K.linewidths(c, mesh, om, ev, ve, 300.0, b, P, workspace=buffer(size - 256))
    if prec != "bf16x3":
        ref = K.tcache_build(c, mesh, om, ev, ve, b, P)
        tc = K.tcache_build(c, mesh, om, ev, ve, b, P, workspace=buffer(size))
        assert torch.equal(tc.row_ptr, ref.row_ptr)
        g, r = (K.tcache_gamma(c, t, om, b.nu_min_thz, [300.0]).cpu().numpy() for t in (tc, ref))
        assert np.max(np.abs(g - r)) <= (1e-10 if prec == "fp64" else 1e-5) * max(r.max(), 1e-300)
        with pytest.raises(K.KaldoError):
            K.tcache_build(c, mesh, om, ev, ve, b, P, workspace=buffer(size - 256))
    c.device_status()
    c.close()


def test_dense_fp64_smaller_workspace():
    """A cell the pruned kernel serves, in a workspace that holds only the dense kernel's phases."""
    m = models.random_cell(44, 4, cutoff=2.4)
    mesh = (4, 6, 4)
    om, ev, ve = (dev(x) for x in oph.phonons(m, mesh))
    b = configs.Broadening(adaptive=True)
    c = K.Crystal.from_model(m)
    want = K.linewidths(c, mesh, om, ev, ve, 300.0, b, K.FP64).cpu().numpy()
    n = 96 * c.nb3
    size = total(8 * n, n, n, 16 * n, 16 * 96 * differences(m))
    assert size < K.linewidths_workspace(c, mesh, K.FP64)
    got = K.linewidths(c, mesh, om, ev, ve, 300.0, b, K.FP64, workspace=buffer(size)).cpu().numpy()
    assert np.max(np.abs(got - want)) <= 1e-10 * want.max()
    with pytest.raises(K.KaldoError):
        K.linewidths(c, mesh, om, ev, ve, 300.0, b, K.FP64, workspace=buffer(size - 256))
    c.device_status()
    c.close()


# 6, 1,008 and 1,050 modes: one block of 1,024 row pointers and two
@pytest.mark.parametrize("mesh", [(1, 1, 1), (4, 6, 7), (5, 5, 7)])
def test_cache_rows_of_both_sweeps(mesh):
    """Row pointers of the sweep by boxes and, in the smaller workspace, in rounds."""
    m = models.diamond()
    om, ev, ve = (dev(x) for x in oph.phonons(m, mesh))
    b = configs.Broadening(adaptive=True)
    c = K.Crystal.from_model(m)
    ref = K.tcache_build(c, mesh, om, ev, ve, b, K.FP64)
    tc = K.tcache_build(c, mesh, om, ev, ve, b, K.FP64,
                        workspace=buffer(crystal_sizes(c, mesh, K.FP64, differences(m))))
    assert torch.equal(tc.row_ptr, ref.row_ptr) and int(ref.row_ptr[-1]) == ref.n_entries
    c.close()


# 1,296, 7,986 and 8,712 modes: two blocks of 1,024 row pointers, eight, and nine
@pytest.mark.parametrize("mesh", [(6, 6, 6), (11, 11, 11), (11, 11, 12)])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 1e-5)])
def test_cache_rows_of_several_blocks(mesh, prec, tol):
    """Every mode's row, by its linewidth."""
    m = models.diamond()
    c = K.Crystal.from_model(m)
    om, ev, ve = K.phonons(c, mesh)
    b = configs.Broadening(adaptive=True)
    P = getattr(K, prec.upper())
    want = K.linewidths(c, mesh, om, ev, ve, 300.0, b, P).cpu().numpy()
    tc = K.tcache_build(c, mesh, om, ev, ve, b, P)
    got = K.tcache_gamma(c, tc, om, b.nu_min_thz, [300.0])[0].cpu().numpy()
    assert int(tc.row_ptr[-1]) == tc.n_entries
    assert np.max(np.abs(got - want)) <= tol * want.max()
    c.close()
