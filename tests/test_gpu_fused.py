"""The fused crystal kernels (partners swept by boxes, or in rounds) against the oracle.

Tolerance: FP64 sums the same terms on both sides, each |V|^2 from at most a
thousand products, so 1e-10 of the largest linewidth leaves two orders; FP32
projects with |V|^2 good to about 2 sqrt(100) 2^-24 ~ 1e-6 of the largest, 1e-5
is the bound of the FP32 form.  The cut is decided in FP64 in both.
"""
import itertools

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

ADAPT = configs.Broadening(adaptive=True)
FIXED = configs.Broadening(adaptive=False, sigma_thz=0.2)
LORENTZ = configs.Broadening(shape=configs.LORENTZ, adaptive=False, sigma_thz=0.2)


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


def wide_cell(n_blk):
    """Two atoms whose Phi3 has one random entry in each of n_blk atom blocks (not symmetric
    in its last two slots)."""
    m = models.random_cell(31, 2)
    rng = np.random.default_rng(n_blk)
    rep = [tuple(int(x) for x in r) for r in m.rep]
    i, j, k, seen = [], [], [], set()
    for l2, l1, jb, kb in itertools.product(range(len(rep)), range(len(rep)), range(2), range(2)):
        key = (jb, kb) + tuple(np.subtract(rep[l1], rep[l2]))
        if key in seen or len(seen) == n_blk:
            continue
        seen.add(key)
        i.append(rng.integers(6))
        j.append((l1 * 2 + jb) * 3 + rng.integers(3))
        k.append((l2 * 2 + kb) * 3 + rng.integers(3))
    return models.Model(**{**m.__dict__, "fc3_i": np.array(i, np.int32), "fc3_j": np.array(j, np.int32),
                           "fc3_k": np.array(k, np.int32), "fc3_val": rng.uniform(-20.0, 20.0, len(i))})


def few_cell():
    """One atom whose Phi3 has one random entry in each of six blocks, four differences up to
    sign."""
    m = models.random_cell(32, 1)
    rep = [tuple(int(x) for x in r) for r in m.rep]
    rng = np.random.default_rng(5)
    at = [rep.index(d) for d in ((0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1))]
    j = [3 * x + rng.integers(3) for x in at]
    k = [3 * rep.index((0, 0, 0)) + rng.integers(3) for _ in at]
    return models.Model(**{**m.__dict__, "fc3_i": rng.integers(0, 3, 6).astype(np.int32),
                           "fc3_j": np.array(j, np.int32), "fc3_k": np.array(k, np.int32),
                           "fc3_val": rng.uniform(-20.0, 20.0, 6)})


# by boxes: diamond and the one-atom cell of four differences; in rounds: the random cells and
# the one of many blocks; boxes that wrap, that do not divide the mesh, thinner than a box, of
# one point
CASES = [("few", (5, 4, 7), ADAPT), ("few", (2, 9, 3), FIXED), ("diamond", (5, 4, 7), ADAPT), ("diamond", (1, 1, 5), FIXED), ("diamond", (9, 2, 1), LORENTZ),
         ("diamond", (6, 6, 6), FIXED), (1, (5, 3, 4), ADAPT), (2, (4, 5, 3), ADAPT), (2, (3, 1, 6), LORENTZ),
         (3, (3, 2, 4), ADAPT), (4, (2, 3, 2), FIXED), ("wide", (3, 3, 2), ADAPT)]


@pytest.mark.parametrize("cell,mesh,b", CASES)
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_fused_matches_oracle(cell, mesh, b, prec, monkeypatch):
    m = (models.diamond() if cell == "diamond" else few_cell() if cell == "few" else
         wide_cell(145) if cell == "wide"
         else models.random_cell(40 + cell, cell, cutoff=2.9 if cell == 4 else 3.6))
    monkeypatch.setenv("KALDO_CRYSTAL_PATH", "fused")
    om, ev, ve = oph.phonons(m, mesh)
    want = olw.crystal_linewidths(m, mesh, om, ev, ve, 300.0, b)
    c = K.Crystal.from_model(m)
    g = K.linewidths(c, mesh, dev(om), dev(ev), dev(ve), 300.0, b, getattr(K, prec.upper()))
    c.device_status()
    tol = 1e-10 if prec == "fp64" else 1e-5
    assert np.max(np.abs(g.cpu().numpy() - want)) <= tol * want.max()
    # a subset writes its own modes and no other
    sub = np.arange(2, om.size, 5, dtype=np.int32)
    gs = K.linewidths(c, mesh, dev(om), dev(ev), dev(ve), 300.0, b, getattr(K, prec.upper()), subset=dev(sub))
    keep = np.zeros(om.size, bool)
    keep[sub] = True
    gs, g = gs.cpu().numpy().reshape(-1), g.cpu().numpy().reshape(-1)
    assert np.max(np.abs(gs - g)[keep]) <= tol * want.max() and np.all(gs[~keep] == 0.0)
    c.close()
