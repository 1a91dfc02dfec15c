"""The count of multiplied 16 x 16 blocks behind the vertex GEMM's rate, against the rule of
the kernel block by block: the tiles of the upper triangle for a symmetric Phi3, either order
of a pair off the diagonal, every block of a diagonal tile in its own order."""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from synthetic import configs  # noqa: E402


@pytest.mark.parametrize("n", [40, 128, 300])
@pytest.mark.parametrize("sym", [True, False])
def test_multiplied_blocks(n, sym):
    om = np.sort(np.random.default_rng(n).uniform(0.5, 60.0, n))
    b = configs.Broadening(adaptive=False, sigma_thz=0.2)
    reach = 2 * (2 * np.pi * b.sigma_thz) * (1 + 1e-12) + 1e-9
    npad = -(-n // 128) * 128
    phys = om / (2 * np.pi) >= b.nu_min_thz
    strips = []
    for k in range(npad // 16):
        f = om[16 * k:16 * k + 16][phys[16 * k:16 * k + 16]]
        strips.append((f.min(), f.max()) if len(f) else None)

    def meets(w, u, v):
        return (w + u[0] - v[1] < reach and w + u[1] - v[0] > -reach) or \
               (w - u[1] - v[1] < reach and w - u[0] - v[0] > -reach)

    blocks = 0
    for w in om[phys]:
        for i, u in enumerate(strips):
            for j, v in enumerate(strips):
                if u is None or v is None or (sym and i // 8 > j // 8):
                    continue
                blocks += meets(w, u, v) or (sym and i // 8 != j // 8 and meets(w, v, u))
    flop, _, n_phys = bench.gamma_point_live_flop(om, b, sym)
    assert flop == blocks * 2.0 * 16 * 16 * npad and n_phys == phys.sum()
