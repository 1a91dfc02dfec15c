"""A cell whose third-order constants hold 200,000 lattice vectors without their negatives
is made in time that grows with their number, not with its square: 12 us a vector at most
(a comparison with every earlier vector took more than twice that at this number).
"""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2602_23728_amd import kaldo as K  # noqa: E402


def cell(n):
    i = np.arange(n)
    rep = np.stack([i // 400, i % 20, i // 20 % 20], axis=1).astype(np.int32)
    fc2 = np.zeros((3, n, 3))
    fc2[:, 0, :] = np.eye(3)
    # (0, j in cell r, k in cell 0): one vector for each r, none its negative
    return K.Crystal(1, np.eye(3) * 3.0, np.ones(1), rep, fc2, np.zeros(n, np.int32),
                     (3 * i).astype(np.int32), np.zeros(n, np.int32), np.full(n, 1e-3))


def test_many_lattice_vectors():
    cell(100).close()  # the device and the library, outside the timing
    t0 = time.monotonic()
    c = cell(200_000)
    took = time.monotonic() - t0
    c.close()
    assert took < 200_000 * 12e-6, took
