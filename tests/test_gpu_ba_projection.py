"""The projection of a bundle-adjustment observation divides in double, each
quotient rounded correctly.  A focal length of 2^50 pixels over points with
x = z, whose u = x (1 / z) is 1 or 1 - 2^-53, turns the last place of 1 / z into
1/8 of a pixel, which the step reports in its cost."""

import numpy as np
import pytest

from test_gpu_ba_windows import _step, gs  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cams", [1, 1100])  # one pass, and two
def test_quotients_are_correctly_rounded(gs, cams):  # noqa: F811
    n, f = 20_000, 2.0 ** 50
    z = np.random.default_rng(4).uniform(0.5, 8.0, n).astype(np.float32)
    X = np.stack([z, np.zeros_like(z), z], 1)
    vm = np.tile(np.eye(4, dtype=np.float32)[:3].reshape(1, 12), (cams, 1))
    intr = np.tile(np.array([[f, 1.0, -f, 0.0]], np.float32), (cams, 1))
    zd = z.astype(np.float64)
    r = f * (zd * (1.0 / zd) - 1.0)
    assert 100 < np.count_nonzero(r) < n
    sc = (X, vm, intr, np.zeros(n, np.int32), np.arange(n, dtype=np.int32), np.zeros((n, 2), np.float32))
    want = np.square(r).sum()  # below delta: sums of the squares, exact in double
    st = _step(gs, sc, max_iter=0)[2]
    assert np.abs(r).max() <= 1.0  # the tests' delta
    assert st[3] == 0 and abs(st[2] - want) <= 1e-6 * want
