"""The one-pass bundle-adjustment step past its end: an iteration that finds the
residual below the tolerance ends the step, and the launches after it, of
either parity, leave the result alone.  Steps with room for exactly the
iterations needed and for up to four more agree to float rounding (the sums
run in double, in no fixed order)."""

import numpy as np
import pytest

from test_gpu_ba_windows import _scene, _step, _tracks, gs  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cams,points", [(40, 500), (300, 20_000)])
def test_launches_after_the_end_change_nothing(gs, cams, points):  # noqa: F811
    sc = _scene(cams, cams, _tracks(points, 30))
    tw, X, st = _step(gs, sc, max_iter=100, tol=1e-4)
    its = int(st[0])
    assert 2 <= its <= 90 and st[1] <= 1e-4
    for more in range(5):
        tw1, X1, st1 = _step(gs, sc, max_iter=its + more, tol=1e-4)
        assert int(st1[0]) == its
        assert np.abs(tw1 - tw).max() <= 1e-6 * np.abs(tw).max()
        assert np.abs(X1 - X).max() <= 1e-6 * np.abs(X).max()
        assert abs(st1[1] - st[1]) <= 1e-4 * st[1]


def test_step_without_a_right_hand_side_ends_at_once(gs):  # noqa: F811
    X, vm, intr, cam, pt, xy = _scene(9, 12, _tracks(50, 12))
    vm = vm.copy().reshape(-1, 3, 4)
    vm[:, 2] *= -1.0  # every observation behind the camera: masked
    tw, dX, st = _step(gs, (X, vm.reshape(-1, 12), intr, cam, pt, xy), max_iter=7)
    assert st[0] == 0 and st[1] == 0 and st[3] == len(cam)
    assert not tw.any() and not dX.any()
