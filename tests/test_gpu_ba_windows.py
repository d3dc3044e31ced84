"""The bundle-adjustment step's passes over windows of observations (at most 64
of consecutive points, a lane each): tracks around and past a window, points
without observations, few and many points, and camera counts on either side of
what one workgroup's LDS holds.  The step solves the damped normal equations,
so what is left of the gradient is a small fraction of it (float32 outputs and
the solver's tolerance: the bound of the full-size tests)."""

import numpy as np
import pytest

import oracle
import scenegen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LDS_CAMS = (160 * 1024 - 256) // 160  # cameras whose data fit one workgroup


@pytest.fixture(scope="module")
def gs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_04847_amd as P
    P.load()
    return P


def _scene(seed, C, lengths):
    """C cameras on a sphere; point i seen by lengths[i] of them."""
    rng = np.random.default_rng(seed)
    vm, intr, _ = scenegen.sphere_cameras(rng, [(640, 480)] * C)
    X = rng.normal(0, 0.4, (len(lengths), 3))
    cam = np.concatenate([rng.choice(C, size=n, replace=False) for n in lengths]).astype(np.int64)
    pt = np.repeat(np.arange(len(lengths)), lengths)
    M = vm.astype(np.float64).reshape(-1, 3, 4)[cam]
    p = np.einsum("nij,nj->ni", M[:, :, :3], X[pt]) + M[:, :, 3]
    f = intr.astype(np.float64)[cam]
    xy = f[:, :2] * p[:, :2] / p[:, 2:] + f[:, 2:] + rng.normal(0, 1.0, (len(cam), 2))
    o = np.lexsort((pt, cam))
    X = X + rng.normal(0, 0.01, X.shape)
    return (X.astype(np.float32), vm, intr, cam[o].astype(np.int32), pt[o].astype(np.int32),
            xy[o].astype(np.float32))


def _step(gs, sc, lm=1e-2, max_iter=300, tol=1e-9, copies=True):
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    X, vm, intr, cam, pt, xy = (t(a) for a in sc)
    Pt, C = X.shape[0], vm.shape[0]
    ctx = gs.Context(max_pairs=Pt + 1, max_isect=1 << 10, max_tiles=16, max_views=1, max_cams=C)
    index = gs.track_point_index(ctx, pt, Pt, *((cam, xy) if copies else ()))
    ba = gs.BundleAdjuster(Pt, C)
    dtw = torch.full((C, 6), 7.0, device="cuda")
    dX = torch.full((Pt, 3), 7.0, device="cuda")
    stats = torch.zeros(5, device="cuda")
    gs.gs_ba_lm_step(ba, X, vm, intr, cam, pt, xy, index, 1.0, lm, 0.01, max_iter, tol, dtw, dX, stats)
    torch.cuda.synchronize()
    return dtw.cpu().numpy(), dX.cpu().numpy(), stats.cpu().numpy()


def _tracks(n, longest, seed=0):
    """Track lengths 2 .. 8, among them empty points, whole and over-long windows."""
    rng = np.random.default_rng(seed)
    lengths = rng.integers(2, 9, n)
    for i, v in zip(range(0, n, 7), (0, 0, 63, 64, 65, 0, longest) * n):
        lengths[i] = min(v, longest)
    return lengths


@pytest.mark.parametrize("copies", [True, False])
@pytest.mark.parametrize("cams,points,longest", [
    (3, 1, 3), (70, 63, 70), (70, 64, 70), (300, 65, 200), (300, 4099, 300), (20, 70_000, 9),
    (LDS_CAMS, 3000, 129), (LDS_CAMS + 1, 3000, 129)])
def test_step_solves_the_normal_equations(gs, cams, points, longest, copies):
    sc = _scene(cams + points, cams, _tracks(points, longest) if points > 1 else np.array([3]))
    dtw, dX, stats = _step(gs, sc, copies=copies)
    X, vm, intr, cam, pt, xy = sc
    g = np.concatenate([a.reshape(-1) for a in oracle.ba_normal_residual(
        X, vm, intr, cam, pt, xy, np.zeros_like(dtw), np.zeros_like(dX), lm_lambda=1e-2)])
    r = np.concatenate([a.reshape(-1) for a in oracle.ba_normal_residual(
        X, vm, intr, cam, pt, xy, dtw, dX, lm_lambda=1e-2)])
    assert np.linalg.norm(r) <= 1e-4 * np.linalg.norm(g)
    assert stats[4] == 0 and stats[3] == 0
    empty = np.setdiff1d(np.arange(points), pt)
    assert np.all(dX[empty] == 0)


@pytest.mark.parametrize("cams", [40, LDS_CAMS + 1])
def test_no_iterations_and_unsorted_observations(gs, cams):
    sc = _scene(5, cams, _tracks(500, 40))
    dtw, dX, stats = _step(gs, sc, max_iter=0)
    assert np.all(dtw == 0) and stats[0] == 0 and stats[1] == 1 and np.any(dX != 0)
    X, vm, intr, cam, pt, xy = sc
    dtw, dX, stats = _step(gs, (X, vm, intr, cam[::-1].copy(), pt[::-1].copy(), xy[::-1].copy()))
    assert stats[4] == 1 and np.all(dtw == 0) and np.all(dX == 0)
