"""The point-major track pass: a wave's 64 points and their observations 64 by
64.  Point counts around 64 and a workgroup's chunks, tracks that are empty,
end at or span several steps of 64, cameras out of range or masked, and camera
counts on either side of what the LDS holds.  Against the FP64 oracle: a pixel
of up to 700 carries four float32 roundings, 2e-4, into a residual of about
half a pixel at least, so 5e-4 of the largest value (sums over a track or a
camera add terms of independent errors).  The loss's error is relative."""

import numpy as np
import pytest

import oracle
import scenegen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

RTOL = 5e-4


@pytest.fixture(scope="module")
def gs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_04847_amd as P
    P.load()
    return P


def _t(a, dtype=torch.float32):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype)


TRACKS = {
    "one point": [1],
    "one long": [200],
    "empty ends": [0, 0] + [3] * 60 + [0, 0],
    "steps of 64": [64, 64, 1, 63, 65, 0, 127, 2, 128],
    "63": [2] * 63,
    "65": [2] * 64 + [5],
    "mixed": [0, 1, 2, 70, 0, 3] * 70,
    "many": [2, 3, 0, 4] * 20000,
}


@pytest.mark.parametrize("cams", [1, 1200, 1201, 2048])
@pytest.mark.parametrize("tracks", TRACKS)
def test_point_major_pass_matches_oracle(gs, tracks, cams):
    rng = np.random.default_rng(31)
    lengths = np.array(TRACKS[tracks])
    Pt, M = len(lengths), int(lengths.sum())
    vm, intr, _ = scenegen.sphere_cameras(rng, [(640, 480)] * cams)
    X = rng.normal(0, 0.4, (Pt, 3)).astype(np.float32)
    pt = np.repeat(np.arange(Pt), lengths).astype(np.int32)
    cam = rng.integers(0, cams, M).astype(np.int32)
    Mv = vm.astype(np.float64).reshape(-1, 3, 4)[cam]
    if Pt > 5:
        X[5] = 50.0 * X[5]                                # behind some of the cameras
    p = np.einsum("nij,nj->ni", Mv[:, :, :3], X[pt].astype(np.float64)) + Mv[:, :, 3]
    f = intr.astype(np.float64)[cam]
    z = np.maximum(np.abs(p[:, 2:]), 0.1)
    xy = (f[:, :2] * p[:, :2] / z + f[:, 2:] + rng.normal(0, 2.0, (M, 2))).astype(np.float32)
    o = np.lexsort((pt, cam))
    cam, pt, xy = cam[o], pt[o], xy[o]
    bad = rng.uniform(size=M) < 0.02 if M > 100 else np.zeros(M, bool)
    # of the thrown point, only the observations clearly behind or well in view
    bad |= (p[o, 2] > -0.5) & ((p[o, 2] < 0.5) | (np.abs(xy).max(1) > 700))
    want = oracle.track(X, vm, intr, cam[~bad], pt[~bad], xy[~bad], delta=1.0, lam=1e-4, jacobians=False)
    cam = np.where(bad, rng.choice([-1, cams, cams + 7], M), cam).astype(np.int32)
    ctx = gs.Context(max_pairs=Pt + 1, max_isect=1 << 10, max_tiles=16, max_views=1, max_cams=cams)
    c, q, x = _t(cam, torch.int32), _t(pt, torch.int32), _t(xy)
    index = gs.track_point_index(ctx, q, Pt, c, x)
    loss = torch.full((1,), 0.5, device="cuda")
    v_X = torch.full((Pt, 3), 0.25, device="cuda")
    v_tw = torch.full((cams, 6), 0.125, device="cuda")
    ctx.reset_status()
    gs.track_reproj_fwd_bwd(ctx, _t(X), _t(vm), _t(intr), c, q, x, 1.0, 1e-4, 0.01, loss, v_X, v_tw,
                            pt_index=index)
    torch.cuda.synchronize()
    assert ctx.status()["n_masked_obs"] == int(want["masked"].sum())
    for got, add, ref, what in ((v_X, 0.25, want["v_X"], "v_X"), (v_tw, 0.125, want["v_twist"], "twists")):
        got = got.cpu().numpy().astype(np.float64) - add
        tol = RTOL * np.abs(ref).max() + 2e-7             # and the rounding of the value added to
        assert np.abs(got - ref).max() <= tol, (what, np.abs(got - ref).max(), tol)
    assert abs(loss.item() - 0.5 - want["loss"]) <= RTOL * want["loss"] + 1e-6
