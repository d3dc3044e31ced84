"""The wave-wide neighbour search of the Gaussian initialisation at the edges of
its parts: leaves of 8 points, waves of 64, no tree up to 24 points, tree steps
of six levels, every k; and points that are not finite, which no other point
may take as a neighbour.  Against brute force in float64; 1e-5 as in the tests
of the call (float32 distances)."""

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_04847_amd as P
    P.load()
    return P


def _scales(gs, pts, k):
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float32)
    ctx = gs.Context(max_pairs=len(pts), max_isect=1 << 10, max_tiles=16, max_views=1)
    out = gs.gs_init_gaussians(ctx, t(pts), t(np.full(pts.shape, 0.5)), sh_degree=0, k=k)
    torch.cuda.synchronize()
    return np.exp(out["log_scales"][0].cpu().numpy().astype(np.float64))


def _points(n, seed):
    """Dense clusters beside a wide cloud."""
    rng = np.random.default_rng(seed)
    c = rng.normal(0, 2, (4, 3))
    p = np.where(rng.uniform(size=(n, 1)) < 0.7, c[rng.integers(0, 4, n)] + rng.normal(0, 0.03, (n, 3)),
                 rng.normal(0, 3, (n, 3)))
    return p.astype(np.float32)


@pytest.mark.parametrize("k", [1, 4, 5, 8])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 23, 24, 25, 26, 63, 64, 65, 80, 81, 96, 97, 512, 513, 520, 4097, 33000])
def test_scales_at_the_edges(gs, n, k):
    pts = _points(n, n)
    idx = np.arange(n) if n < 5000 else np.random.default_rng(0).choice(n, 1500, replace=False)
    want = np.maximum(oracle.knn_mean_dist(pts, k, queries=np.sort(idx)), 1e-7)
    got = _scales(gs, pts, k)[np.sort(idx)]
    assert np.max(np.abs(got / want - 1)) <= 1e-5


@pytest.mark.parametrize("n", [40, 300, 5000])
def test_points_that_are_not_finite_are_no_neighbours(gs, n):
    pts = _points(n, 7)
    bad = np.random.default_rng(1).permutation(n)[: n // 8]
    dirty = pts.copy()
    dirty[bad[::2], 0] = np.nan
    dirty[bad[1::2], 1] = np.inf
    fine = np.setdiff1d(np.arange(n), bad)
    got = _scales(gs, dirty, 4)[fine]
    want = np.maximum(oracle.knn_mean_dist(pts[fine], 4, queries=np.arange(len(fine))), 1e-7)
    assert np.max(np.abs(got / want - 1)) <= 1e-5
