"""Points without finite neighbours (not a number, infinite, or so far apart that
their squared distances overflow) have no bound to search by and walk the whole
tree, whose first step takes fewer nodes than a wave has lanes (at these sizes
2, 16, 2 and 4): only nodes that are there may be read.  Their own scale is
infinite; the others' are those of brute force in float64 over the ordinary
points (1e-5 as in the tests of the call)."""

import numpy as np
import pytest

import oracle
from test_gpu_init_waves import _points, _scales, gs  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["nan", "inf", "far"])
@pytest.mark.parametrize("n,k", [(600, 4), (5000, 8), (40_000, 4), (100_000, 4)])
def test_points_without_a_bound(gs, n, k, kind):  # noqa: F811
    pts = _points(n, n)
    bad = np.random.default_rng(2).permutation(n)[:20]
    dirty = pts.copy()
    if kind == "far":
        dirty[bad] = np.random.default_rng(3).normal(size=(20, 3)) * 1e25
    else:
        dirty[bad, np.arange(20) % 3] = np.nan if kind == "nan" else np.inf
    got = _scales(gs, dirty, k)
    assert np.all(np.isinf(got[bad]))
    fine = np.setdiff1d(np.arange(n), bad)
    q = np.sort(np.random.default_rng(0).choice(len(fine), 400, replace=False))
    want = np.maximum(oracle.knn_mean_dist(pts[fine], k, queries=q), 1e-7)
    assert np.max(np.abs(got[fine[q]] / want - 1)) <= 1e-5
