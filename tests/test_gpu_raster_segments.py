"""The backward's segments: a tile's gradient sums are those of one wave over
its whole list, bit for bit, however the list is cut.  One view is taken as it
is (few tiles: every list in up to 16 segments) and with rows appended (more
tiles than that: only heavy lists are cut, into up to 8), over lists from
nothing to many times a batch of 64.  Gaussians that meet at most two tiles get
at most two atomic additions a component, whose order does not matter, so their
gradients are compared bit for bit; the others to the rounding of float atomics."""

import numpy as np
import pytest

import scenegen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

KEYS = ("means", "log_scales", "quats", "opacity_logit", "sh")


@pytest.fixture(scope="module")
def gs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_04847_amd as P
    P.load()
    return P


def _t(a, dtype=torch.float32):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype)


def _grads(gs, sc, wh, tile, w):
    from paper_2603_04847_amd import _lib as L
    N = sc["means"].shape[1]
    ctx = gs.Context(max_pairs=N, max_isect=2_000_000, max_tiles=20_000, max_views=1)
    p = {k: _t(sc[k]) for k in KEYS}
    g = L.make_gaussians(*(p[k] for k in KEYS), sc["sh_degree"])
    cams = L.Cameras(_t(sc["viewmat"]), _t(sc["intr"]), np.array([wh], np.int32))
    s = gs.default_settings(tile_w=tile[0], tile_h=tile[1])
    P = cams.n_pixels
    rgb, T = torch.empty((P, 3), device="cuda"), torch.empty((P,), device="cuda")
    last = torch.empty((P,), device="cuda", dtype=torch.int32)
    L.gs_project(ctx, g, cams, s)
    L.gs_bin_sort(ctx, cams, N, s)
    L.gs_render_fwd(ctx, cams, s, None, rgb, T, last)
    v = torch.zeros((P, 3), device="cuda")
    v[:len(w)] = _t(w)
    out = {k: torch.empty_like(p[k]) for k in KEYS}
    v_tw = torch.zeros((1, 6), device="cuda")
    L.gs_render_bwd(ctx, g, cams, s, None, T, last, v, L.make_grads(*(out[k] for k in KEYS)), v_tw)
    torch.cuda.synchronize()
    st = ctx.status()
    assert st["flags"] == 0
    b = ctx.buffers()
    ids = L.copy_to_host(b["isect_ids"], st["n_isect"], np.int32).view(np.uint32) & 0x0FFFFFFF
    tiles = np.bincount(ids, minlength=N)
    img = {k: a.cpu().numpy()[:len(w)] for k, a in (("rgb", rgb), ("T", T), ("last", last))}
    ctx.close()
    return {k: a.cpu().numpy() for k, a in out.items()}, tiles, img


@pytest.mark.parametrize("tile", [(16, 16), (16, 8), (8, 8), (32, 16)])
@pytest.mark.parametrize("n", [60, 2000, 60000])
def test_a_tiles_sums_do_not_depend_on_its_segments(gs, tile, n):
    sc = scenegen.frustum_scene(61, 256, 192, 300.0, 300.0, n, 1, -4.6, 0.4, sh_sd=0.2)
    if n > 2000:                                  # one long list: a third of them in one corner
        k = n // 3
        sc["means"][:, :k] = sc["means"][:, :1] + 0.02 * (sc["means"][:, :k] - sc["means"][:, :1])
    w = np.random.default_rng(3).normal(size=(256 * 192, 3)).astype(np.float32)
    a, _, ia = _grads(gs, sc, (256, 192), tile, w)
    b, tiles, ib = _grads(gs, sc, (256, 2400), tile, w)
    for k in ia:
        assert np.array_equal(ia[k], ib[k]), k
    few = tiles <= 2
    assert few.sum() > n // 4
    for k in KEYS:
        assert np.array_equal(a[k][..., few], b[k][..., few]), k
        assert np.abs(a[k] - b[k]).max() <= 1e-4 * np.abs(a[k]).max(), k
