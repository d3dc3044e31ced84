"""The raster's waves per part of a tile and the backward's plan: image sizes on
either side of the one whose parts are all resident at once (4096 waves), tile
loads from nothing to a dense cluster, ragged edges, every tile shape.  The
forward by parts equals the counting forward (one wave per tile) bit for bit;
the gradients meet the oracle's within the repository's parity rule (1e-4 of
the group's largest, ambiguous pixels left out)."""

import numpy as np
import pytest

import oracle
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


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float32)


def _scene(W, H, N):
    """Splats over the view, two thirds of them small and close together."""
    sc = scenegen.frustum_scene(11, W, H, 1.2 * W, 1.2 * W, N, 1, -2.6, 0.5, sh_sd=0.2,
                                random_world=False)
    n = 2 * N // 3
    c = sc["means"][:, :1]
    sc["means"][:, :n] = c + 0.15 * (sc["means"][:, :n] - c)
    sc["log_scales"][:, :n] -= 1.0
    sc["opacity_logit"][:n] -= 2.0  # long lists before the pixels stop
    return sc


def _run(gs, sc, settings, w):
    from paper_2603_04847_amd.splat import Splatter
    N = sc["means"].shape[1]
    ctx = gs.Context(max_pairs=N, max_isect=4_000_000, max_tiles=20_000, max_views=1)
    sp = Splatter(ctx, settings)
    params = {k: _t(sc[k]) for k in KEYS}
    rgb, T, last, cams = sp.forward(params, 1, _t(sc["viewmat"]), _t(sc["intr"]), sc["wh"])
    assert ctx.status()["flags"] == 0
    grads = sp.backward(params, 1, cams, T, last, _t(w)) if w is not None else None
    torch.cuda.synchronize()
    return rgb.cpu().numpy(), T.cpu().numpy(), last.cpu().numpy(), grads


@pytest.mark.parametrize("lazy", [0, 1])
@pytest.mark.parametrize("tile,order", [((16, 16), 0), ((16, 8), 1), ((8, 8), 2), ((32, 16), 2),
                                        ((32, 16), 1)])
@pytest.mark.parametrize("W,H", [(33, 17), (512, 512), (521, 515), (1030, 530)])
def test_parts_forward_equals_tiles_forward(gs, W, H, tile, order, lazy):
    sc = _scene(W, H, 3000)
    run = lambda stats: _run(gs, sc, gs.default_settings(
        tile_w=tile[0], tile_h=tile[1], tile_order=order, lazy_lists=lazy, eval_stats=stats), None)
    a, b = run(0), run(1)
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("W,H", [(33, 17), (256, 256), (521, 515)])
def test_gradients_of_parts_and_plan(gs, W, H):
    sc = _scene(W, H, 700)
    amb = oracle.render_fwd_bwd(sc)["ambiguous"]
    w = np.random.default_rng(0).normal(size=(W * H, 3))
    w[amb] = 0
    want = oracle.render_fwd_bwd(sc, v_rgb=w)["grads"]
    for tile, order in (((16, 16), 0), ((16, 8), 1), ((8, 8), 0), ((32, 16), 2)):
        s = gs.default_settings(tile_w=tile[0], tile_h=tile[1], tile_order=order, lazy_lists=1)
        grads, tw = _run(gs, sc, s, w)[3]
        for k in (*KEYS, "twist"):
            got = (tw if k == "twist" else grads[k]).cpu().numpy()
            err = np.abs(got - want[k]).max()
            assert err <= 1e-4 * np.abs(want[k]).max(), (k, tile, err)
