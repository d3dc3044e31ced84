"""The forward takes a wave per tile or a wave per part of a tile by the number
of tiles and of pairs: on either side of each line of that rule (8192 tiles;
32768 tiles; 8 pairs a tile) the image, transmittance and last contributors are
those of the counting forward bit for bit, and the part of the lazy lists that it
writes serves the backward (gradients as with whole lists, to the order of float
atomics)."""

import numpy as np
import pytest

import scenegen
from test_gpu_raster_parts import KEYS, _t, gs  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _run(gs, sc, settings, w):  # noqa: F811
    from paper_2603_04847_amd.splat import Splatter
    N = sc["means"].shape[1]
    ctx = gs.Context(max_pairs=N, max_isect=60_000_000, max_tiles=33_000, max_views=1)
    sp = Splatter(ctx, settings)
    params = {k: _t(sc[k]) for k in KEYS}
    rgb, T, last, cams = sp.forward(params, 1, _t(sc["viewmat"]), _t(sc["intr"]), sc["wh"])
    assert ctx.status()["flags"] == 0
    grads = sp.backward(params, 1, cams, T, last, w)[0]
    out = [x.cpu().numpy() for x in (rgb, T, last)], {k: grads[k].cpu().numpy() for k in KEYS}
    ctx.close()
    return out


@pytest.mark.parametrize("W,H,N", [
    (724, 720, 3000), (728, 728, 3000),            # tiles of 8x8: 8190 and 8281
    (728, 728, 66_000), (728, 728, 67_000),        # 8281: just under 8 pairs a tile, and over
    (1448, 1448, 300_000), (1449, 1448, 300_000),  # 32761 and 32942
])
@pytest.mark.parametrize("lazy", [0, 1])
def test_forward_on_either_side_of_the_rule(gs, W, H, N, lazy):  # noqa: F811
    sc = scenegen.frustum_scene(11, W, H, 1.2 * W, 1.2 * W, N, 1, -4.5, 0.5, sh_sd=0.2, random_world=False)
    w = _t(np.random.default_rng(1).normal(size=(W * H, 3)))
    run = lambda stats, lz: _run(gs, sc, gs.default_settings(
        tile_w=8, tile_h=8, lazy_lists=lz, eval_stats=stats), w)
    (a, ga), (b, gb) = run(0, lazy), run(1, 0)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    for k in KEYS:
        assert np.abs(ga[k] - gb[k]).max() <= 1e-4 * np.abs(gb[k]).max(), k
