"""The raster backward runs the tiles in natural order where the settings say so
(gs_settings.tile_order = 0).  A splat's tiles add their gradient sums in floats
as they run, so the order shows in what an addition loses: the first eight tiles
of a 4096x4096 view (one on each die, whose starts are not at one time) add 2^25
each of something to a splat over the whole view, the last eight take it away,
and thousands of tiles between (further from both than the chip holds waves at
once) add 1 each.  In natural order every 1 is lost beside the large sum (less
than an eighth of its last place) and nothing is left but that place; run
heaviest first, the tiles between, which a second splat makes the heavier, would
come first and their sum stay.  Waves may add out of turn, so one of eight
passes has to show the order; heaviest first, none would."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIDE, TILE = 4096, 16
BIG = 2.0 ** 25


@pytest.fixture(scope="module")
def gs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_04847_amd as P
    P.load()
    return P


def test_backward_runs_in_natural_order(gs):
    from paper_2603_04847_amd.splat import Splatter
    f = lambda a: torch.tensor(a, device="cuda", dtype=torch.float32)
    fx = 300.0
    # on the axis: one splat over the whole view, and behind it one 450 pixels
    # wide (its alpha passes 1/255 out to 1400), which no corner meets
    sd, z = np.array([20000.0, 450.0]), np.array([2.0, 3.0])
    means = np.zeros((3, 2))
    means[2] = z
    quats = np.zeros((4, 2))
    quats[0] = 1.0
    params = dict(means=f(means), log_scales=f(np.tile(np.log(sd * z / fx), (3, 1))), quats=f(quats),
                  opacity_logit=f([-3.9, 0.0]), sh=f(np.zeros((1, 3, 2))))
    ctx = gs.Context(max_pairs=2, max_isect=400_000, max_tiles=(SIDE // TILE) ** 2, max_views=1)
    sp = Splatter(ctx, gs.default_settings(tile_order=0))
    view = np.eye(4)[None, :3].reshape(1, 12)
    rgb, T, last, cams = sp.forward(params, 0, f(view), f([[fx, fx, SIDE / 2, SIDE / 2]]),
                                    np.array([[SIDE, SIDE]], np.int32))
    assert ctx.status()["flags"] == 0
    last = last.view(SIDE, SIDE)
    v = torch.zeros((SIDE, SIDE, 3), device="cuda")
    p = TILE // 2
    q = slice(p, 8 * TILE, TILE)
    v[p, q, 0] = BIG
    v[SIDE - 1 - p, SIDE - 8 * TILE + TILE - 1 - p::TILE, 0] = -BIG  # mirror images: the same alpha
    assert torch.count_nonzero(v) == 16 and last[p, q].max() == 1
    y, x = slice(68 * TILE + p, 188 * TILE, TILE), slice(78 * TILE + p, 178 * TILE, TILE)
    v[y, x, 0] = 1.0
    assert last[y, x].min() == 2
    n = v[y, x, 0].numel()
    alpha = 1.0 / (1.0 + np.exp(3.9))
    kept = []
    for _ in range(8):
        grads, _ = sp.backward(params, 0, cams, T, last.reshape(-1), v.reshape(-1, 3))
        got = float(grads["sh"][0, 0, 0]) / 0.28209479177387814  # of the colour
        kept.append(got / (n * alpha))  # (alpha falls by 1% to the corners)
    ctx.close()
    assert min(abs(x) for x in kept) <= 0.05, kept
