"""The projection writes a wave's records as one run: the records of the first
N Gaussians of a scene are those of the whole scene, bit for bit, where the
last wave is full, holds one or lacks one, over two views and with culled and
non-finite Gaussians among them (their opacity word is zero)."""

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


def _records(gs, sc, n):
    from paper_2603_04847_amd import _lib as L
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float32)
    ctx = gs.Context(max_pairs=2 * n, max_isect=1 << 16, max_tiles=1 << 12, max_views=2)
    p = {k: t(sc[k][..., :n]) for k in KEYS}
    cams = L.Cameras(t(sc["viewmat"]), t(sc["intr"]), sc["wh"])
    L.gs_project(ctx, L.make_gaussians(*(p[k] for k in KEYS), sc["sh_degree"]), cams, gs.default_settings())
    torch.cuda.synchronize()
    rec = L.copy_to_host(ctx.buffers()["records"], 2 * n * 12, np.float32).reshape(2, n, 12).copy()
    ctx.close()
    rec[rec[..., 3] == 0] = 0.0      # of a culled pair only the first four words are written
    return rec


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 255, 257, 320])
def test_records_of_a_partial_wave(gs, n):
    sc = scenegen.blob_scene(41, [(203, 150), (96, 64)], 321, sh_degree=2)
    sc["means"][0, 5] = np.nan
    sc["sh"][1, 2, 60] = np.inf
    whole = _records(gs, sc, 321)
    assert (whole[..., 3] > 0).sum() > 200 and (whole[..., 3] == 0).any()
    got = _records(gs, sc, n)
    assert np.array_equal(got.view(np.uint32), whole[:, :n].copy().view(np.uint32))
