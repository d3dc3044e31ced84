"""The one-pass sort of the block entries: lists bit for bit those of the
oracle at block counts on either side of each of its digit widths and of its
limit (2047 blocks and the unused slots' id; more take two passes), with
fewer entries than a tile of 8192, several tiles, and capacities past 2^25,
where eight tiles share one column of counts.  A block of 8x8 tiles is 32x32
pixels."""

import numpy as np
import pytest

import oracle
import scenegen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# blocks across and down: 63, 64, 255, 256, 511, 512, 1023, 1024, 2047, 2048
GRIDS = [(9, 7), (8, 8), (17, 15), (16, 16), (73, 7), (32, 16), (33, 31), (32, 32), (89, 23), (64, 32)]


@pytest.fixture(scope="module")
def gs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_04847_amd as P
    P.load()
    return P


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float32)


@pytest.mark.parametrize("n,cap", [(40, 1 << 13), (2000, 3_000_000), (6000, 40_000_000)])
@pytest.mark.parametrize("grid", GRIDS)
def test_lists_match_the_oracle(gs, grid, n, cap):
    wh = np.array([[32 * grid[0], 32 * grid[1]]], np.int32)
    r = scenegen.synthetic_records(17, 1, wh, n, tile=(8, 8))
    rec = np.zeros((n, 12), np.float32)
    rec[:, 0:2] = r["mean2d"]
    rec[:, 2] = r["depth"]
    rec[:, 3] = np.where(r["valid"] > 0, r["opacity"], 0.0)
    rec[:, 4:7] = r["conic"]
    rec[:, 7:10] = r["rgb"]
    ranges_o, ids_o, masks_o = oracle.bin_sort(wh, (8, 8), r["valid"], r["mean2d"], r["conic"], r["opacity"],
                                               r["depth"], with_masks=True)
    ctx = gs.Context(max_pairs=n, max_isect=cap, max_tiles=16 * grid[0] * grid[1], max_views=1)
    cams = gs.Cameras(_t(np.zeros((1, 12))), _t(np.zeros((1, 4))), wh)
    s = gs.default_settings(tile_w=8, tile_h=8)
    drec = _t(rec)
    for rep in range(2):
        gs.gs_bin_sort(ctx, cams, n, s, drec)
        st = ctx.status()
        assert st["flags"] == 0 and st["n_isect"] == len(ids_o) > n // 2
        b = ctx.buffers()
        T = b["n_tiles"]
        ranges = gs._lib.copy_to_host(b["tile_ranges"], 2 * T, np.int32).reshape(T, 2)
        ent = gs._lib.copy_to_host(b["isect_ids"], len(ids_o), np.int32).view(np.uint32)
        assert np.array_equal(ranges, ranges_o.astype(np.int32)), rep
        assert np.array_equal(ent & 0x0FFFFFFF, ids_o.astype(np.uint32)), rep
        assert np.array_equal(ent >> 28, masks_o.astype(np.uint32)), rep
    ctx.close()
