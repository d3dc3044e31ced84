"""The one-workgroup depth sort of at most 16384 pairs, with the scan of their
counts: lists bit for bit the oracle's at its edges (waves, thousands, its
limit and one more), over depths that need from no digit to all, equal depths
(ties by pair index), and with none, some or all of the pairs culled."""

import numpy as np
import pytest

import oracle
import scenegen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_04847_amd as P
    P.load()
    return P


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float32)


def _depths(rng, kind, n):
    if kind == "scene":
        return rng.uniform(0.3, 20.0, n)
    if kind == "wide":                       # 32 bits of key range, nearly
        return 10.0 ** rng.uniform(-37, 38, n)
    if kind == "ties":
        return rng.choice([1.0, 1.0000001, 2.5], n)
    return np.full(n, 3.0)                   # "equal"


@pytest.mark.parametrize("depths", ["scene", "wide", "ties", "equal"])
@pytest.mark.parametrize("n", [1, 64, 65, 1023, 1025, 9999, 16383, 16384, 16385])
def test_lists_match_the_oracle(gs, n, depths):
    rng = np.random.default_rng(n)
    wh = np.array([[203, 150]], np.int32)
    r = scenegen.synthetic_records(19, 1, wh, n, tile=(16, 16))
    r["depth"] = _depths(rng, depths, n).astype(np.float32)
    r["valid"] = np.where(rng.uniform(size=n) < 0.2, 0, r["valid"])
    _check(gs, wh, n, r)


def test_all_culled(gs):
    wh = np.array([[203, 150]], np.int32)
    r = scenegen.synthetic_records(19, 1, wh, 2000, tile=(16, 16))
    r["valid"] = np.zeros_like(r["valid"])
    _check(gs, wh, 2000, r)


def _check(gs, wh, n, r):
    rec = np.zeros((n, 12), np.float32)
    rec[:, 0:2] = r["mean2d"]
    rec[:, 2] = r["depth"]
    rec[:, 3] = np.where(r["valid"] > 0, r["opacity"], 0.0)
    rec[:, 4:7] = r["conic"]
    rec[:, 7:10] = r["rgb"]
    ranges_o, ids_o, masks_o = oracle.bin_sort(wh, (16, 16), r["valid"], r["mean2d"], r["conic"], r["opacity"],
                                               r["depth"], with_masks=True)
    ctx = gs.Context(max_pairs=n, max_isect=4_000_000, max_tiles=1000, max_views=1)
    cams = gs.Cameras(_t(np.zeros((1, 12))), _t(np.zeros((1, 4))), wh)
    gs.gs_bin_sort(ctx, cams, n, gs.default_settings(), _t(rec))
    st = ctx.status()
    assert st["flags"] == 0 and st["n_isect"] == len(ids_o)
    b = ctx.buffers()
    T = b["n_tiles"]
    ranges = gs._lib.copy_to_host(b["tile_ranges"], 2 * T, np.int32).reshape(T, 2)
    assert np.array_equal(ranges, ranges_o.astype(np.int32))
    if len(ids_o):
        ent = gs._lib.copy_to_host(b["isect_ids"], len(ids_o), np.int32).view(np.uint32)
        assert np.array_equal(ent & 0x0FFFFFFF, ids_o.astype(np.uint32))
        assert np.array_equal(ent >> 28, masks_o.astype(np.uint32))
    ctx.close()
