// Front-to-back compositing over the depth-sorted tile lists, its backward,
// and the photometric L1 term.
//
// A tile of TW x TH pixels is PPL = TW*TH/64 slots of 64 pixels, each slot in
// fixed tile quadrants; every list entry carries the quadrants its splat
// reaches.  The forward gives each slot (a part of the tile) a wave, one pixel a
// lane; the backward gives a wave a whole tile, PPL pixels a lane, or for the
// heaviest tiles a segment of its list.  Lists are consumed in batches of 64: each lane loads
// one splat record (a gather of 40 B) and stages it in the wave's own LDS
// region; the wave then walks the batch reading each splat's parameters with
// broadcast LDS loads (one address for all lanes), synchronising only with
// itself, while the next batch's records and the entries after it are in
// flight.  The backward walks the lists back to front from each pixel's last
// contributor, recovering the transmittance by division, and sums the splats'
// nine 2D gradients over the whole wave (DPP and lane-swap steps) before one
// lane per component issues the global atomic.
#include <algorithm>

#include "gs_internal.h"

namespace gs {

namespace {

__device__ __forceinline__ int tile_view(const ViewTable& vt, int t) {
    int v = 0;
    while (v + 1 < vt.V && t >= vt.tile_off[v + 1]) v++;
    return v;
}

// Pixel of slot k of a lane inside a TW x TH tile, and the quadrants (TW/2 x
// TH/2 blocks, bit qx + 2 qy) that slot's 64 pixels lie in.  Slots are laid out
// so each one stays inside fixed quadrants: a splat whose entry mask misses
// them is skipped by the whole wave at once.
template <int TW, int TH>
struct TileMap {
    static constexpr int PPL = TW * TH / kWave;
    static_assert(PPL == 1 || PPL == 2 || PPL == 4 || PPL == 8, "tile shape");
    __device__ static __forceinline__ void pixel(int l, int k, int& x, int& y) {
        if constexpr (PPL == 1) {          // 8x8
            x = l % 8;
            y = l / 8;
        } else if constexpr (PPL == 2) {   // 16x8: two 8x8 halves
            x = 8 * k + l % 8;
            y = l / 8;
        } else if constexpr (PPL == 4) {   // 16x16: one 8x8 quadrant per slot
            x = (k % 2) * 8 + l % 8;
            y = (k / 2) * 8 + l / 8;
        } else {                            // 32x16: two 16x4 bands per 16x8 quadrant
            const int q = k / 2;
            x = (q % 2) * 16 + l % 16;
            y = (q / 2) * 8 + (k % 2) * 4 + l / 16;
        }
    }
    static constexpr uint32_t quads(int k) {
        return PPL == 1 ? 0xFu : PPL == 2 ? ((1u << k) | (1u << (k + 2)))
                        : PPL == 4 ? (1u << k) : (1u << (k / 2));
    }
};

// The tile of this workgroup.  Orders 0 and 1 number the workgroups like the
// tiles (1 through the heaviest-first permutation).  Order 2 is for the L2
// caches: workgroups are dealt round-robin over the chip's 8 XCDs, each with
// its own L2, so workgroups b, b + 8, b + 16, ... share one.  Tiles are walked
// block by block (4 x 4 tiles, row-major inside the block) and each block's
// 16 tiles go to 16 consecutive workgroups of one XCD: neighbouring tiles,
// which share most of their splats, read them through the same L2.  Returns
// false for a workgroup whose slot falls outside the view (edge blocks).
constexpr int kXcds = 8;
constexpr int kBlockTileCount = kBlockTiles * kBlockTiles;

__device__ __forceinline__ bool block_tile(int b, const uint32_t* order, int mode, const ViewTable& vt,
                                           int& t) {
    if (mode != 2) {
        t = order ? (int)order[b] : b;
        return true;
    }
    const int x = b % kXcds, j = b / kXcds;
    const int s = ((j / kBlockTileCount) * kXcds + x) * kBlockTileCount + j % kBlockTileCount;
    const int gb = s / kBlockTileCount, w = s % kBlockTileCount;
    if (gb >= vt.block_off[vt.V]) return false;
    int v = 0;
    while (v + 1 < vt.V && gb >= vt.block_off[v + 1]) v++;
    const int lb = gb - vt.block_off[v];
    const int tx = (lb % vt.bx[v]) * kBlockTiles + w % kBlockTiles;
    const int ty = (lb / vt.bx[v]) * kBlockTiles + w / kBlockTiles;
    const int gy = (vt.tile_off[v + 1] - vt.tile_off[v]) / vt.gx[v];
    if (tx >= vt.gx[v] || ty >= gy) return false;
    t = vt.tile_off[v] + ty * vt.gx[v] + tx;
    return true;
}

// One splat record as a lane loads it: position, opacity, the base-2 conic,
// colour.
struct LaneSplat {
    float mx, my, o, a, b, c, cr, cg, cb;
};

__device__ __forceinline__ LaneSplat load_splat(const float4* __restrict__ rec, uint32_t pair) {
    const int64_t p = pair;
    const float4 ra = rec[3 * p], rb = rec[3 * p + 1];
    const float2 rc = *reinterpret_cast<const float2*>(rec + 3 * p + 2);
    const ConicE2 q = conic_e2(rb.x, rb.y, rb.z);
    return {ra.x, ra.y, ra.w, q.a, q.b, q.c, rb.w, rc.x, rc.y};
}

// A batch's splats staged in LDS, one entry per lane as three float4:
// (mx, my, o, -), (a, b, c, r), (g, b, -, -).  Entry i is then read by the
// whole wave from one address (a broadcast), not gathered by readlane.
struct BatchLds {
    float4 f[3][kWave];
};

__device__ __forceinline__ void stage_splat(BatchLds& sb, const LaneSplat& ls) {
    const int lane = threadIdx.x;
    sb.f[0][lane] = make_float4(ls.mx, ls.my, ls.o, 0.f);
    sb.f[1][lane] = make_float4(ls.a, ls.b, ls.c, ls.cr);
    sb.f[2][lane] = make_float4(ls.cg, ls.cb, 0.f, 0.f);
}

// One batch's list entries, loaded by every lane (index clamped into the
// list, which is not empty) and zeroed outside [s, e): the load stays
// unconditional, so the compiler's wait bookkeeping sees it on every path.
__device__ __forceinline__ uint32_t batch_ids(const int32_t* __restrict__ ids, int b, int s, int e) {
    const int j = b + (int)threadIdx.x;
    const uint32_t id = (uint32_t)ids[min(max(j, s), e - 1)];
    return (j >= s && j < e) ? id : 0u;
}

// Where a forward over lazy lists draws its tiles' entries from: the sorted
// block lists (pair; low and high 32 bits of the 64-bit quadrant mask), the
// block ranges, and the tile lists it writes what it reads into.
struct BlockSrc {
    const uint32_t* pair;
    const uint32_t* mlo;
    const uint32_t* mhi;
    const int32_t* branges;
    uint32_t* tids;
};

// Block-list entries a lazy forward keeps in flight (loads of 64 each), and
// the LDS ring its filtered entries queue in: at most 63 waiting plus one
// refill of kPull * 64.
constexpr int kPull = 8;
constexpr uint32_t kRing = 1024;
static_assert(kRing >= kWave - 1 + kPull * kWave, "ring");

// The counting forward (gs_settings.eval_stats): a wave per tile, PPL pixels a
// lane, which also counts what the tile read and evaluated.  The plain forward
// is k_render_fwd_part below; both give the same image bit for bit.
template <int TW, int TH, bool LAZY>
__global__ __launch_bounds__(64) void k_render_fwd_stats(const float4* __restrict__ rec,
                                                   const int32_t* __restrict__ ids,
                                                   const int32_t* __restrict__ ranges,
                                                   const uint32_t* __restrict__ order, ViewTable vt,
                                                   RasterParams rp, const float* __restrict__ bg,
                                                   float* __restrict__ out_rgb,
                                                   float* __restrict__ out_T,
                                                   int32_t* __restrict__ out_last,
                                                   int32_t* __restrict__ tile_contrib,
                                                   int32_t* __restrict__ tile_entries,
                                                   int32_t* __restrict__ tile_evals, int mode,
                                                   BlockSrc src) {
    using TM = TileMap<TW, TH>;
    constexpr int PPL = TM::PPL;
    int t;
    if (!block_tile(blockIdx.x, order, mode, vt, t)) return;
    const int v = tile_view(vt, t);
    const int lt = t - vt.tile_off[v];
    const int gx = vt.gx[v], W = vt.W[v], H = vt.H[v];
    const int tx = lt % gx, ty = lt / gx;
    const int lane = threadIdx.x;
    const float amin = rp.alpha_min, amax = rp.alpha_max, tmin = rp.t_min;
    float fx[PPL], fy[PPL], T[PPL], C0[PPL], C1[PPL], C2[PPL];
    int last[PPL];
    // per slot: entries met so far whose mask covers the slot's quadrants (the
    // same for the whole wave), and its value at each pixel's last contributor
    int qn[PPL], lastq[PPL];
    // the pixel's alpha gate: alpha_min while it composites, 2 (above every
    // alpha) once it has stopped or when it lies outside the view, so one
    // compare both gates and skips
    float gmin[PPL];
#pragma unroll
    for (int k = 0; k < PPL; k++) {
        int x, y;
        TM::pixel(lane, k, x, y);
        const int px = tx * TW + x, py = ty * TH + y;
        fx[k] = px + 0.5f;
        fy[k] = py + 0.5f;
        gmin[k] = (px < W && py < H) ? amin : 2.f;
        T[k] = 1.f;
        C0[k] = C1[k] = C2[k] = 0.f;
        last[k] = 0;
        qn[k] = lastq[k] = 0;
    }
    const int s = ranges[2 * t];
    int e = ranges[2 * t + 1];
    int ncontrib = 0, nent = 0;
    __shared__ BatchLds sb;
    // Lazy lists: the tile's list is its block's list filtered by the tile's
    // four mask bits (the definition of the tile lists).  Block entries are
    // loaded kPull * 64 at a time, one load ahead; the entries that meet the
    // tile queue in an LDS ring in list order (qt queued, qh handed out, both
    // wave-uniform) and are handed out 64 at a time, each batch written to the
    // tile list as it is drawn, so the backward finds every entry up to the
    // last contributor.
    __shared__ uint32_t s_ring[LAZY ? kRing : 1];
    uint32_t lp[kPull], lm[kPull];
    int bpf = 0, bend = 0, msh = 0;
    uint32_t qh = 0, qt = 0;
    const uint32_t* mw = nullptr;
    auto pull = [&](int p0) {
        bpf = p0;
#pragma unroll
        for (int u = 0; u < kPull; u++) {
            const int j = min(p0 + u * kWave + lane, bend - 1);
            lp[u] = src.pair[j];
            lm[u] = mw[j];
        }
    };
    auto take = [&]() {
#pragma unroll
        for (int u = 0; u < kPull; u++) {
            const uint32_t w = lm[u];
            uint32_t m4 = ((w >> msh) & 3u) | (((w >> (msh + 8)) & 3u) << 2);
            m4 = bpf + u * kWave + lane < bend ? m4 : 0u;
            const uint64_t bal = __ballot(m4 != 0u);
            // set bits of bal below this lane
            const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            if (m4) s_ring[(qt + below) % kRing] = lp[u] | (m4 << kPairBits);
            qt += (uint32_t)__popcll(bal);
        }
        bpf += kPull * kWave;
    };
    // the next `want` entries (got < want only if the block list ran out
    // first, which the exact list lengths rule out)
    auto draw = [&](int want, int& got) -> uint32_t {
        while ((int)(qt - qh) < want && bpf < bend) {
            take();
            if (bpf < bend) pull(bpf);
        }
        got = min(want, (int)(qt - qh));
        wave_lds_sync();
        const uint32_t id = lane < got ? s_ring[(qh + (uint32_t)lane) % kRing] : 0u;
        qh += (uint32_t)got;
        return id;
    };
    // Two-deep pipeline: while a batch composites, the next batch's records
    // are in flight (their entries arrived during the batch before) and the
    // entries of the batch after that are requested.
    uint32_t id_cur = 0u, id_nxt = 0u;
    if constexpr (LAZY) {
        const int sx = tx % kBlockTiles, sy = ty % kBlockTiles;
        const int B = vt.block_off[v] + (ty / kBlockTiles) * vt.bx[v] + tx / kBlockTiles;
        // the block's entries are requested without waiting for the tile range
        bend = src.branges[2 * B + 1];
        bpf = src.branges[2 * B];
        mw = sy < 2 ? src.mlo : src.mhi;
        msh = 16 * (sy % 2) + 2 * sx;
        if (bpf < bend) pull(bpf);
        if (s < e) {
            const int want = min(kWave, e - s);
            int got;
            id_cur = draw(want, got);
            if (got < want) e = s + got;
            if (lane < got) src.tids[s + lane] = id_cur;
        }
    } else {
        id_cur = s < e ? batch_ids(ids, s, s, e) : 0u;
        id_nxt = s < e ? batch_ids(ids, s + kWave, s, e) : 0u;
    }
    LaneSplat ls_cur = {};
    if (lane < e - s) ls_cur = load_splat(rec, id_cur & kPairMask);
    for (int b = s; b < e; b += kWave) {
        bool alive = false;
#pragma unroll
        for (int k = 0; k < PPL; k++) alive |= gmin[k] <= 1.f;
        if (__ballot(alive) == 0) break;
        const uint32_t id = id_cur;
        const int nb = min(kWave, e - b);
        wave_lds_sync();  // the previous batch is read
        stage_splat(sb, ls_cur);
        ls_cur = {};
        if constexpr (LAZY) {
            const int want = min(kWave, e - (b + kWave));
            if (want > 0) {
                int got;
                id_cur = draw(want, got);
                if (got < want) e = b + kWave + got;
                if (lane < got) {
                    src.tids[b + kWave + lane] = id_cur;
                    ls_cur = load_splat(rec, id_cur & kPairMask);
                }
            }
        } else {
            if (lane < e - (b + kWave)) ls_cur = load_splat(rec, id_nxt & kPairMask);
            id_cur = id_nxt;
            id_nxt = batch_ids(ids, b + 2 * kWave, s, e);
        }
        wave_lds_sync();
        nent += nb;
        for (int i = 0; i < nb; i++) {
            const uint32_t m = (uint32_t)bcast((int)id, i) >> kPairBits;
            const float4 f0 = sb.f[0][i], f1 = sb.f[1][i], f2 = sb.f[2][i];
            const float mx = f0.x, my = f0.y, o = f0.z;
            const float qa = f1.x, qb = f1.y, qc = f1.z, cr = f1.w, cg = f2.x, cb = f2.y;
            const int pos = b + i - s + 1;
#pragma unroll
            for (int k = 0; k < PPL; k++) {
                if (!(m & TM::quads(k))) continue;  // wave-uniform
                qn[k]++;
                if (__ballot(gmin[k] <= 1.f) == 0) continue;  // wave-uniform: the slot has stopped
                const float dx = mx - fx[k];
                const float dy = my - fy[k];
                // listed splats have positive-definite conics (binning drops the
                // rest), so sigma >= 0 needs no test of its own
                const float e2 = splat_e2(qa, qb, qc, dx, dy);
                // min(amax, o 2^e2) as one median (the product is >= 0)
                const float alpha = __builtin_amdgcn_fmed3f(o * __builtin_amdgcn_exp2f(e2), 0.f, amax);
                const float Tn = T[k] * (1.f - alpha);
                // the gate (never passed by a stopped pixel); then the splat
                // that would take T below t_min stops the pixel instead of
                // contributing.  Decided without branches, one branch for the
                // update.
                const bool gate = alpha >= gmin[k];
                const bool stop = gate && Tn < tmin;
                gmin[k] = stop ? 2.f : gmin[k];
                if (gate && !stop) {
                    const float w = alpha * T[k];
                    C0[k] = __builtin_fmaf(cr, w, C0[k]);
                    C1[k] = __builtin_fmaf(cg, w, C1[k]);
                    C2[k] = __builtin_fmaf(cb, w, C2[k]);
                    T[k] = Tn;
                    last[k] = pos;
                    lastq[k] = qn[k];
                    ncontrib++;
                }
            }
        }
    }
    // workload statistics of the tile : contributing
    // (pixel, splat) pairs, list entries read, and (pixel, entry) evaluations
    // up to each pixel's last contributor over the entries covering its quadrant
    int nev = 0;
#pragma unroll
    for (int k = 0; k < PPL; k++) nev += lastq[k];
    for (int sh = 32; sh > 0; sh >>= 1) {
        ncontrib += __shfl_xor(ncontrib, sh, kWave);
        nev += __shfl_xor(nev, sh, kWave);
    }
    if (lane == 0) {
        tile_contrib[t] = ncontrib;
        tile_entries[t] = nent;
        tile_evals[t] = nev;
    }
    const float b0 = bg ? bg[0] : 0.f, b1 = bg ? bg[1] : 0.f, b2 = bg ? bg[2] : 0.f;
#pragma unroll
    for (int k = 0; k < PPL; k++) {
        int x, y;
        TM::pixel(lane, k, x, y);
        const int px = tx * TW + x, py = ty * TH + y;
        if (px < W && py < H) {
            const int64_t pix = (int64_t)vt.pix_off[v] + (int64_t)py * W + px;
            out_rgb[3 * pix] = C0[k] + T[k] * b0;
            out_rgb[3 * pix + 1] = C1[k] + T[k] * b1;
            out_rgb[3 * pix + 2] = C2[k] + T[k] * b2;
            out_T[pix] = T[k];
            out_last[pix] = last[k];
        }
    }
}

// What the raster backward reads and writes.
struct BwdArgs {
    const float4* rec;
    const int32_t* ids;
    const int32_t* ranges;
    const float* bg;
    const float* T_final;
    const int32_t* last;
    const float* v_rgb;
    float* grad_geo;
    float* grad_col;
    float* snap;  // pixel states at the segments' ends (see chain_bwd)
    int segs;     // segments of a heavy tile at most
    RasterParams rp;
};

// A heavy tile's list is walked in at most g.segs segments of whole batches.
__device__ __forceinline__ int seg_length(const BwdArgs& g, int lmax) {
    return ((lmax + g.segs - 1) / g.segs + kWave - 1) / kWave * kWave;
}
// the states at the end of segment `seg` of the heavy tile in slot `slot`: [2][pixels]
template <int PIXELS>
__device__ __forceinline__ float* snap_at(const BwdArgs& g, int slot, int seg) {
    return g.snap + ((int64_t)slot * (g.segs - 1) + seg) * (2 * PIXELS);
}

// Tile t by one wave: all of it, or (SEG) segment `seg` of the heavy tile in
// slot `slot`, whose pixels start from the states that the chain left.
template <int TW, int TH, bool SEG>
__device__ __forceinline__ void tile_bwd(const BwdArgs& g, const ViewTable& vt, int t, BatchLds& sb, int slot = 0,
                                         int seg = 0) {
    using TM = TileMap<TW, TH>;
    constexpr int PPL = TM::PPL;
    const float4* __restrict__ rec = g.rec;
    const int32_t* __restrict__ ids = g.ids;
    const float* bg = g.bg;
    const int v = tile_view(vt, t);
    const int lt = t - vt.tile_off[v];
    const int gx = vt.gx[v], W = vt.W[v], H = vt.H[v];
    const int tx = lt % gx, ty = lt / gx;
    const int lane = threadIdx.x;
    const float b0 = bg ? bg[0] : 0.f, b1 = bg ? bg[1] : 0.f, b2 = bg ? bg[2] : 0.f;
    float fx[PPL], fy[PPL], Tc[PPL], V0[PPL], V1[PPL], V2[PPL], VS[PPL];
    int L[PPL];
    int lmax = 0;
#pragma unroll
    for (int k = 0; k < PPL; k++) {
        int x, y;
        TM::pixel(lane, k, x, y);
        const int px = tx * TW + x, py = ty * TH + y;
        fx[k] = px + 0.5f;
        fy[k] = py + 0.5f;
        L[k] = 0;
        Tc[k] = 1.f;
        V0[k] = V1[k] = V2[k] = 0.f;
        if (px < W && py < H) {
            const int64_t pix = (int64_t)vt.pix_off[v] + (int64_t)py * W + px;
            L[k] = g.last[pix];
            Tc[k] = g.T_final[pix];
            V0[k] = g.v_rgb[3 * pix];
            V1[k] = g.v_rgb[3 * pix + 1];
            V2[k] = g.v_rgb[3 * pix + 2];
        }
        // VS = dL/dC . S, S = sum over later splats of colour alpha T, plus
        // T_final bg (the background term seeds it)
        VS[k] = Tc[k] * (V0[k] * b0 + V1[k] * b1 + V2[k] * b2);
        lmax = max(lmax, L[k]);
    }
    // per slot, the largest `last` of its pixels: past it the whole wave skips
    // the slot (all its pixels are behind their last contributor)
    // (wave-uniform: read from the first lane, so the loops below stay scalar)
    int Lk[PPL];
#pragma unroll
    for (int k = 0; k < PPL; k++) Lk[k] = __builtin_amdgcn_readfirstlane(wave_max_i(L[k]));
    lmax = __builtin_amdgcn_readfirstlane(wave_max_i(lmax));
    const int s = g.ranges[2 * t], e = g.ranges[2 * t + 1];
    lmax = min(lmax, e - s);  // a pixel's last contributor lies inside its tile's list
    if (lmax <= 0) return;
    const float amin = g.rp.alpha_min, amax = g.rp.alpha_max;
    int low = s, top = s + lmax;  // entries [s, top) can matter; this wave's are [low, top)
    if (SEG) {
        const int len = seg_length(g, lmax), end = (seg + 1) * len;
        if (seg * len >= lmax) return;
        low = s + seg * len;
        top = min(top, s + end);
        const float* snap = snap_at<TW * TH>(g, slot, seg);
#pragma unroll
        for (int k = 0; k < PPL; k++)
            if (end < min(Lk[k], e - s)) {  // wave-uniform: the slot's pixels reach past the end
                Tc[k] = snap[k * kWave + lane];
                VS[k] = snap[TW * TH + k * kWave + lane];
            }
    }
    // The gradient component this lane adds after the wave sums E of two splats
    // (the first in lanes 0-31, the second in 32-63; see wave_sums_t): 0 mean.x,
    // 1 mean.y, 2 A, 3 B, 4 C, 5 opacity, 6 r, 7 g, 8 b, -1 none.
    // It is E (kS o + kE) + o ln2 ((ua a + ub b) QX + (vb b + vc c) QY) with
    // QX, QY the first two moments, so every lane runs the same instructions.
    const int comp = sum_lane_comp<2>(lane);
    float* const grad = comp < kGradGeo ? g.grad_geo + comp : g.grad_col + (comp - kGradGeo);
    const int gstep = comp < kGradGeo ? kGradGeo : kGradCol;
    const float kS = (comp == 2 || comp == 4) ? -0.5f : comp == 3 ? -1.f : 0.f;
    const float kE = comp >= 5 ? 1.f : 0.f;
    const float ua = comp == 0 ? 2.f : 0.f, ub = comp == 1 ? 1.f : 0.f;
    const float vb = comp == 0 ? 1.f : 0.f, vc = comp == 1 ? 2.f : 0.f;
    int b = low + ((top - low - 1) / kWave) * kWave;
    // the same two-deep pipeline as the forward, walking down: the batches
    // after the first (partial) one are full
    uint32_t id_cur = batch_ids(ids, b, s, top);
    uint32_t id_nxt = batch_ids(ids, b - kWave, s, top);
    LaneSplat ls_cur = {};
    if (lane < top - b) ls_cur = load_splat(rec, id_cur & kPairMask);
    for (; b >= low; b -= kWave) {
        const uint32_t id = id_cur;
        const int nb = min(kWave, top - b);
        wave_lds_sync();  // the previous batch is read
        stage_splat(sb, ls_cur);
        ls_cur = {};
        if (b - kWave >= low) ls_cur = load_splat(rec, id_nxt & kPairMask);
        id_cur = id_nxt;
        id_nxt = batch_ids(ids, b - 2 * kWave, s, top);
        wave_lds_sync();
        // Two splats at a time: their nine sums each are then taken over the
        // wave in one butterfly and added by one atomic instruction, which
        // costs 35 instructions a splat where one by one it was 51.
        for (int i = nb - 1; i >= 0; i -= 2) {
            // per-lane sums over the lane's pixels: q dx, q dy, q dx^2, q dx dy,
            // q dy^2 and q, q = dL/dalpha e^-sigma (zero where alpha is
            // clamped), then the colour weights; the exponent's gradient is
            // -o q, so the mean and conic gradients follow from these after the
            // wave sum
            float a[2][9];
            float4 f0[2], f1[2];
            bool any = false;
#pragma unroll
            for (int u = 0; u < 2; u++) {
#pragma unroll
                for (int c = 0; c < 9; c++) a[u][c] = 0.f;
                const int j = max(i - u, 0);
                const uint32_t m = i >= u ? (uint32_t)bcast((int)id, j) >> kPairBits : 0u;
                f0[u] = sb.f[0][j];
                f1[u] = sb.f[1][j];
                const float4 f2 = sb.f[2][j];
                const float mx = f0[u].x, my = f0[u].y, o = f0[u].z;
                const float qa = f1[u].x, qb = f1[u].y, qc = f1[u].z, cr = f1[u].w, cg = f2.x, cb = f2.y;
                const int pos = b + j - s;
#pragma unroll
                for (int k = 0; k < PPL; k++) {
                    if (!(m & TM::quads(k)) || pos >= Lk[k]) continue;  // wave-uniform
                    const float dx = mx - fx[k];
                    const float dy = my - fy[k];
                    const float e2 = splat_e2(qa, qb, qc, dx, dy);
                    const float ex = __builtin_amdgcn_exp2f(e2);
                    const float araw = o * ex;
                    const float alpha = __builtin_amdgcn_fmed3f(araw, 0.f, amax);
                    // same decisions as the forward: before the pixel's last
                    // contributor and above the alpha gate
                    const bool live = pos < L[k] && alpha >= amin;
                    if (live) {
                        any = true;
                        const float iom = __builtin_amdgcn_rcpf(1.f - alpha);
                        const float Tb = Tc[k] * iom;  // transmittance in front of this splat
                        const float w = alpha * Tb;
                        a[u][6] = __builtin_fmaf(w, V0[k], a[u][6]);
                        a[u][7] = __builtin_fmaf(w, V1[k], a[u][7]);
                        a[u][8] = __builtin_fmaf(w, V2[k], a[u][8]);
                        const float Vc = __builtin_fmaf(V2[k], cb, __builtin_fmaf(V1[k], cg, V0[k] * cr));
                        // dL/dalpha = T (dL/dC . c) - (dL/dC . S) / (1 - alpha)
                        const float va = __builtin_fmaf(Tb, Vc, -(iom * VS[k]));
                        VS[k] = __builtin_fmaf(w, Vc, VS[k]);
                        Tc[k] = Tb;
                        const float q = araw < amax ? va * ex : 0.f;  // clamped alpha passes no gradient
                        a[u][5] += q;
                        const float qx = q * dx, qy = q * dy;
                        a[u][0] += qx;
                        a[u][1] += qy;
                        a[u][2] = __builtin_fmaf(qx, dx, a[u][2]);
                        a[u][3] = __builtin_fmaf(qx, dy, a[u][3]);
                        a[u][4] = __builtin_fmaf(qy, dy, a[u][4]);
                    }
                }
            }
            if (__ballot(any) == 0) continue;
            const float E = wave_sums_t(a);
            const float QX = dpp_f<0x150>(E), QY = dpp_f<0x154>(E);  // lanes 0 and 4 of the row: m_x, m_y
            if (comp >= 0) {
                // With vs = -o q the sums of vs dx, vs dy, ... are -o times the
                // moments; A = -2 a / log2(e), B = -b / log2(e), C = -2 c / log2(e).
                const bool second = lane >= kWave / 2;
                const float o = second ? f0[1].z : f0[0].z;
                const float qa = second ? f1[1].x : f1[0].x, qb = second ? f1[1].y : f1[0].y,
                            qc = second ? f1[1].z : f1[0].z;
                const float mean = __builtin_fmaf(__builtin_fmaf(ua, qa, ub * qb), QX,
                                                  __builtin_fmaf(vb, qb, vc * qc) * QY);
                const float val = __builtin_fmaf(o * kLn2, mean, E * __builtin_fmaf(kS, o, kE));
                const uint32_t p0 = (uint32_t)bcast((int)id, i), p1 = (uint32_t)bcast((int)id, max(i - 1, 0));
                const int64_t p = (second ? p1 : p0) & kPairMask;
                if (val != 0.f) atomicAdd(grad + gstep * p, val);
            }
        }
    }
}

// ---- one wave per part of a tile
//
// An entry costs a wave an LDS round trip and its own dependent arithmetic,
// about 250 cycles however little there is to do, and a tile's list is one
// serial chain: 256 tiles were one wave on each CU.  So each slot of the TileMap
// (64 pixels, one a lane) gets a wave of its own, which queues only the entries
// whose mask meets the part's quadrants (with their places in the tile's list,
// which `last` counts by) and takes the queued entries kGroup at a time: their
// LDS loads and exponents overlap, and only the transmittance runs serially.
// Every pixel sees the same operations in the same order as with a wave per
// tile.  VALU-bound where the chip is full (the CUs busy 99% of the launch).
// Forward, a wave per tile -> per part: 256x256 and 10k splats 84 -> 23 us (10k
// blob splats 339 -> 97); 4 x 1237x822 (16x16 tiles) 519 -> 476; 8 uneven
// views 977 -> 850; 4 x 1600x1066 (32x16) 1175 -> 930; one 1237x822 view 96 ->
// 97: so every launch takes the parts.
constexpr int kGroup = 4;
static_assert(kWave % kGroup == 0, "groups fill a batch");

// The slot and the part of this workgroup: a slot's parts are kXcds apart, so
// they run together on one XCD.
template <int PPL>
__device__ __forceinline__ void part_slot(int& slot, int& part) {
    const int x = blockIdx.x;
    slot = x / (kXcds * PPL) * kXcds + x % kXcds;
    part = x / kXcds % PPL;
}

// The queue of a part's entries in LDS: (pair | mask << 28) and place in the
// tile's list; at most 63 waiting plus one refill of PULL * 64.
template <int PULL>
struct PartRing {
    static constexpr uint32_t kSize = 128 * PULL;
    static_assert(kSize >= kWave - 1 + PULL * kWave, "ring");
    uint32_t id[kSize];
    uint32_t pos[kSize];
};
// The backward's loads are of a list it reads every entry of: fewer in flight,
// for a ring that leaves the LDS to four waves a SIMD.
constexpr int kPullBwd = 4;

template <int TW, int TH, bool LAZY>
__global__ __launch_bounds__(64) void k_render_fwd_part(const float4* __restrict__ rec,
                                                        const int32_t* __restrict__ ids,
                                                        const int32_t* __restrict__ ranges,
                                                        const uint32_t* __restrict__ order, int n_slots,
                                                        ViewTable vt, RasterParams rp,
                                                        const float* __restrict__ bg,
                                                        float* __restrict__ out_rgb,
                                                        float* __restrict__ out_T,
                                                        int32_t* __restrict__ out_last, int mode,
                                                        BlockSrc src) {
    using TM = TileMap<TW, TH>;
    int slot, part, t;
    part_slot<TM::PPL>(slot, part);
    if (slot >= n_slots || !block_tile(slot, order, mode, vt, t)) return;
    const int v = tile_view(vt, t);
    const int lt = t - vt.tile_off[v];
    const int gx = vt.gx[v], W = vt.W[v], H = vt.H[v];
    const int tx = lt % gx, ty = lt / gx;
    const int lane = threadIdx.x;
    const float amin = rp.alpha_min, amax = rp.alpha_max, tmin = rp.t_min;
    int x, y;
    TM::pixel(lane, part, x, y);
    const int px = tx * TW + x, py = ty * TH + y;
    const float fx = px + 0.5f, fy = py + 0.5f;
    // alpha_min while the pixel composites, 2 once it has stopped (or outside)
    float gmin = (px < W && py < H) ? amin : 2.f;
    float T = 1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f;
    int last = 0;
    const uint32_t quads = TM::quads(part);
    const int s = ranges[2 * t], e = ranges[2 * t + 1];
    __shared__ BatchLds sb;
    __shared__ PartRing<kPull> ring;
    uint32_t lp[kPull], lm[kPull];
    // next: the first entry not yet taken; end: of the block's list (lazy) or
    // the tile's
    int next = s, end = e, msh = 0;
    uint32_t qh = 0, qt = 0;
    int place = 0;  // entries of the tile's list taken so far (lazy)
    const uint32_t* mw = nullptr;
    if constexpr (LAZY) {
        const int sx = tx % kBlockTiles, sy = ty % kBlockTiles;
        const int B = vt.block_off[v] + (ty / kBlockTiles) * vt.bx[v] + tx / kBlockTiles;
        next = src.branges[2 * B];
        end = s < e ? src.branges[2 * B + 1] : next;
        mw = sy < 2 ? src.mlo : src.mhi;
        msh = 16 * (sy % 2) + 2 * sx;
    }
    auto pull = [&]() {
#pragma unroll
        for (int u = 0; u < kPull; u++) {
            const int j = min(next + u * kWave + lane, end - 1);
            lp[u] = LAZY ? src.pair[j] : (uint32_t)ids[j];
            if (LAZY) lm[u] = mw[j];
        }
    };
    auto take = [&]() {
#pragma unroll
        for (int u = 0; u < kPull; u++) {
            const int j = next + u * kWave + lane;
            uint32_t id, pos, m4;
            if (LAZY) {
                m4 = ((lm[u] >> msh) & 3u) | (((lm[u] >> (msh + 8)) & 3u) << 2);
                m4 = j < end ? m4 : 0u;
                const uint64_t bal = __ballot(m4 != 0u);
                pos = (uint32_t)place + __builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                id = lp[u] | (m4 << kPairBits);
                // every part of the tile writes the same entries
                if (m4 && (int)pos < e - s) src.tids[s + (int)pos] = id;
                place += __popcll(bal);
            } else {
                id = lp[u];
                pos = (uint32_t)(j - s);
                m4 = j < end ? id >> kPairBits : 0u;
            }
            const bool hit = (m4 & quads) != 0u;
            const uint64_t bal = __ballot(hit);
            const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            if (hit) {
                ring.id[(qt + below) % ring.kSize] = id;
                ring.pos[(qt + below) % ring.kSize] = pos;
            }
            qt += (uint32_t)__popcll(bal);
        }
        next += kPull * kWave;
    };
    // the next queued entries, up to 64: their count and this lane's
    auto draw = [&](uint32_t& id, uint32_t& pos) -> int {
        while (qt - qh < (uint32_t)kWave && next < end) {
            take();
            if (next < end) pull();
        }
        const int got = (int)min(qt - qh, (uint32_t)kWave);
        wave_lds_sync();
        id = pos = 0u;
        if (lane < got) {
            id = ring.id[(qh + (uint32_t)lane) % ring.kSize];
            pos = ring.pos[(qh + (uint32_t)lane) % ring.kSize];
        }
        qh += (uint32_t)got;
        return got;
    };
    if (next < end) pull();
    uint32_t id, pos;
    int nb = draw(id, pos);
    LaneSplat ls = {};
    if (lane < nb) ls = load_splat(rec, id & kPairMask);
    while (nb > 0 && __ballot(gmin <= 1.f) != 0) {
        wave_lds_sync();  // the previous batch is read
        stage_splat(sb, ls);
        sb.f[2][lane].z = __uint_as_float(pos);
        // the next batch's records are in flight while this one composites
        ls = {};
        const int nn = draw(id, pos);
        if (lane < nn) ls = load_splat(rec, id & kPairMask);
        wave_lds_sync();
        for (int i = 0; i < nb; i += kGroup) {
            float al[kGroup], cr[kGroup], cg[kGroup], cb[kGroup];
            int ps[kGroup];
#pragma unroll
            for (int u = 0; u < kGroup; u++) {
                // (entries past the batch are staged as zeros: alpha 0)
                const float4 f0 = sb.f[0][i + u], f1 = sb.f[1][i + u], f2 = sb.f[2][i + u];
                const float e2 = splat_e2(f1.x, f1.y, f1.z, f0.x - fx, f0.y - fy);
                al[u] = __builtin_amdgcn_fmed3f(f0.z * __builtin_amdgcn_exp2f(e2), 0.f, amax);
                cr[u] = f1.w;
                cg[u] = f2.x;
                cb[u] = f2.y;
                ps[u] = (int)__float_as_uint(f2.z) + 1;
            }
#pragma unroll
            for (int u = 0; u < kGroup; u++) {
                const float Tn = T * (1.f - al[u]);
                const bool gate = al[u] >= gmin;
                const bool stop = gate && Tn < tmin;
                const bool adds = gate && !stop;
                gmin = stop ? 2.f : gmin;
                const float w = adds ? al[u] * T : 0.f;
                C0 = __builtin_fmaf(cr[u], w, C0);
                C1 = __builtin_fmaf(cg[u], w, C1);
                C2 = __builtin_fmaf(cb[u], w, C2);
                T = adds ? Tn : T;
                last = adds ? ps[u] : last;
            }
            if (__ballot(gmin <= 1.f) == 0) break;
        }
        nb = nn;
    }
    if (px < W && py < H) {
        const float b0 = bg ? bg[0] : 0.f, b1 = bg ? bg[1] : 0.f, b2 = bg ? bg[2] : 0.f;
        const int64_t pix = (int64_t)vt.pix_off[v] + (int64_t)py * W + px;
        out_rgb[3 * pix] = C0 + T * b0;
        out_rgb[3 * pix + 1] = C1 + T * b1;
        out_rgb[3 * pix + 2] = C2 + T * b2;
        out_T[pix] = T;
        out_last[pix] = last;
    }
}

// What the pixels of part `part` of heavy tile t carry down the list, their
// transmittance Tc and VS, without the gradients: left at each segment's end
// (`snap`), from where the segments are then walked at once.  A tile's sums are
// those of a wave with the whole tile, bit for bit: a wave a part, each adding
// its own sums, is as exact but rounds otherwise, and what cancels in the
// sums of needle-like splats made that 1e-3 of the gradients' rms on single ones.
template <int TW, int TH>
__device__ __forceinline__ void chain_bwd(const BwdArgs& g, const ViewTable& vt, int t, int part, int slot,
                                          BatchLds& sb, PartRing<kPullBwd>& ring) {
    using TM = TileMap<TW, TH>;
    const float4* __restrict__ rec = g.rec;
    const int32_t* __restrict__ ids = g.ids;
    const float* bg = g.bg;
    const int v = tile_view(vt, t);
    const int lt = t - vt.tile_off[v];
    const int gx = vt.gx[v], W = vt.W[v], H = vt.H[v];
    const int tx = lt % gx, ty = lt / gx;
    const int lane = threadIdx.x;
    const float b0 = bg ? bg[0] : 0.f, b1 = bg ? bg[1] : 0.f, b2 = bg ? bg[2] : 0.f;
    int x, y;
    TM::pixel(lane, part, x, y);
    const int px = tx * TW + x, py = ty * TH + y;
    const float fx = px + 0.5f, fy = py + 0.5f;
    int L = 0;
    float Tc = 1.f, V0 = 0.f, V1 = 0.f, V2 = 0.f;
    if (px < W && py < H) {
        const int64_t pix = (int64_t)vt.pix_off[v] + (int64_t)py * W + px;
        L = g.last[pix];
        Tc = g.T_final[pix];
        V0 = g.v_rgb[3 * pix];
        V1 = g.v_rgb[3 * pix + 1];
        V2 = g.v_rgb[3 * pix + 2];
    }
    float VS = Tc * (V0 * b0 + V1 * b1 + V2 * b2);
    const int s = g.ranges[2 * t], e = g.ranges[2 * t + 1];
    int most = 0;  // the tile's largest `last`, which sets the segments
#pragma unroll
    for (int k = 0; k < TM::PPL; k++) {
        int kx, ky;
        TM::pixel(lane, k, kx, ky);
        kx += tx * TW;
        ky += ty * TH;
        if (kx < W && ky < H) most = max(most, g.last[(int64_t)vt.pix_off[v] + (int64_t)ky * W + kx]);
    }
    // a pixel's last contributor lies inside its tile's list
    most = min(__builtin_amdgcn_readfirstlane(wave_max_i(most)), e - s);
    const int lmax = min(__builtin_amdgcn_readfirstlane(wave_max_i(L)), e - s);
    if (lmax <= 0) return;
    const int len = seg_length(g, most);
    int seg = (lmax - 1) / len - 1;  // the next segment to end, at entry (seg + 1) len
    if (seg < 0) return;
    auto leave = [&]() {
        float* p = snap_at<TW * TH>(g, slot, seg);
        p[part * kWave + lane] = Tc;
        p[TW * TH + part * kWave + lane] = VS;
        seg--;
    };
    const float amin = g.rp.alpha_min, amax = g.rp.alpha_max;
    const uint32_t quads = TM::quads(part);
    uint32_t lp[kPullBwd];
    int next = s + lmax - 1;  // the first entry not yet taken, walking down
    uint32_t qh = 0, qt = 0;
    auto pull = [&]() {
#pragma unroll
        for (int u = 0; u < kPullBwd; u++) lp[u] = (uint32_t)ids[max(next - u * kWave - lane, s)];
    };
    auto take = [&]() {
#pragma unroll
        for (int u = 0; u < kPullBwd; u++) {
            const int j = next - u * kWave - lane;
            const bool hit = j >= s && ((lp[u] >> kPairBits) & quads) != 0u;
            const uint64_t bal = __ballot(hit);
            const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            if (hit) {
                ring.id[(qt + below) % ring.kSize] = lp[u];
                ring.pos[(qt + below) % ring.kSize] = (uint32_t)(j - s);
            }
            qt += (uint32_t)__popcll(bal);
        }
        next -= kPullBwd * kWave;
    };
    auto draw = [&](uint32_t& id, uint32_t& pos) -> int {
        while (qt - qh < (uint32_t)kWave && next >= s) {
            take();
            if (next >= s) pull();
        }
        const int got = (int)min(qt - qh, (uint32_t)kWave);
        wave_lds_sync();
        id = pos = 0u;
        if (lane < got) {
            id = ring.id[(qh + (uint32_t)lane) % ring.kSize];
            pos = ring.pos[(qh + (uint32_t)lane) % ring.kSize];
        }
        qh += (uint32_t)got;
        return got;
    };
    pull();
    uint32_t id, pos;
    int nb = draw(id, pos);
    LaneSplat ls = {};
    if (lane < nb) ls = load_splat(rec, id & kPairMask);
    while (nb > 0) {
        wave_lds_sync();  // the previous batch is read
        stage_splat(sb, ls);
        sb.f[2][lane].z = __uint_as_float(pos);
        ls = {};
        const int nn = draw(id, pos);
        if (lane < nn) ls = load_splat(rec, id & kPairMask);
        wave_lds_sync();
        for (int i = 0; i < nb; i += kGroup) {
            float al[kGroup], iom[kGroup], Vc[kGroup];
            int at[kGroup];
            bool live[kGroup];
#pragma unroll
            for (int u = 0; u < kGroup; u++) {
                const float4 f0 = sb.f[0][i + u], f1 = sb.f[1][i + u], f2 = sb.f[2][i + u];
                const float dx = f0.x - fx;
                const float dy = f0.y - fy;
                const float ex = __builtin_amdgcn_exp2f(splat_e2(f1.x, f1.y, f1.z, dx, dy));
                al[u] = __builtin_amdgcn_fmed3f(f0.z * ex, 0.f, amax);
                iom[u] = __builtin_amdgcn_rcpf(1.f - al[u]);
                Vc[u] = __builtin_fmaf(V2, f2.y, __builtin_fmaf(V1, f2.x, V0 * f1.w));
                at[u] = (int)__float_as_uint(f2.z);
                live[u] = at[u] < L && al[u] >= amin;
            }
            auto step = [&](int u) {
                const float Tb = Tc * iom[u];  // transmittance in front of this splat
                VS = live[u] ? __builtin_fmaf(al[u] * Tb, Vc[u], VS) : VS;
                Tc = live[u] ? Tb : Tc;
            };
            // (of a short last group, the unused entries' alpha is zero)
            const int rest = min(kGroup, nb - i);
            const int lowest = (int)__builtin_amdgcn_readfirstlane(__float_as_uint(sb.f[2][i + rest - 1].z));
            if (lowest >= (seg + 1) * len) {
#pragma unroll
                for (int u = 0; u < kGroup; u++) step(u);
            } else {
#pragma unroll
                for (int u = 0; u < kGroup; u++) {
                    const int p = __builtin_amdgcn_readfirstlane(at[u]);
                    if (u < rest)
                        while (seg >= 0 && p < (seg + 1) * len) leave();
                    step(u);
                }
                if (seg < 0) return;
            }
        }
        nb = nn;
    }
    while (seg >= 0) leave();
}

// ---- the backward's launch
//
// Tiles differ a hundredfold in the entries their pixels reach back through,
// and a wave has a tile to itself: the launch lasted as long as its heaviest
// tiles, with the CUs busy three quarters of it on the 150-camera step and a
// fifth of it on 256 tiles.  So the tiles are launched heaviest first by what
// the backward will walk (the largest `last` of a tile's pixels, read here
// from the image the caller passes), and those much heavier than a wave's fair
// share of the launch are walked in segments at once, from the states that a
// chain over the list left at the segments' ends (chain_bwd).
// Weights are bucketed, 16 buckets an octave like gs_settings.tile_order's.
// us, a wave per tile in the settings' order -> this (weights and plan, 20-30
// us, not counted): 4 x 1237x822 920 -> 690, 4 x 1600x1066 (32x16) 1250 -> 1065, 8
// uneven views 1149 -> 1185, one 1237x822 view of blobs 346 -> 303.
constexpr int kWeightBuckets = 513;
constexpr int kWeightThreads = 1024;
constexpr int kWaveSlots = 4096;  // waves of the backward the chip holds at once
// A tile is heavy past kShare times the launch's weight over kWaveSlots; so at
// most kWaveSlots / kShare tiles are.  The chain is work on top of the tile's
// own, about half of it, so too many are a loss and too few leave the tail: us
// at kShare 2, 3, 4 on 4 x 1237x822 803, 686, 692, on 4 x 1600x1066 1240, 1065,
// 1041, on 8 uneven views 1103, 1189, 1185, on one 1237x822 view of blobs 240, 303,
// 354.
constexpr int kShare = 3;
constexpr int kMaxHeavy = kBwdHeavy;
static_assert(kMaxHeavy >= kWaveSlots / kShare, "as many as can pass kShare");

// (walked entries, their bucket; no entries: bucket 0)
__device__ __forceinline__ uint32_t weight_bucket(uint32_t n) {
    if (n == 0) return 0;
    const int lg = 31 - __clz((int)n);
    const uint32_t m = lg >= 4 ? (n >> (lg - 4)) & 15u : (n << (4 - lg)) & 15u;
    return 1u + 16u * (uint32_t)lg + m;
}

__device__ __forceinline__ float bucket_weight(int b) {  // of a bucket's lower end
    return b <= 0 ? 0.f : __builtin_ldexpf(1.f + (float)((b - 1) & 15) / 16.f, (b - 1) >> 4);
}

// each tile's weight bucket, a wave per tile
template <int TW, int TH>
__global__ __launch_bounds__(256) void k_bwd_weights(ViewTable vt, const int32_t* __restrict__ ranges,
                                                     const int32_t* __restrict__ last, int T,
                                                     uint32_t* __restrict__ bucket) {
    using TM = TileMap<TW, TH>;
    const int t = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + threadIdx.x / kWave));
    const int lane = threadIdx.x % kWave;
    if (t >= T) return;
    const int v = tile_view(vt, t);
    const int lt = t - vt.tile_off[v];
    const int gx = vt.gx[v], W = vt.W[v], H = vt.H[v];
    const int tx = lt % gx, ty = lt / gx;
    int m = 0;
#pragma unroll
    for (int k = 0; k < TM::PPL; k++) {
        int x, y;
        TM::pixel(lane, k, x, y);
        const int px = tx * TW + x, py = ty * TH + y;
        if (px < W && py < H) m = max(m, last[(int64_t)vt.pix_off[v] + (int64_t)py * W + px]);
    }
    m = min(wave_max_i(m), ranges[2 * t + 1] - ranges[2 * t]);
    if (lane == 0) bucket[t] = weight_bucket((uint32_t)max(m, 0));
}

// The order of the tiles with anything to walk, heaviest bucket first, their
// number and the heavy ones' (plan[0], plan[1]).  One workgroup; each thread
// keeps kHold tiles' loads in flight (12 us on 16224 tiles).
__global__ __launch_bounds__(kWeightThreads) void k_bwd_plan(const uint32_t* __restrict__ bucket, int T,
                                                             uint32_t* __restrict__ order,
                                                             uint32_t* __restrict__ plan) {
    constexpr int kHold = 8;
    __shared__ uint32_t s_n[kWeightBuckets];
    __shared__ uint32_t s_w[kWeightThreads / kWave];
    __shared__ float s_t[kWeightThreads / kWave];
    __shared__ uint32_t s_heavy;
    const int tid = threadIdx.x, lane = tid % kWave, w = tid / kWave;
    if (tid < kWeightBuckets) s_n[tid] = 0;
    if (tid == 0) s_heavy = 0;
    __syncthreads();
    auto each = [&](auto f) {
        for (int t0 = 0; t0 < T; t0 += kHold * kWeightThreads) {
            uint32_t b[kHold];
#pragma unroll
            for (int h = 0; h < kHold; h++) {
                const int t = t0 + h * kWeightThreads + tid;
                b[h] = t < T ? bucket[t] : 0u;
            }
#pragma unroll
            for (int h = 0; h < kHold; h++)
                if (b[h]) f(t0 + h * kWeightThreads + tid, b[h]);
        }
    };
    each([&](int, uint32_t b) { atomicAdd(&s_n[b], 1u); });
    __syncthreads();
    // exclusive scan from the heaviest bucket down: thread i takes bucket
    // kWeightBuckets - 1 - i; and the launch's whole weight
    const int qb = kWeightBuckets - 1 - tid;
    const uint32_t c = qb > 0 ? s_n[qb] : 0u;
    const float mine = (float)c * bucket_weight(qb);
    uint32_t inc = c;
    float tot = mine;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t x = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += x;
        tot += __shfl_xor(tot, off, kWave);
    }
    if (lane == kWave - 1) {
        s_w[w] = inc;
        s_t[w] = tot;
    }
    __syncthreads();
    uint32_t before = 0, all = 0;
    tot = 0.f;
    for (int i = 0; i < kWeightThreads / kWave; i++) {
        if (i < w) before += s_w[i];
        all += s_w[i];
        tot += s_t[i];
    }
    if (qb > 0) {
        s_n[qb] = before + inc - c;
        if (c && bucket_weight(qb) * kWaveSlots > kShare * tot) atomicMax(&s_heavy, before + inc);
    }
    __syncthreads();
    if (tid == 0) {
        plan[0] = all;
        plan[1] = min(s_heavy, (uint32_t)kMaxHeavy);
    }
    each([&](int t, uint32_t b) { order[atomicAdd(&s_n[b], 1u)] = (uint32_t)t; });
}

// The heavy tiles' chains first (a tile's parts kXcds workgroups apart, so they
// share an L2), then the other tiles, whole.  Without a plan (plan NULL) the
// first `heavy` tiles are.
template <int TW, int TH>
__global__ __launch_bounds__(64) void k_render_bwd(BwdArgs g, ViewTable vt, int T,
                                                   const uint32_t* __restrict__ order,
                                                   const uint32_t* __restrict__ plan, int heavy) {
    constexpr int PPL = TileMap<TW, TH>::PPL;
    __shared__ BatchLds sb;
    __shared__ PartRing<kPullBwd> ring;
    const int n = plan ? (int)plan[0] : T;
    if (plan) heavy = (int)plan[1];
    const int x = blockIdx.x;
    const int parts = (heavy + kXcds - 1) / kXcds * kXcds * PPL;
    if (x < parts) {
        const int slot = x / (kXcds * PPL) * kXcds + x % kXcds;
        if (slot >= heavy) return;
        chain_bwd<TW, TH>(g, vt, order ? (int)order[slot] : slot, x / kXcds % PPL, slot, sb, ring);
    } else {
        const int slot = heavy + x - parts;
        if (slot >= n) return;
        tile_bwd<TW, TH, false>(g, vt, order ? (int)order[slot] : slot, sb);
    }
}

// The heavy tiles' segments, a wave each.
template <int TW, int TH>
__global__ __launch_bounds__(64) void k_render_bwd_segs(BwdArgs g, ViewTable vt, const uint32_t* __restrict__ order,
                                                        const uint32_t* __restrict__ plan, int heavy) {
    __shared__ BatchLds sb;
    if (plan) heavy = (int)plan[1];
    const int x = blockIdx.x;
    const int slot = x / (kXcds * g.segs) * kXcds + x % kXcds;
    if (slot >= heavy) return;
    tile_bwd<TW, TH, true>(g, vt, order ? (int)order[slot] : slot, sb, slot, x / kXcds % g.segs);
}

constexpr int kL1Blocks = 1024;

__global__ __launch_bounds__(256) void k_l1(const float* __restrict__ rgb,
                                            const float* __restrict__ target,
                                            float* __restrict__ v_rgb, ViewTable vt,
                                            double* __restrict__ loss_acc) {
    __shared__ float s_w[4];
    const int64_t P = vt.pix_off[vt.V];
    float part = 0.f;
    for (int64_t pix = (int64_t)blockIdx.x * 256 + threadIdx.x; pix < P;
         pix += (int64_t)gridDim.x * 256) {
        int v = 0;
        while (v + 1 < vt.V && pix >= vt.pix_off[v + 1]) v++;
        const float wgt = 1.f / (3.f * (float)(vt.pix_off[v + 1] - vt.pix_off[v]) * (float)vt.V);
#pragma unroll
        for (int ch = 0; ch < 3; ch++) {
            const float d = rgb[3 * pix + ch] - target[3 * pix + ch];
            v_rgb[3 * pix + ch] = d > 0.f ? wgt : (d < 0.f ? -wgt : 0.f);
            part += fabsf(d) * wgt;
        }
    }
    // one double atomic per block
    const float s = wave_sum(part);
    if (__lane_id() == 0) s_w[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double tot = (double)s_w[0] + s_w[1] + s_w[2] + s_w[3];
        if (tot != 0.0) atomicAdd(loss_acc, tot);
    }
}

// workgroups of a raster launch: one per tile, or for the XCD order one per
// slot of every 4 x 4 block, rounded to whole rounds over the XCDs
unsigned raster_grid(const Ctx* c, const ViewTable& vt, int mode) {
    if (mode != 2) return (unsigned)c->n_tiles;
    const int64_t slots = (int64_t)vt.block_off[vt.V] * kBlockTileCount;
    const int64_t round = (int64_t)kXcds * kBlockTileCount;
    return (unsigned)((slots + round - 1) / round * round);
}

template <int TW, int TH, bool LAZY>
void fwd_launch(Ctx* c, const ViewTable& vt, const RasterParams& rp, const float* bg, float* rgb,
                float* T_final, int32_t* last, const uint32_t* order, int mode, const BlockSrc& src,
                hipStream_t st) {
    const float4* rec = reinterpret_cast<const float4*>(c->rec);
    const int32_t* ids = reinterpret_cast<const int32_t*>(c->tids);
    const unsigned slots = raster_grid(c, vt, mode);
    constexpr int PPL = TileMap<TW, TH>::PPL;
    if (rp.eval_stats)
        hipLaunchKernelGGL((k_render_fwd_stats<TW, TH, LAZY>), dim3(slots), dim3(64), 0, st, rec, ids, c->tranges,
                           order, vt, rp, bg, rgb, T_final, last, c->tile_contrib, c->tile_entries,
                           c->tile_evals, mode, src);
    else
        hipLaunchKernelGGL((k_render_fwd_part<TW, TH, LAZY>), dim3((slots + kXcds - 1) / kXcds * kXcds * PPL),
                           dim3(64), 0, st, rec, ids, c->tranges, order, (int)slots, vt, rp, bg, rgb, T_final,
                           last, mode, src);
}

template <int TW, int TH>
hipError_t fwd_impl(Ctx* c, const ViewTable& vt, const RasterParams& rp, const float* bg,
                    float* rgb, float* T_final, int32_t* last, const uint32_t* order, int mode,
                    hipStream_t st) {
    BlockSrc src = {};
    if (c->lists_lazy) {
        const int sd = c->block_side;
        src = {c->iv[sd], c->im[sd], c->im[sd] + c->cap.max_isect, c->ranges, c->tids};
        fwd_launch<TW, TH, true>(c, vt, rp, bg, rgb, T_final, last, order, mode, src, st);
    } else {
        fwd_launch<TW, TH, false>(c, vt, rp, bg, rgb, T_final, last, order, mode, src, st);
    }
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess && c->lists_lazy) c->lists_filled = true;
    return e;
}

// Tiles whose chains are all resident at once are all walked in segments, unplanned
// (256 tiles of 16x16, 10k blob splats 514 -> 178 us; 476 of 32x16, 1.4M splats 1290);
// more are planned.  Past 2^20 tiles (the plan is one workgroup's) none is split.
template <int TW, int TH>
hipError_t bwd_impl(Ctx* c, const ViewTable& vt, const RasterParams& rp, const float* bg,
                    const float* T_final, const int32_t* last, const float* v_rgb, hipStream_t st) {
    constexpr int PPL = TileMap<TW, TH>::PPL;
    const int T = (int)c->n_tiles;
    const int all = (int64_t)T * PPL <= kWaveSlots ? T : 0;
    const BwdArgs g = {reinterpret_cast<const float4*>(c->rec), reinterpret_cast<const int32_t*>(c->tids),
                       c->tranges, bg, T_final, last, v_rgb, c->grad2d,
                       c->grad2d + kGradGeo * c->cap.max_pairs, c->snap, all ? 2 * kBwdSegs : kBwdSegs, rp};
    const auto segments = [&](int tiles, const uint32_t* order, const uint32_t* plan, int heavy) {
        hipLaunchKernelGGL((k_render_bwd_segs<TW, TH>), dim3((unsigned)((tiles + kXcds - 1) / kXcds * kXcds * g.segs)),
                           dim3(64), 0, st, g, vt, order, plan, heavy);
    };
    if (all || T > (1 << 20)) {
        const unsigned grid = all ? (unsigned)((T + kXcds - 1) / kXcds * kXcds * PPL) : (unsigned)T;
        hipLaunchKernelGGL((k_render_bwd<TW, TH>), dim3(grid), dim3(64), 0, st, g, vt, T, nullptr, nullptr, all);
        if (all) segments(T, nullptr, nullptr, all);
        return hipGetLastError();
    }
    uint32_t* bucket = c->tk[0];
    uint32_t* order = c->tk[1];
    uint32_t* plan = c->scalars + kScalarPlan;
    hipLaunchKernelGGL((k_bwd_weights<TW, TH>), dim3((unsigned)((T + 3) / 4)), dim3(256), 0, st, vt, c->tranges,
                       last, T, bucket);
    hipLaunchKernelGGL(k_bwd_plan, dim3(1), dim3(kWeightThreads), 0, st, bucket, T, order, plan);
    const unsigned grid = (unsigned)(T + (PPL - 1) * std::min(T, kMaxHeavy) + kXcds * PPL);
    hipLaunchKernelGGL((k_render_bwd<TW, TH>), dim3(grid), dim3(64), 0, st, g, vt, T, order, plan, 0);
    segments(std::min(T, kMaxHeavy), order, plan, 0);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_render_fwd(Ctx* c, const ViewTable& vt, const RasterParams& rp, const float* bg,
                             float* rgb, float* T_final, int32_t* last, hipStream_t st) {
    if (c->n_tiles <= 0) return hipSuccess;
    const uint32_t* order = c->ordered ? c->tile_order : nullptr;
    const int mode = rp.tile_order == 2 ? 2 : (order ? 1 : 0);
    const int TW = rp.tile_w, TH = rp.tile_h;
    if (TW == 16 && TH == 16) return fwd_impl<16, 16>(c, vt, rp, bg, rgb, T_final, last, order, mode, st);
    if (TW == 16 && TH == 8) return fwd_impl<16, 8>(c, vt, rp, bg, rgb, T_final, last, order, mode, st);
    if (TW == 8 && TH == 8) return fwd_impl<8, 8>(c, vt, rp, bg, rgb, T_final, last, order, mode, st);
    if (TW == 32 && TH == 16) return fwd_impl<32, 16>(c, vt, rp, bg, rgb, T_final, last, order, mode, st);
    return hipErrorInvalidValue;
}

hipError_t launch_render_bwd(Ctx* c, const ViewTable& vt, const RasterParams& rp, const float* bg,
                             const float* T_final, const int32_t* last, const float* v_rgb,
                             hipStream_t st) {
    if (c->n_tiles <= 0) return hipSuccess;
    // lazy lists with no forward since the bin step: write them in full first
    if (c->lists_lazy && !c->lists_filled) {
        const hipError_t e = launch_expand_lists(c, st);
        if (e != hipSuccess) return e;
    }
    const int TW = rp.tile_w, TH = rp.tile_h;
    if (TW == 16 && TH == 16) return bwd_impl<16, 16>(c, vt, rp, bg, T_final, last, v_rgb, st);
    if (TW == 16 && TH == 8) return bwd_impl<16, 8>(c, vt, rp, bg, T_final, last, v_rgb, st);
    if (TW == 8 && TH == 8) return bwd_impl<8, 8>(c, vt, rp, bg, T_final, last, v_rgb, st);
    if (TW == 32 && TH == 16) return bwd_impl<32, 16>(c, vt, rp, bg, T_final, last, v_rgb, st);
    return hipErrorInvalidValue;
}

hipError_t launch_l1(Ctx* c, const ViewTable& vt, const float* rgb, const float* target,
                     float* v_rgb, float* loss, hipStream_t st) {
    const int64_t P = vt.pix_off[vt.V];
    if (P > 0) {
        const unsigned nb = (unsigned)std::min<int64_t>((P + 255) / 256, kL1Blocks);
        hipLaunchKernelGGL(k_l1, dim3(nb), dim3(256), 0, st, rgb, target, v_rgb, vt, c->loss_acc);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_flush_acc(c->loss_acc, loss, 1, st);
}

}  // namespace gs
