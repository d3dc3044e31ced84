// Gaussians from SfM points: mean = the point, an isotropic scale equal to
// the mean distance to its k nearest other points, identity rotation, one
// opacity, and the point's colour in the degree-0 SH band.
//
// The k nearest neighbours are exact and come from a bounding-volume
// hierarchy over the points in Morton order (10 bits per axis over the
// bounding cube).  Leaves hold kLeaf consecutive points of that order; the
// tree over the leaves is complete and implicit (heap numbering: node v has
// children 2v and 2v+1, the leaves are NL..2NL-1, padded with empty boxes) and
// stores each node's axis-aligned box of its points.  Because the boxes are
// the points' own boxes and the leaves split by count, not by space, the
// search adapts to the density: clustered scenes (dense blobs next to sparse
// outliers) cost about the same per point as uniform ones.  A wave
// searches for 64 consecutive points of the order at once.  It first takes its
// own leaves and kSide on either side of them (almost always near) as
// candidates, which bounds each point's k-th distance; it then walks the tree
// six levels at a step, a lane testing one of a node's 64 descendants there
// (contiguous in heap order) against the boxes of the wave's four rows of 16
// points, and the points testing each survivor, skipping every box farther than
// all their k-th distances.  The box distances are computed with the same float
// operations as the point distances and are monotone in them, so no point
// nearer than the bound is ever skipped.
#include <math.h>

#include <algorithm>

#include "gs_internal.h"

namespace gs {

namespace {

constexpr int kBlock = 256;
constexpr int kMaxK = GS_INIT_MAX_K;
constexpr int kLeaf = 8;           // points per leaf
constexpr int kSide = 2;           // leaves on either side of a wave's own taken first
constexpr int kBoxBlocks = 1024;   // blocks of the bounding-box reduction
constexpr int kUpBlock = 256;      // nodes per block in the bottom-up box pass
constexpr float kSMin = 1e-7f;     // smallest scale (coincident points)

// up to here a wave takes every leaf first, and there is no tree
constexpr int kNoTree = (kSide + 1) * kLeaf;

// Morton cells: origin and 1024 / (side of the bounding cube)
struct Grid {
    float ox, oy, oz, ih;
};

// the wave's least lo and greatest hi, in every lane
__device__ __forceinline__ void wave_box(float (&lo)[3], float (&hi)[3]) {
#pragma unroll
    for (int a = 0; a < 3; a++)
        for (int off = 32; off > 0; off >>= 1) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], off, kWave));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], off, kWave));
        }
}

// per block: min and max of x, y, z
__global__ __launch_bounds__(kBlock) void k_box_partial(const float* __restrict__ pts, int n,
                                                        float* __restrict__ part) {
    __shared__ float s[6][kBlock / kWave];
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const float v = pts[3 * (int64_t)i + a];
            lo[a] = fminf(lo[a], v);
            hi[a] = fmaxf(hi[a], v);
        }
    }
    wave_box(lo, hi);
    const int w = threadIdx.x / kWave;
    if (__lane_id() == 0)
        for (int a = 0; a < 3; a++) {
            s[a][w] = lo[a];
            s[3 + a][w] = hi[a];
        }
    __syncthreads();
    if (threadIdx.x < 6) {
        const bool mx = threadIdx.x >= 3;
        float v = s[threadIdx.x][0];
        for (int q = 1; q < kBlock / kWave; q++) v = mx ? fmaxf(v, s[threadIdx.x][q]) : fminf(v, s[threadIdx.x][q]);
        part[6 * blockIdx.x + threadIdx.x] = v;
    }
}

// The Morton grid: 1024 cells per axis over the bounding cube (the order only
// serves locality; the search does not depend on the cells).  One wave.
__global__ __launch_bounds__(kWave) void k_grid(const float* __restrict__ part, int nb, Grid* __restrict__ g) {
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int b = threadIdx.x; b < nb; b += kWave)
#pragma unroll
        for (int a = 0; a < 3; a++) {
            lo[a] = fminf(lo[a], part[6 * b + a]);
            hi[a] = fmaxf(hi[a], part[6 * b + 3 + a]);
        }
    wave_box(lo, hi);
    if (threadIdx.x != 0) return;
    const float e = fmaxf(hi[0] - lo[0], fmaxf(hi[1] - lo[1], hi[2] - lo[2]));
    Grid G;
    G.ox = lo[0];
    G.oy = lo[1];
    G.oz = lo[2];
    G.ih = (e > 0.f && e < INFINITY) ? 1024.f / e : 0.f;  // all points coincide: one cell
    *g = G;
}

__device__ __forceinline__ uint32_t cell_of(float v, float o, float ih) {
    const float c = (v - o) * ih;
    return c >= 1023.f ? 1023u : (c > 0.f ? (uint32_t)c : 0u);  // NaN goes to 0
}

// 10 bits spread to every third bit
__device__ __forceinline__ uint32_t spread3(uint32_t v) {
    v &= 1023u;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__global__ __launch_bounds__(kBlock) void k_cell_keys(const float* __restrict__ pts, int n,
                                                      const Grid* __restrict__ gp,
                                                      uint32_t* __restrict__ keys,
                                                      uint32_t* __restrict__ vals) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const Grid g = *gp;
    const uint32_t cx = cell_of(pts[3 * (int64_t)i], g.ox, g.ih);
    const uint32_t cy = cell_of(pts[3 * (int64_t)i + 1], g.oy, g.ih);
    const uint32_t cz = cell_of(pts[3 * (int64_t)i + 2], g.oz, g.ih);
    keys[i] = spread3(cx) | (spread3(cy) << 1) | (spread3(cz) << 2);
    vals[i] = (uint32_t)i;
}

// points in sorted order (x, y, z, -), the last leaf filled up with points that
// are near nothing
__global__ __launch_bounds__(kBlock) void k_gather(const float* __restrict__ pts, int n,
                                                   const uint32_t* __restrict__ vals,
                                                   float4* __restrict__ sp) {
    const int j = blockIdx.x * kBlock + threadIdx.x;
    if (j >= (n + kLeaf - 1) / kLeaf * kLeaf) return;
    if (j >= n) {
        sp[j] = make_float4(INFINITY, INFINITY, INFINITY, 0.f);
        return;
    }
    const int64_t q = vals[j];
    sp[j] = make_float4(pts[3 * q], pts[3 * q + 1], pts[3 * q + 2], 0.f);
}

// The k <= K smallest squared distances seen, ascending, in the last k places
// (the first K - k hold -inf, so the k-th is always the last).
template <int K>
struct TopK {
    float d[K];
    // v: not a NaN
    __device__ __forceinline__ void push(float v) {
#pragma unroll
        for (int i = 0; i < K; i++) {
            const float t = fminf(d[i], v);
            v = fmaxf(d[i], v);
            d[i] = t;
        }
    }
};

// leaf boxes: tree[2v] = (min x, y, z, -), tree[2v + 1] = (max x, y, z, -);
// padded leaves get an empty box (+inf, -inf), which every bound skips
__global__ __launch_bounds__(kBlock) void k_leaf_box(const float4* __restrict__ sp, int n, int NL,
                                                     float4* __restrict__ tree) {
    const int l = blockIdx.x * kBlock + threadIdx.x;
    if (l >= NL) return;
    float4 lo = make_float4(INFINITY, INFINITY, INFINITY, 0.f);
    float4 hi = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.f);
    const int a = l * kLeaf, b = min(n, a + kLeaf);
    for (int i = a; i < b; i++) {
        const float4 p = sp[i];
        lo.x = fminf(lo.x, p.x);
        lo.y = fminf(lo.y, p.y);
        lo.z = fminf(lo.z, p.z);
        hi.x = fmaxf(hi.x, p.x);
        hi.y = fmaxf(hi.y, p.y);
        hi.z = fmaxf(hi.z, p.z);
    }
    tree[2 * (int64_t)(NL + l)] = lo;
    tree[2 * (int64_t)(NL + l) + 1] = hi;
}

// Boxes of the inner nodes from their children, up to nine levels per launch:
// block b makes the nodes m + 256 b .. m + 256 b + 255 of level [m, 2m) (the
// level below is done), then their parents from its own results in LDS, and
// so on while it holds more than one node.  m is a power of two.
__global__ __launch_bounds__(kUpBlock) void k_tree_up(float4* __restrict__ tree, int m) {
    __shared__ float4 slo[kUpBlock], shi[kUpBlock];
    const int t = threadIdx.x;
    int cnt = min(kUpBlock, m);
    int base = m + blockIdx.x * kUpBlock;
    float4 lo, hi;
    if (t < cnt) {
        const int64_t c = 2 * (int64_t)(base + t);
        const float4 l0 = tree[2 * c], h0 = tree[2 * c + 1], l1 = tree[2 * c + 2], h1 = tree[2 * c + 3];
        lo = make_float4(fminf(l0.x, l1.x), fminf(l0.y, l1.y), fminf(l0.z, l1.z), 0.f);
        hi = make_float4(fmaxf(h0.x, h1.x), fmaxf(h0.y, h1.y), fmaxf(h0.z, h1.z), 0.f);
        tree[2 * (int64_t)(base + t)] = lo;
        tree[2 * (int64_t)(base + t) + 1] = hi;
        slo[t] = lo;
        shi[t] = hi;
    }
    while (cnt > 1) {
        __syncthreads();
        cnt >>= 1;
        base >>= 1;
        if (t < cnt) {
            const float4 l0 = slo[2 * t], h0 = shi[2 * t], l1 = slo[2 * t + 1], h1 = shi[2 * t + 1];
            lo = make_float4(fminf(l0.x, l1.x), fminf(l0.y, l1.y), fminf(l0.z, l1.z), 0.f);
            hi = make_float4(fmaxf(h0.x, h1.x), fmaxf(h0.y, h1.y), fmaxf(h0.z, h1.z), 0.f);
        }
        __syncthreads();
        if (t < cnt) {
            slo[t] = lo;
            shi[t] = hi;
            tree[2 * (int64_t)(base + t)] = lo;
            tree[2 * (int64_t)(base + t) + 1] = hi;
        }
    }
}

__device__ __forceinline__ float dist2(float4 o, float4 p) {
    const float dx = o.x - p.x, dy = o.y - p.y, dz = o.z - p.z;
    return __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
}

// squared distance from p to a box; for any point q in the box each axis
// difference is at least the box's, in float too (rounding is monotone), so
// this never exceeds dist2(q, p)
__device__ __forceinline__ float box_dist2(float4 lo, float4 hi, float4 p) {
    const float ex = fmaxf(fmaxf(lo.x - p.x, p.x - hi.x), 0.f);
    const float ey = fmaxf(fmaxf(lo.y - p.y, p.y - hi.y), 0.f);
    const float ez = fmaxf(fmaxf(lo.z - p.z, p.z - hi.z), 0.f);
    return __builtin_fmaf(ex, ex, __builtin_fmaf(ey, ey, ez * ez));
}

// The greatest of v in each row of 16 lanes, in all of its lanes.
__device__ __forceinline__ float row_max(float v) {
    v = fmaxf(v, dpp_f<0xB1>(v));
    v = fmaxf(v, dpp_f<0x4E>(v));
    v = fmaxf(v, dpp_f<0x124>(v));  // row_ror:4
    return fmaxf(v, dpp_f<0x128>(v));
}

// The search of a wave's 64 points (one a lane, in sorted order).
template <int K>
struct Search {
    const float4* __restrict__ sp;
    const float4* __restrict__ tree;
    int NL, nl, l0, l1;  // leaves 0 .. nl - 1 hold points; l0 .. l1 - 1 are taken
    float4 p;
    TopK<K> best;
    bool open;                  // whether the point has anything to look for
    float glo[4][3], ghi[4][3]; // the boxes of the wave's rows

    // the largest squared distance of interest
    __device__ __forceinline__ float bound() const { return open ? best.d[K - 1] : -1.f; }

    // the 8 points of a leaf, each read by all lanes from one address; j: this
    // lane's own place in the order, or -1 where the leaf does not hold it
    __device__ __forceinline__ void leaf(int l, int j) {
        const float4* o = sp + l * kLeaf;
#pragma unroll
        for (int i = 0; i < kLeaf; i++) {
            const float d2 = dist2(o[i], p);
            const bool nearer = d2 < best.d[K - 1] && l * kLeaf + i != j;  // (a NaN is not)
            if (__ballot(nearer) != 0) best.push(nearer ? d2 : INFINITY);
        }
    }

    // Node v's descendants `width` nodes of heap order wide (64, or fewer for
    // the root's step), D such steps above the leaves: lane i tests descendant
    // v width + i against the rows' boxes and largest bounds; the points then
    // test each survivor.
    template <int D>
    __device__ __forceinline__ void visit(int v, int width) {
        const int lane = threadIdx.x % kWave;
        const int c0 = v * width;
        const float rb = row_max(bound());
        float4 lo = make_float4(INFINITY, INFINITY, INFINITY, 0.f), hi = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.f);
        if (lane < width) {
            lo = tree[2 * (int64_t)(c0 + lane)];
            hi = tree[2 * (int64_t)(c0 + lane) + 1];
        }
        bool near = false;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const float ex = fmaxf(fmaxf(lo.x - ghi[r][0], glo[r][0] - hi.x), 0.f);
            const float ey = fmaxf(fmaxf(lo.y - ghi[r][1], glo[r][1] - hi.y), 0.f);
            const float ez = fmaxf(fmaxf(lo.z - ghi[r][2], glo[r][2] - hi.z), 0.f);
            near |= __builtin_fmaf(ex, ex, __builtin_fmaf(ey, ey, ez * ez)) <= bcast(rb, 16 * r);
        }
        near = near && lane < width;  // (no box is near only where the bounds are finite)
        if (D == 1) {
            const int l = c0 + lane - NL;
            near = near && l < nl && (unsigned)(l - l0) >= (unsigned)(l1 - l0);
        }
        uint64_t todo = __ballot(near);
        while (todo) {
            const int b = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            const float4 l = make_float4(bcast(lo.x, b), bcast(lo.y, b), bcast(lo.z, b), 0.f);
            const float4 h = make_float4(bcast(hi.x, b), bcast(hi.y, b), bcast(hi.z, b), 0.f);
            if (__ballot(box_dist2(l, h, p) <= bound()) == 0) continue;
            if constexpr (D == 1)
                leaf(c0 + b - NL, -1);
            else
                visit<D - 1>(c0 + b, kWave);
        }
    }
};

// A wave per 64 points, in sorted order; the mean of the k nearest distances
// goes to s[original index].  With n <= kNoTree there is no tree.
// VALU-bound (about 14000 instructions a wave): a wave's points share the tree's
// and the leaves' loads, and a leaf's points reach the lanes from one address.
// 1.5M clustered points, k = 4, under the profiler: 930 us; 3800 with a thread
// per point walking the tree by itself (its lanes on unlike nodes, a dependent
// load each step); 2130 with the wave's points bounded by their 16 sorted
// neighbours and prefiltered by one box.
template <int K, int STEPS>
__global__ __launch_bounds__(kBlock) void k_knn(const uint32_t* __restrict__ vals,
                                                const float4* __restrict__ sp, int n, int k,
                                                const float4* __restrict__ tree, int NL, int levels,
                                                float* __restrict__ s) {
    const int j = blockIdx.x * kBlock + threadIdx.x;
    const int w0 = __builtin_amdgcn_readfirstlane(j - threadIdx.x % kWave);  // the wave's first point
    if (w0 >= n) return;
    const bool mine = j < n;
    const int nl = (n + kLeaf - 1) / kLeaf;
    Search<K> S;
    S.sp = sp;
    S.tree = tree;
    S.NL = NL;
    S.nl = nl;
    S.l0 = max(w0 / kLeaf - kSide, 0);
    S.l1 = min(w0 / kLeaf + kWave / kLeaf + kSide, nl);
    const int kk = min(k, n - 1);
    S.p = sp[min(j, n - 1)];
#pragma unroll
    for (int i = 0; i < K; i++) S.best.d[i] = mine && i >= K - kk ? INFINITY : -INFINITY;
    for (int l = S.l0; l < S.l1; l++) S.leaf(l, j);
    // (nothing to look for when all its neighbours coincide with it)
    S.open = mine && kk > 0 && S.best.d[K - 1] > 0.f;
    if (n > kNoTree && __ballot(S.open) != 0) {
        const float x[3] = {S.p.x, S.p.y, S.p.z};
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const float lo = -row_max(S.open ? -x[a] : -INFINITY), hi = row_max(S.open ? x[a] : -INFINITY);
#pragma unroll
            for (int r = 0; r < 4; r++) {
                S.glo[r][a] = bcast(lo, 16 * r);
                S.ghi[r][a] = bcast(hi, 16 * r);
            }
        }
        // steps of six levels, the odd ones at the root
        S.template visit<STEPS>(1, 1 << (levels - 6 * (STEPS - 1)));
    }
    if (!mine) return;
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < K; i++) m += i >= K - kk ? sqrtf(S.best.d[i]) : 0.f;
    m = kk > 0 ? m / (float)kk : 0.f;
    s[vals[j]] = fmaxf(m, kSMin);
}

// the Gaussians, coalesced in the original order
__global__ __launch_bounds__(kBlock) void k_init_write(const float* __restrict__ pts,
                                                       const float* __restrict__ rgb, int n, int K,
                                                       float opacity_logit,
                                                       const float* __restrict__ s,
                                                       float* __restrict__ means,
                                                       float* __restrict__ log_scales,
                                                       float* __restrict__ quats,
                                                       float* __restrict__ logit,
                                                       float* __restrict__ sh) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    // rgb = 0.5 + C0 sh_0 with C0 = 1 / (2 sqrt(pi)), the renderer's colour rule
    constexpr float kInvC0 = 3.5449077018110318f;  // 2 sqrt(pi)
    const float ls = logf(s[i]);
#pragma unroll
    for (int a = 0; a < 3; a++) {
        means[(int64_t)a * n + i] = pts[3 * (int64_t)i + a];
        log_scales[(int64_t)a * n + i] = ls;
    }
    quats[i] = 1.f;
    quats[(int64_t)n + i] = 0.f;
    quats[2 * (int64_t)n + i] = 0.f;
    quats[3 * (int64_t)n + i] = 0.f;
    logit[i] = opacity_logit;
    for (int c = 0; c < K; c++)
#pragma unroll
        for (int ch = 0; ch < 3; ch++)
            sh[((int64_t)c * 3 + ch) * n + i] = c == 0 ? (rgb[3 * (int64_t)i + ch] - 0.5f) * kInvC0 : 0.f;
}

}  // namespace

hipError_t launch_init_gaussians(Ctx* c, const float* pts, const float* rgb, int n, int k,
                                 float opacity, int sh_degree, float* means, float* log_scales,
                                 float* quats, float* logit, float* sh, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int nb = std::min((n + kBlock - 1) / kBlock, kBoxBlocks);
    float* part = c->aux;
    Grid* grid = reinterpret_cast<Grid*>(c->aux + 6 * kBoxBlocks);
    hipLaunchKernelGGL(k_box_partial, dim3(nb), dim3(kBlock), 0, st, pts, n, part);
    hipLaunchKernelGGL(k_grid, dim3(1), dim3(64), 0, st, part, nb, grid);
    const unsigned g = (unsigned)((n + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_cell_keys, dim3(g), dim3(kBlock), 0, st, pts, n, grid, c->pk[0], c->pv[0]);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int side = radix_sort_pairs(c->pk[0], c->pv[0], c->pk[1], c->pv[1], n, nullptr, 0, 30,
                                      c->hist, c->scan_scratch, c->diag + kDiagFlags, st, &e);
    if (e != hipSuccess) return e;
    const uint32_t* vals = c->pv[side];
    // sorted points, then the tree, in the record buffer (12 floats per pair):
    // 128 nl bytes and, past kNoTree points, 64 NL < 128 nl (nl = ceil(n / 8))
    const int nl = (n + kLeaf - 1) / kLeaf;
    float4* sp = reinterpret_cast<float4*>(c->rec);
    float4* tree = sp + (int64_t)nl * kLeaf;
    float* s = reinterpret_cast<float*>(c->cnt);
    hipLaunchKernelGGL(k_gather, dim3(g), dim3(kBlock), 0, st, pts, n, vals, sp);
    int NL = 0, levels = 0;
    if (n > kNoTree) {
        NL = 1;
        while (NL < nl) NL *= 2, levels++;
        hipLaunchKernelGGL(k_leaf_box, dim3((NL + kBlock - 1) / kBlock), dim3(kBlock), 0, st, sp, n, NL,
                           tree);
        for (int m = NL / 2; m >= 1; m /= 2 * kUpBlock)
            hipLaunchKernelGGL(k_tree_up, dim3(std::max(1, m / kUpBlock)), dim3(kUpBlock), 0, st, tree, m);
    }
    const auto knn = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(g), dim3(kBlock), 0, st, vals, sp, n, k, tree, NL, levels, s);
    };
    const int steps = (levels + 5) / 6;  // (n <= max_pairs <= 2^26: at most 23 levels)
    if (k <= 4) knn(steps <= 1 ? k_knn<4, 1> : steps == 2 ? k_knn<4, 2> : steps == 3 ? k_knn<4, 3> : k_knn<4, 4>);
    else knn(steps <= 1 ? k_knn<kMaxK, 1> : steps == 2 ? k_knn<kMaxK, 2> : steps == 3 ? k_knn<kMaxK, 3> : k_knn<kMaxK, 4>);
    const float lg = logf(opacity / (1.f - opacity));
    const int K = (sh_degree + 1) * (sh_degree + 1);
    hipLaunchKernelGGL(k_init_write, dim3(g), dim3(kBlock), 0, st, pts, rgb, n, K, lg, s, means,
                       log_scales, quats, logit, sh);
    return hipGetLastError();
}

}  // namespace gs
