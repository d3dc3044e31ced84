// One Levenberg-Marquardt step of bundle adjustment on the track
// reprojection term: poses (left twists at the current pose) and points,
// Huber cost on the squared reprojection error, iteratively reweighted.
//
// With r the residual of an observation, s = |r|^2, w = rho'(s) and
// J = [J_pose | J_X] its Jacobian, the normal equations are
//   [U  W] [dc]   [-g_c]      U = sum w J_pose^T J_pose (+ lambda diag),
//   [W' V] [dX] = [-g_X],     V = sum w J_X^T J_X (+ lambda diag),
//                             W = sum w J_pose^T J_X, g = sum w J^T r.
// Points are eliminated (V is block diagonal, 3x3 per point): the reduced
// camera system S dc = b with S = U - W V^-1 W', b = -g_c + W V^-1 g_X is
// solved by conjugate gradients preconditioned with the inverse 6x6 diagonal
// blocks of S, then dX = -V^-1 (g_X + W' dc).  S is never formed: a product
// S p takes u_k = V_k^-1 sum W'_o p over a point's observations and then
// U p - sum W_o u_k over a camera's, recomputing each observation's Jacobian
// blocks from the parameters (12 B read per observation, instead of the 144 B
// its blocks would take).  All arithmetic is double.
// With few enough cameras for their data to fit one workgroup's LDS, both
// sums are one pass by point and one launch per iteration (k_ba_cg); with
// more, one pass by point and one by camera, and a launch for the update.
// The iteration count is fixed at launch (a graph-capturable step); once the
// residual is below tol |b| a device flag turns the remaining launches into
// no-ops.
#include <math.h>

#include <algorithm>

#include "gs_internal.h"

struct gs_ba {
    int64_t max_points;
    int32_t max_cams;
    int32_t lds_cams; // cameras whose data fit the LDS of one workgroup (k_ba_cg)
    double* pt;       // V^-1 [Pt][6] (sym), then rows [Pt][12] (kRow)
    double* cam;      // per camera: U (21), L (21), 9 vectors of 6, 16 floats
    void* win;        // windows of k_ba_cg, at most one per point and one more per wave
    int32_t* cam_off; // [max_cams + 1]
    double* sc;       // [16] scalars
};

namespace gs {

namespace {

constexpr int kBlock = 256;
constexpr int kVec = 1024;  // threads of the single-workgroup vector kernels and of k_ba_cg
constexpr int kCgBlocks = 256;  // most workgroups of k_ba_cg: one per CU
constexpr int kCgWaves = kCgBlocks * (kVec / kWave);
constexpr int kPt = 18, kCam = 104;  // doubles of workspace per point and per camera
// A point's row: V^-1 (6), V^-1 g_X (3), and X (3 floats), in whose place the
// two-pass path later keeps u (3).  The passes by camera gather whole rows; the
// passes by point read V^-1 from the array of its own.
constexpr int kRow = 12;
// Camera workspace: U [21][n_cams], then L [21][n_cams] (the Cholesky factor of
// S_ii, its diagonal stored as reciprocals; 0 for a fixed camera), then the
// vectors of the conjugate gradients, 6 per camera ([6][n_cams] in k_ba_cg,
// whose threads read them by camera; [n_cams][6] on the two-pass path, which
// gathers them), and the cameras' floats.
enum { vX = 0, vR = 1, vR1 = 2, vP = 3, vP1 = 4, vAp = 5, vAp1 = 6, vAp2 = 7, vZ = 8, vCams = 9 };
__host__ __device__ inline int64_t off_l(int n_cams) { return (int64_t)21 * n_cams; }
__host__ __device__ inline int64_t off_vec(int n_cams, int v) { return (int64_t)(42 + 6 * v) * n_cams; }
// scalars (sRZ and sEnd: two, by the parity of the iteration; sPap: three, like
// A p).  sDone ends the two-pass path, sEnd k_ba_cg.
enum { sRZ = 0, sBB = 2, sDone = 3, sIt = 4, sCost = 5, sMasked = 6, sUnsorted = 7, sRR = 8, sPap = 9, sEnd = 12 };
// LDS of k_ba_cg: per camera its 16 floats, its 6 of p and its 6 sums of W u
constexpr int kLdsPerCam = 16 * 4 + 6 * 8 + 6 * 8;
constexpr int kLdsFixed = 2 * (kVec / kWave) * 8;

struct BaObs {
    const float* X;
    const float* viewmat;
    const float* intr;
    float4* cams;  // [n_cams][4]: the rows of [R|t], then fx, fy, cx, cy (k_ba_ranges)
    const int32_t* obs_cam;
    const int32_t* obs_pt;
    const float* obs_xy;
    int Pt, n_cams, M;
    double delta, near_plane, lambda;
};

struct Lin {
    bool ok;
    double r0, r1, w, rho;
    double Jp[12], Jx[6];
};

// A camera's 16 floats.
struct CamData {
    float4 q[4];
};

__device__ __forceinline__ CamData load_cam(const BaObs& a, int ci) {
    CamData c;
#pragma unroll
    for (int q = 0; q < 4; q++) c.q[q] = a.cams[4 * (int64_t)ci + q];
    return c;
}

// The quads of the cameras in LDS are 64 B apart; quad q of camera c sits in
// slot (q + c / 4) mod 4, so 16 consecutive cameras' quads fall in 16
// different bank groups.
__device__ __forceinline__ int cam_slot(int c, int q) { return 4 * c + ((q + (c >> 2)) & 3); }

__device__ __forceinline__ CamData lds_cam(const float4* s_cam, int c) {
    CamData d;
#pragma unroll
    for (int q = 0; q < 4; q++) d.q[q] = s_cam[cam_slot(c, q)];
    return d;
}

// 1/x of normal positive x: the hardware's estimate (about 2^-26) and two Newton
// steps, the second of which rounds correctly what the first left within an ulp
// or two, in half the instructions of a division, which also minds the ends of
// the range.
__device__ __forceinline__ double recip(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}

// Projection of one observation: camera point p, J_pi = [[a00, 0, a02],
// [0, a11, a12]] = [[fx/z, 0, -fx x/z^2], [0, fy/z, -fy y/z^2]], residual and
// weight.
struct Proj {
    bool ok;
    double R[9], p[3], a00, a02, a11, a12, r0, r1, w, rho;
};

__device__ __forceinline__ void project(const BaObs& a, const CamData& cam, double X0, double X1,
                                        double X2, float2 xy, Proj& P) {
#pragma unroll
    for (int i = 0; i < 3; i++) {
        P.R[3 * i] = cam.q[i].x;
        P.R[3 * i + 1] = cam.q[i].y;
        P.R[3 * i + 2] = cam.q[i].z;
        P.p[i] = P.R[3 * i] * X0 + P.R[3 * i + 1] * X1 + P.R[3 * i + 2] * X2 + (double)cam.q[i].w;
    }
    P.ok = P.p[2] >= a.near_plane;
    if (!P.ok) return;
    const double fx = cam.q[3].x, fy = cam.q[3].y, cx = cam.q[3].z, cy = cam.q[3].w;
    const double iz = recip(P.p[2]), u = P.p[0] * iz, v = P.p[1] * iz;
    P.r0 = fx * u + cx - (double)xy.x;
    P.r1 = fy * v + cy - (double)xy.y;
    const double s = P.r0 * P.r0 + P.r1 * P.r1;
    if (s <= a.delta * a.delta) {
        P.w = 1.0;
        P.rho = s;
    } else {
        const double rs = sqrt(s);
        P.w = a.delta / rs;
        P.rho = 2.0 * a.delta * rs - a.delta * a.delta;
    }
    P.a00 = fx * iz;
    P.a02 = -P.a00 * u;
    P.a11 = fy * iz;
    P.a12 = -P.a11 * v;
}

__device__ __forceinline__ void linearise(const BaObs& a, const CamData& cam, double X0, double X1,
                                          double X2, float2 xy, Lin& L) {
    Proj P;
    project(a, cam, X0, X1, X2, xy, P);
    L.ok = P.ok;
    if (!L.ok) return;
    L.r0 = P.r0;
    L.r1 = P.r1;
    L.w = P.w;
    L.rho = P.rho;
    // J_pose = J_pi [I | -[p]x]
    L.Jp[0] = P.a00; L.Jp[1] = 0.0; L.Jp[2] = P.a02;
    L.Jp[3] = P.a02 * P.p[1];
    L.Jp[4] = P.a00 * P.p[2] - P.a02 * P.p[0];
    L.Jp[5] = -P.a00 * P.p[1];
    L.Jp[6] = 0.0; L.Jp[7] = P.a11; L.Jp[8] = P.a12;
    L.Jp[9] = -P.a11 * P.p[2] + P.a12 * P.p[1];
    L.Jp[10] = -P.a12 * P.p[0];
    L.Jp[11] = P.a11 * P.p[0];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        L.Jx[c] = P.a00 * P.R[c] + P.a02 * P.R[6 + c];
        L.Jx[3 + c] = P.a11 * P.R[3 + c] + P.a12 * P.R[6 + c];
    }
}

__device__ __forceinline__ void linearise(const BaObs& a, int o, int ci, int k, Lin& L) {
    linearise(a, load_cam(a, ci), a.X[3 * (int64_t)k], a.X[3 * (int64_t)k + 1], a.X[3 * (int64_t)k + 2],
              make_float2(a.obs_xy[2 * (int64_t)o], a.obs_xy[2 * (int64_t)o + 1]), L);
}

// symmetric 3x3 (00 01 02 11 12 22) and 6x6 (row-major lower triangle, 21)
__device__ __forceinline__ int tri6(int i, int j) { return i >= j ? i * (i + 1) / 2 + j : j * (j + 1) / 2 + i; }

template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* s) {
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
#pragma unroll
    for (int j = 0; j < NV; j++)
        for (int off = 32; off > 0; off >>= 1) v[j] += __shfl_xor(v[j], off, kWave);
    if (lane == 0)
#pragma unroll
        for (int j = 0; j < NV; j++) s[w * NV + j] = v[j];
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int j = 0; j < NV; j++) {
            double t = 0.0;
            for (int q = 0; q < kBlock / kWave; q++) t += s[q * NV + j];
            v[j] = t;
        }
}

__device__ __forceinline__ int lower_bound_i(const int32_t* a, int n, int key) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// camera ranges of the observations (sorted by camera), the sort check, and
// the cameras' floats packed for 16-byte loads (a lane gathering them as twelve
// and four words kept the passes by point waiting on the L1)
__global__ __launch_bounds__(kBlock) void k_ba_ranges(BaObs a, int32_t* __restrict__ cam_off,
                                                      double* __restrict__ sc) {
    const int tid = blockIdx.x * kBlock + threadIdx.x;
    if (tid <= a.n_cams) cam_off[tid] = lower_bound_i(a.obs_cam, a.M, tid);
    if (tid < a.n_cams) {
        const float* v = a.viewmat + 12 * (int64_t)tid;
        const float* f = a.intr + 4 * (int64_t)tid;
#pragma unroll
        for (int q = 0; q < 3; q++)
            a.cams[4 * (int64_t)tid + q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        a.cams[4 * (int64_t)tid + 3] = make_float4(f[0], f[1], f[2], f[3]);
    }
    for (int o = tid; o + 1 < a.M; o += gridDim.x * kBlock)
        if (a.obs_cam[o] > a.obs_cam[o + 1]) sc[sUnsorted] = 1.0;
}

// A window: consecutive points with observations, of at most 64
// observations in all, one for each lane.  Bit l of `heads` is set where lane
// l holds the first observation of a point.  heads = 0: one point of more than
// 64 observations.  The window after a wave's last one closes it: only its o0
// counts.
struct alignas(16) Window {
    unsigned long long heads;
    int k0, o0;  // its first point and observation
};

// A wave's points: an equal share, whatever the grid.
__device__ __forceinline__ void wave_share(int Pt, int64_t wave, int64_t waves, int& begin, int& end) {
    begin = (int)(Pt * wave / waves);
    end = (int)(Pt * (wave + 1) / waves);
}

// cut each wave's points into windows (one wave each; `waves` of its readers)
__global__ __launch_bounds__(kWave) void k_ba_windows(int Pt, const int32_t* __restrict__ pt_off,
                                                      Window* __restrict__ win, int32_t* __restrict__ n_win) {
    constexpr int kChunk = 512;
    __shared__ int s_off[kChunk + 1];
    __shared__ unsigned long long s_heads;
    const int lane = threadIdx.x;
    int k, end, n = 0;
    wave_share(Pt, blockIdx.x, gridDim.x, k, end);
    Window* w = win + k + blockIdx.x;
    int o0 = k < end ? pt_off[k] : 0;
    int base = k, top = k;  // s_off holds the offsets of points base .. top
    while (k < end) {
        if (min(k + kWave, end) > top) {
            __syncthreads();
            base = k;
            top = min(k + kChunk, end);
            for (int i = lane; i <= top - base; i += kWave) s_off[i] = pt_off[base + i];
            __syncthreads();
        }
        const int m = min(k + lane, end - 1) - base;
        const int b = s_off[m], e = s_off[m + 1];
        const bool some = e > b;
        if (!(__ballot(some) & 1)) {  // a point without observations is in no window
            k++;
            continue;
        }
        // points up to the first that is empty or does not fit
        const uint64_t stop = __ballot(k + lane >= end || !some || e - o0 > kWave);
        const int np = stop ? __ffsll((unsigned long long)stop) - 1 : kWave;
        if (lane == 0) s_heads = 0;
        __syncthreads();
        if (lane < np) atomicOr(&s_heads, 1ull << (b - o0));
        __syncthreads();
        if (lane == 0) w[n] = Window{s_heads, k, o0};
        __syncthreads();
        n++;
        const int step = max(np, 1);
        o0 = __shfl(e, step - 1, kWave);
        k += step;
    }
    if (lane == 0) {
        w[n] = Window{0, end, o0};
        n_win[blockIdx.x] = n;
    }
}

// The segment (point) a lane of a window of `cnt` observations belongs to: its
// first and last lane.
struct Segment {
    int head, tail;
};

__device__ __forceinline__ Segment segment_of(uint64_t heads, int cnt, int lane) {
    const uint64_t upto = ~0ull >> (63 - lane);
    const uint64_t above = heads & ~upto;
    return Segment{63 - __clzll((long long)(heads & upto)),
                   above ? __ffsll((unsigned long long)above) - 2 : cnt - 1};
}

// the index of lane's point in a window
__device__ __forceinline__ int point_of(const Window& w) {
    const uint64_t h = w.heads >> 1;  // the number of heads at lanes 1 .. lane
    return w.k0 + __builtin_amdgcn_mbcnt_hi((uint32_t)(h >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)h, 0));
}

// What a lane reads for its observation of a window, ahead of its use.
struct Slot {
    int cam, k;  // cam: -1 where the lane has none
    float2 xy;
    float X[3];
};

__device__ __forceinline__ void read_pixel(const BaObs& a, const int32_t* __restrict__ pt_obs, int j, int k,
                                           Slot& s) {
    s.k = k;
    const int64_t o = pt_obs ? pt_obs[j] : j;  // no index: the arrays are point-major
    s.cam = a.obs_cam[o];
    s.xy = make_float2(a.obs_xy[2 * o], a.obs_xy[2 * o + 1]);
    if (s.cam < 0 || s.cam >= a.n_cams) s.cam = -1;
#pragma unroll
    for (int i = 0; i < 3; i++) s.X[i] = a.X[3 * (int64_t)k + i];
}

__device__ __forceinline__ void read_slot(const BaObs& a, const int32_t* __restrict__ pt_obs, const Window& w,
                                          int o1, int lane, Slot& s) {
    s.cam = -1;
    s.k = w.k0;
    if (w.heads == 0 || w.o0 + lane >= o1) return;
    read_pixel(a, pt_obs, w.o0 + lane, point_of(w), s);
}

// one observation's share of its point's V (6, sym) and g_X (3)
__device__ __forceinline__ void add_normal(const Proj& P, double (&v)[9]) {
    double J0[3], J1[3], w0[3], w1[3];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        J0[c] = P.a00 * P.R[c] + P.a02 * P.R[6 + c];
        J1[c] = P.a11 * P.R[3 + c] + P.a12 * P.R[6 + c];
        w0[c] = P.w * J0[c];
        w1[c] = P.w * J1[c];
        v[6 + c] += w0[c] * P.r0 + w1[c] * P.r1;
    }
    v[0] += w0[0] * J0[0] + w1[0] * J1[0];
    v[1] += w0[0] * J0[1] + w1[0] * J1[1];
    v[2] += w0[0] * J0[2] + w1[0] * J1[2];
    v[3] += w0[1] * J0[1] + w1[1] * J1[1];
    v[4] += w0[1] * J0[2] + w1[1] * J1[2];
    v[5] += w0[2] * J0[2] + w1[2] * J1[2];
}

// V damped and inverted by the adjugate, V^-1 g_X; a point with no observation
// is held fixed (zeros)
__device__ __forceinline__ void write_point(const BaObs& a, int k, double (&v)[9], double* __restrict__ pt) {
    v[0] *= 1.0 + a.lambda;
    v[3] *= 1.0 + a.lambda;
    v[5] *= 1.0 + a.lambda;
    const double c00 = v[3] * v[5] - v[4] * v[4], c01 = v[2] * v[4] - v[1] * v[5],
                 c02 = v[1] * v[4] - v[2] * v[3], c11 = v[0] * v[5] - v[2] * v[2],
                 c12 = v[1] * v[2] - v[0] * v[4], c22 = v[0] * v[3] - v[1] * v[1];
    const double det = v[0] * c00 + v[1] * c01 + v[2] * c02;
    const bool ok = det > 0.0;
    const double id = ok ? 1.0 / det : 0.0;
    const double q[6] = {c00 * id, c01 * id, c02 * id, c11 * id, c12 * id, c22 * id};
    double* vi = pt + 6 * (int64_t)k;
    double* e = pt + 6 * (int64_t)a.Pt + kRow * (int64_t)k;
#pragma unroll
    for (int i = 0; i < 6; i++) e[i] = vi[i] = ok ? q[i] : 0.0;
    e[6] = ok ? q[0] * v[6] + q[1] * v[7] + q[2] * v[8] : 0.0;
    e[7] = ok ? q[1] * v[6] + q[3] * v[7] + q[4] * v[8] : 0.0;
    e[8] = ok ? q[2] * v[6] + q[4] * v[7] + q[5] * v[8] : 0.0;
    float* x = reinterpret_cast<float*>(e + 9);
#pragma unroll
    for (int i = 0; i < 3; i++) x[i] = a.X[3 * (int64_t)k + i];
}

// Per point: V and V^-1 g_X; the cost and the masked count.  A lane takes one
// observation of a window and the nine sums of a point run over its lanes.
// Bound by the gathers of the cameras' floats and the 144 B written per point:
// 1.5M points, 6.5M observations take 187 us, as much as with a thread per
// point (160-190), but the pass then shares the windows and no wave waits for
// its longest track.
__global__ __launch_bounds__(kBlock) void k_ba_points(BaObs a, const int32_t* __restrict__ pt_off,
                                                      const int32_t* __restrict__ pt_obs,
                                                      const Window* __restrict__ win,
                                                      const int32_t* __restrict__ n_win,
                                                      double* __restrict__ pt, double* __restrict__ sc) {
    __shared__ double s_red[(kBlock / kWave) * 2];
    const int lane = threadIdx.x % kWave;
    const int wave =
        __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave));
    int kb, ke;
    wave_share(a.Pt, wave, (int64_t)gridDim.x * (kBlock / kWave), kb, ke);
    const Window* w = win + kb + wave;
    const int nw = n_win[wave];
    double cost = 0.0, masked = 0.0;
    // one observation: adds to v, the cost and the masked count
    auto take = [&](const Slot& s, double (&v)[9]) {
        if (s.cam < 0) return;
        Proj P;
        project(a, load_cam(a, s.cam), s.X[0], s.X[1], s.X[2], s.xy, P);
        if (!P.ok) {
            masked += 1.0;
            return;
        }
        cost += P.rho;
        add_normal(P, v);
    };
    for (int k = kb + lane; k < ke; k += kWave)
        if (pt_off[k] == pt_off[k + 1]) {
            double v[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
            write_point(a, k, v, pt);
        }
    Window cur = w[0], next = w[min(1, nw)];
    Slot s, s1;
    read_slot(a, pt_obs, cur, nw > 0 ? next.o0 : cur.o0, lane, s);
    for (int i = 0; i < nw; i++) {
        const Window after = w[min(i + 2, nw)];
        s1.cam = -1;
        if (i + 1 < nw) read_slot(a, pt_obs, next, after.o0, lane, s1);
        const int cnt = next.o0 - cur.o0;
        double v[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        if (cur.heads != 0) {
            take(s, v);
            const Segment g = segment_of(cur.heads, cnt, lane);
            seg_sum(v, lane, g.head);
            if (lane < cnt && lane == g.tail) write_point(a, s.k, v, pt);
        } else {
            for (int j = lane; j < cnt; j += kWave) {
                Slot l;
                read_pixel(a, pt_obs, cur.o0 + j, cur.k0, l);
                take(l, v);
            }
#pragma unroll
            for (int e = 0; e < 9; e++)
                for (int off = 32; off > 0; off >>= 1) v[e] += __shfl_xor(v[e], off, kWave);
            if (lane == 0) write_point(a, cur.k0, v, pt);
        }
        cur = next;
        next = after;
        s = s1;
    }
    double v[2] = {cost, masked};
    block_sum<2>(v, s_red);
    if (threadIdx.x == 0) {
        if (v[0] != 0.0) atomicAdd(&sc[sCost], v[0]);
        if (v[1] != 0.0) atomicAdd(&sc[sMasked], v[1]);
    }
}

// A point's row and its pixel as k_ba_cams reads them, an observation ahead.
struct BaRow {
    bool any;
    float2 xy;
    float X[3];
    double q[9];
};

__device__ __forceinline__ void read_row(const BaObs& a, const double* __restrict__ pt, int k, int o, BaRow& r) {
    r.any = k >= 0 && k < a.Pt;
    if (!r.any) return;
    const double* q = pt + 6 * (int64_t)a.Pt + kRow * (int64_t)k;
#pragma unroll
    for (int i = 0; i < 9; i++) r.q[i] = q[i];
    const float* x = reinterpret_cast<const float*>(q + 9);
#pragma unroll
    for (int i = 0; i < 3; i++) r.X[i] = x[i];
    r.xy = make_float2(a.obs_xy[2 * (int64_t)o], a.obs_xy[2 * (int64_t)o + 1]);
}

// per camera (one workgroup): U (damped), S_ii = U - sum W V^-1 W' and its
// Cholesky factor, b = -g_c + sum W V^-1 g_X
__global__ __launch_bounds__(kBlock) void k_ba_cams(BaObs a, const int32_t* __restrict__ cam_off,
                                                    const double* __restrict__ pt,
                                                    double* __restrict__ cam, bool planar) {
    __shared__ double s_red[(kBlock / kWave) * 54];
    const int c = blockIdx.x;
    const CamData cam_c = load_cam(a, c);
    double v[54];  // U (21), corr (21), g_c (6), W V^-1 g_X (6)
#pragma unroll
    for (int j = 0; j < 54; j++) v[j] = 0.0;
    const int end = cam_off[c + 1];
    int o = cam_off[c] + threadIdx.x;
    BaRow row, next;
    int k1 = o + kBlock < end ? a.obs_pt[o + kBlock] : -1;  // two ahead: the row's index
    read_row(a, pt, o < end ? a.obs_pt[o] : -1, o, next);
    for (; o < end; o += kBlock) {
        row = next;
        read_row(a, pt, k1, o + kBlock, next);
        k1 = o + 2 * kBlock < end ? a.obs_pt[o + 2 * kBlock] : -1;
        if (!row.any) continue;
        const double* q = row.q;
        const double* vg = row.q + 6;
        Lin L;
        linearise(a, cam_c, row.X[0], row.X[1], row.X[2], row.xy, L);
        if (!L.ok) continue;
        // M2 = J_X V^-1 J_X' (2x2), e = J_X V^-1 g_X (2)
        double JV[2][3];
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const double* J = L.Jx + 3 * r;
            JV[r][0] = J[0] * q[0] + J[1] * q[1] + J[2] * q[2];
            JV[r][1] = J[0] * q[1] + J[1] * q[3] + J[2] * q[4];
            JV[r][2] = J[0] * q[2] + J[1] * q[4] + J[2] * q[5];
        }
        const double m00 = JV[0][0] * L.Jx[0] + JV[0][1] * L.Jx[1] + JV[0][2] * L.Jx[2];
        const double m01 = JV[0][0] * L.Jx[3] + JV[0][1] * L.Jx[4] + JV[0][2] * L.Jx[5];
        const double m11 = JV[1][0] * L.Jx[3] + JV[1][1] * L.Jx[4] + JV[1][2] * L.Jx[5];
        const double e0 = L.Jx[0] * vg[0] + L.Jx[1] * vg[1] + L.Jx[2] * vg[2];
        const double e1 = L.Jx[3] * vg[0] + L.Jx[4] * vg[1] + L.Jx[5] * vg[2];
        const double w2 = L.w * L.w;
#pragma unroll
        for (int i = 0; i < 6; i++) {
            const double pi0 = L.Jp[i], pi1 = L.Jp[6 + i];
#pragma unroll
            for (int j = 0; j <= i; j++) {
                const double pj0 = L.Jp[j], pj1 = L.Jp[6 + j];
                v[tri6(i, j)] += L.w * (pi0 * pj0 + pi1 * pj1);
                v[21 + tri6(i, j)] += w2 * (pi0 * (m00 * pj0 + m01 * pj1) + pi1 * (m01 * pj0 + m11 * pj1));
            }
            v[42 + i] += L.w * (pi0 * L.r0 + pi1 * L.r1);
            v[48 + i] += L.w * (pi0 * e0 + pi1 * e1);
        }
    }
    block_sum<54>(v, s_red);
    if (threadIdx.x != 0) return;
    const int n = a.n_cams;
    bool live = false;
#pragma unroll
    for (int i = 0; i < 6; i++) live |= v[tri6(i, i)] > 0.0;
    double S[21];
#pragma unroll
    for (int i = 0; i < 6; i++) v[tri6(i, i)] *= 1.0 + a.lambda;
#pragma unroll
    for (int e = 0; e < 21; e++) {
        cam[(int64_t)e * n + c] = v[e];
        S[e] = v[e] - v[21 + e];
    }
    // Cholesky S = L L' (lower, packed like the matrix); a camera with no
    // observation (or a block that is not positive) is held fixed: L = 0
    bool ok = live;
    for (int i = 0; i < 6 && ok; i++) {
        for (int j = 0; j <= i; j++) {
            double sum = S[tri6(i, j)];
            for (int m = 0; m < j; m++) sum -= S[tri6(i, m)] * S[tri6(j, m)];
            if (i == j) {
                if (!(sum > 0.0)) {
                    ok = false;
                    break;
                }
                S[tri6(i, i)] = 1.0 / sqrt(sum);
            } else {
                S[tri6(i, j)] = sum * S[tri6(j, j)];
            }
        }
    }
    double* l = cam + off_l(n);
#pragma unroll
    for (int e = 0; e < 21; e++) l[(int64_t)e * n + c] = ok ? S[e] : 0.0;
    double* r = cam + off_vec(n, vR);
    double* ap = cam + off_vec(n, vAp);
#pragma unroll
    for (int i = 0; i < 6; i++) {
        const int64_t e = planar ? (int64_t)i * n + c : 6 * (int64_t)c + i;
        r[e] = ok ? -v[42 + i] + v[48 + i] : 0.0;  // b, the first residual
        ap[e] = 0.0;                               // k_ba_cg adds into it
    }
}

// z = (L L')^-1 r of a camera (0 for a fixed one), reciprocals on L's diagonal
__device__ __forceinline__ void precond(const double (&L)[21], const double (&r)[6], double (&z)[6]) {
#pragma unroll
    for (int i = 0; i < 6; i++) {
        double s = r[i];
#pragma unroll
        for (int m = 0; m < i; m++) s -= L[tri6(i, m)] * z[m];
        z[i] = s * L[tri6(i, i)];
    }
#pragma unroll
    for (int i = 5; i >= 0; i--) {
        double s = z[i];
#pragma unroll
        for (int m = i + 1; m < 6; m++) s -= L[tri6(m, i)] * z[m];
        z[i] = s * L[tri6(i, i)];
    }
}

__device__ __forceinline__ void load_l(const double* l, int n, double (&L)[21]) {
#pragma unroll
    for (int e = 0; e < 21; e++) L[e] = l[(int64_t)e * n];
}

__device__ __forceinline__ double block_dot(double v, double* s) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    __syncthreads();
    if (lane == 0) s[w] = v;
    __syncthreads();
    double t = 0.0;
    for (int q = 0; q < kVec / kWave; q++) t += s[q];
    return t;
}

// two dot products at once (s: 2 kVec / kWave words, not in use before)
__device__ __forceinline__ void block_dot2(double& v, double& w, double* s) {
    for (int off = 32; off > 0; off >>= 1) {
        v += __shfl_xor(v, off, kWave);
        w += __shfl_xor(w, off, kWave);
    }
    constexpr int kW = kVec / kWave;
    if (threadIdx.x % kWave == 0) {
        s[threadIdx.x / kWave] = v;
        s[kW + threadIdx.x / kWave] = w;
    }
    __syncthreads();
    v = w = 0.0;
    for (int q = 0; q < kW; q++) {
        v += s[q];
        w += s[kW + q];
    }
}

// x = 0, r = b, z = P r, p = z
__global__ __launch_bounds__(kVec) void k_ba_pcg_init(int n_cams, double* __restrict__ cam,
                                                      double* __restrict__ sc) {
    __shared__ double s[kVec / kWave];
    double rz = 0.0, bb = 0.0;
    for (int c = threadIdx.x; c < n_cams; c += kVec) {
        double r[6], z[6], L[21];
#pragma unroll
        for (int i = 0; i < 6; i++) r[i] = cam[off_vec(n_cams, vR) + 6 * (int64_t)c + i];
        load_l(cam + off_l(n_cams) + c, n_cams, L);
        precond(L, r, z);
#pragma unroll
        for (int i = 0; i < 6; i++) {
            cam[off_vec(n_cams, vX) + 6 * (int64_t)c + i] = 0.0;
            cam[off_vec(n_cams, vP) + 6 * (int64_t)c + i] = z[i];
            rz += r[i] * z[i];
            bb += r[i] * r[i];
        }
    }
    rz = block_dot(rz, s);
    bb = block_dot(bb, s);
    if (threadIdx.x == 0) {
        sc[sRZ] = rz;
        sc[sBB] = bb;
        sc[sRR] = bb;
        sc[sIt] = 0.0;
        sc[sDone] = (bb > 0.0 && !(sc[sUnsorted] > 0.0)) ? 0.0 : 1.0;
    }
}

// u_k = V_k^-1 sum_o W_o' src_cam(o)   (src: the camera vector)
__global__ __launch_bounds__(kBlock) void k_ba_pt_apply(BaObs a, const int32_t* __restrict__ pt_off,
                                                        const int32_t* __restrict__ pt_obs,
                                                        const double* __restrict__ src,
                                                        double* __restrict__ pt,
                                                        const double* __restrict__ sc, int force) {
    if (!force && sc[sDone] > 0.0) return;
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k >= a.Pt) return;
    double t[3] = {0, 0, 0};
    for (int j = pt_off[k]; j < pt_off[k + 1]; j++) {
        const int o = pt_obs ? pt_obs[j] : j;  // no index: the arrays are point-major
        const int ci = a.obs_cam[o];
        if (ci < 0 || ci >= a.n_cams) continue;
        Lin L;
        linearise(a, o, ci, k, L);
        if (!L.ok) continue;
        const double* x = src + 6 * (int64_t)ci;
        double jp0 = 0.0, jp1 = 0.0;
#pragma unroll
        for (int i = 0; i < 6; i++) {
            jp0 += L.Jp[i] * x[i];
            jp1 += L.Jp[6 + i] * x[i];
        }
#pragma unroll
        for (int c = 0; c < 3; c++) t[c] += L.w * (L.Jx[c] * jp0 + L.Jx[3 + c] * jp1);
    }
    const double* q = pt + 6 * (int64_t)k;
    double* u = pt + 6 * (int64_t)a.Pt + kRow * (int64_t)k + 9;
    u[0] = q[0] * t[0] + q[1] * t[1] + q[2] * t[2];
    u[1] = q[1] * t[0] + q[3] * t[1] + q[4] * t[2];
    u[2] = q[2] * t[0] + q[4] * t[1] + q[5] * t[2];
}

// Ap_c = U_c p_c - sum_o W_o u_k(o)   (one workgroup per camera)
__global__ __launch_bounds__(kBlock) void k_ba_cam_apply(BaObs a, const int32_t* __restrict__ cam_off,
                                                         const double* __restrict__ pt,
                                                         double* __restrict__ cam,
                                                         const double* __restrict__ sc) {
    __shared__ double s_red[(kBlock / kWave) * 6];
    if (sc[sDone] > 0.0) return;
    const int c = blockIdx.x;
    double v[6] = {0, 0, 0, 0, 0, 0};
    for (int o = cam_off[c] + threadIdx.x; o < cam_off[c + 1]; o += kBlock) {
        const int k = a.obs_pt[o];
        if (k < 0 || k >= a.Pt) continue;
        Lin L;
        linearise(a, o, c, k, L);
        if (!L.ok) continue;
        const double* u = pt + 6 * (int64_t)a.Pt + kRow * (int64_t)k + 9;
        const double e0 = L.Jx[0] * u[0] + L.Jx[1] * u[1] + L.Jx[2] * u[2];
        const double e1 = L.Jx[3] * u[0] + L.Jx[4] * u[1] + L.Jx[5] * u[2];
#pragma unroll
        for (int i = 0; i < 6; i++) v[i] -= L.w * (L.Jp[i] * e0 + L.Jp[6 + i] * e1);
    }
    block_sum<6>(v, s_red);
    if (threadIdx.x != 0) return;
    const int n = a.n_cams;
    const bool live = cam[off_l(n) + c] > 0.0;
    const double* pc = cam + off_vec(n, vP) + 6 * (int64_t)c;
#pragma unroll
    for (int i = 0; i < 6; i++) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < 6; j++) s += cam[(int64_t)tri6(i, j) * n + c] * pc[j];
        cam[off_vec(n, vAp) + 6 * (int64_t)c + i] = live ? s + v[i] : 0.0;
    }
}

// one conjugate-gradient update; sets the done flag on convergence
__global__ __launch_bounds__(kVec) void k_ba_pcg_update(int n_cams, double* __restrict__ cam,
                                                        double* __restrict__ sc, double tol2) {
    __shared__ double s[kVec / kWave];
    if (sc[sDone] > 0.0) return;
    double* x = cam + off_vec(n_cams, vX);
    double* r = cam + off_vec(n_cams, vR);
    double* z = cam + off_vec(n_cams, vZ);
    double* p = cam + off_vec(n_cams, vP);
    const double* ap = cam + off_vec(n_cams, vAp);
    const int n6 = 6 * n_cams;
    double pap = 0.0;
    for (int i = threadIdx.x; i < n6; i += kVec) pap += p[i] * ap[i];
    pap = block_dot(pap, s);
    const double rz = sc[sRZ];
    const double alpha = pap > 0.0 ? rz / pap : 0.0;
    double rr = 0.0, rz1 = 0.0;
    for (int c = threadIdx.x; c < n_cams; c += kVec) {
        double rc[6], zc[6], L[21];
#pragma unroll
        for (int i = 0; i < 6; i++) {
            const int64_t e = 6 * (int64_t)c + i;
            x[e] += alpha * p[e];
            rc[i] = r[e] - alpha * ap[e];
            r[e] = rc[i];
            rr += rc[i] * rc[i];
        }
        load_l(cam + off_l(n_cams) + c, n_cams, L);
        precond(L, rc, zc);
#pragma unroll
        for (int i = 0; i < 6; i++) {
            z[6 * (int64_t)c + i] = zc[i];
            rz1 += rc[i] * zc[i];
        }
    }
    rr = block_dot(rr, s);
    rz1 = block_dot(rz1, s);
    const bool done = !(pap > 0.0) || rr <= tol2 * sc[sBB];
    if (!done) {
        const double beta = rz > 0.0 ? rz1 / rz : 0.0;
        for (int c = threadIdx.x; c < n_cams; c += kVec)
#pragma unroll
            for (int i = 0; i < 6; i++) {
                const int64_t e = 6 * (int64_t)c + i;
                p[e] = z[e] + beta * p[e];
            }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        sc[sIt] += 1.0;
        sc[sRR] = rr;
        sc[sRZ] = rz1;
        if (done) sc[sDone] = 1.0;
    }
}

// The conjugate-gradient state a workgroup of k_ba_cg holds: thread c keeps
// camera c's rows (n_cams <= the workgroup).
struct Cg {
    double x[6], p[6];  // x is formed only where `with_x` asks for it
    double rr, bb, its;
    bool done;
};

// The update that ends iteration it - 1 and opens iteration `it`: from A p of
// the last iteration to the new r, z and p (it = 0: r = b, p = z).  Every
// workgroup computes it for itself, in the same order, so all agree without a
// grid-wide wait; workgroup 0 stores it.  Vectors that one launch reads and
// another workgroup of it writes alternate between two buffers, A p between
// three (read, added into, cleared for the next).
__device__ __forceinline__ void cg_open(int it, int n, double* __restrict__ cam, double* __restrict__ sc,
                                        double tol2, double* s_red, bool with_x, Cg& g) {
    const int c = threadIdx.x;
    const bool mine = c < n, first = blockIdx.x == 0;
    double r[6] = {0, 0, 0, 0, 0, 0}, z[6] = {0, 0, 0, 0, 0, 0}, pp[6] = {0, 0, 0, 0, 0, 0};
    double rz = 0.0, alpha = 0.0, pap = 0.0, L[21];
    if (mine) load_l(cam + off_l(n) + c, n, L);
    if (it == 0) {
        if (mine)
#pragma unroll
            for (int i = 0; i < 6; i++) r[i] = cam[off_vec(n, vR) + (int64_t)i * n + c];
    } else {
        const int q = (it - 1) & 1, w = (it - 1) % 3;
        double ap[6] = {0, 0, 0, 0, 0, 0};
        if (mine) {
            const bool live = L[0] > 0.0;
#pragma unroll
            for (int i = 0; i < 6; i++) {
                r[i] = cam[off_vec(n, vR + q) + (int64_t)i * n + c];
                pp[i] = cam[off_vec(n, vP + q) + (int64_t)i * n + c];
                ap[i] = live ? cam[off_vec(n, vAp + w) + (int64_t)i * n + c] : 0.0;
            }
        }
        pap = sc[sPap + w];
        rz = sc[sRZ + q];
        alpha = pap > 0.0 ? rz / pap : 0.0;
#pragma unroll
        for (int i = 0; i < 6; i++) r[i] -= alpha * ap[i];
    }
    double rr = 0.0, rz1 = 0.0;
    if (mine) {
        precond(L, r, z);
#pragma unroll
        for (int i = 0; i < 6; i++) {
            rr += r[i] * r[i];
            rz1 += r[i] * z[i];
        }
    }
    block_dot2(rr, rz1, s_red);
    const double bb = it == 0 ? rr : sc[sBB];
    const bool done = it == 0 ? !(bb > 0.0) || sc[sUnsorted] > 0.0 : !(pap > 0.0) || rr <= tol2 * bb;
    const double beta = it > 0 && rz > 0.0 ? rz1 / rz : 0.0;
#pragma unroll
    for (int i = 0; i < 6; i++) g.p[i] = z[i] + beta * pp[i];
    if (mine && (with_x || first)) {
#pragma unroll
        for (int i = 0; i < 6; i++)
            g.x[i] = it == 0 ? 0.0 : cam[off_vec(n, vX) + (int64_t)i * n + c] + alpha * pp[i];
    }
    g.rr = rr;
    g.bb = bb;
    g.its = it;
    g.done = done;
    if (with_x || !first) return;  // the last launch stores the step itself
    if (mine) {
#pragma unroll
        for (int i = 0; i < 6; i++) {
            cam[off_vec(n, vX) + (int64_t)i * n + c] = g.x[i];
            if (it > 0) cam[off_vec(n, vR + (it & 1)) + (int64_t)i * n + c] = r[i];
            cam[off_vec(n, vP + (it & 1)) + (int64_t)i * n + c] = g.p[i];
            cam[off_vec(n, vAp + (it + 1) % 3) + (int64_t)i * n + c] = 0.0;
        }
    }
    if (threadIdx.x == 0) {
        sc[sRZ + (it & 1)] = rz1;
        sc[sPap + (it + 1) % 3] = 0.0;
        if (it == 0) sc[sBB] = bb;
        sc[sRR] = rr;
        sc[sIt] = (double)it;
        sc[sEnd + (it & 1)] = done ? 1.0 : 0.0;
    }
}

// q = [I | -[p]x] x
__device__ __forceinline__ void twist_at(const Proj& P, const double* x, double (&q)[3]) {
    q[0] = x[0] + x[4] * P.p[2] - x[5] * P.p[1];
    q[1] = x[1] + x[5] * P.p[0] - x[3] * P.p[2];
    q[2] = x[2] + x[3] * P.p[1] - x[4] * P.p[0];
}

// h = w J_pi' J_pi q
__device__ __forceinline__ void weigh(const Proj& P, const double (&q)[3], double (&h)[3]) {
    const double e0 = P.w * (P.a00 * q[0] + P.a02 * q[2]);
    const double e1 = P.w * (P.a11 * q[1] + P.a12 * q[2]);
    h[0] = P.a00 * e0;
    h[1] = P.a11 * e1;
    h[2] = P.a02 * e0 + P.a12 * e1;
}

// the point's part of an observation's product: R' h, h from the camera's x
__device__ __forceinline__ void to_point(const Proj& P, const double* x, double (&t)[3]) {
    double q[3], h[3];
    twist_at(P, x, q);
    weigh(P, q, h);
#pragma unroll
    for (int i = 0; i < 3; i++) t[i] = P.R[i] * h[0] + P.R[3 + i] * h[1] + P.R[6 + i] * h[2];
}

// the camera's part: -(h, p x h), h from the point's u, added to its sums
// (n apart)
__device__ __forceinline__ void to_camera(const Proj& P, const double (&u)[3], double* v, int n) {
    double q[3], h[3];
#pragma unroll
    for (int i = 0; i < 3; i++) q[i] = P.R[3 * i] * u[0] + P.R[3 * i + 1] * u[1] + P.R[3 * i + 2] * u[2];
    weigh(P, q, h);
    atomicAdd(&v[0], -h[0]);
    atomicAdd(&v[n], -h[1]);
    atomicAdd(&v[2 * n], -h[2]);
    atomicAdd(&v[3 * n], P.p[2] * h[1] - P.p[1] * h[2]);
    atomicAdd(&v[4 * n], P.p[0] * h[2] - P.p[2] * h[0]);
    atomicAdd(&v[5 * n], P.p[1] * h[0] - P.p[0] * h[1]);
}

__device__ __forceinline__ void solve_point(const double* q, double (&t)[3]) {
    const double t0 = t[0], t1 = t[1], t2 = t[2];
    t[0] = q[0] * t0 + q[1] * t1 + q[2] * t2;
    t[1] = q[1] * t0 + q[3] * t1 + q[4] * t2;
    t[2] = q[2] * t0 + q[4] * t1 + q[5] * t2;
}

__device__ __forceinline__ void write_dx(const BaObs& a, const double* __restrict__ pt, int k,
                                         const double (&u)[3], bool bad, float* __restrict__ d_X) {
    const double* g = pt + 6 * (int64_t)a.Pt + kRow * (int64_t)k + 6;
#pragma unroll
    for (int i = 0; i < 3; i++) d_X[3 * (int64_t)k + i] = bad ? 0.f : (float)(-(g[i] + u[i]));
}

// a point of more than 64 observations, 64 at a time: once for u, once for the
// cameras
template <bool LAST>
__device__ __forceinline__ void long_point(const BaObs& a, const int32_t* __restrict__ pt_obs,
                                        const double* __restrict__ pt, const float4* s_cam,
                                        const double* s_vec, double* s_acc, int k, int o0, int o1, bool bad,
                                        float* __restrict__ d_X, double& quad) {
    const int lane = threadIdx.x % kWave;
    double t[3] = {0.0, 0.0, 0.0};
    for (int walk = 0; walk < (LAST ? 1 : 2); walk++) {
        for (int j = o0 + lane; j < o1; j += kWave) {
            Slot s;
            read_pixel(a, pt_obs, j, k, s);
            if (s.cam < 0) continue;
            const int c = s.cam;
            Proj P;
            project(a, lds_cam(s_cam, c), s.X[0], s.X[1], s.X[2], s.xy, P);
            if (!P.ok) continue;
            if (walk == 0) {
                double y[3];
                to_point(P, s_vec + 6 * c, y);
#pragma unroll
                for (int i = 0; i < 3; i++) t[i] += y[i];
            } else {
                to_camera(P, t, s_acc + c, a.n_cams);
            }
        }
        if (walk == 0) {
#pragma unroll
            for (int i = 0; i < 3; i++)
                for (int off = 32; off > 0; off >>= 1) t[i] += __shfl_xor(t[i], off, kWave);
            const double y[3] = {t[0], t[1], t[2]};
            solve_point(pt + 6 * (int64_t)k, t);
            if (lane == 0) quad += y[0] * t[0] + y[1] * t[1] + y[2] * t[2];
            if (LAST && lane == 0) write_dx(a, pt, k, t, bad, d_X);
        }
    }
}

// One conjugate-gradient iteration in one launch: the update of the last one
// (cg_open), then A p = U p - sum W_o u_k in one pass over the observations by
// point.  A lane takes one observation of a window: its product with p is
// summed over the point's lanes, u_k = V_k^-1 times that sum, and W_o u_k goes
// to the camera's sum, so an observation is projected once and every array is
// read in order, the next window's part while this one is computed.  The
// cameras' poses, p and the sums sit in LDS (160 B a camera; one workgroup
// fills a CU), and the sums leave by one double atomic per camera entry and
// workgroup.  Bound by the double-precision arithmetic: about 300 instructions
// per 64 observations.
// 1000 cameras and 6.5M observations: 106 us an iteration (13 of them the update); 390 as a
// pass by point (one thread per point, 31% of lanes active), a pass by camera
// (each observation gathering X and u of a random point) and an update kernel;
// 200 with a thread walking its points' observations twice, once for u and
// once for the cameras.
// LAST: x of the last update, then d_twist = x, d_X = -(V^-1 g_X + u(x)) and
// the statistics.
template <bool LAST>
__global__ __launch_bounds__(kVec) void k_ba_cg(BaObs a, const int32_t* __restrict__ pt_off,
                                                const int32_t* __restrict__ pt_obs,
                                                const double* __restrict__ pt, double* __restrict__ cam,
                                                const Window* __restrict__ win,
                                                const int32_t* __restrict__ n_win, double* __restrict__ sc,
                                                int it, double tol2, float* __restrict__ d_twist,
                                                float* __restrict__ d_X, float* __restrict__ stats) {
    extern __shared__ double s_dyn[];
    const int n = a.n_cams;
    double* s_red = s_dyn;                                // [2 kVec / kWave]
    double* s_vec = s_dyn + kLdsFixed / 8;                // [n][6]: p, or x in the last launch
    double* s_acc = s_vec + 6 * n;                        // [6][n]: sum of W u
    float4* s_cam = reinterpret_cast<float4*>(s_acc + (LAST ? 0 : 6 * n));  // [n][4]
    const int tid = threadIdx.x;
    // whether an earlier launch found the end: a word that no workgroup of this
    // launch writes, so all waves of all workgroups see the same
    const bool ended = it > 0 && sc[sEnd + ((it - 1) & 1)] > 0.0;
    if (!LAST && ended) {
        if (blockIdx.x == 0 && tid == 0) sc[sEnd + (it & 1)] = 1.0;
        return;
    }
    if (tid < n) {
        const CamData cd = load_cam(a, tid);
#pragma unroll
        for (int q = 0; q < 4; q++) s_cam[cam_slot(tid, q)] = cd.q[q];
    }
    Cg g;
    if (LAST && ended) {
        g.done = true;
        g.rr = sc[sRR];
        g.bb = sc[sBB];
        g.its = sc[sIt];
        if (tid < n)
#pragma unroll
            for (int i = 0; i < 6; i++) g.x[i] = cam[off_vec(n, vX) + (int64_t)i * n + tid];
    } else {
        cg_open(it, n, cam, sc, tol2, s_red, LAST, g);
        if (!LAST && g.done) return;
    }
    const bool bad = sc[sUnsorted] > 0.0;
    double pup = 0.0;  // p' U p of this thread's camera
    if (tid < n) {
        const double* w = LAST ? g.x : g.p;
#pragma unroll
        for (int i = 0; i < 6; i++) s_vec[6 * tid + i] = w[i];
        if (!LAST) {
            // U p of the cameras dealt to this workgroup, 0 for the others
            const bool own = tid % (int)gridDim.x == (int)blockIdx.x;
#pragma unroll
            for (int i = 0; i < 6; i++) {
                double s = 0.0;
                if (own)
#pragma unroll
                    for (int j = 0; j < 6; j++) s += cam[(int64_t)tri6(i, j) * n + tid] * g.p[j];
                s_acc[i * n + tid] = s;
                pup += s * g.p[i];
            }
        } else if (blockIdx.x == 0) {
#pragma unroll
            for (int i = 0; i < 6; i++) d_twist[6 * tid + i] = bad ? 0.f : (float)g.x[i];
        }
    }
    if (LAST && blockIdx.x == 0 && tid == 0 && stats) {
        stats[0] = (float)g.its;
        stats[1] = g.bb > 0.0 ? (float)sqrt(g.rr / g.bb) : 0.f;
        stats[2] = (float)sc[sCost];
        stats[3] = (float)sc[sMasked];
        stats[4] = bad ? 1.f : 0.f;
    }
    __syncthreads();
    const int lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane((int)blockIdx.x * (kVec / kWave) + tid / kWave);
    int kb, ke;
    wave_share(a.Pt, wave, (int64_t)gridDim.x * (kVec / kWave), kb, ke);
    if (LAST) {  // points without observations are in no window
        const double zero[3] = {0.0, 0.0, 0.0};
        for (int k = kb + lane; k < ke; k += kWave)
            if (pt_off[k] == pt_off[k + 1]) write_dx(a, pt, k, zero, bad, d_X);
    }
    const Window* w = win + kb + wave;
    const int nw = n_win[wave];
    Window cur = w[0], next = w[min(1, nw)];
    bool any_long = false;
    double quad = 0.0;  // this lane's share of p' W V^-1 W' p
    Slot s, s1;
    double Vi[6], Vi1[6];
    auto read = [&](const Window& x, int o1, Slot& s, double (&Vi)[6]) {
        read_slot(a, pt_obs, x, o1, lane, s);
        if (x.heads != 0 && x.o0 + lane < o1)
#pragma unroll
            for (int e = 0; e < 6; e++) Vi[e] = pt[6 * (int64_t)s.k + e];
    };
    read(cur, nw > 0 ? next.o0 : cur.o0, s, Vi);
    for (int i = 0; i < nw; i++) {
        const Window after = w[min(i + 2, nw)];
        s1.cam = -1;
        if (i + 1 < nw) read(next, after.o0, s1, Vi1);
        if (cur.heads == 0) {
            any_long = true;
        } else {
            Proj P;
            P.ok = false;
            if (s.cam >= 0) project(a, lds_cam(s_cam, s.cam), s.X[0], s.X[1], s.X[2], s.xy, P);
            double y[3] = {0.0, 0.0, 0.0};
            if (P.ok) to_point(P, s_vec + 6 * s.cam, y);
            double t[3] = {y[0], y[1], y[2]};
            const int cnt = next.o0 - cur.o0;
            const Segment g = segment_of(cur.heads, cnt, lane);
            seg_sum(t, lane, g.head);
            if (LAST) {
                if (lane < cnt && lane == g.tail) {
                    solve_point(Vi, t);
                    write_dx(a, pt, s.k, t, bad, d_X);
                }
            } else {
#pragma unroll
                for (int i = 0; i < 3; i++) t[i] = __shfl(t[i], g.tail, kWave);
                if (P.ok) {
                    double u[3] = {t[0], t[1], t[2]};
                    solve_point(Vi, u);
                    to_camera(P, u, s_acc + s.cam, n);
                    // this lane's share of p' W V^-1 W' p: y = its own product
                    quad += y[0] * u[0] + y[1] * u[1] + y[2] * u[2];
                }
            }
        }
        cur = next;
        next = after;
        s = s1;
#pragma unroll
        for (int e = 0; e < 6; e++) Vi[e] = Vi1[e];
    }
    if (any_long)
        for (int i = 0; i < nw; i++)
            if (w[i].heads == 0)
                long_point<LAST>(a, pt_obs, pt, s_cam, s_vec, s_acc, w[i].k0, w[i].o0, w[i + 1].o0, bad, d_X, quad);
    if (LAST) return;
    // p' A p: the points' part and, of this workgroup's cameras, p' U p
    quad = block_dot(pup - quad, s_red);  // its barriers also end the sums
    if (tid == 0) atomicAdd(&sc[sPap + it % 3], quad);
    double* ap = cam + off_vec(n, vAp + it % 3);
    const int n6 = 6 * n;
    const int start = (int)((int64_t)n6 * blockIdx.x / gridDim.x);  // workgroups begin at unlike entries
    for (int i = tid; i < n6; i += kVec) {
        const int e = i + start < n6 ? i + start : i + start - n6;
        if (s_acc[e] != 0.0) atomicAdd(&ap[e], s_acc[e]);
    }
}

// the step of the two-pass path: d_twist = x, d_X = -(V^-1 g_X + u(x)); statistics
__global__ __launch_bounds__(kBlock) void k_ba_finish(int n_cams, int Pt, const double* __restrict__ cam,
                                                      const double* __restrict__ pt,
                                                      const double* __restrict__ sc,
                                                      float* __restrict__ d_twist, float* __restrict__ d_X,
                                                      float* __restrict__ stats) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const bool bad = sc[sUnsorted] > 0.0;
    if (i < 6 * n_cams) d_twist[i] = bad ? 0.f : (float)cam[off_vec(n_cams, vX) + i];
    if (i < 3 * Pt) {
        const double* q = pt + 6 * (int64_t)Pt + kRow * (int64_t)(i / 3);
        d_X[i] = bad ? 0.f : (float)(-(q[6 + i % 3] + q[9 + i % 3]));
    }
    if (i == 0 && stats) {
        stats[0] = (float)sc[sIt];
        stats[1] = sc[sBB] > 0.0 ? (float)sqrt(sc[sRR] / sc[sBB]) : 0.f;
        stats[2] = (float)sc[sCost];
        stats[3] = (float)sc[sMasked];
        stats[4] = bad ? 1.f : 0.f;
    }
}

__global__ void k_ba_clear(double* __restrict__ sc) {
    if (threadIdx.x < 16) sc[threadIdx.x] = 0.0;
}

}  // namespace

hipError_t launch_ba_step(gs_ba* ba, const BaInputs& in, float* d_twist, float* d_X, float* stats,
                          hipStream_t st) {
    BaObs a;
    a.X = in.X;
    a.viewmat = in.viewmat;
    a.intr = in.intr;
    a.cams = reinterpret_cast<float4*>(ba->cam + off_vec(in.n_cams, vCams));
    a.obs_cam = in.obs_cam;
    a.obs_pt = in.obs_pt;
    a.obs_xy = in.obs_xy;
    a.Pt = in.Pt;
    a.n_cams = in.n_cams;
    a.M = in.M;
    a.delta = in.delta;
    a.near_plane = in.near_plane;
    a.lambda = in.lambda;
    // the point passes read the point-major copies in order when there are
    // some (no index then), else the caller's arrays through the index
    BaObs ap = a;
    const int32_t* pidx = in.pt_obs;
    if (in.pm_cam && in.pm_xy) {
        ap.obs_cam = in.pm_cam;
        ap.obs_xy = in.pm_xy;
        pidx = nullptr;
    }
    const unsigned gp = (unsigned)std::max((in.Pt + kBlock - 1) / kBlock, 1);
    // the passes by window: equal shares of the points, at least a wave's worth
    const unsigned wg = (unsigned)std::min(std::max((in.Pt + kWave - 1) / kWave, 1), kCgBlocks);
    int32_t* n_win = static_cast<int32_t*>(ba->win);
    Window* win = reinterpret_cast<Window*>(n_win + kCgWaves);
    const bool fused = in.n_cams > 0 && in.n_cams <= ba->lds_cams;  // the rule is at k_ba_cg below
    const unsigned gr = (unsigned)std::min(std::max((std::max(in.M, in.n_cams + 1) + kBlock - 1) / kBlock, 1), 4096);
    hipLaunchKernelGGL(k_ba_clear, dim3(1), dim3(64), 0, st, ba->sc);
    hipLaunchKernelGGL(k_ba_ranges, dim3(gr), dim3(kBlock), 0, st, a, ba->cam_off, ba->sc);
    hipLaunchKernelGGL(k_ba_windows, dim3(wg * (kVec / kWave)), dim3(kWave), 0, st, in.Pt, in.pt_off, win, n_win);
    hipLaunchKernelGGL(k_ba_points, dim3(wg * (kVec / kBlock)), dim3(kBlock), 0, st, ap, in.pt_off, pidx, win,
                       n_win, ba->pt, ba->sc);
    if (in.n_cams > 0)
        hipLaunchKernelGGL(k_ba_cams, dim3(in.n_cams), dim3(kBlock), 0, st, a, ba->cam_off, ba->pt, ba->cam, fused);
    const double tol2 = (double)in.tol * (double)in.tol;
    // The one-pass path wherever the cameras fit the LDS (1022 of them in 160
    // KB): 1000 cameras and 6.5M observations, 21 iterations of at most 100,
    // took 2.56 ms a step against 8.8 on two passes; 150 cameras and 430k
    // observations 594 us against 1510, of which the launches after
    // convergence are 185 (2.3 us each, whatever their grid).
    if (fused) {
        const size_t lds = kLdsFixed + (size_t)kLdsPerCam * in.n_cams;
        for (int it = 0; it < in.max_iter; it++)
            hipLaunchKernelGGL(k_ba_cg<false>, dim3(wg), dim3(kVec), lds, st, ap, in.pt_off, pidx, ba->pt,
                               ba->cam, win, n_win, ba->sc, it, tol2, d_twist, d_X, stats);
        hipLaunchKernelGGL(k_ba_cg<true>, dim3(wg), dim3(kVec), lds, st, ap, in.pt_off, pidx, ba->pt, ba->cam,
                           win, n_win, ba->sc, in.max_iter, tol2, d_twist, d_X, stats);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_ba_pcg_init, dim3(1), dim3(kVec), 0, st, in.n_cams, ba->cam, ba->sc);
    for (int it = 0; it < in.max_iter; it++) {
        hipLaunchKernelGGL(k_ba_pt_apply, dim3(gp), dim3(kBlock), 0, st, ap, in.pt_off, pidx,
                           ba->cam + off_vec(in.n_cams, vP), ba->pt, ba->sc, 0);
        if (in.n_cams > 0)
            hipLaunchKernelGGL(k_ba_cam_apply, dim3(in.n_cams), dim3(kBlock), 0, st, a, ba->cam_off, ba->pt,
                               ba->cam, ba->sc);
        hipLaunchKernelGGL(k_ba_pcg_update, dim3(1), dim3(kVec), 0, st, in.n_cams, ba->cam, ba->sc, tol2);
    }
    // back-substitution for the points with the final camera step
    hipLaunchKernelGGL(k_ba_pt_apply, dim3(gp), dim3(kBlock), 0, st, ap, in.pt_off, pidx,
                       ba->cam + off_vec(in.n_cams, vX), ba->pt, ba->sc, 1);
    const int nout = std::max(6 * in.n_cams, 3 * in.Pt);
    hipLaunchKernelGGL(k_ba_finish, dim3((unsigned)std::max((nout + kBlock - 1) / kBlock, 1)), dim3(kBlock), 0, st,
                       in.n_cams, in.Pt, ba->cam, ba->pt, ba->sc, d_twist, d_X, stats);
    return hipGetLastError();
}

}  // namespace gs

extern "C" {

gs_status gs_ba_create(gs_ba** out, int64_t max_points, int32_t max_cams) {
    if (!out) return GS_ERR_INVALID_ARG;
    *out = nullptr;
    if (max_points < 0 || max_cams < 0) return GS_ERR_INVALID_ARG;
    if (max_points > ((int64_t)1 << 28) || max_cams > GS_BA_MAX_CAMS) return GS_ERR_CAPACITY;
    gs_ba* b = new gs_ba();
    b->max_points = max_points;
    b->max_cams = max_cams;
    hipError_t e = hipMalloc((void**)&b->pt, sizeof(double) * gs::kPt * (size_t)std::max<int64_t>(max_points, 1));
    if (e == hipSuccess)
        e = hipMalloc((void**)&b->cam, sizeof(double) * gs::kCam * (size_t)std::max(max_cams, 1));
    if (e == hipSuccess)
        e = hipMalloc(&b->win, sizeof(int32_t) * gs::kCgWaves +
                                   sizeof(gs::Window) * ((size_t)max_points + gs::kCgWaves));
    if (e == hipSuccess) e = hipMalloc((void**)&b->cam_off, sizeof(int32_t) * ((size_t)max_cams + 1));
    if (e == hipSuccess) e = hipMalloc((void**)&b->sc, sizeof(double) * 16);
    // the cameras a workgroup's LDS holds, and at most one per thread
    int dev = 0, lds = 0;
    if (e == hipSuccess) e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    b->lds_cams = std::min(std::max((lds - gs::kLdsFixed) / gs::kLdsPerCam, 0), gs::kVec);
    if (e != hipSuccess) {
        gs_ba_destroy(b);
        return GS_ERR_HIP;
    }
    *out = b;
    return GS_OK;
}

gs_status gs_ba_destroy(gs_ba* b) {
    if (!b) return GS_ERR_INVALID_ARG;
    hipDeviceSynchronize();
    if (b->pt) hipFree(b->pt);
    if (b->cam) hipFree(b->cam);
    if (b->win) hipFree(b->win);
    if (b->cam_off) hipFree(b->cam_off);
    if (b->sc) hipFree(b->sc);
    delete b;
    return GS_OK;
}

gs_status gs_ba_lm_step(gs_ba* b, const float* X, int32_t Pt, const float* viewmat, const float* intr,
                        int32_t n_cams, const int32_t* obs_cam, const int32_t* obs_pt,
                        const float* obs_xy, int32_t M, const int32_t* pt_off, const int32_t* pt_obs,
                        const int32_t* pm_cam, const float* pm_xy, float delta, float lm_lambda,
                        float near_plane, int32_t max_iter, float tol, float* d_twist, float* d_X,
                        float* stats, void* stream) {
    if (!b || Pt < 0 || n_cams < 0 || M < 0 || max_iter < 0) return GS_ERR_INVALID_ARG;
    if ((int64_t)Pt > b->max_points || n_cams > b->max_cams) return GS_ERR_CAPACITY;
    if (!(delta > 0.f) || !(lm_lambda > 0.f) || !(near_plane > 0.f) || !(tol >= 0.f)) return GS_ERR_INVALID_ARG;
    if ((n_cams > 0 && (!viewmat || !intr || !d_twist)) || (Pt > 0 && (!X || !pt_off || !d_X)) ||
        (M > 0 && (!obs_cam || !obs_pt || !obs_xy || !pt_obs)))
        return GS_ERR_INVALID_ARG;
    if ((pm_cam == nullptr) != (pm_xy == nullptr)) return GS_ERR_INVALID_ARG;  // both or neither
    gs::BaInputs in;
    in.X = X;
    in.viewmat = viewmat;
    in.intr = intr;
    in.obs_cam = obs_cam;
    in.obs_pt = obs_pt;
    in.obs_xy = obs_xy;
    in.pt_off = pt_off;
    in.pt_obs = pt_obs;
    in.pm_cam = pm_cam;
    in.pm_xy = pm_xy;
    in.Pt = Pt;
    in.n_cams = n_cams;
    in.M = M;
    in.delta = delta;
    in.lambda = lm_lambda;
    in.near_plane = near_plane;
    in.max_iter = max_iter;
    in.tol = tol;
    return gs::launch_ba_step(b, in, d_twist, d_X, stats, (hipStream_t)stream) == hipSuccess ? GS_OK
                                                                                           : GS_ERR_HIP;
}

}  // extern "C"
