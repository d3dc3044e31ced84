// The stochastic density control of the joint step (MCMC densification):
// relocation of dead Gaussians onto live ones drawn in proportion to their
// opacity, with the opacity and scale rule that keeps a source's combined
// contribution, and the noise added to the means after an update.  The
// random numbers come in as arguments.
//
// Draws are exact integer arithmetic: each live Gaussian weighs
// floor(o 2^24) (o from the logit in double), the weights' inclusive prefix
// sums are 64-bit (a block pass, one workgroup for the block totals), and dead
// Gaussian j takes the first index whose prefix exceeds floor(u_j W), found by
// binary search over the blocks, then in one.
//
// What moves is 59 rows of parameters and 118 of moments (SH degree 3), a
// fifth of their words at random places: the rows are taken one after another
// by the whole chip, so that a row's gathers find it in the cache and each line
// is written once, and the dead are listed in order, so that every lane has one.
#include <math.h>

#include <algorithm>

#include "gs_internal.h"

namespace gs {

namespace {

constexpr int kBlock = 1024;      // items (and threads) per block of the prefix sums
constexpr int kMaxCopies = 51;    // copies counted in the opacity and scale rule
constexpr double kWeightScale = 16777216.0;  // 2^24

// Rows of N floats: of the parameters, or of both moments.
constexpr int kMaxRows = 11 + 3 * 16;
template <int MAX>
struct Rows {
    float* p[MAX];
    int n;
};

__device__ __forceinline__ double opacity_of(float logit) { return 1.0 / (1.0 + exp(-(double)logit)); }

__device__ __forceinline__ uint64_t block_incl_scan_u64(uint64_t v, uint64_t* s, uint64_t& total) {
    // inclusive scan over kBlock threads: waves by shuffles, then the waves' totals
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    for (int off = 1; off < kWave; off <<= 1) {
        const uint64_t t = __shfl_up(v, off, kWave);
        if (lane >= off) v += t;
    }
    if (lane == kWave - 1) s[w] = v;
    __syncthreads();
    uint64_t before = 0, tot = 0;
    for (int q = 0; q < kBlock / kWave; q++) {
        if (q < w) before += s[q];
        tot += s[q];
    }
    __syncthreads();
    total = tot;
    return v + before;
}

// threads of the wave below this one that `on` holds for
__device__ __forceinline__ int rank_in(uint64_t on) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(on >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)on, 0u));
}

// The threads of the block that `on` holds for, listed in order in s_list
// (their thread indices); returns their number.
__device__ __forceinline__ int block_list(bool on, int* s_list, int* s_n) {
    const int w = threadIdx.x / kWave;
    const uint64_t bal = __ballot(on);
    if (threadIdx.x % kWave == 0) s_n[w] = __popcll(bal);
    __syncthreads();
    int before = 0, all = 0;
    for (int q = 0; q < kBlock / kWave; q++) {
        if (q < w) before += s_n[q];
        all += s_n[q];
    }
    if (on) s_list[before + rank_in(bal)] = threadIdx.x;
    __syncthreads();
    return all;
}

// per item: its weight's prefix within the block, no draws yet; per block: the
// weights' sum and the number of dead
__global__ __launch_bounds__(kBlock) void k_mc_weights(const float* __restrict__ logit, int N, float t_dead,
                                                       uint64_t* __restrict__ cdf, uint64_t* __restrict__ bsum,
                                                       uint64_t* __restrict__ bdead,
                                                       uint32_t* __restrict__ count) {
    __shared__ uint64_t s[kBlock / kWave];
    __shared__ int s_d[kBlock / kWave];
    const int i = blockIdx.x * kBlock + threadIdx.x;
    uint64_t w = 0;
    bool dead = false;
    if (i < N) {
        const double o = opacity_of(logit[i]);
        dead = !(o > (double)t_dead);
        if (!dead) w = (uint64_t)floor(o * kWeightScale);
    }
    const uint64_t bal = __ballot(dead);
    if (threadIdx.x % kWave == 0) s_d[threadIdx.x / kWave] = __popcll(bal);
    uint64_t tot;
    const uint64_t inc = block_incl_scan_u64(w, s, tot);  // (its barriers also order s_d)
    if (i < N) {
        cdf[i] = inc;
        count[i] = 0u;
    }
    if (threadIdx.x == 0) {
        int d = 0;
        for (int q = 0; q < kBlock / kWave; q++) d += s_d[q];
        bsum[blockIdx.x] = tot;
        bdead[blockIdx.x] = (uint64_t)d;
    }
}

// one workgroup: exclusive prefixes of the block sums, the totals last
__global__ __launch_bounds__(kBlock) void k_mc_block_offsets(uint64_t* __restrict__ bsum,
                                                             uint64_t* __restrict__ bdead, int nb,
                                                             int32_t* __restrict__ n_moved) {
    __shared__ uint64_t s[kBlock / kWave];
    uint64_t carry[2] = {0, 0};
    for (int base = 0; base < nb; base += kBlock) {
        const int b = base + threadIdx.x;
#pragma unroll
        for (int a = 0; a < 2; a++) {
            uint64_t* x = a ? bdead : bsum;
            const uint64_t v = b < nb ? x[b] : 0;
            uint64_t tot;
            const uint64_t inc = block_incl_scan_u64(v, s, tot);
            if (b < nb) x[b] = carry[a] + inc - v;
            carry[a] += tot;
        }
    }
    if (threadIdx.x != 0) return;
    if (carry[0] == 0) carry[1] = 0;  // no live Gaussian: nothing moves
    bsum[nb] = carry[0];
    bdead[nb] = carry[1];
    if (n_moved) *n_moved = (int32_t)carry[1];
}

// the first place in [0, n) where a[place] > v (n if there is none)
__device__ __forceinline__ int first_above(const uint64_t* __restrict__ a, int n, uint64_t v) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] > v) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// Each dead Gaussian draws its source; the dead and their sources are listed
// in order.
__global__ __launch_bounds__(kBlock) void k_mc_draw(const float* __restrict__ logit, int N, float t_dead,
                                                    const float* __restrict__ u,
                                                    const uint64_t* __restrict__ cdf,
                                                    const uint64_t* __restrict__ bsum,
                                                    const uint64_t* __restrict__ bdead, int nb,
                                                    int32_t* __restrict__ src, uint32_t* __restrict__ count,
                                                    int2* __restrict__ list) {
    __shared__ int s_list[kBlock], s_n[kBlock / kWave];
    const int i0 = blockIdx.x * kBlock, i = i0 + threadIdx.x;
    const uint64_t W = bsum[nb];
    const bool dead = i < N && W > 0 && !(opacity_of(logit[i]) > (double)t_dead);
    if (i < N && !dead) src[i] = -1;
    const int nd = block_list(dead, s_list, s_n);
    if ((int)threadIdx.x >= nd) return;
    const int d = i0 + s_list[threadIdx.x];
    const uint64_t tv = (uint64_t)floor((double)u[d] * (double)W);
    const int b = first_above(bsum + 1, nb, tv);  // bsum[b + 1]: the prefix to the end of block b
    int s = N - 1;
    if (b < nb) {
        const int n = min(kBlock, N - b * kBlock);
        s = min(b * kBlock + first_above(cdf + (int64_t)b * kBlock, n, tv - bsum[b]), N - 1);
    }
    atomicAdd(&count[s], 1u);
    src[d] = s;
    list[bdead[blockIdx.x] + threadIdx.x] = make_int2(d, s);
}

// Below one dead in a hundred the moments are cleared by the list of the dead
// instead of the words of what moved: 5M Gaussians, us a call by the list and by
// the words, at 0.05% dead 176 and 422, 0.5% 494 and 588, 1% 789 and 771, 2%
// 1279 and 1164.
__device__ __forceinline__ bool few_dead(int n, int N) { return (int64_t)100 * n < N; }

// Sources: the opacity and scale of their n copies,
//   o' = 1 - (1 - o)^(1/n),  scale *= o / sum_{i=1..n} sum_{k<i} C(i-1, k) (-1)^k o'^(k+1) / sqrt(k+1),
// the double sum taken as sum_{k<n} C(n, k+1) (-1)^k o'^(k+1) / sqrt(k+1) (the
// binomials sum up a diagonal, and are exact in double to n = 51).  Per 64
// items, a word of which of them moved (dead or source), where k_mc_zero reads it.
__global__ __launch_bounds__(kBlock) void k_mc_sources(float* __restrict__ logit, float* __restrict__ ls, int N,
                                                       const uint32_t* __restrict__ count,
                                                       const int32_t* __restrict__ src,
                                                       const uint64_t* __restrict__ n_dead,
                                                       uint64_t* __restrict__ moved) {
    const int nd = (int)*n_dead;
    if (nd == 0) return;  // uniform over the launch
    __shared__ int s_list[kBlock], s_n[kBlock / kWave];
    __shared__ double s_rs[kMaxCopies];
    const int i0 = blockIdx.x * kBlock, i = i0 + threadIdx.x;
    if (threadIdx.x < kMaxCopies) s_rs[threadIdx.x] = rsqrt((double)(threadIdx.x + 1));
    const bool source = i < N && count[i] != 0u;
    if (!few_dead(nd, N)) {
        const uint64_t mv = __ballot(source || (i < N && src[i] >= 0));
        if (threadIdx.x % kWave == 0 && i < N) moved[i / kWave] = mv;
    }
    const int ns = block_list(source, s_list, s_n);
    if ((int)threadIdx.x >= ns) return;
    const int j = i0 + s_list[threadIdx.x];
    const int n = (int)min(count[j] + 1u, (uint32_t)kMaxCopies);
    const double o = opacity_of(logit[j]);
    const double op = 1.0 - pow(1.0 - o, 1.0 / n);
    double denom = 0.0, c = 1.0, pw = op;
    for (int k = 0; k < n; k++) {
        c = c * (double)(n - k) / (double)(k + 1);  // C(n, k + 1)
        denom += ((k & 1) ? -c : c) * pw * s_rs[k];
        pw *= op;
    }
    const double lf = log(o / denom);
    logit[j] = (float)log(op / (1.0 - op));
#pragma unroll
    for (int a = 0; a < 3; a++) {
        float& l = ls[(int64_t)a * N + j];
        l = (float)((double)l + lf);
    }
}

// Dead Gaussians: copies of their (updated) source.  blockIdx.y is the row, so
// the chip works within a few rows at a time (20 MB each for 5M Gaussians),
// which the last-level cache holds: bound by the random lines the gathers take
// from it and the partial lines written.  5M Gaussians, a fifth dead, 59 rows,
// us by the rows a thread takes together: 1 1218, 2 1263, 4 1289, 8 1303, 16
// 1312, all 1742; a thread per Gaussian, dead or not, walking all rows and then
// the moments' took 2975.  A row's workgroups cost a launch with few or no dead
// 0.2 ns each whatever they find: us with none and with a fifth dead, by
// workgroups a row, 256 5 and 1354, 512 8 and 1320, 1024 14 and 1271, 2048 27 and
// 1218.
constexpr unsigned kCopyBlocks = 512;

__global__ __launch_bounds__(256) void k_mc_copy(Rows<kMaxRows> rows, const int2* __restrict__ list,
                                                 const uint64_t* __restrict__ n_dead) {
    const int n = (int)*n_dead;
    float* row = rows.p[blockIdx.y];
    for (int e = blockIdx.x * 256 + threadIdx.x; e < n; e += gridDim.x * 256) {
        const int2 ds = list[e];
        row[ds.x] = row[ds.y];
    }
}

// The moments of everything that moved restart at zero.  Bound by the partial
// lines written (37% of the words at random: every line): 5M Gaussians, 118 rows,
// a fifth dead 971 us with 256 workgroups a row, 8 with none dead; a thread per
// item 916 and 489, which made a call with none dead four times as long.
constexpr unsigned kZeroBlocks = 256;

__global__ __launch_bounds__(256) void k_mc_zero(Rows<2 * kMaxRows> rows, int N,
                                                 const uint64_t* __restrict__ moved,
                                                 const int2* __restrict__ list,
                                                 const uint64_t* __restrict__ n_dead) {
    const int n = (int)*n_dead;
    float* row = rows.p[blockIdx.y];
    const int first = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
    if (few_dead(n, N)) {
        for (int e = first; e < n; e += step) {
            const int2 ds = list[e];
            row[ds.x] = 0.f;
            row[ds.y] = 0.f;
        }
        return;
    }
    for (int i = first; i < N; i += step)
        if (moved[i / kWave] >> (i % kWave) & 1) row[i] = 0.f;
}

// mu += scale sigmoid(-k (o - t)) Sigma eta
__global__ __launch_bounds__(256) void k_mc_noise(float* __restrict__ means, const float* __restrict__ ls,
                                                  const float* __restrict__ quats,
                                                  const float* __restrict__ logit, int N,
                                                  const float* __restrict__ eta, float scale, float k,
                                                  float t) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    float q[4];
    float qn = 0.f;
#pragma unroll
    for (int a = 0; a < 4; a++) {
        q[a] = quats[(int64_t)a * N + i];
        qn += q[a] * q[a];
    }
    const float iq = rsqrtf(qn);
    const float w = q[0] * iq, x = q[1] * iq, y = q[2] * iq, z = q[3] * iq;
    const float R[9] = {1.f - 2.f * (y * y + z * z), 2.f * (x * y - w * z), 2.f * (x * z + w * y),
                        2.f * (x * y + w * z), 1.f - 2.f * (x * x + z * z), 2.f * (y * z - w * x),
                        2.f * (x * z - w * y), 2.f * (y * z + w * x), 1.f - 2.f * (x * x + y * y)};
    float s2[3];
#pragma unroll
    for (int a = 0; a < 3; a++) s2[a] = expf(2.f * ls[(int64_t)a * N + i]);
    const float o = 1.f / (1.f + expf(-logit[i]));
    const float gate = 1.f / (1.f + expf(k * (o - t)));
    const float e[3] = {eta[i], eta[(int64_t)N + i], eta[2 * (int64_t)N + i]};
    // Sigma eta = R diag(s^2) R^T eta
    float rt[3];
#pragma unroll
    for (int c = 0; c < 3; c++) rt[c] = s2[c] * (R[c] * e[0] + R[3 + c] * e[1] + R[6 + c] * e[2]);
#pragma unroll
    for (int a = 0; a < 3; a++)
        means[(int64_t)a * N + i] += scale * gate * (R[3 * a] * rt[0] + R[3 * a + 1] * rt[1] + R[3 * a + 2] * rt[2]);
}

}  // namespace

hipError_t launch_mcmc_relocate(Ctx* c, const gs_gaussian_adam* state, int N, int sh_degree,
                                const float* u, float t_dead, int32_t* src, int32_t* n_moved,
                                hipStream_t st) {
    if (N <= 0) return hipSuccess;
    const int K = (sh_degree + 1) * (sh_degree + 1);
    const int rows[5] = {3, 3, 4, 1, 3 * K};
    Rows<kMaxRows> par = {};
    Rows<2 * kMaxRows> mom = {};
    for (int q = 0; q < 5; q++)
        for (int r = 0; r < rows[q]; r++) {
            par.p[par.n++] = state->params[q] + (int64_t)r * N;
            mom.p[mom.n++] = state->exp_avg[q] + (int64_t)r * N;
            mom.p[mom.n++] = state->exp_avg_sq[q] + (int64_t)r * N;
        }
    // workspace in the record buffer (48 B per item, at least 128): prefixes and
    // the list of the dead (8 B per item each), counts and sources (4 B each; the
    // caller's src array, if given), the moved words, block sums
    const int nb = (N + kBlock - 1) / kBlock;
    const size_t nw = ((size_t)N + kWave - 1) / kWave;
    uint64_t* cdf = reinterpret_cast<uint64_t*>(c->rec);
    int2* list = reinterpret_cast<int2*>(cdf + N);
    uint64_t* moved = reinterpret_cast<uint64_t*>(list + N);
    uint64_t* bsum = moved + nw;
    uint64_t* bdead = bsum + nb + 1;
    uint32_t* count = reinterpret_cast<uint32_t*>(bdead + nb + 1);
    if (!src) src = reinterpret_cast<int32_t*>(count + N);
    const dim3 gb(nb), tb(kBlock);
    hipLaunchKernelGGL(k_mc_weights, gb, tb, 0, st, par.p[10], N, t_dead, cdf, bsum, bdead, count);
    hipLaunchKernelGGL(k_mc_block_offsets, dim3(1), tb, 0, st, bsum, bdead, nb, n_moved);
    hipLaunchKernelGGL(k_mc_draw, gb, tb, 0, st, par.p[10], N, t_dead, u, cdf, bsum, bdead, nb, src, count,
                       list);
    hipLaunchKernelGGL(k_mc_sources, gb, tb, 0, st, par.p[10], par.p[3], N, count, src, bdead + nb,
                       moved);
    const unsigned g = (unsigned)((N + 255) / 256);
    hipLaunchKernelGGL(k_mc_copy, dim3(std::min(g, kCopyBlocks), par.n), dim3(256), 0, st, par, list, bdead + nb);
    hipLaunchKernelGGL(k_mc_zero, dim3(std::min(g, kZeroBlocks), mom.n), dim3(256), 0, st, mom, N, moved, list,
                       bdead + nb);
    return hipGetLastError();
}

hipError_t launch_mcmc_noise(float* means, const float* log_scales, const float* quats,
                             const float* logit, int N, const float* eta, float scale, float k, float t,
                             hipStream_t st) {
    if (N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mc_noise, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, means, log_scales,
                       quats, logit, N, eta, scale, k, t);
    return hipGetLastError();
}

}  // namespace gs
