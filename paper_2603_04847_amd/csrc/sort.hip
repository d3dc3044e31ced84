// Device-wide exclusive scan (single pass) and stable LSD radix sort of (u32 key, u32 value)
// pairs, written for wave64: digit ranks inside a wave come from ballots
// (match-any over the digit bits), across waves from LDS counters, and each
// block stages its items in LDS so the global scatter writes contiguous runs.
#include <type_traits>

#include "gs_internal.h"

namespace gs {

namespace {

constexpr int kThreads = 256;
constexpr int kItems = 16;
constexpr int kTile = kThreads * kItems;  // 4096 items per block
constexpr int kWaves = kThreads / kWave;

// ------------------------------------------------------------------ scan

// shifts by 1, 2, 4 and 8 inside the rows of 16 lanes, then the rows' carries
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);
    return v;
}

// exclusive scan of one value per thread over the block; returns the block total
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* s_w, uint32_t& total) {
    const int lane = __lane_id(), w = threadIdx.x / kWave;
    uint32_t inc = wave_incl_scan(v);
    if (lane == kWave - 1) s_w[w] = inc;
    __syncthreads();
    uint32_t before = 0, tot = 0;
    for (int i = 0; i < (int)(blockDim.x / kWave); i++) {
        if (i < w) before += s_w[i];
        tot += s_w[i];
    }
    __syncthreads();
    total = tot;
    return before + inc - v;
}

// Single-pass scan with decoupled look-back.  Tiles of kScanTile items are taken
// in launch order from a counter, so every tile a workgroup waits on belongs
// to a workgroup that is already running.  A tile publishes its own total
// (flag kAgg), then its first wave reads the words of the 64 preceding tiles
// at once and adds back to the nearest one that carries an inclusive prefix
// (flag kIncl), which it then publishes for itself.  The last workgroup to
// finish clears the words and counters, so the workspace is clean for the
// next scan without a separate fill.
//
// Workspace (u32 words): [0] tile counter, [1] finished counter, then one
// 64-bit word per tile from word kScanHeader: flag << 32 | value.
constexpr int kScanHeader = 64;
constexpr uint32_t kAgg = 1u, kIncl = 2u;
// bound on the polls of one look-back (each ~1 us): a wait that never ends is
// reported (GS_FLAG_SCAN_STALLED) instead of hanging the device
constexpr int kSpinLimit = 1 << 21;

__device__ __forceinline__ uint64_t ld_word(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_word(uint64_t* p, uint32_t flag, uint32_t v) {
    __hip_atomic_store(p, ((uint64_t)flag << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// Called by one whole wave: the sum of the values of tiles [0, t) (mod 2^32).
__device__ uint32_t wave_lookback(const uint64_t* words, int64_t t, uint32_t* flags) {
    const int lane = __lane_id();
    uint32_t excl = 0;
    int64_t top = t - 1;
    int polls = 0;
    while (top >= 0) {
        const int64_t idx = top - lane;
        const uint64_t w = idx >= 0 ? ld_word(words + idx) : ((uint64_t)kIncl << 32);
        const uint32_t flag = (uint32_t)(w >> 32);
        const uint64_t incl = __ballot(flag == kIncl);
        const uint64_t none = __ballot(flag == 0u);
        const int first = incl ? __builtin_ctzll(incl) : kWave;  // nearest inclusive tile
        const uint64_t need = first >= kWave - 1 ? ~0ull : ((2ull << first) - 1ull);
        if (none & need) {
            if (++polls > kSpinLimit) {
                if (lane == 0 && flags) {
                    atomicOr(flags, (uint32_t)GS_FLAG_SCAN_STALLED);
                    __atomic_thread_fence(__ATOMIC_RELEASE);
                }
                return excl;
            }
            __builtin_amdgcn_s_sleep(2);
            continue;
        }
        excl += wave_sum_u32(lane <= first ? (uint32_t)w : 0u);
        if (first < kWave) break;
        top -= kWave;
    }
    return excl;
}

// A scan whose look-back gave up (GS_FLAG_SCAN_STALLED) has offsets that are
// not to be trusted: the check then treats the list as overflowed, so every
// later stage writes nothing.
__device__ __forceinline__ void cap_check(uint32_t t, const CapCheck& c, const uint32_t* flags) {
    if (!c.used) return;
    const bool stalled =
        flags && (__hip_atomic_load(flags, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) &
                  (uint32_t)GS_FLAG_SCAN_STALLED) != 0u;
    const bool prev_over = c.prev_total && *c.prev_total != 0u && *c.prev_used == 0u;
    const bool over = prev_over || stalled || (int64_t)t > c.cap;
    *c.used = over ? 0u : t;
    if (prev_over) return;
    c.diag[kDiagIsectTotal] = t;
    c.diag[kDiagIsectUsed] = over ? 0u : t;
    if (over) atomicOr(&c.diag[kDiagFlags], (uint32_t)GS_FLAG_ISECT_OVERFLOW);
}

// 32 items per thread, read and written as 16-byte vectors: 8192 per tile of
// 256 threads.  Scans past kWideScan items use tiles of 1024 threads (32768
// items): the tickets and the look-back chain are per tile, and on the 20M
// offsets of the large scene the wide tiles take 0.05 ms off the binning
// (smaller scans lose parallelism with them).
constexpr int kScanItems = 32;
constexpr int kScanTile = kThreads * kScanItems;
constexpr int kWideThreads = 1024;
constexpr int64_t kWideScan = (int64_t)1 << 23;

// The length is max_n, or, with d_cnt, mul * (ceil(*d_cnt / per) + add)
// clamped to max_n (a count only the device knows: the grid covers max_n and
// tiles past the length only take their tickets).
template <int THREADS, bool UNPACK = false>
__global__ __launch_bounds__(THREADS) void k_scan(uint32_t* __restrict__ data, int64_t max_n,
                                                   const uint32_t* __restrict__ d_cnt, int64_t per,
                                                   int64_t mul, int64_t add,
                                                   uint32_t* __restrict__ total_out,
                                                   uint32_t* __restrict__ ws,
                                                   uint32_t* __restrict__ flags, CapCheck chk,
                                                   ScanUnpack un) {
    constexpr int TILE = THREADS * kScanItems;
    __shared__ uint32_t s_w[THREADS / kWave];
    __shared__ uint32_t s_t, s_excl, s_last;
    uint64_t* words = reinterpret_cast<uint64_t*>(ws + kScanHeader);
    int64_t n = max_n;
    if (d_cnt) n = min(max_n, mul * (((int64_t)*d_cnt + per - 1) / per + add));
    const int64_t ntiles = (n + TILE - 1) / TILE;
    // a grid of one needs neither ticket nor clearing, each a round trip to
    // memory (5.5 -> 4.6 us)
    const bool lone = THREADS == kThreads && gridDim.x == 1;
    if (!lone) {
        if (threadIdx.x == 0) s_t = atomicAdd(&ws[0], 1u);
        __syncthreads();
    }
    const int64_t t = lone ? 0 : s_t;
    if (t >= ntiles) {
        if (t == 0 && threadIdx.x == 0) {
            if (total_out) *total_out = 0u;
            cap_check(0u, chk, flags);
        }
    } else {
        const int64_t base = t * TILE + (int64_t)threadIdx.x * kScanItems;
        const bool full = base + kScanItems <= n;
        uint32_t v[kScanItems];
        const uint32_t* in = UNPACK ? un.src : data;
        if (full) {
            const uint4* p = reinterpret_cast<const uint4*>(in + base);
#pragma unroll
            for (int i = 0; i < kScanItems / 4; i++) {
                const uint4 q = p[i];
                v[4 * i] = q.x;
                v[4 * i + 1] = q.y;
                v[4 * i + 2] = q.z;
                v[4 * i + 3] = q.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < kScanItems; i++) v[i] = base + i < n ? in[base + i] : 0u;
        }
        if (UNPACK) {
            const uint32_t esc = ~0u >> un.pbits, pmask = (1u << un.pbits) - 1u;
#pragma unroll
            for (int i = 0; i < kScanItems; i++) {
                const uint32_t c = v[i] >> un.pbits;
                v[i] = c == esc ? un.cnt[v[i] & pmask] : c;
            }
        }
        uint32_t s = 0;
#pragma unroll
        for (int i = 0; i < kScanItems; i++) s += v[i];
        uint32_t tot;
        uint32_t ex = block_excl_scan(s, s_w, tot);
        if (threadIdx.x < kWave) {
            if (threadIdx.x == 0 && !lone) st_word(words + t, t == 0 ? kIncl : kAgg, tot);
            const uint32_t excl = t > 0 ? wave_lookback(words, t, flags) : 0u;
            if (threadIdx.x == 0) {
                if (t > 0) st_word(words + t, kIncl, excl + tot);
                s_excl = excl;
                if (t == ntiles - 1) {
                    if (total_out) *total_out = excl + tot;
                    cap_check(excl + tot, chk, flags);
                }
            }
        }
        __syncthreads();
        ex += s_excl;
#pragma unroll
        for (int i = 0; i < kScanItems; i++) {
            const uint32_t x = v[i];
            v[i] = ex;
            ex += x;
        }
        if (full) {
            uint4* p = reinterpret_cast<uint4*>(data + base);
#pragma unroll
            for (int i = 0; i < kScanItems / 4; i++)
                p[i] = make_uint4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
        } else {
#pragma unroll
            for (int i = 0; i < kScanItems; i++)
                if (base + i < n) data[base + i] = v[i];
        }
    }
    if (lone) return;
    // every tile has finished its look-back once all have taken a ticket here
    if (threadIdx.x == 0) s_last = atomicAdd(&ws[1], 1u) == gridDim.x - 1;
    __syncthreads();
    if (s_last) {
        for (int64_t k = threadIdx.x; k < ntiles; k += THREADS) st_word(words + k, 0u, 0u);
        if (threadIdx.x == 0) {
            __hip_atomic_store(&ws[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&ws[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ------------------------------------------------------------------ radix sort

__device__ __forceinline__ uint32_t dev_count(const uint32_t* d_n, int64_t max_n) {
    if (!d_n) return (uint32_t)max_n;
    uint32_t n = *d_n;
    return n < (uint64_t)max_n ? n : (uint32_t)max_n;
}

// lanes of the wave holding the same digit of `bits` bits (among lanes with `valid`)
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid, int bits) {
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < bits; b++) {
        const bool bit = (d >> b) & 1u;
        const uint64_t m = __ballot(bit);
        peers &= bit ? m : ~m;
    }
    return peers;
}

// Items of a block: wave w owns the contiguous chunk [base + 64 ITEMS w,
// base + 64 ITEMS (w+1)), read 64 at a time; so (wave, step, lane) order is
// index order and ranks can be kept per wave without block barriers.
template <int ITEMS>
__device__ __forceinline__ int64_t item_index(int64_t base, int w, int i, int lane) {
    return base + (int64_t)w * (kWave * ITEMS) + i * kWave + lane;
}

// Per-block digit counts, digit-major: hist[d * nb + block] with nb the number
// of blocks that hold items (the live count), so the scan covers only those.
// All loads of a thread are issued before the first count.  Counts need no
// ranks: for 7- and 8-bit digits each item is one LDS add, and a wave whose
// valid items share one digit (common in the top digit of clustered keys)
// adds them at once; narrower digits of clustered keys (the block ids) would
// pile many adds onto a few addresses, so there one lane per distinct digit
// adds the count its ballot match found.
template <int ITEMS>
__global__ __launch_bounds__(kThreads) void k_radix_hist(const uint32_t* __restrict__ keys,
                                                         const uint32_t* __restrict__ d_n,
                                                         int64_t max_n, int shift, int bits,
                                                         uint32_t* __restrict__ hist) {
    constexpr int TILE = kThreads * ITEMS;
    __shared__ uint32_t s_h[kWaves][256];
    const uint32_t n = dev_count(d_n, max_n);
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
    const uint32_t mask = (1u << bits) - 1u;
    for (int q = 0; q < kWaves; q++) s_h[q][tid] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * TILE;
    if (base < n) {
        uint32_t k[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            const int64_t j = item_index<ITEMS>(base, w, i, lane);
            k[i] = j < n ? keys[j] : 0u;
        }
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            const bool valid = item_index<ITEMS>(base, w, i, lane) < n;
            const uint32_t d = (k[i] >> shift) & mask;
            if (bits > 6) {
                const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
                if (__ballot(valid && d != d0) == 0) {
                    const uint64_t live = __ballot(valid);
                    if (lane == 0 && live) atomicAdd(&s_h[w][d0], (uint32_t)__popcll(live));
                } else if (valid) {
                    atomicAdd(&s_h[w][d], 1u);
                }
            } else {
                const uint64_t peers = match_digit(d, valid, bits);
                if (valid && (peers & lanemask_lt()) == 0) atomicAdd(&s_h[w][d], (uint32_t)__popcll(peers));
            }
        }
    }
    __syncthreads();
    const int64_t nb = ((int64_t)n + TILE - 1) / TILE;
    if (tid <= (int)mask && (int64_t)blockIdx.x < nb)
        hist[(int64_t)tid * nb + blockIdx.x] = s_h[0][tid] + s_h[1][tid] + s_h[2][tid] + s_h[3][tid];
}

// Value arrays moved with the keys: NV words per item, one array each.
template <int NV>
struct ValArrays {
    const uint32_t* in[NV];
    uint32_t* out[NV];
};

// The block of items a scattering workgroup takes, of nb (nb: none).
// Workgroups go round the eight dies in launch order, each die with an L2 of
// its own.  A block's run of one digit ends inside a line that the next block's
// run goes on with, so consecutive blocks run on one die, which fills the line
// before it goes to memory: bandwidth-bound, 63M entries of four words 473 ->
// 396 us, 20M of two 120 -> 95, 4M of two 29 -> 21 (with the blocks taken in
// launch order first).  The digit counts gain nothing by it (35 -> 50 us, the
// counts of 20M keys) and keep the launch order.
constexpr int kXcds = 8;
__device__ __forceinline__ int64_t xcd_block(int64_t nb) {
    const int64_t per = (nb + kXcds - 1) / kXcds;
    const int64_t i = blockIdx.x / kXcds;
    return i < per ? (int64_t)(blockIdx.x % kXcds) * per + i : nb;
}

template <int ITEMS, int NV>
__global__ __launch_bounds__(kThreads) void k_radix_scatter(
    const uint32_t* __restrict__ kin, uint32_t* __restrict__ kout, ValArrays<NV> va,
    const uint32_t* __restrict__ d_n, int64_t max_n, int shift, int bits,
    const uint32_t* __restrict__ hist) {
    constexpr int TILE = kThreads * ITEMS;
    __shared__ uint32_t s_h[kWaves][256];  // per-wave digit counts, then offsets
    __shared__ uint32_t s_start[256];
    __shared__ uint32_t s_glob[256];
    __shared__ uint32_t s_w[kWaves];
    __shared__ uint32_t s_key[TILE];
    __shared__ uint32_t s_val[NV][TILE];
    const uint32_t n = dev_count(d_n, max_n);
    const int64_t nb = ((int64_t)n + TILE - 1) / TILE;
    const int64_t blk = xcd_block(nb);
    if (blk >= nb) return;  // uniform over the block
    const int64_t base = blk * TILE;
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
    const uint32_t mask = (1u << bits) - 1u;
    uint32_t k[ITEMS], v[NV][ITEMS];
    uint16_t rank[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
        const int64_t j = item_index<ITEMS>(base, w, i, lane);
        k[i] = j < n ? kin[j] : 0u;
#pragma unroll
        for (int c = 0; c < NV; c++) v[c][i] = j < n ? va.in[c][j] : 0u;
    }
    for (int q = 0; q < kWaves; q++) s_h[q][tid] = 0;
    s_glob[tid] = tid <= (int)mask ? hist[(int64_t)tid * nb + blk] : 0u;
    __syncthreads();
    // stable rank inside the wave's chunk: earlier steps (LDS count) + earlier lanes
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
        const bool valid = item_index<ITEMS>(base, w, i, lane) < n;
        const uint32_t d = (k[i] >> shift) & mask;
        const uint64_t peers = match_digit(d, valid, bits);
        const uint32_t before = s_h[w][d];
        rank[i] = (uint16_t)(before + (uint32_t)__popcll(peers & lanemask_lt()));
        if (valid && (peers & lanemask_lt()) == 0) s_h[w][d] = before + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    // per digit: offsets of the waves, then the block-wide exclusive scan
    uint32_t run = 0;
    for (int q = 0; q < kWaves; q++) {
        const uint32_t c = s_h[q][tid];
        s_h[q][tid] = run;
        run += c;
    }
    uint32_t tot;
    s_start[tid] = block_excl_scan(run, s_w, tot);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
        if (item_index<ITEMS>(base, w, i, lane) < n) {
            const uint32_t d = (k[i] >> shift) & mask;
            const uint32_t pos = s_start[d] + s_h[w][d] + rank[i];
            s_key[pos] = k[i];
#pragma unroll
            for (int c = 0; c < NV; c++) s_val[c][pos] = v[c][i];
        }
    }
    __syncthreads();
    const uint32_t cnt = (uint32_t)min((int64_t)TILE, (int64_t)n - base);
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
        const uint32_t j = i * kThreads + tid;
        if (j < cnt) {
            const uint32_t key = s_key[j];
            const uint32_t d = (key >> shift) & mask;
            const uint32_t g = s_glob[d] + (j - s_start[d]);
            if (g < n) {  // always, unless a digit scan gave up (flagged)
                kout[g] = key;
#pragma unroll
                for (int c = 0; c < NV; c++) va.out[c][g] = s_val[c][j];
            }
        }
    }
}

// ------------------------------------------------------------------ one pass over block ids
//
// A counting sort of entries of three words by keys below `digits` (at most
// kWideDigits): counts, their scan, one scatter, which moves every word once
// (the keys' own order is known then from the counts, which give the ranges, so
// they are not written).  A block's run of a digit is short, nine items at a
// thousand digits, and the next blocks, on the same die, fill its lines.
// Bandwidth-bound: 63M entries, 885 blocks, 68 us of counts and 426 of scatter
// (28 B an entry, 4.1 TB/s) against 974 for two passes of 5 bits over all four
// words and a search of the sorted keys for the ranges; 2.6M entries, 261
// blocks, 41 against 78.  A tile of 8192 in 512 threads of 16 items: two
// workgroups a CU, one staging while the other ranks (1024 threads of 8: 568).
constexpr int kWideBlock = 512;
constexpr int kWideItems = 16;
constexpr int kWideTile = kWideBlock * kWideItems;
constexpr int kWideWaves = kWideBlock / kWave;

// Counts of `ch` consecutive tiles, digit-major over the groups: hist[d * groups
// + group]; and, where a group is more than one tile, each tile's counts of
// the group's tiles before it, rows[tile * digits + d] (below 2^16).  A group's
// counts go to as many lines as there are digits, so few groups are few
// partial lines; the rows are written in order.
__global__ __launch_bounds__(kWideBlock) void k_wide_hist(const uint32_t* __restrict__ keys,
                                                             const uint32_t* __restrict__ d_n, int64_t max_n,
                                                             int digits, int ch, uint16_t* __restrict__ rows,
                                                             uint32_t* __restrict__ hist) {
    __shared__ uint32_t s_h[kWideDigits];
    const uint32_t n = dev_count(d_n, max_n);
    const int64_t nb = ((int64_t)n + kWideTile - 1) / kWideTile, groups = (nb + ch - 1) / ch;
    if (blockIdx.x >= groups) return;  // uniform over the block
    const int tid = threadIdx.x;
    for (int d = tid; d < digits; d += kWideBlock) s_h[d] = 0u;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * ch, t1 = min(t0 + ch, nb);
    for (int64_t t = t0; t < t1; t++) {
        const int64_t base = t * kWideTile;
        uint4 k[kWideItems / 4];
#pragma unroll
        for (int i = 0; i < kWideItems / 4; i++) {
            const int64_t j = base + 4 * (i * kWideBlock + tid);
            if (j + 4 <= n) {
                k[i] = *reinterpret_cast<const uint4*>(keys + j);
            } else {
                k[i].x = j < n ? keys[j] : ~0u;
                k[i].y = j + 1 < n ? keys[j + 1] : ~0u;
                k[i].z = j + 2 < n ? keys[j + 2] : ~0u;
                k[i].w = ~0u;
            }
        }
        if (ch > 1) {
            for (int d = tid; d < digits; d += kWideBlock) rows[t * digits + d] = (uint16_t)s_h[d];
            __syncthreads();
        }
        const uint32_t top = (uint32_t)digits;  // unused places hold ~0
        if (digits > 64) {
#pragma unroll
            for (int i = 0; i < kWideItems / 4; i++) {
                if (k[i].x < top) atomicAdd(&s_h[k[i].x], 1u);
                if (k[i].y < top) atomicAdd(&s_h[k[i].y], 1u);
                if (k[i].z < top) atomicAdd(&s_h[k[i].z], 1u);
                if (k[i].w < top) atomicAdd(&s_h[k[i].w], 1u);
            }
        } else {  // few addresses: one lane per distinct digit adds its lanes
            auto add = [&](uint32_t d) {
                const uint64_t peers = match_digit(d, d < top, 6);
                if (d < top && (peers & lanemask_lt()) == 0) atomicAdd(&s_h[d], (uint32_t)__popcll(peers));
            };
#pragma unroll
            for (int i = 0; i < kWideItems / 4; i++) {
                add(k[i].x);
                add(k[i].y);
                add(k[i].z);
                add(k[i].w);
            }
        }
        __syncthreads();
    }
    for (int d = tid; d < digits; d += kWideBlock) hist[(int64_t)d * groups + blockIdx.x] = s_h[d];
}

// LDS: the digits' offsets, then the waves' digit counts, in whose place the
// tile is staged once the items' places are known.
__host__ __device__ inline size_t wide_lds(int digits) {
    const size_t dp = ((size_t)digits + 3) / 4 * 4;
    const size_t counts = sizeof(uint16_t) * kWideWaves * dp, stage = (sizeof(uint16_t) + sizeof(uint32_t)) * kWideTile;
    return sizeof(uint32_t) * dp + (counts > stage ? counts : stage);
}

// a word at a byte offset (of arrays of at most 2^30 words)
template <typename T>
__device__ __forceinline__ T& word_at(T* p, uint32_t at) {
    using C = std::conditional_t<std::is_const_v<T>, const char, char>;
    return *reinterpret_cast<T*>(reinterpret_cast<C*>(p) + at);
}

template <int BITS>
__global__ __launch_bounds__(kWideBlock, 4) void k_wide_scatter(
    const uint32_t* __restrict__ keys, ValArrays<3> va, const uint32_t* __restrict__ d_n, int64_t max_n,
    int digits, int ch, const uint16_t* __restrict__ rows, const uint32_t* __restrict__ hist,
    int32_t* __restrict__ ranges) {
    extern __shared__ __attribute__((aligned(16))) uint32_t s_wide[];
    __shared__ uint32_t s_w[kWideWaves];
    const uint32_t n = dev_count(d_n, max_n);
    const int64_t nb = ((int64_t)n + kWideTile - 1) / kWideTile, groups = (nb + ch - 1) / ch;
    const int64_t blk = xcd_block(nb);
    if (blk >= nb) return;  // uniform over the block
    const uint32_t base = (uint32_t)(blk * kWideTile);  // below n
    const int dp = (digits + 3) / 4 * 4;
    uint32_t* s_off = s_wide;                                   // [dp]
    uint16_t* s_cnt = reinterpret_cast<uint16_t*>(s_wide + dp);  // [waves][dp]
    uint32_t* s_val = s_wide + dp;                              // [tile], over the counts
    uint16_t* s_dig = reinterpret_cast<uint16_t*>(s_val + kWideTile);
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
    const uint32_t first = base + (uint32_t)(w * kWave * kWideItems + lane);  // a wave's items: 64 at a time
    // every load below is one base and a 32-bit offset (at most 2^30 items)
    uint32_t k[kWideItems], v[3][kWideItems];
#pragma unroll
    for (int i = 0; i < kWideItems; i++) {
        k[i] = word_at(keys, 4u * min(first + i * kWave, n - 1u));
    }
    for (int d = tid; d < kWideWaves * dp / 2; d += kWideBlock) s_val[d] = 0u;
    __syncthreads();
    // stable rank inside the wave's chunk: earlier steps (LDS count) + earlier lanes
#pragma unroll
    for (int i = 0; i < kWideItems; i++) {
        const bool valid = first + i * kWave < n;
        const uint32_t d = min(k[i], (uint32_t)digits - 1u);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < BITS; b++) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t before = s_cnt[w * dp + d];
        const uint32_t below = (uint32_t)__popcll(peers & lanemask_lt());
        if (valid && below == 0) s_cnt[w * dp + d] = (uint16_t)(before + (uint32_t)__popcll(peers));
        k[i] = d | (before + below) << 16;  // both below 2^16
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // the values, while the digits are scanned
#pragma unroll
    for (int i = 0; i < kWideItems; i++) {
        const uint32_t at = 4u * min(first + i * kWave, n - 1u);
#pragma unroll
        for (int c = 0; c < 3; c++) v[c][i] = word_at(va.in[c], at);
    }
    // four digits a thread: offsets of the waves, then the scan over the digits
    uint32_t run[4] = {0u, 0u, 0u, 0u};
    const int d0 = 4 * tid;
    if (d0 < digits) {
#pragma unroll 4
        for (int q = 0; q < kWideWaves; q++) {
            uint2* p = reinterpret_cast<uint2*>(s_cnt + q * dp + d0);
            const uint2 c = *p;
            *p = make_uint2(run[0] | run[1] << 16, run[2] | run[3] << 16);
            run[0] += c.x & 0xFFFFu;
            run[1] += c.x >> 16;
            run[2] += c.y & 0xFFFFu;
            run[3] += c.y >> 16;
        }
    }
    uint32_t tot;
    uint32_t start = block_excl_scan(run[0] + run[1] + run[2] + run[3], s_w, tot);
    if (d0 < digits) {
        uint32_t st[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            st[e] = start;
            start += run[e];
            if (d0 + e < digits) {
                uint32_t g = hist[(int64_t)(d0 + e) * groups + blk / ch];
                if (ch > 1) g += rows[blk * digits + d0 + e];
                s_off[d0 + e] = g - st[e];
            }
        }
#pragma unroll 4
        for (int q = 0; q < kWideWaves; q++) {  // no field reaches 2^16: a tile holds 2^13 items
            uint2* p = reinterpret_cast<uint2*>(s_cnt + q * dp + d0);
            uint2 c = *p;
            c.x += st[0] | st[1] << 16;
            c.y += st[2] | st[3] << 16;
            *p = c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kWideItems; i++) k[i] += (uint32_t)s_cnt[w * dp + (k[i] & 0xFFFFu)] << 16;
    __syncthreads();  // the counts make room for the staged tile
    const uint32_t cnt = min((uint32_t)kWideTile, n - base);
#pragma unroll
    for (int i = 0; i < kWideItems; i++)
        if (first + i * kWave < n) {
            s_dig[k[i] >> 16] = (uint16_t)k[i];
            s_val[k[i] >> 16] = v[0][i];
        }
    __syncthreads();
    uint32_t to[kWideItems];
#pragma unroll
    for (int i = 0; i < kWideItems; i++) {
        const uint32_t j = i * kWideBlock + tid;
        const uint32_t g = j < cnt ? s_off[s_dig[j]] + j : ~0u;
        to[i] = g < n ? 4u * g : ~0u;  // past n only if the scan gave up (flagged)
    }
#pragma unroll
    for (int c = 0; c < 3; c++) {
        if (c > 0) {
#pragma unroll
            for (int i = 0; i < kWideItems; i++)
                if (first + i * kWave < n) s_val[k[i] >> 16] = v[c][i];
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < kWideItems; i++)
            if (to[i] != ~0u) word_at(va.out[c], to[i]) = s_val[i * kWideBlock + tid];
        if (c < 2) __syncthreads();
    }
    // the ranges of all keys but the last, from the scanned counts
    if (blk == 0)
        for (int d = tid; d < digits - 1; d += kWideBlock) {
            ranges[2 * d] = (int32_t)min(hist[(int64_t)d * groups], n);
            ranges[2 * d + 1] = (int32_t)min(hist[(int64_t)(d + 1) * groups], n);
        }
}

// ------------------------------------------------------------------ a small sort in one workgroup
//
// At most kSmallSort packed pairs sorted by depth key and their entry counts
// scanned, all in one workgroup's LDS: where the general path is four passes
// of three launches and a scan, each a few microseconds whatever its size.
// Keys are taken from the smallest visible one up, the culled pairs' just past
// the largest, so the digits cover the range there is: three passes of nine
// bits for a depth range of sixteen octaves.  Every wave owns a run of
// 64 `steps` items, as in k_radix_scatter; places past the end are culled keys,
// which sort last.  Bound by one CU's arithmetic (the ballots of the ranks): 2000
// pairs 58 -> 16 us of kernels, 10000 75 -> 36, 16384 67 -> 52, each in one
// launch instead of thirteen; what the LDS holds is the limit.
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;
constexpr int kSmallItems = (int)(kSmallSort / kSmallThreads);
constexpr int kSmallBits = 9;
constexpr int kSmallDigits = 1 << kSmallBits;

__global__ __launch_bounds__(kSmallThreads) void k_small_sort(const uint32_t* __restrict__ kin,
                                                              uint32_t* __restrict__ kout,
                                                              uint32_t* __restrict__ vout, int n, int steps,
                                                              ScanUnpack un, uint32_t* __restrict__ off,
                                                              uint32_t* __restrict__ total_out,
                                                              uint32_t* __restrict__ flags, CapCheck chk) {
    extern __shared__ __attribute__((aligned(16))) uint32_t s_items[];  // [2][1024 steps]
    __shared__ uint16_t s_cnt[kSmallWaves][kSmallDigits];
    __shared__ uint32_t s_w[kSmallWaves], s_lo[kSmallWaves], s_hi[kSmallWaves];
    uint32_t* s_key = s_items;
    uint32_t* s_val = s_items + kSmallThreads * steps;
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
    const int first = w * kWave * steps + lane;  // item i of the thread: first + 64 i
    uint32_t k[kSmallItems], v[kSmallItems], rank[kSmallItems];
    uint32_t lo = ~0u, hi = 0u;
#pragma unroll
    for (int i = 0; i < kSmallItems; i++) {
        if (i < steps) {
            const int j = first + i * kWave;
            k[i] = j < n ? kin[j] : ~0u;
            v[i] = j < n ? un.src[j] : 0u;
        }
    }
#pragma unroll
    for (int i = 0; i < kSmallItems; i++) {
        if (i < steps) {
            lo = min(lo, k[i]);
            hi = max(hi, k[i] == ~0u ? 0u : k[i]);
        }
    }
    for (int m = 32; m > 0; m >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, m, kWave));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, m, kWave));
    }
    if (lane == 0) {
        s_lo[w] = lo;
        s_hi[w] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSmallWaves; q++) {
        lo = min(lo, s_lo[q]);
        hi = max(hi, s_hi[q]);
    }
    const uint32_t top = lo == ~0u ? 0u : hi - lo + 1u;  // a culled pair's key
    const int width = top ? 32 - __clz((int)top) : 0;
    const int passes = (width + kSmallBits - 1) / kSmallBits;
    const int bits = passes ? (width + passes - 1) / passes : 0;
#pragma unroll
    for (int i = 0; i < kSmallItems; i++)
        if (i < steps) k[i] = k[i] == ~0u ? top : k[i] - lo;
    for (int p = 0; p < passes; p++) {
        const int shift = p * bits;
        const uint32_t mask = (1u << bits) - 1u;
        for (int d = tid; d < kSmallWaves * kSmallDigits / 2; d += kSmallThreads)
            reinterpret_cast<uint32_t*>(&s_cnt[0][0])[d] = 0u;
        __syncthreads();
        // stable rank inside the wave's run: earlier steps (LDS count) + earlier lanes
#pragma unroll
        for (int i = 0; i < kSmallItems; i++) {
            if (i < steps) {
                const uint32_t d = (k[i] >> shift) & mask;
                const uint64_t peers = match_digit(d, true, bits);
                const uint32_t before = s_cnt[w][d];
                const uint32_t below = (uint32_t)__popcll(peers & lanemask_lt());
                rank[i] = before + below;
                if (below == 0) s_cnt[w][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
            }
        }
        __syncthreads();
        // a digit a thread: offsets of the waves after the smaller digits' items
        uint32_t c[kSmallWaves], run = 0;
        if (tid < kSmallDigits)
#pragma unroll
            for (int q = 0; q < kSmallWaves; q++) {
                c[q] = run;
                run += s_cnt[q][tid];
            }
        uint32_t tot;
        const uint32_t start = block_excl_scan(run, s_w, tot);
        if (tid < kSmallDigits)
#pragma unroll
            for (int q = 0; q < kSmallWaves; q++) s_cnt[q][tid] = (uint16_t)(start + c[q]);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSmallItems; i++) {
            if (i < steps) {
                const uint32_t to = s_cnt[w][(k[i] >> shift) & mask] + rank[i];
                s_key[to] = k[i];
                s_val[to] = v[i];
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSmallItems; i++) {
            if (i < steps) {
                k[i] = s_key[first + i * kWave];
                v[i] = s_val[first + i * kWave];
            }
        }
    }
    // the sorted pairs, and the scan of their counts
    const uint32_t esc = ~0u >> un.pbits, pmask = (1u << un.pbits) - 1u;
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kSmallItems; i++) {
        if (i < steps) {
            const int j = first + i * kWave;
            uint32_t c = v[i] >> un.pbits;
            if (c == esc) c = un.cnt[v[i] & pmask];
            const uint32_t inc = wave_incl_scan(c);
            rank[i] = sum + inc - c;
            sum += (uint32_t)bcast((int)inc, kWave - 1);
            if (j < n) {
                kout[j] = k[i] == top ? ~0u : k[i] + lo;
                vout[j] = v[i];
            }
        }
    }
    if (lane == 0) s_w[w] = sum;
    __syncthreads();
    uint32_t base = 0, total = 0;
#pragma unroll
    for (int q = 0; q < kSmallWaves; q++) {
        base += q < w ? s_w[q] : 0u;
        total += s_w[q];
    }
#pragma unroll
    for (int i = 0; i < kSmallItems; i++)
        if (i < steps && first + i * kWave < n) off[first + i * kWave] = base + rank[i];
    if (tid == 0) {
        *total_out = total;
        cap_check(total, chk, flags);
    }
}

}  // namespace

size_t scan_scratch_words(int64_t max_n) {
    return (size_t)kScanHeader + 2 * (size_t)((max_n + kScanTile - 1) / kScanTile) + 16;
}

namespace {

hipError_t scan_launch(uint32_t* data, int64_t max_n, const uint32_t* d_cnt, int64_t per, int64_t mul,
                       int64_t add, uint32_t* total_out, uint32_t* scratch, uint32_t* flags,
                       hipStream_t st, const CapCheck* chk, const ScanUnpack* un = nullptr) {
    CapCheck ck = {};
    if (chk) ck = *chk;
    // nothing to scan: done, unless a capacity check must still see the 0 total
    if (max_n <= 0 && !ck.used) return hipSuccess;
    if (max_n < 0) max_n = 0;
    // whole-tile vector accesses need 16-byte alignment
    if (reinterpret_cast<uintptr_t>(data) % 16 != 0 || (d_cnt && (per <= 0 || mul <= 0 || add < 0)) ||
        (un && (reinterpret_cast<uintptr_t>(un->src) % 16 != 0 || un->pbits < 1 || un->pbits > 31)))
        return hipErrorInvalidValue;
    const ScanUnpack u = un ? *un : ScanUnpack{nullptr, nullptr, 1};
    if (max_n > kWideScan) {
        const int64_t ntw = (max_n + kWideThreads * kScanItems - 1) / (kWideThreads * kScanItems);
        if (un)
            hipLaunchKernelGGL((k_scan<kWideThreads, true>), dim3((unsigned)ntw), dim3(kWideThreads), 0, st, data,
                               max_n, d_cnt, per, mul, add, total_out, scratch, flags, ck, u);
        else
            hipLaunchKernelGGL((k_scan<kWideThreads, false>), dim3((unsigned)ntw), dim3(kWideThreads), 0, st, data,
                               max_n, d_cnt, per, mul, add, total_out, scratch, flags, ck, u);
        return hipGetLastError();
    }
    const int64_t nt = std::max<int64_t>((max_n + kScanTile - 1) / kScanTile, 1);
    if (nt > ((int64_t)1 << 31)) return hipErrorInvalidValue;
    if (un)
        hipLaunchKernelGGL((k_scan<kThreads, true>), dim3((unsigned)nt), dim3(kThreads), 0, st, data, max_n, d_cnt,
                           per, mul, add, total_out, scratch, flags, ck, u);
    else
        hipLaunchKernelGGL((k_scan<kThreads, false>), dim3((unsigned)nt), dim3(kThreads), 0, st, data, max_n, d_cnt,
                           per, mul, add, total_out, scratch, flags, ck, u);
    return hipGetLastError();
}

}  // namespace

hipError_t exclusive_scan_u32_dev(uint32_t* data, int64_t max_n, const uint32_t* d_cnt, int64_t per,
                                  int64_t mul, int64_t add, uint32_t* total_out, uint32_t* scratch,
                                  uint32_t* flags, hipStream_t st) {
    return scan_launch(data, max_n, d_cnt, per, mul, add, total_out, scratch, flags, st, nullptr);
}

hipError_t exclusive_scan_u32(uint32_t* data, int64_t n, uint32_t* total_out, uint32_t* scratch,
                              uint32_t* flags, hipStream_t st, const CapCheck* chk) {
    return scan_launch(data, n, nullptr, 1, 1, 0, total_out, scratch, flags, st, chk);
}

hipError_t exclusive_scan_u32_unpack(uint32_t* data, const ScanUnpack& un, int64_t n, uint32_t* total_out,
                                     uint32_t* scratch, uint32_t* flags, hipStream_t st, const CapCheck* chk) {
    return scan_launch(data, n, nullptr, 1, 1, 0, total_out, scratch, flags, st, chk, &un);
}

// sized for the smallest block (2048 items)
size_t radix_hist_words(int64_t max_n) { return (size_t)256 * ((max_n + kTile / 2 - 1) / (kTile / 2)) + 16; }

namespace {

// one pass over `bits` bits at `shift`; blocks of 256 x ITEMS items
template <int ITEMS, int NV>
hipError_t radix_pass(const uint32_t* ki, uint32_t* ko, const ValArrays<NV>& va, int64_t max_n,
                      const uint32_t* d_n, int shift, int bits, uint32_t* hist,
                      uint32_t* scan_scratch, uint32_t* flags, hipStream_t st) {
    const uint32_t nb = (uint32_t)((max_n + kThreads * ITEMS - 1) / (kThreads * ITEMS));
    const uint32_t grid = (nb + kXcds - 1) / kXcds * kXcds;
    hipLaunchKernelGGL(k_radix_hist<ITEMS>, dim3(nb), dim3(kThreads), 0, st, ki, d_n, max_n, shift,
                       bits, hist);
    hipError_t e = exclusive_scan_u32_dev(hist, ((int64_t)1 << bits) * nb, d_n, kThreads * ITEMS,
                                          (int64_t)1 << bits, 0, nullptr, scan_scratch, flags, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_radix_scatter<ITEMS, NV>), dim3(grid), dim3(kThreads), 0, st, ki, ko, va,
                       d_n, max_n, shift, bits, hist);
    return hipGetLastError();
}

// LSD passes of equal digit widths (at most 8 bits) over [lo, hi); K[2] and
// V[c][2] are the ping-pong buffers; returns the side holding the result
template <int NV>
int radix_sort_impl(uint32_t* K[2], uint32_t* V[NV][2], int64_t max_n, const uint32_t* d_n, int lo,
                    int hi, uint32_t* hist, uint32_t* scan_scratch, uint32_t* flags, hipStream_t st,
                    hipError_t* err) {
    *err = hipSuccess;
    if (max_n <= 0 || hi <= lo) return 0;
    const int total = hi - lo;
    const int passes = (total + 7) / 8;
    int cur = 0;
    int shift = lo;
    for (int p = 0; p < passes; p++) {
        const int bits = (total - (shift - lo) + (passes - p) - 1) / (passes - p);
        ValArrays<NV> va;
        for (int c = 0; c < NV; c++) {
            va.in[c] = V[c][cur];
            va.out[c] = V[c][cur ^ 1];
        }
        // large single-value inputs (the depth sort, whose one value word
        // packs the pair and its entry count): 4096 items per block (on the
        // 20M pairs of the large scene 0.06 ms faster over the four passes
        // than 8192, and 0.08 ms faster than 2048); the block sort of a list
        // capacity past 2^27 4096 (fewer digit counts to scan); the others
        // 2048: a sort of a few million items still gives every CU several
        // blocks, and a block sort of tens of millions of entries gains from
        // the shorter blocks (measured: at 70M capacity 2048 beats 4096 by
        // 15 us, at 333M it loses by 120 us)
        if (NV == 1 && max_n > ((int64_t)1 << 22))
            *err = radix_pass<16, NV>(K[cur], K[cur ^ 1], va, max_n, d_n, shift, bits, hist,
                                      scan_scratch, flags, st);
        else if (NV == 3 && max_n > ((int64_t)1 << 27))
            *err = radix_pass<16, NV>(K[cur], K[cur ^ 1], va, max_n, d_n, shift, bits, hist,
                                      scan_scratch, flags, st);
        else
            *err = radix_pass<8, NV>(K[cur], K[cur ^ 1], va, max_n, d_n, shift, bits, hist,
                                     scan_scratch, flags, st);
        if (*err != hipSuccess) return cur;
        shift += bits;
        cur ^= 1;
    }
    return cur;
}

}  // namespace

int radix_sort_pairs(uint32_t* ka, uint32_t* va, uint32_t* kb, uint32_t* vb, int64_t max_n,
                     const uint32_t* d_n, int lo, int hi, uint32_t* hist, uint32_t* scan_scratch,
                     uint32_t* flags, hipStream_t st, hipError_t* err) {
    uint32_t* K[2] = {ka, kb};
    uint32_t* V[1][2] = {{va, vb}};
    return radix_sort_impl<1>(K, V, max_n, d_n, lo, hi, hist, scan_scratch, flags, st, err);
}

int radix_sort_kv3(uint32_t* K[2], uint32_t* V[3][2], int64_t max_n, const uint32_t* d_n, int lo,
                   int hi, uint32_t* hist, uint32_t* scan_scratch, uint32_t* flags, hipStream_t st,
                   hipError_t* err) {
    return radix_sort_impl<3>(K, V, max_n, d_n, lo, hi, hist, scan_scratch, flags, st, err);
}

bool wide_sort_kv3(const uint32_t* keys, uint32_t* V[3][2], int64_t max_n, const uint32_t* d_n, int64_t digits,
                   uint32_t* scratch, int64_t scratch_words, uint32_t* scan_scratch, uint32_t* flags,
                   int32_t* ranges, hipStream_t st, hipError_t* err) {
    *err = hipSuccess;
    if (digits < 1 || digits > kWideDigits || max_n <= 0) return false;
    const int64_t nb = (max_n + kWideTile - 1) / kWideTile;
    const int ch = max_n > ((int64_t)1 << 25) ? 8 : 1;
    const int64_t groups = (nb + ch - 1) / ch;
    const int64_t hist_words = (digits * groups + 3) / 4 * 4, row_words = ch > 1 ? (digits * nb + 1) / 2 : 0;
    if (hist_words + row_words > scratch_words) return false;
    uint32_t* hist = scratch;
    uint16_t* rows = reinterpret_cast<uint16_t*>(scratch + hist_words);
    hipLaunchKernelGGL(k_wide_hist, dim3((unsigned)groups), dim3(kWideBlock), 0, st, keys, d_n, max_n,
                       (int)digits, ch, rows, hist);
    *err = exclusive_scan_u32_dev(hist, digits * groups, d_n, (int64_t)kWideTile * ch, digits, 0, nullptr,
                                  scan_scratch, flags, st);
    if (*err != hipSuccess) return true;
    ValArrays<3> va;
    for (int c = 0; c < 3; c++) {
        va.in[c] = V[c][0];
        va.out[c] = V[c][1];
    }
    const dim3 grid((unsigned)((nb + kXcds - 1) / kXcds * kXcds));
    const size_t lds = wide_lds((int)digits);
    auto scatter = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(kWideBlock), lds, st, keys, va, d_n, max_n, (int)digits, ch, rows,
                           hist, ranges);
    };
    if (digits <= 64) scatter(k_wide_scatter<6>);
    else if (digits <= 256) scatter(k_wide_scatter<8>);
    else if (digits <= 512) scatter(k_wide_scatter<9>);
    else if (digits <= 1024) scatter(k_wide_scatter<10>);
    else scatter(k_wide_scatter<11>);
    *err = hipGetLastError();
    return true;
}

hipError_t small_sort_scan(const uint32_t* keys, uint32_t* kout, uint32_t* vout, int64_t n, const ScanUnpack& un,
                           uint32_t* off, uint32_t* total_out, uint32_t* flags, hipStream_t st,
                           const CapCheck& chk) {
    if (n < 1 || n > kSmallSort) return hipErrorInvalidValue;
    const int steps = (int)((n + kSmallThreads - 1) / kSmallThreads);
    hipLaunchKernelGGL(k_small_sort, dim3(1), dim3(kSmallThreads), 2 * sizeof(uint32_t) * kSmallThreads * steps, st,
                       keys, kout, vout, (int)n, steps, un, off, total_out, flags, chk);
    return hipGetLastError();
}

}  // namespace gs
