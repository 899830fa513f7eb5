// kernels.hip -- gfx950 kernels of the per-view 4pi track finder.
//
// Pipeline (paper Sec. 2, tracking paragraph; hash cells after the Sec. 3
// footnote), for a batch of views packed one after another:
//   bin      bounding box per view, counting sort of grains into cells
//   seeds    all pairs closer than R, ordered by line class (one wave per
//            anchor grain)
//   count    grains within r of each seed's infinite line (one lane per seed,
//            over line grids filled per class; small calls over the cells)
//   members  grain lists of the seeds that reach n_min
//   merge    exclusive association, rounds of deterministic reservations
//   fit      track order, grain order, least-squares direction
// Every geometric decision is exact integer arithmetic; floating point only
// chooses which cells to visit and carries a safety margin.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "deal.h"
#include "emt_dev.h"
#include "seed_rows.h"

namespace emt {

namespace {

// Tuning constants; -D on the compiler line overrides them (the counting
// kernel's tiles come from tile_table.h, through emt_dev.h).
constexpr float kMargin = 4.0f;  // units added to every cell window
constexpr int kScanItems = 8;
constexpr int kScanTile = kBlock * kScanItems;

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

__device__ __forceinline__ unsigned long long lanes_below() {
    return (1ull << lane_id()) - 1ull;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ __forceinline__ float wave_min(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o));
    return v;
}

__device__ __forceinline__ float wave_max(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

// Make this lane's global writes visible to the other lanes of its wave.
__device__ __forceinline__ void wave_sync_mem() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Adds a workgroup's total of wave-uniform values v (one per wave) to one
// of the kPartSlots counters of total `which`: the waves' values are summed
// in LDS, then one atomic per workgroup, the workgroups spread over the
// counters. Every thread of the workgroup must call it (it synchronises the
// workgroup twice).
__device__ __forceinline__ void add_spread(unsigned long long *part64, int which,
                                           unsigned long long v) {
    __shared__ unsigned long long s_part[16];  // waves of the largest workgroup
    if (lane_id() == 0) s_part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (uint32_t w = 0; w < blockDim.x / 64; ++w) t += s_part[w];
        if (t)
            atomicAdd(&part64[(which * kPartSlots + (int)(blockIdx.x % kPartSlots)) * kPartStride], t);
    }
    __syncthreads();  // s_part is free again for the next call
}

// (__ballot turns its argument into an integer and compares that)
__device__ __forceinline__ unsigned long long ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

__device__ __forceinline__ uint32_t grid_tid() { return blockIdx.x * blockDim.x + threadIdx.x; }
__device__ __forceinline__ uint32_t grid_threads() { return gridDim.x * blockDim.x; }

// Inclusive prefix sum over the 64 lanes with DPP row shifts and row
// broadcasts (no LDS traffic).
__device__ __forceinline__ uint32_t wave_incl_scan_dpp(uint32_t x) {
    uint32_t v = x;
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint32_t uniform(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

__device__ __forceinline__ unsigned long long uniform(unsigned long long x) {
    return ((unsigned long long)uniform((uint32_t)(x >> 32)) << 32) | uniform((uint32_t)x);
}

// ------------------------------------------------------------------ scan

// Exclusive scan inside one block of kThreads threads.
template <int kThreads = kBlock>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *total) {
    __shared__ uint32_t wsum[kThreads / 64];
    const uint32_t incl = wave_incl_scan_dpp(v);
    const int w = threadIdx.x >> 6;
    if (lane_id() == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t off = 0, tot = 0;
    for (int i = 0; i < kThreads / 64; ++i) {
        if (i < w) off += wsum[i];
        tot += wsum[i];
    }
    __syncthreads();
    *total = tot;
    return off + incl - v;
}

template <int kThreads = kBlock>
__device__ __forceinline__ uint32_t block_sum(uint32_t v) {
    __shared__ uint32_t wsum[kThreads / 64];
    v = wave_sum(v);
    if (lane_id() == 0) wsum[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t tot = 0;
    for (int i = 0; i < kThreads / 64; ++i) tot += wsum[i];
    __syncthreads();
    return tot;
}

__device__ __forceinline__ uint32_t scan_len(const uint32_t *n_dev, uint32_t n_cap) {
    if (!n_dev) return n_cap;
    const uint32_t n = *n_dev;
    return n < n_cap ? n : n_cap;
}

// Items [base, base + kItems) of an array of n, zero past its end; base is a
// multiple of kItems and the array starts on a 16-byte boundary.
template <int kItems>
__device__ __forceinline__ void load_items(const uint32_t *in, uint32_t base, uint32_t n,
                                           uint32_t (&v)[kItems]) {
    if (kItems % 4 == 0 && base + kItems <= n) {
#pragma unroll
        for (int k = 0; k < kItems; k += 4) {
            const uint4 q = *reinterpret_cast<const uint4 *>(in + base + k);
            v[k] = q.x;
            v[k + 1] = q.y;
            v[k + 2] = q.z;
            v[k + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kItems; ++k) v[k] = base + k < n ? in[base + k] : 0u;
    }
}

template <int kItems>
__device__ __forceinline__ void store_items(uint32_t *out, uint32_t base, uint32_t n,
                                            const uint32_t (&v)[kItems]) {
    if (kItems % 4 == 0 && base + kItems <= n) {
#pragma unroll
        for (int k = 0; k < kItems; k += 4)
            *reinterpret_cast<uint4 *>(out + base + k) =
                make_uint4(v[k], v[k + 1], v[k + 2], v[k + 3]);
    } else {
#pragma unroll
        for (int k = 0; k < kItems; ++k)
            if (base + k < n) out[base + k] = v[k];
    }
}

// What the last workgroup of a scan does with the total.
enum ScanEnd { kEndTotal, kEndSeeds, kEndMembers };
struct ScanOut {
    uint32_t *out, *total;  // total may be null
    Counters *cnt;
    const unsigned long long *part64;
    unsigned long long seed_cap;
};

// Called by every lane of one wave, once per scan of n items.
template <ScanEnd kEnd>
__device__ __forceinline__ void scan_end(const ScanOut &o, uint32_t n, uint32_t total) {
    if constexpr (kEnd == kEndTotal) {
        if (lane_id() != 0) return;
        if (o.total) *o.total = total;
    } else if constexpr (kEnd == kEndSeeds) {
        // The seed total of the uint32 scan, replaced by the exact 64-bit
        // count (saturated to 2^32 - 1), and the number of seeds the later
        // stages take: none when they do not fit the seed buffer (the host
        // then re-runs the call with a larger one, or fails if no buffer can
        // hold them). One of the spread partial sums per lane.
        const unsigned long long t = wave_sum(o.part64[lane_id() * kPartStride]);
        if (lane_id() != 0) return;
        Counters *cnt = o.cnt;
        cnt->seeds64 = t;
        const uint32_t ns = t > 0xffffffffull ? 0xffffffffu : (uint32_t)t;
        cnt->n_seeds = ns;
        cnt->n_seeds_ok = ns <= o.seed_cap ? ns : 0u;
        cnt->pass_words = (uint32_t)(((unsigned long long)cnt->n_seeds_ok + 31ull) / 32ull);
    } else {
        // Likewise for the member entries (the scan of candidate counts): a
        // total that wrapped reads as an overflow, so no stage uses the
        // wrapped offsets. The counting kernel's tests and hits too (it has
        // finished).
        const unsigned long long m = wave_sum(o.part64[(kPartSlots + lane_id()) * kPartStride]);
        const unsigned long long t = wave_sum(o.part64[(2 * kPartSlots + lane_id()) * kPartStride]);
        const unsigned long long h = wave_sum(o.part64[(3 * kPartSlots + lane_id()) * kPartStride]);
        if (lane_id() != 0) return;
        Counters *cnt = o.cnt;
        cnt->tests = t;
        cnt->hits = h;
        cnt->members64 = m;
        cnt->n_members = m > 0xffffffffull ? 0xffffffffu : (uint32_t)m;
    }
    o.out[n] = total;
}

// The sum of each tile of kBlock * kItems items (their popcounts with kPopc).
template <bool kPopc, int kItems>
__global__ void __launch_bounds__(kBlock) k_scan_part(const uint32_t *in, const uint32_t *n_dev,
                                                      uint32_t n_cap, uint32_t *part) {
    const uint32_t n = scan_len(n_dev, n_cap);
    if (blockIdx.x * (kBlock * kItems) >= n) return;
    uint32_t v[kItems], sum = 0;
    load_items(in, (blockIdx.x * kBlock + threadIdx.x) * kItems, n, v);
#pragma unroll
    for (int k = 0; k < kItems; ++k) sum += kPopc ? (uint32_t)__popc(v[k]) : v[k];
    sum = block_sum(sum);
    if (threadIdx.x == 0) part[blockIdx.x] = sum;
}

// The tiles' sums to exclusive offsets, where there are too many of them for
// every later workgroup to add up those before its own.
constexpr int kScanBlock = 1024;
__global__ void __launch_bounds__(kScanBlock) k_scan_parts(uint32_t *part, uint32_t tile,
                                                           const uint32_t *n_dev, uint32_t n_cap) {
    const uint32_t n = scan_len(n_dev, n_cap);
    const uint32_t nb = n / tile + (n % tile != 0 ? 1u : 0u);
    uint32_t carry = 0;
    for (uint32_t base = 0; base < nb; base += kScanBlock * 4) {
        const uint32_t at = base + threadIdx.x * 4;
        uint32_t v[4], tot;
        load_items(part, at, nb, v);
        uint32_t run = carry + block_excl_scan<kScanBlock>(v[0] + v[1] + v[2] + v[3], &tot);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t x = v[k];
            v[k] = run;
            run += x;
        }
        store_items(part, at, nb, v);
        carry += tot;
    }
}

// Offset of this workgroup's tile: the sum of the earlier tiles, or what
// k_scan_parts left. Called by the whole workgroup. Nothing is before the first
// tile, and where there are no items at all nobody has written its place.
template <bool kDirect>
__device__ __forceinline__ uint32_t tile_offset(const uint32_t *part) {
    if (blockIdx.x == 0) return 0u;
    if constexpr (!kDirect) return part[blockIdx.x];
    uint32_t sum = 0;
#pragma unroll 4
    for (uint32_t i = threadIdx.x; i < blockIdx.x; i += kBlock) sum += part[i];
    return block_sum(sum);
}

template <bool kDirect, ScanEnd kEnd>
__global__ void __launch_bounds__(kBlock) k_scan_apply(const uint32_t *in, const uint32_t *n_dev,
                                                       uint32_t n_cap, const uint32_t *part,
                                                       ScanOut o) {
    const uint32_t n = scan_len(n_dev, n_cap);
    if (blockIdx.x > 0 && blockIdx.x * kScanTile >= n) return;
    const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    uint32_t v[kScanItems], sum = 0;
    load_items(in, base, n, v);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) sum += v[k];
    const uint32_t off = tile_offset<kDirect>(part);
    uint32_t tot;
    uint32_t run = off + block_excl_scan(sum, &tot);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const uint32_t x = v[k];
        v[k] = run;
        run += x;
    }
    store_items(o.out, base, n, v);
    if (n - blockIdx.x * kScanTile <= (uint32_t)kScanTile && threadIdx.x < 64)
        scan_end<kEnd>(o, n, off + tot);
}

template <ScanEnd kEnd>
__global__ void __launch_bounds__(kScanBlock) k_scan_one(const uint32_t *in, const uint32_t *n_dev,
                                                         uint32_t n_cap, ScanOut o) {
    const uint32_t n = scan_len(n_dev, n_cap);
    uint32_t carry = 0;
    for (uint32_t first = 0; first < n; first += kScanBlock * kScanItems) {
        const uint32_t base = first + threadIdx.x * kScanItems;
        uint32_t v[kScanItems], sum = 0, tot;
        load_items(in, base, n, v);
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) sum += v[k];
        uint32_t run = carry + block_excl_scan<kScanBlock>(sum, &tot);
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const uint32_t x = v[k];
            v[k] = run;
            run += x;
        }
        store_items(o.out, base, n, v);
        carry += tot;
    }
    if (threadIdx.x < 64) scan_end<kEnd>(o, n, carry);
}

// Bound by launches: a scan is one to three kernels of 3 to 5 us. Up to
// kScanDirect tiles a workgroup adds up the sums before its own (32 KB from L2
// at most; with 256 tiles one c2 view 735 us, with 2048 713, one c5 view 3541,
// with more 3509; calls of eight c5 views do not care). Up to kScanOne items
// one workgroup scans alone, 8192 at a time: one view of 900 grains 177 us, 182
// without, and no difference between 16 and 128 thousand.
constexpr uint32_t kScanDirect = 8192;
constexpr uint32_t kScanOne = 32768;

// o.out[i] = sum of in[0..i) for i <= n, n = min(*n_dev, n_cap) (n_cap if no
// n_dev), then kEnd with the total. In and out start on 16-byte boundaries.
template <ScanEnd kEnd>
void scan_excl(const uint32_t *in, const uint32_t *n_dev, uint32_t n_cap, uint32_t *part,
               const ScanOut &o, hipStream_t s) {
    if (n_cap <= kScanOne) {
        k_scan_one<kEnd><<<1, kScanBlock, 0, s>>>(in, n_dev, n_cap, o);
        return;
    }
    const uint32_t nb = n_cap / kScanTile + 1;
    k_scan_part<false, kScanItems><<<nb, kBlock, 0, s>>>(in, n_dev, n_cap, part);
    if (nb <= kScanDirect) {
        k_scan_apply<true, kEnd><<<nb, kBlock, 0, s>>>(in, n_dev, n_cap, part, o);
    } else {
        k_scan_parts<<<1, kScanBlock, 0, s>>>(part, kScanTile, n_dev, n_cap);
        k_scan_apply<false, kEnd><<<nb, kBlock, 0, s>>>(in, n_dev, n_cap, part, o);
    }
}

// ------------------------------------------------------------------- bin

// The call's sizes and view records, from the host's mapped memory, and
// everything that starts at zero. (A copy command a table cost 3 us each.)
__global__ void __launch_bounds__(kBlock) k_zero(DevPtrs d) {
    __shared__ BatchDesc s_desc;  // the host's words, read once a workgroup
    constexpr uint32_t kDescWords = sizeof(BatchDesc) / 4, kGridWords = sizeof(ViewGrid) / 4;
    const uint32_t tid = grid_tid();
    if (threadIdx.x < kDescWords) {
        const uint32_t w = reinterpret_cast<const uint32_t *>(d.in_desc)[threadIdx.x];
        reinterpret_cast<uint32_t *>(&s_desc)[threadIdx.x] = w;
        if (blockIdx.x == 0) reinterpret_cast<uint32_t *>(d.desc)[threadIdx.x] = w;
    }
    __syncthreads();
    const uint32_t n_views = s_desc.n_views, n_cells = s_desc.n_cells;
    if (tid == 0) {
        Counters z = {};
        *d.cnt = z;
        d.view_tr_off[0] = 0;
    }
    const uint32_t *in = reinterpret_cast<const uint32_t *>(d.in_grids);
    uint32_t *grids = reinterpret_cast<uint32_t *>(d.grids);
    for (uint32_t i = tid; i < n_views * kGridWords; i += grid_threads()) grids[i] = in[i];
    for (uint32_t i = tid; i < (uint32_t)kGrabWords; i += grid_threads()) d.grab[i] = 0;
    for (uint32_t i = tid; i < (uint32_t)kPartWords; i += grid_threads()) d.part64[i] = 0;
    for (uint32_t v = tid; v < n_views; v += grid_threads()) {
        d.view_seeds[v] = 0;
        d.view_cand[v] = 0;
        d.view_ntr[v] = 0;
        d.view_cursor[v] = 0;
        d.view_tail[v] = 0;
    }
    for (uint32_t i = tid; i < n_cells; i += grid_threads()) d.cell_count[i] = 0;
}

// The views' grains into one packed array, the bounding box of every view
// (grid origin) and the view index of each grain. A view is read from where
// it is, in device memory or the host's mapped memory, as consecutive words:
// of a tile of kBlock grains a thread reads words t, kBlock + t and
// 2 kBlock + t, which are one x, one y and one z as kBlock = 1 (mod 3). (A
// copy command a view cost 2.3 us: 150 us for 64 views.)
__global__ void __launch_bounds__(kBlock) k_bbox(int32_t *xyz, const int32_t *const *src,
                                                 ViewGrid *grids, uint32_t *view_of,
                                                 const BatchDesc *desc) {
    static_assert(kBlock % 3 == 1, "a thread's words are of three axes");
    const uint32_t v = blockIdx.y;
    if (v >= desc->n_views) return;
    const uint32_t off = grids[v].grain_off, n = grids[v].n;
    const uint32_t first = threadIdx.x % 3u;  // axis of the thread's first word
    int l[3] = {INT32_MAX, INT32_MAX, INT32_MAX};
    int h[3] = {INT32_MIN, INT32_MIN, INT32_MIN};
    if (blockIdx.x * kBlock < n) {
        const int32_t *in = src[v];
        int32_t *out = xyz + 3 * (size_t)off;
        for (uint32_t t = blockIdx.x * kBlock; t < n; t += gridDim.x * kBlock) {
            if (t + threadIdx.x < n) view_of[(size_t)off + t + threadIdx.x] = v;
            const uint32_t end = 3u * min(n - t, (uint32_t)kBlock);
#pragma unroll
            for (uint32_t m = 0; m < 3; ++m) {
                const uint32_t w = m * kBlock + threadIdx.x;
                if (w >= end) continue;
                const int x = in[3 * (size_t)t + w];
                out[3 * (size_t)t + w] = x;
                l[m] = min(l[m], x);
                h[m] = max(h[m], x);
            }
        }
    }
    // word m of a thread is of axis (first + m) mod 3
    int lo[3], hi[3];
#pragma unroll
    for (uint32_t m = 0; m < 3; ++m) {
        const uint32_t k = m + 3u - first;
        lo[m] = k % 3u == 0 ? l[0] : k % 3u == 1 ? l[1] : l[2];
        hi[m] = k % 3u == 0 ? h[0] : k % 3u == 1 ? h[1] : h[2];
    }
    for (int m = 0; m < 3; ++m) {
        for (int o = 32; o > 0; o >>= 1) {
            lo[m] = min(lo[m], __shfl_xor(lo[m], o));
            hi[m] = max(hi[m], __shfl_xor(hi[m], o));
        }
    }
    // one atomic per workgroup and value: atomics on the six words of a
    // view serialise in L2, so they are reduced across the waves first
    __shared__ int s_box[kBlock / 64][6];
    const int wave = threadIdx.x >> 6;
    if (lane_id() == 0)
        for (int m = 0; m < 3; ++m) {
            s_box[wave][m] = lo[m];
            s_box[wave][3 + m] = hi[m];
        }
    __syncthreads();
    if (threadIdx.x < 6 && n > 0) {
        const int m = (int)threadIdx.x;
        int b = s_box[0][m];
        for (int w = 1; w < kBlock / 64; ++w)
            b = m < 3 ? min(b, s_box[w][m]) : max(b, s_box[w][m]);
        if (m < 3)
            atomicMin(&grids[v].lo[m], b);
        else
            atomicMax(&grids[v].hi[m - 3], b);
    }
}

// Cell geometry per view: the requested edges, doubled until the grid has at
// most cell_cap cells. A view whose span exceeds the limit is marked: its
// grains still go through the binning (into one cell, so every later view
// keeps its place in the sorted arrays) but it produces no seeds.
__global__ void k_grid(ViewGrid *grids, LineGrid *lines, uint32_t *pool, uint32_t *coarse,
                       int nc, const BatchDesc *desc, Params P) {
    const uint32_t v = grid_tid();
    if (v >= desc->n_views) return;
    ViewGrid G = grids[v];
    long long span[3];
    for (int m = 0; m < 3; ++m) {
        if (G.n == 0) {
            G.lo[m] = 0;
            G.hi[m] = 0;
        }
        span[m] = (long long)G.hi[m] - (long long)G.lo[m];
        if (span[m] > kSpanMax) G.err = 1;
    }
    // cell edges: fixed, or by the view's grain density (bounding box)
    int b = 0;
    const double vol_um3 = (double)(span[0] + 1) * (double)(span[1] + 1) *
                           (double)(span[2] + 1) * 1e-6;
    const double per_1000 = 1000.0 * (double)G.n / vol_um3;
    double edge = kCellEdge0;
    while (b < kCellBuckets - 1 && per_1000 >= edge) {
        ++b;
        edge *= 2.0;
    }
    for (int m = 0; m < 3; ++m) G.cell[m] = P.auto_cells ? P.cell_tab[b][m] : P.cell_req[m];
    if (G.err) {
        for (int m = 0; m < 3; ++m) {
            G.cell[m] = 1;
            G.dims[m] = 1;
        }
        grids[v] = G;
        return;
    }
    for (;;) {
        long long tot = 1;
        for (int m = 0; m < 3; ++m) {
            G.dims[m] = (int)(span[m] / G.cell[m] + 1);
            tot *= G.dims[m];
        }
        if (tot <= (long long)G.cell_cap) break;
        for (int m = 0; m < 3; ++m) G.cell[m] *= 2;
    }
    grids[v] = G;
    if (nc == 1) return;  // the lines are not classed
    // the grid used unless its lists overflow their share, and a coarser one
    // whose lists cannot: a rectangle covers at most 2 x 2 cells, six words
    lines[2 * v] = line_grid(G.n, span, P.line_tab[b], nc, P.r, 2.0 / 3.0);
    lines[2 * v + 1] = line_grid(G.n, span, P.line_tab[b], nc, P.r, 2.0);
    for (int i = 0; i < 2 * nc; ++i) pool[(size_t)v * 2 * nc + i] = 0u;
    coarse[v] = 0u;
}

__device__ __forceinline__ int axis_cell(const ViewGrid &G, int m, int x) {
    const long long c = ((long long)x - (long long)G.lo[m]) / G.cell[m];
    return (int)(c < 0 ? 0 : (c >= G.dims[m] ? G.dims[m] - 1 : c));
}

__device__ __forceinline__ uint32_t cell_index(const ViewGrid &G, int x, int y, int z) {
    const int cx = axis_cell(G, 0, x), cy = axis_cell(G, 1, y), cz = axis_cell(G, 2, z);
    return G.cell_off + (uint32_t)((cz * G.dims[1] + cy) * G.dims[0] + cx);
}

__global__ void __launch_bounds__(kBlock) k_hist(const int32_t *xyz, const ViewGrid *grids,
                                                 uint32_t *cell_of, uint32_t *rank,
                                                 uint32_t *cell_count, const BatchDesc *desc) {
    const uint32_t v = blockIdx.y;
    if (v >= desc->n_views) return;
    const ViewGrid G = grids[v];
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < G.n; i += gridDim.x * blockDim.x) {
        const size_t g = (size_t)G.grain_off + i;
        const uint32_t c = cell_index(G, xyz[3 * g], xyz[3 * g + 1], xyz[3 * g + 2]);
        cell_of[g] = c;
        rank[g] = atomicAdd(&cell_count[c], 1u);
    }
}

// Sorted grains: coordinates relative to the view origin (0 .. 2^18) and
// the input index within the view.
__global__ void __launch_bounds__(kBlock) k_scatter(const int32_t *xyz, const ViewGrid *grids,
                                                    const uint32_t *cell_of, const uint32_t *rank,
                                                    const uint32_t *cell_start, int4 *sg,
                                                    const BatchDesc *desc) {
    const uint32_t v = blockIdx.y;
    if (v >= desc->n_views) return;
    const ViewGrid G = grids[v];
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < G.n; i += gridDim.x * blockDim.x) {
        const size_t g = (size_t)G.grain_off + i;
        const uint32_t pos = cell_start[cell_of[g]] + rank[g];
        const int x = xyz[3 * g] - G.lo[0], y = xyz[3 * g + 1] - G.lo[1], z = xyz[3 * g + 2] - G.lo[2];
        sg[pos] = make_int4(x, y, z, (int)i);
    }
}

// ------------------------------------------- line walk over the binned cells
//
// Which cells can hold a grain within r of the infinite line p(t) = g + t d?
// If |k - p(t*)| <= r then |k_m - p_m(t*)| <= r on every axis. Cells along x
// are contiguous in memory, so the walk enumerates (y, z) pencils: for each
// (y, z) cell that the projected line, widened by r on each axis, crosses,
// it takes the parameter interval during which p_y and p_z stay within r of
// that cell, and the x range p_x covers on it, widened by r. That x range is
// one contiguous run of sorted grains. The traversal steps along the larger
// of |d_y|, |d_z| (axis e), and for each e cell across the f cells the line
// can reach. FP32 values only choose cells: every bound is widened by
// kMargin units, more than the rounding of any coordinate below 2^20, and
// the exact integer predicate decides each grain.
struct Run {
    uint32_t k, e;
};

struct Pencil {
    // Per line, precomputed so a pencil costs few instructions: the line is
    // oriented so that x grows with t; e and f cell intervals in t are stored
    // low end first; x and f are kept in cell units (t * ds + gs) with the
    // widening folded in; rows advance by fixed strides.
    float tlo, thi;                  // t range within rr of the grid box
    float ue_lo0, ue_step, ue_w;     // e cell j: t in [ue_lo0 + j ue_step, + ue_w]
    float uf_lo0, uf_step, uf_w;     // f cell j likewise
    float dfs, gfs, rrf, fnf;        // f in cell units, its widening, nf
    float dxs, gxs_lo, gxs_hi, fnx;  // x in cell units minus / plus widening, nx
    int nx, nf, ie1;
    uint32_t off, se, sf;            // view's first cell, row strides of e and f
    // walk state: e cell ie of [.., ie1], f cells [jf, jf1] of it
    int ie, jf, jf1;
    uint32_t row_e;                  // off + ie * se
    float ta, tb;
    bool live;

    // No divisions: reciprocals (within 1 ulp) are covered by the kMargin
    // widening.
    // ext >= 0: a finite cylinder, whose grains project at most ext units
    // beyond the seed grains; the walk then covers only that stretch.
    __device__ __forceinline__ void init(const ViewGrid *__restrict__ Gp, int4 g, int idx, int idy,
                                         int idz, int r, int ext) {
        nx = Gp->dims[0];
        const int ny = Gp->dims[1];
        const int nz = Gp->dims[2];
        const int cxi = Gp->cell[0], cyi = Gp->cell[1], czi = Gp->cell[2];
        off = Gp->cell_off;
        const float rr = (float)r + kMargin;
        // the line is undirected: take the direction with d_x >= 0
        const bool flipped = idx < 0;
        if (idx < 0) {
            idx = -idx;
            idy = -idy;
            idz = -idz;
        }
        const float icx = __builtin_amdgcn_rcpf((float)cxi);
        const float gx = (float)g.x, dx = (float)idx;
        const float gy = (float)g.y, gz = (float)g.z, dy = (float)idy, dz = (float)idz;
        const float ix = idx ? __builtin_amdgcn_rcpf(dx) : 0.0f;
        const float iy = idy ? __builtin_amdgcn_rcpf(dy) : 0.0f;
        const float iz = idz ? __builtin_amdgcn_rcpf(dz) : 0.0f;
        // parameter range in which the line is within rr of the grid box
        constexpr float kBig = 1.0e38f;
        float t1, t2;
        tlo = -kBig;
        thi = kBig;
        if (idx) {
            t1 = (-rr - gx) * ix;
            t2 = ((float)(nx * cxi - 1) + rr - gx) * ix;
            tlo = fmaxf(tlo, fminf(t1, t2));
            thi = fminf(thi, fmaxf(t1, t2));
        }
        if (idy) {
            t1 = (-rr - gy) * iy;
            t2 = ((float)(ny * cyi - 1) + rr - gy) * iy;
            tlo = fmaxf(tlo, fminf(t1, t2));
            thi = fminf(thi, fmaxf(t1, t2));
        }
        if (idz) {
            t1 = (-rr - gz) * iz;
            t2 = ((float)(nz * czi - 1) + rr - gz) * iz;
            tlo = fmaxf(tlo, fminf(t1, t2));
            thi = fminf(thi, fmaxf(t1, t2));
        }
        if (ext >= 0) {
            // the seed grains sit at t = 0 and t = 1 (t = -1 once flipped);
            // grains of the cylinder project within (ext + rr) / |d| beyond
            // them (widened for the approximate reciprocal square root)
            const float reach = ((float)ext + rr) * 1.001f *
                                __builtin_amdgcn_rsqf(dx * dx + dy * dy + dz * dz);
            const float s0 = flipped ? -1.0f : 0.0f;
            tlo = fmaxf(tlo, s0 - reach);
            thi = fminf(thi, s0 + 1.0f + reach);
        }
        const bool e_is_y = abs(idy) >= abs(idz);
        const float ge = e_is_y ? gy : gz;
        const float de = e_is_y ? dy : dz;
        const float ie_ = e_is_y ? iy : iz;
        const float ce = (float)(e_is_y ? cyi : czi);
        const int ne = e_is_y ? ny : nz;
        const float gf = e_is_y ? gz : gy;
        const float df = e_is_y ? dz : dy;
        const float if_ = e_is_y ? iz : iy;
        const float cf = (float)(e_is_y ? czi : cyi);
        nf = e_is_y ? nz : ny;
        se = e_is_y ? (uint32_t)nx : (uint32_t)(nx * ny);
        sf = e_is_y ? (uint32_t)(nx * ny) : (uint32_t)nx;
        const float ice = __builtin_amdgcn_rcpf(ce);
        const float icf = __builtin_amdgcn_rcpf(cf);
        // cell j of an axis with direction d != 0 is met for parameters
        // between (j c - rr - g)/d and ((j+1) c - 1 + rr - g)/d, the first
        // the lower one when d > 0; with d == 0 every visited cell is met for
        // all parameters
        if (de != 0.0f) {
            const float a0 = (-rr - ge) * ie_, w = (ce - 1.0f + 2.0f * rr) * ie_;
            ue_step = ce * ie_;
            ue_lo0 = de > 0.0f ? a0 : a0 + w;
            ue_w = fabsf(w);
        } else {
            ue_lo0 = -kBig;
            ue_step = 0.0f;
            ue_w = 2.0f * kBig;
        }
        if (df != 0.0f) {
            const float a0 = (-rr - gf) * if_, w = (cf - 1.0f + 2.0f * rr) * if_;
            uf_step = cf * if_;
            uf_lo0 = df > 0.0f ? a0 : a0 + w;
            uf_w = fabsf(w);
        } else {
            uf_lo0 = -kBig;
            uf_step = 0.0f;
            uf_w = 2.0f * kBig;
        }
        dfs = df * icf;
        gfs = gf * icf;
        rrf = rr * icf;
        fnf = (float)nf;
        dxs = dx * icx;
        gxs_lo = (gx - rr) * icx;
        gxs_hi = (gx + rr) * icx;
        fnx = (float)nx;
        // e cells the widened projection touches
        const float ea = ge + tlo * de, eb = ge + thi * de;
        const float elo = (de != 0.0f ? fminf(ea, eb) : ge) - rr;
        const float ehi = (de != 0.0f ? fmaxf(ea, eb) : ge) + rr;
        int ie0 = max(0, (int)floorf(fmaxf(elo * ice, -1.0f)));
        ie1 = min(ne - 1, (int)floorf(fminf(ehi * ice, (float)ne)));
        ie = ie0 - 1;
        jf = 1;
        jf1 = 0;
        row_e = 0;
        ta = tb = 0.0f;
        live = ie0 <= ie1 && tlo <= thi;
    }

    // One move of the walk, straight-line: step to the next e cell when the
    // current one is used up, then take the next f cell of it. Fills out
    // with that pencil's run or an empty run; the two cell_start loads are
    // issued but not waited on. Truncation is the floor for lower bounds
    // (clamped at 0); for upper ones it can only add a cell, which costs
    // tests, not results.
    __device__ __forceinline__ void fetch(const uint32_t *__restrict__ cs, Run &out) {
        // set-up of e cell ie + 1, taken if the current one is used up
        const bool step_e = jf > jf1;
        const int ien = ie + 1;
        const float elo = fmaf((float)ien, ue_step, ue_lo0);
        const float tan_ = fmaxf(tlo, elo), tbn = fminf(thi, elo + ue_w);
        const float fa = fmaf(tan_, dfs, gfs), fb = fmaf(tbn, dfs, gfs);
        const int jf0n = (int)fmaxf(fminf(fa, fb) - rrf, 0.0f);
        const int jf1n = min(nf - 1, (int)fmaxf(fminf(fmaxf(fa, fb) + rrf, fnf), -1.0f));
        if (step_e) {
            ie = ien;
            ta = tan_;
            tb = tbn;
            jf = tan_ <= tbn ? jf0n : 1;
            jf1 = tan_ <= tbn ? jf1n : 0;
            row_e = off + (uint32_t)ien * se;
        }
        live = live && ie <= ie1;
        const int j = jf;
        const float flo = fmaf((float)j, uf_step, uf_lo0);
        const float tc = fmaxf(ta, flo), td = fminf(tb, flo + uf_w);
        // x grows with t, so [tc, td] maps to [x(tc), x(td)]
        const int x0 = (int)fmaxf(fmaf(tc, dxs, gxs_lo), 0.0f);
        const int x1 = min(nx - 1, (int)fmaxf(fminf(fmaf(td, dxs, gxs_hi), fnx), -1.0f));
        const bool ok = live && j <= jf1 && tc <= td && x0 <= x1;
        jf = j + 1;
        const uint32_t row = row_e + (uint32_t)j * sf;
        // 32-bit byte offsets from the table base (the table is far below
        // 4 GB), so the loads take a scalar base and one vector offset
        const char *base = reinterpret_cast<const char *>(cs);
        const uint32_t b0 = (row + (uint32_t)x0) * 4u, b1 = (row + (uint32_t)x1 + 1u) * 4u;
        out.k = ok ? *reinterpret_cast<const uint32_t *>(base + b0) : 0u;
        out.e = ok ? *reinterpret_cast<const uint32_t *>(base + b1) : 0u;
    }
};

// Acceptance variants.
//
// Finite cylinder: grain k also needs t = g_k.d in [lo, hi], lo = g_i.d - F,
// hi = g_i.d + |d|^2 + F, F = floor(cyl_ext |d|) = isqrt(cyl_ext^2 |d|^2):
// t is an integer, so t - g_i.d >= -cyl_ext |d| iff t >= g_i.d - F, and
// likewise above. Coordinates are in [0, 2^18] and |d| < 2^12, so |t| < 2^31
// and the 24-bit products are exact; the bounds are clamped to int32.
__device__ __forceinline__ int2 axial_bounds(int4 gi, int dx, int dy, int dz, int ext) {
    const long long D = (long long)dx * dx + (long long)dy * dy + (long long)dz * dz;
    const long long e2D = (long long)ext * ext * D;  // < 2^59
    long long F = (long long)sqrt((double)e2D);
    while (F > 0 && F * F > e2D) --F;
    while ((F + 1) * (F + 1) <= e2D) ++F;
    const long long gd = (long long)gi.x * dx + (long long)gi.y * dy + (long long)gi.z * dz;
    const long long lo = gd - F, hi = gd + D + F;
    return make_int2((int)max(lo, -2147483647ll - 1), (int)min(hi, 2147483647ll));
}

__device__ __forceinline__ bool axial_ok(int4 h, int4 A, int2 b) {
    const int t = __mul24(h.x, A.x) + __mul24(h.y, A.y) + __mul24(h.z, A.z);
    return t >= b.x && t <= b.y;
}

// Grain-count threshold of a seed with direction d: n_min + ceil(b tan(theta)),
// b = thr_num / thr_den, tan(theta) = sqrt(dx^2 + dy^2) / |dz|, capped at
// thr_max when set; dz = 0 needs the cap (no cap: unreachable). The ceiling
// m = ceil(sqrt(Q) / K), Q = thr_num^2 (dx^2 + dy^2), K = thr_den |dz|, is the
// smallest m >= 0 with (m K)^2 >= Q: a double estimate, corrected with exact
// integer squares (m K < 2^23).
__device__ __forceinline__ uint32_t seed_threshold(int dx, int dy, int dz, const Params &P) {
    if (P.thr_num == 0) return (uint32_t)P.n_min;
    const uint32_t cap = P.thr_max > 0 ? (uint32_t)P.thr_max : 0xffffffffu;
    const long long K = (long long)P.thr_den * (dz < 0 ? -dz : dz);
    if (K == 0) return cap;
    const long long Q =
        (long long)P.thr_num * P.thr_num * ((long long)dx * dx + (long long)dy * dy);
    long long m = (long long)ceil(sqrt((double)Q) / (double)K);
    while (m > 0 && (m - 1) * K * (m - 1) * K >= Q) --m;
    while (m * K * m * K < Q) ++m;
    const long long t = (long long)P.n_min + m;
    return t < (long long)cap ? (uint32_t)t : cap;
}

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ----------------------------------------------------------------- seeds

// The line class of direction d (up to the rounding at the bins' edges, where
// both classes list the line's grains): its face, and its slopes' bins.
__device__ __forceinline__ int line_face(int ax, int ay, int az) {
    return (ax >= ay && ax >= az) ? 0 : (ay >= az ? 1 : 2);
}

__device__ __forceinline__ int line_bin(float slope, int sub) {
    return max(0, min(sub - 1, (int)((slope + 1.0f) * (0.5f * (float)sub))));
}

__device__ __forceinline__ int line_class(float dx, float dy, float dz, int ns) {
    const bool x = fabsf(dx) >= fabsf(dy) && fabsf(dx) >= fabsf(dz), z = fabsf(dy) < fabsf(dz);
    const int a = x ? 0 : (z ? 2 : 1);
    const float ida = __builtin_amdgcn_rcpf(x ? dx : z ? dz : dy);
    const float su = (x ? dy : dx) * ida, sv = (x || !z ? dz : dy) * ida;
    return (a * ns + line_bin(su, ns)) * ns + line_bin(sv, ns);
}

// The order of a class's seeds: their anchors by tiles of the plane across
// the class's middle direction (positions moved along it to the middle of the
// view), row by row. Lines of one class through one tile stay close together
// all the way, so the waves that count them read the same records and words.
// One workgroup per view and class sorts the anchors by counting, in LDS.
constexpr int kOrderBlock = 1024;
constexpr int kTiles = 2048;

// The grains of each face in the order k_line_fill and the tests read them:
// by groups of slabs, and in a group by square tiles of at least 20 um, u
// fastest. line_tiles: slabs a group, groups, tiles along u and v.
struct LineTiles {
    int gs, ng, tu, tv;
    float it;  // 1 / tile edge
};

__device__ __forceinline__ int line_key_cap(uint32_t n) { return (int)min((uint32_t)kLineKeys, n); }

__device__ __forceinline__ uint32_t *line_keys(const DevPtrs &d, const ViewGrid &G, uint32_t v,
                                               int a) {
    return d.lkey + 3 * ((size_t)G.grain_off + v) + (size_t)a * (line_key_cap(G.n) + 1);
}

__device__ LineTiles line_tiles(const ViewGrid &G, const LineGrid &L, int a) {
    LineTiles T;
    const int cap = line_key_cap(G.n);
    const int ns = L.ns[a], au = line_u(a), av = line_v(a);
    T.gs = (ns + cap - 1) / cap;
    T.ng = (ns + T.gs - 1) / T.gs;
    const float su = (float)(G.hi[au] - G.lo[au]) + 1.0f, sv = (float)(G.hi[av] - G.lo[av]) + 1.0f;
    float edge = fmaxf(2000.0f, sqrtf(su * sv * (float)T.ng / (float)cap));
    for (;;) {
        T.it = 1.0f / edge;
        T.tu = (int)(su * T.it) + 1;
        T.tv = (int)(sv * T.it) + 1;
        if ((long long)T.ng * T.tu * T.tv <= cap) return T;
        edge *= 1.25f;
    }
}

// One face's grains, sorted by counting in LDS (one workgroup).
__device__ void line_sort(const DevPtrs &d, const ViewGrid &G, uint32_t v, int a, uint32_t *s_key,
                          uint32_t *s_wave) {
    const LineGrid &L = d.lines[2 * v];
    const LineTiles T = line_tiles(G, L, a);
    const int gw = T.gs * L.w;  // a group's thickness
    auto key_of = [&](const int4 &g) {
        const int ga = a == 0 ? g.x : a == 1 ? g.y : g.z;
        const float gu = (float)(a == 0 ? g.y : g.x), gv = (float)(a == 2 ? g.y : g.z);
        const int iu = min(T.tu - 1, (int)(gu * T.it)), iv = min(T.tv - 1, (int)(gv * T.it));
        return ((ga / gw) * T.tv + iv) * T.tu + iu;
    };
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const uint32_t n = G.n, goff = G.grain_off;
    constexpr int kPer = kLineKeys / kOrderBlock;
    for (int i = threadIdx.x; i < kLineKeys; i += kOrderBlock) s_key[i] = 0u;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += kOrderBlock)
        atomicAdd(&s_key[key_of(d.sg[goff + i])], 1u);
    __syncthreads();
    uint32_t c[kPer], sum = 0;
    for (int i = 0; i < kPer; ++i) sum += c[i] = s_key[kPer * threadIdx.x + i];
    const uint32_t incl = wave_incl_scan_dpp(sum);
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = incl - sum;
    for (int w = 0; w < wave; ++w) before += s_wave[w];
    uint32_t *start = line_keys(d, G, v, a);
    for (int i = 0; i < kPer; ++i) {
        const int key = kPer * threadIdx.x + i;
        s_key[key] = before;
        if (key <= line_key_cap(n)) start[key] = before;
        before += c[i];
    }
    if (threadIdx.x == kOrderBlock - 1 && line_key_cap(n) == kLineKeys) start[kLineKeys] = before;
    __syncthreads();
    float4 *out = d.lsg + 3 * (size_t)goff + (size_t)a * n;
    for (uint32_t i = threadIdx.x; i < n; i += kOrderBlock) {
        const int4 g = d.sg[goff + i];
        out[atomicAdd(&s_key[key_of(g)], 1u)] =
            make_float4((float)(a == 0 ? g.x : a == 1 ? g.y : g.z), (float)(a == 0 ? g.y : g.x),
                        (float)(a == 2 ? g.y : g.z), __uint_as_float(i));
    }
}

__global__ void __launch_bounds__(kOrderBlock) k_line_order(DevPtrs d) {
    __shared__ uint32_t s_tile[kLineKeys > kTiles ? kLineKeys : kTiles];
    __shared__ uint32_t s_wave[kOrderBlock / 64];
    const uint32_t v = blockIdx.y;
    if (v >= d.desc->n_views) return;
    const ViewGrid *G = &d.grids[v];
    const uint32_t n = G->n, goff = G->grain_off;
    if (G->err || n < 2) return;
    if (blockIdx.x < 3) {
        line_sort(d, *G, v, (int)blockIdx.x, s_tile, s_wave);
        return;
    }
    const int nsub = d.lines[2 * v].sub, cls = (int)blockIdx.x - 3;
    if (cls >= 3 * nsub * nsub) return;
    const int a = cls / (nsub * nsub), sub = cls % (nsub * nsub);
    const int au = line_u(a), av = line_v(a);
    const float delta = 1.0f / (float)nsub;
    const float su0 = (float)(2 * (sub / nsub) + 1) * delta - 1.0f;
    const float sv0 = (float)(2 * (sub % nsub) + 1) * delta - 1.0f;
    const float half = 0.5f * (float)(G->hi[a] - G->lo[a]);
    const float ru = (float)(G->hi[au] - G->lo[au]) + 2.0f * fabsf(su0) * half + 1.0f;
    const float rv = (float)(G->hi[av] - G->lo[av]) + 2.0f * fabsf(sv0) * half + 1.0f;
    // about kTiles / 2 square tiles; no more than kTiles whatever the shape
    const float edge = fmaxf(sqrtf(ru * rv * (2.0f / kTiles)), fmaxf(ru, rv) * (4.0f / kTiles));
    const float ie = 1.0f / edge;
    const int tu = min((int)(ru * ie) + 1, kTiles / 2);
    const int tv = min((int)(rv * ie) + 1, kTiles / tu);
    auto tile_of = [&](const int4 &g) {
        const float h = (float)(a == 0 ? g.x : a == 1 ? g.y : g.z) - half;
        const float u = (float)(a == 0 ? g.y : g.x) - su0 * h + fabsf(su0) * half;
        const float w = (float)(a == 2 ? g.y : g.z) - sv0 * h + fabsf(sv0) * half;
        const int iu = max(0, min(tu - 1, (int)(u * ie))), iv = max(0, min(tv - 1, (int)(w * ie)));
        return iv * tu + iu;
    };
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < kTiles; i += kOrderBlock) s_tile[i] = 0u;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += kOrderBlock) atomicAdd(&s_tile[tile_of(d.sg[goff + i])], 1u);
    __syncthreads();
    const uint32_t c0 = s_tile[2 * threadIdx.x], c1 = s_tile[2 * threadIdx.x + 1];
    const uint32_t incl = wave_incl_scan_dpp(c0 + c1);
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = incl - c0 - c1;
    for (int w = 0; w < wave; ++w) before += s_wave[w];
    s_tile[2 * threadIdx.x] = before;
    s_tile[2 * threadIdx.x + 1] = before + c0;
    __syncthreads();
    uint32_t *rank = d.lrank + (size_t)d.nc * goff + (size_t)cls * n;
    for (uint32_t i = threadIdx.x; i < n; i += kOrderBlock)
        rank[i] = atomicAdd(&s_tile[tile_of(d.sg[goff + i])], 1u);
}
static_assert(kTiles == 2 * kOrderBlock, "two tiles a thread");

constexpr uint32_t kSeedRun = 64;
constexpr uint32_t kSeedWords = 64;  // one a lane: 4096 elements
// Seeds of an anchor put in order in LDS before they are written: its classes'
// seeds lie 48 bytes here and there, and written as they were found the open
// lines of all waves outgrew the L2 (write pass of 32 c5 views 8.8 -> 6.4 ms, of
// 8 1.75 -> 1.45; 384: 7.1, 768: 6.3 but one c2 view 105 -> 113 us in all).
constexpr uint32_t kSeedStage = 512;

// One wave per anchor grain p (a sorted position); lanes take the (y, z)
// rows of the cell box overlapping [g_p - (R-1), g_p + (R-1)]. Every grain q
// of those rows at a higher sorted position with 0 < |g_q - g_p|^2 < R^2
// makes a seed, stored with the lower input index first. A first pass counts
// the seeds of every anchor and line class, a scan turns the counts into
// offsets, and a second pass writes them: no shared counter, and the seed list
// comes out by view, class and anchor. Bound by VALU issue (the count pass by
// itself, the write pass also by its partly written lines, 7.8 GB for 5.2 GB of
// seeds with 32 c5 views): finding an element's row by counting row ends instead
// of a search over the row starts, cell bounds by reciprocals and the pair test
// in FP32 took 8 c5 views' passes from 2.9 to 2.45 ms, one c2 view's from 74 to
// 52 us. The write pass puts an anchor's seeds in order in LDS first
// (kSeedStage).
template <bool kWrite>
__global__ void __launch_bounds__(kBlock) k_seeds(DevPtrs d, Caps c, Params P) {
    // per wave: for each row that has grains, the sorted position of its first
    // minus the row's first flat element (so that grain = dk[r] + element); a
    // bit for every element that ends a row
    __shared__ uint32_t s_rows[kBlock / 64][65];
    __shared__ unsigned long long s_ends[kBlock / 64][kSeedWords];
    // per wave and class: the anchor's seeds so far, or where the next goes
    __shared__ uint32_t s_cls[kBlock / 64][kLineClasses];
    // write pass: the anchor's seeds by class, each its partner (top bit: the
    // anchor comes first) and where it goes
    __shared__ uint2 s_out[kWrite ? kBlock / 64 : 1][kWrite ? kSeedStage : 1];
    __shared__ uint32_t s_dst[kWrite ? kBlock / 64 : 1][kLineClasses];
    uint32_t *cls_s = s_cls[threadIdx.x >> 6];
    const int lane = lane_id();
    // workgroups are dealt to the XCDs in turn: each XCD takes runs of
    // kSeedRun workgroups' consecutive anchors, whose seeds share lines in
    // its L2
    const uint32_t wi = blockIdx.x >> 3;
    const uint32_t wg = ((wi / kSeedRun) * 8u + (blockIdx.x & 7u)) * kSeedRun + wi % kSeedRun;
    const uint32_t gw = wg * (kBlock / 64) + (threadIdx.x >> 6);
    const uint32_t nw = grid_threads() >> 6;
    const int R1 = P.R - 1;
    const float R2 = (float)(P.R * P.R);
    const uint32_t n_total = d.desc->n_total;
    // the write pass has nothing to do when the seeds overflow their buffer
    if (kWrite && d.cnt->n_seeds_ok == 0) return;
    if constexpr (kWrite) {
        // the candidate bit mask starts clear; the counting kernel sets the
        // bits of the seeds that reach their threshold
        const uint32_t nwd = d.cnt->pass_words;
        for (uint32_t w = grid_tid(); w < nwd; w += grid_threads()) d.pass[w] = 0u;
    }
    unsigned long long wave_total = 0;  // count pass: seeds of this wave's anchors
    for (uint32_t p = gw; p < n_total; p += nw) {
        const uint32_t v = d.view_of[p];
        const ViewGrid *G = &d.grids[v];
        // the anchor's places in its view's table of classes by ordered anchors
        const uint32_t tab = (uint32_t)d.nc * G->grain_off, rel = p - G->grain_off;
        uint32_t at = 0;
        static_assert(kLineClasses <= 64, "one class a lane");
        // (one class, anchors in place, where the lines are not classed)
        const int nsub = d.nc > 1 ? d.lines[2 * v].sub : 0;
        if (lane < 3 * nsub * nsub && !G->err)
            at = tab + (uint32_t)lane * G->n + d.lrank[tab + (uint32_t)lane * G->n + rel];
        else if (lane < d.nc)
            at = tab + (uint32_t)lane * G->n + rel;
        wave_lds_sync();  // the previous anchor's are read
        uint32_t n_seeds = 0;
        if constexpr (kWrite) {
            const uint32_t o0 = lane < d.nc ? d.seed_off[at] : 0u;
            const uint32_t len = lane < d.nc ? d.seed_off[at + 1u] - o0 : 0u;
            const uint32_t incl = wave_incl_scan_dpp(len);
            n_seeds = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            if (lane < d.nc) {
                cls_s[lane] = incl - len;
                s_dst[threadIdx.x >> 6][lane] = o0 - (incl - len);
            }
        } else if (lane < d.nc) {
            cls_s[lane] = 0u;
        }
        wave_lds_sync();
        uint32_t mine = 0;
        auto put = [&](bool first, uint32_t q, uint32_t dst) {
            if (dst < c.seed_cap) d.seeds[dst] = first ? make_uint2(p, q) : make_uint2(q, p);
        };
        if (!G->err) {
            const int nx = G->dims[0], ny = G->dims[1], nz = G->dims[2];
            const int cx = G->cell[0], cy = G->cell[1], cz = G->cell[2];
            const uint32_t off = G->cell_off;
            const int4 g = d.sg[p];
            // the box's first and last cells, to the cell or one too wide
            // (reciprocals; coordinates are below 2^18, and the pair test and
            // the least position decide what a wider box adds)
            constexpr float kLess = 1.0f - 0x1p-20f, kMore = kRowsMore;
            const float icx = __builtin_amdgcn_rcpf((float)cx), icy = __builtin_amdgcn_rcpf((float)cy),
                        icz = __builtin_amdgcn_rcpf((float)cz);
            const int x0 = (int)((float)max(0, g.x - R1) * (icx * kLess));
            const int y0 = (int)((float)max(0, g.y - R1) * (icy * kLess));
            const int z0 = (int)((float)max(0, g.z - R1) * (icz * kLess));
            const int x1 = min(nx - 1, (int)((float)(g.x + R1) * (icx * kMore)));
            const int y1 = min(ny - 1, (int)((float)(g.y + R1) * (icy * kMore)));
            const int z1 = min(nz - 1, (int)((float)(g.z + R1) * (icz * kMore)));
            // each unordered pair once, from the grain with the lower sorted
            // position: rows of the box that sort before the anchor's own row
            // hold only lower positions, and in its row the scan starts past it
            const int yp = min(ny - 1, (int)((float)g.y * (icy * kLess)));
            const int zp = min(nz - 1, (int)((float)g.z * (icz * kLess)));
            const int nyr = y1 - y0 + 1;
            const float inyr = __builtin_amdgcn_rcpf((float)nyr) * kMore;
            const int nrows = nyr * (z1 - z0 + 1);
            const int row_p = (zp - z0) * nyr + (yp - y0);
            // the rows' grains are taken as one flat range: lane L tests
            // elements b + L and b + 64 + L of each trip, so every lane has
            // grains whatever the row lengths. An element is of the row
            // numbered by the row ends before it: those of earlier words are
            // counted as the trips go on, those of its own by two instructions
            // on the word, which is the same for all lanes.
            uint32_t *dk_s = s_rows[threadIdx.x >> 6];
            unsigned long long *ends_s = s_ends[threadIdx.x >> 6];
            for (int rb = row_p; rb < nrows; rb += 64) {
                const int rr = rb + lane;
                uint32_t k0 = 0, k1 = 0;
                if (rr < nrows) {
                    const int rz = row_layer(rr, nyr, inyr);
                    const int y = y0 + rr - rz * nyr, z = z0 + rz;
                    const uint32_t row = off + (uint32_t)((z * ny + y) * nx);
                    k0 = max(d.cell_start[row + x0], p + 1);
                    k1 = d.cell_start[row + x1 + 1];
                }
                const uint32_t len = k1 > k0 ? k1 - k0 : 0u;
                const uint32_t incl = wave_incl_scan_dpp(len);
                const uint32_t T = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                const unsigned long long some = ballot(len > 0);
                const uint32_t slot = __builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u));
                wave_lds_sync();  // the previous block's readers are done
                if (len) dk_s[slot] = k0 - (incl - len);
                uint32_t rows = 0;  // rows that end before word e0
                for (uint32_t e0 = 0; e0 < T; e0 += 64 * kSeedWords) {
                    ends_s[lane] = 0ull;
                    wave_lds_sync();
                    const uint32_t end = incl - 1u - e0;
                    if (len && end < 64 * kSeedWords) atomicOr(&ends_s[end >> 6], 1ull << (end & 63u));
                    wave_lds_sync();
                    // the grain of flat element i, of word m (past the end the
                    // anchor itself, which makes no pair)
                    auto grain_of = [&](uint32_t i, unsigned long long m) -> uint32_t {
                        const uint32_t r = __builtin_amdgcn_mbcnt_hi(
                            (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, rows));
                        rows += (uint32_t)__popcll(m);
                        return i < T ? dk_s[r] + i : p;
                    };
                    // |g_h - g|^2 in (0, R^2): R^2 is at most 2^24, so a sum below
                    // it is exact in FP32 and any other stays at or above it
                    auto pairs = [&](const int4 &h, float3 &e) {
                        e = make_float3((float)(h.x - g.x), (float)(h.y - g.y), (float)(h.z - g.z));
                        const float D = fmaf(e.x, e.x, fmaf(e.y, e.y, e.z * e.z));
                        return D > 0.0f && D < R2;
                    };
                    // stored lower input index first: that grain is the
                    // seed's i (the fit's origin and key order)
                    auto take = [&](bool ok, const int4 &h, const float3 &e, uint32_t q) {
                        if (!ok) return;
                        const int cls = nsub ? line_class(e.x, e.y, e.z, nsub) : 0;
                        const uint32_t slot = atomicAdd(&cls_s[cls], 1u);
                        if constexpr (kWrite) {
                            const uint32_t dst = s_dst[threadIdx.x >> 6][cls] + slot;
                            const uint32_t first = h.w > g.w ? 0x80000000u : 0u;
                            if (slot < kSeedStage)
                                s_out[threadIdx.x >> 6][slot] = make_uint2(q | first, dst);
                            else
                                put(first != 0u, q, dst);
                        }
                    };
                    // two elements a lane per trip: their row searches and grain
                    // loads are in flight together
                    const uint32_t e1 = min(T, e0 + 64 * kSeedWords);
                    for (uint32_t b = e0; b < e1; b += 128) {
                        const uint32_t i0 = b + (uint32_t)lane, i1 = i0 + 64;
                        const unsigned long long *word = ends_s + ((b - e0) >> 6);
                        const uint32_t q0 = grain_of(i0, uniform(word[0]));
                        const uint32_t q1 = grain_of(i1, uniform(word[1]));
                        const int4 h0 = d.sg[q0], h1 = d.sg[q1];
                        float3 d0, d1;
                        const bool ok0 = pairs(h0, d0), ok1 = pairs(h1, d1);
                        take(ok0, h0, d0, q0);
                        take(ok1, h1, d1, q1);
                        if (!kWrite) mine += (ok0 ? 1u : 0u) + (ok1 ? 1u : 0u);
                    }
                    wave_lds_sync();  // the words have been read
                }
            }
        }
        wave_lds_sync();
        if constexpr (kWrite) {
            const uint32_t m = min(n_seeds, kSeedStage);
            for (uint32_t i = (uint32_t)lane; i < m; i += 64) {
                const uint2 o = s_out[threadIdx.x >> 6][i];
                put((int)o.x < 0, o.x & 0x7fffffffu, o.y);
            }
        } else {
            if (lane < d.nc) d.seed_cnt[at] = cls_s[lane];
            wave_total += wave_sum(mine);
        }
    }
    if constexpr (!kWrite) add_spread(d.part64, 0, wave_total);
}

// ------------------------------------------------------- count / members


// Line grids (line_grid.h): filling the cells.
//
// A record covers a block of 8 x 4 cells of a plane: x has a bit for every
// cell that lists grains, cell 0's the topmost, y + 1 is the list word of its
// last such cell, the others following in falling cell order: with the bit of
// the cell asked for shifted to the top, the sign says whether it lists any and
// the bits left count the words from y. A cell's word is its grain, or for several
// grains x = kLineList and y the first of their words; those are the grains,
// with kLineList on all but the last. A grain's word holds its coordinates, so
// that the test needs no other load: 19 bits along the face's axis, 12 bits
// each, signed, of u and v from the record's multiple of its edge, and its
// position in the view (20 bits). Cells too large for that (not packed) hold
// the place among the face's sorted grains in x and the position in y.
constexpr uint32_t kLineList = 0x80000000u;

__device__ __forceinline__ uint2 line_pack(int a, int u, int v, uint32_t rel) {
    return make_uint2((uint32_t)a | (((uint32_t)u & 0xfffu) << 19),
                      ((uint32_t)v & 0xfffu) | (rel << 12));
}
constexpr int kLineBlock = 256;
static_assert(kLineBlock == (int)kLineBand, "one record a thread");

// A class's list words: its first, from d.lent.
__device__ __forceinline__ size_t line_pool(uint32_t nc, uint32_t grain_off, uint32_t n,
                                            uint32_t cls) {
    return (size_t)kLineEnt * ((size_t)nc * grain_off + (size_t)cls * n);
}

// The grid a view's lines walk: the coarser one if a class's list words did
// not fit.
__device__ __forceinline__ bool line_coarse(const DevPtrs &d, uint32_t v) {
    return d.lcoarse[v] != 0u;
}

__device__ __forceinline__ const LineGrid *line_grid_of(const DevPtrs &d, uint32_t v) {
    return &d.lines[2 * v + (line_coarse(d, v) ? 1 : 0)];
}

// One workgroup fills a band of at most kLineBand records of one plane: it
// counts the grains of every cell in LDS, takes the band's words of the
// class's pool, and places the grains. The grains that can reach the band are
// a range of the face's sorted grains. kPass 1 fills the coarser grid of the views that need it.
template <int kPass>
__global__ void __launch_bounds__(kLineBlock) k_line_fill(DevPtrs d, Params P) {
    // 33 words a record keep the threads' counts in different banks
    __shared__ uint32_t s_cell[kLineBand * 33];
    __shared__ uint32_t s_wave[kLineBlock / 64], s_base;
    const uint32_t v = blockIdx.z;
    if (v >= d.desc->n_views) return;
    if (kPass == 1 && !line_coarse(d, v)) return;
    const ViewGrid G = d.grids[v];
    if (G.err || G.n < 2) return;
    const LineGrid L = d.lines[2 * v + kPass];
    const int nsub = L.sub, cls = (int)blockIdx.y;
    if (cls >= 3 * nsub * nsub) return;
    const int a = cls / (nsub * nsub), sub = cls % (nsub * nsub);
    const LineTiles T = line_tiles(G, d.lines[2 * v], a);
    const int gw = T.gs * d.lines[2 * v].w;
    const uint32_t *start = line_keys(d, G, v, a);
    const float4 *sorted = d.lsg + 3 * (size_t)G.grain_off + (size_t)a * G.n;
    const int span_v = G.hi[line_v(a)] - G.lo[line_v(a)];
    const float delta = 1.0f / (float)nsub;
    const float su0 = (float)(2 * (sub / nsub) + 1) * delta - 1.0f;
    const float sv0 = (float)(2 * (sub % nsub) + 1) * delta - 1.0f;
    const float su = fabsf(su0) + delta, sv = fabsf(sv0) + delta;
    const float hu0 = line_half(P.r, su, L.margin), hv0 = line_half(P.r, sv, L.margin);
    const int ns = L.ns[a], nu = L.nu[a], nv = L.nv[a], bu = L.bu[a];
    const uint32_t plane = L.plane[a];
    uint2 *recs = d.lrec + (size_t)line_recs(d.nc) * G.grain_off + L.face_off[a] +
                  (size_t)sub * ns * plane;
    uint2 *ent = d.lent + line_pool((uint32_t)d.nc, G.grain_off, G.n, (uint32_t)cls);
    uint32_t *pool = d.lpool + (size_t)(2 * v + kPass) * d.nc + cls;
    const int nbv = (nv + 3) / 4;
    const int brows = max(1, min(nbv, (int)kLineBand / bu));  // record rows a band
    const int nbands = (nbv + brows - 1) / brows;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    constexpr int kW = kLineBlock / 64;
    for (uint32_t i = threadIdx.x; i < kLineBand * 33; i += kLineBlock) s_cell[i] = 0u;
    __syncthreads();
    for (int item = blockIdx.x; item < ns * nbands; item += gridDim.x) {
        const int k = item / nbands, r0 = (item % nbands) * brows, r1 = min(nbv, r0 + brows);
        const int b0 = 4 * r0, b1 = min(nv, 4 * r1);  // cell rows of the band
        // the sorted grains of the slab that can reach the band
        const int a0 = k * L.w, a1 = a0 + L.w;
        const int g0 = a0 / gw, g1 = min((a1 - 1) / gw, T.ng - 1);
        int t0 = 0, t1 = T.tv - 1;
        if (g0 == g1) {
            t0 = max(0, min(t1, (int)((float)max(0, b0 * L.c - 2 * L.reach) * T.it)));
            t1 = max(0, min(t1, (int)((float)min(span_v, b1 * L.c) * T.it)));
        }
        const uint32_t i0 = start[(g0 * T.tv + t0) * T.tu], i1 = start[(g1 * T.tv + t1 + 1) * T.tu];
        const float fa0 = (float)a0, fa1 = (float)a1, mid = fa0 + 0.5f * (float)L.w;
        // calls at(cell, record's column and row, grain, its place) for every
        // cell of the band that lists a grain
        auto each = [&](auto at) {
            for (uint32_t i = i0 + threadIdx.x; i < i1; i += kLineBlock) {
                const float4 g = sorted[i];
                if (g.x < fa0 || g.x >= fa1) continue;
                const float h = g.x - mid;
                int ju0, ju1, jv0, jv1;
                line_cells(L, g.y, h, su0, delta, hu0, 0, nu - 1, ju0, ju1);
                line_cells(L, g.z, h, sv0, delta, hv0, b0, b1 - 1, jv0, jv1);
                for (int jv = jv0; jv <= jv1; ++jv) {
                    const int row = ((jv >> 2) - r0) * bu, in = (jv & 3) << 3;
                    for (int ju = ju0; ju <= ju1; ++ju)
                        at((uint32_t)((row + (ju >> 3)) * 33 + in + (ju & 7)), ju >> 3, jv >> 2, g, i);
                }
            }
        };
        each([&](uint32_t cell, int, int, const float4 &, uint32_t) { atomicAdd(&s_cell[cell], 1u); });
        __syncthreads();
        // each thread one record: its bits, and how many words its cells need
        const uint32_t n_rec = (uint32_t)((r1 - r0) * bu);
        uint32_t *mine = s_cell + threadIdx.x * 33;
        uint32_t bits = 0, words = 0;
#pragma unroll 8
        for (int i = 0; i < 32; ++i) {
            const uint32_t n = mine[i];
            bits |= n ? 0x80000000u >> i : 0u;
            words += n < 2u ? n : n + 1u;
        }
        const uint32_t incl = wave_incl_scan_dpp(words);
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        uint32_t before = incl - words, total = 0;
        for (int w = 0; w < kW; ++w) {
            before += w < wave ? s_wave[w] : 0u;
            total += s_wave[w];
        }
        if (threadIdx.x == 0) {
            s_base = atomicAdd(pool, total);
            if (s_base + total > kLineEnt * G.n) d.lcoarse[v] = 1u;
        }
        __syncthreads();
        const uint32_t base = s_base + before;
        const bool room = s_base + total <= kLineEnt * G.n;
        uint32_t lists = 0;  // the cells of this record that list several grains
        if (threadIdx.x < n_rec) {
            recs[(size_t)k * plane + (size_t)r0 * bu + threadIdx.x] =
                make_uint2(room ? bits : 0u, base - 1u);
            uint32_t word = base, list = base + (uint32_t)__popc(bits);
            for (uint32_t rest = room ? bits : 0u; rest; rest &= rest - 1u) {
                const int i = 32 - __ffs(rest);
                const uint32_t n = mine[i];
                if (n == 1) {
                    mine[i] = word;
                } else {
                    ent[word] = make_uint2(kLineList, list);
                    mine[i] = kLineList | list;
                    lists |= 1u << i;
                    list += n;
                }
                ++word;
            }
        }
        __syncthreads();
        if (room)
            each([&](uint32_t cell, int cu8, int rv4, const float4 &g, uint32_t place) {
                const uint32_t at = atomicAdd(&s_cell[cell], 1u);
                const uint32_t rel = __float_as_uint(g.w);
                uint2 w = make_uint2(place, rel);
                if (L.packed)
                    w = line_pack((int)g.x, (int)g.y - 8 * L.c * cu8, (int)g.z - 4 * L.c * rv4, rel);
                w.x |= at & kLineList;
                ent[at & ~kLineList] = w;
            });
        __syncthreads();
        for (; lists; lists &= lists - 1u) {
            const uint32_t last = (mine[__ffs(lists) - 1] & ~kLineList) - 1u;
            ent[last].x &= ~kLineList;
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < n_rec * 33; i += kLineBlock) s_cell[i] = 0u;
        __syncthreads();
    }
}

// Bound by VALU issue and by the cache lines the record and word loads touch
// (8 c5 views: VALU 76 % busy, 0.84 L1 accesses a cycle; L2 hits 95 %). One
// lookup a slab and 16 tests a seed replace the 20 cell pencils and 84 tests
// of a walk over the binned cells: 11.9 against 26.0 ms for the 163 M seeds of
// 8 c5 views, and 225 against 500 us for the 3.3 M of one c2 view.
//
// Counting: a wave counts 64 lines at a time, one a lane. The lines of one
// class (nearly always all 64) step through its slabs together, so that what
// describes the class stays in scalar registers and the lanes, whose lines
// run side by side, read neighbouring records. The words of the cells they
// find go into a queue of the wave in LDS, and whenever it holds 64 of them
// every lane tests one grain against the line it was found for (in LDS too),
// so the test runs with all lanes whatever the lines hold.
constexpr int kFetch = EMT_COUNT_FETCH;            // slabs walked per step
constexpr int kCountBlock = EMT_COUNT_THREADS;     // threads of a workgroup
constexpr int kCountWaves = kCountBlock / 64;
constexpr uint32_t kChunkSeeds = EMT_CHUNK_SEEDS;  // most seeds a workgroup takes at a time
// Seeds from which XCDs work apart. Apart / in turn, us a call: one c2 view (3.3 M
// seeds) 729 / 720, four (12.8 M) 1793 / 1870, one c5 view (20 M) 3271 / 3394, 16
// and 32 c3 views (26, 51 M) 3618 / 3688, 6482 / 6628, 3, 8 and 16 c5 views (61,
// 162, 326 M) 8207 / 8672, 20930 / 22320, 42300 / 45000. In turn is the better
// side for a single small view only; the line is well on the safe side of it.
constexpr uint32_t kApartSeeds = 50000000;
// at most 63 words are left in the queue before a step's are added, and a
// test adds back at most one for each it takes
constexpr uint32_t kQueue = 64u * (kFetch + 1);
// queued: position in the class's pool, lane of the line, and whether the
// word is one of a cell's list (else a cell's first); the cell, u << 16 | v
constexpr uint32_t kItemLane = 24, kItemList = 1u << 31;
static_assert((unsigned long long)kLineEnt * kNMax <= 1ull << kItemLane, "pool positions");

template <bool kFinite, bool kEmit>
struct CountLds {
    float4 la[64];  // dx, dy, dz, tlo
    float4 lc[64];  // -ex, -ey, -ez, thi
    uint32_t lp[64];             // sorted position of g_i (the int64 test)
    uint32_t cnt[64];
    int2 pc[kFinite ? 64 : 1];   // finite cylinder: bounds of g_k.d
    uint2 mo[kEmit ? 64 : 1];    // listing members: where they go, how many
    uint2 queue[kQueue];
};

// The counting test in FP32, decided exactly. With coordinates in [0, 2^18]
// (exact floats) and |d| < 2^12, c = g_k x d - g_i x d is formed by two
// fused multiply-adds a component from d, -d and the rounded -(g_i x d).
// Each rounding is at most 2^-24 of a magnitude below 2^18 (1 + sqrt 2)|d|,
// so each component is within 0.06 |d| of the exact one and |c| within
// 0.104 |d|. A grain is certainly inside when the FP32 |c|^2 is at most
// tlo = (r - 1/8)^2 |d|^2 and certainly outside above thi = (r + 1/8)^2
// |d|^2, both widened by 2^-20 (tlo < 0 when r = 0); in between the test is
// redone in int64. The widening covers the rounding of the FP32 sum of
// squares (within 5 * 2^-24 relative) and of the FP32 products forming tlo
// and thi (|d|^2 < 2^26 rounded, a square, two products: within 4 * 2^-24).
// The components of g_i x d are differences of two 24-bit products below
// 2^18 * 4095, so they are exact in int32.
__device__ __forceinline__ void line_consts(int4 gi, int dx, int dy, int dz, int r, float4 &A,
                                            float4 &C) {
    const float Df = (float)(dx * dx + dy * dy + dz * dz);  // |d| < 2^12: exact in int32
    const float rlo = (float)r - 0.125f, rhi = (float)r + 0.125f;  // exact
    const float tlo = r > 0 ? rlo * rlo * Df * (1.0f - 0x1p-20f) : -1.0f;
    const float thi = rhi * rhi * Df * (1.0f + 0x1p-20f);
    const int ex = __mul24(gi.y, dz) - __mul24(gi.z, dy);
    const int ey = __mul24(gi.z, dx) - __mul24(gi.x, dz);
    const int ez = __mul24(gi.x, dy) - __mul24(gi.y, dx);
    A = make_float4((float)dx, (float)dy, (float)dz, tlo);
    C = make_float4((float)-ex, (float)-ey, (float)-ez, thi);
}

// Seeds for the waves of a workgroup, a chunk of consecutive ones at a time.
// Chunks are dealt to the XCDs in turn (as workgroups are), so all XCDs have
// the same mix of long and short lines; or, from kApartSeeds on, each XCD has
// an eighth of the list, so that its L2 holds the records and words of views
// of its own; candidates always (a third of their loads hit L2 when dealt in
// turn; the members stage of 8 c5 views 2.24 -> 1.70 ms). Which chunk is whose
// is deal.h's: every chunk has one taker, as two listing the same candidate
// would write its members at once. A workgroup whose XCD has no chunk left
// takes those of the others. The waves of a workgroup take `step` seeds at a
// time from its chunk: they stay close together in the class's order and so
// share the CU's cache. range: the chunk's next seed and, in the upper half,
// its end.
struct Feed {
    unsigned long long range;
    uint32_t lock, done;
    Deal deal;  // (here rather than in registers, which the walk needs)
};

// The next chunk, by one lane of the wave that holds the feed's lock; 0 if
// there is none left.
__device__ __forceinline__ unsigned long long next_chunk(uint32_t *grab, const Deal &D) {
    const uint32_t wgs = gridDim.x / kXcds;
    for (uint32_t t = 0; t < kXcds; ++t) {
        const uint32_t x = (blockIdx.x + t) % kXcds, mine = deal_share(D, x);
        uint32_t *ctr = grab + 16 * x;
        const uint32_t cur = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (wgs + cur >= mine) continue;
        const unsigned long long r = deal_range(D, x, wgs + atomicAdd(ctr, 1u));
        if (r) return r;
    }
    return 0ull;
}

// Takes the next seeds [next, next + n) for the calling wave, n <= step.
// Returns false when every range is used up; n = 0 with true if another wave
// of the workgroup is fetching a chunk. Wave-uniform.
__device__ __forceinline__ bool take_seeds(Feed &F, uint32_t *grab, uint32_t step, uint32_t &next,
                                           uint32_t &n) {
    uint32_t s = 0, m = 0, ok = 1;
    if (lane_id() == 0) {
        volatile Feed *V = &F;
        unsigned long long r = V->range;
        if ((uint32_t)r < (uint32_t)(r >> 32)) {
            r = atomicAdd(&F.range, (unsigned long long)step);
            s = (uint32_t)r;
            const uint32_t e = (uint32_t)(r >> 32);
            m = s < e ? min(step, e - s) : 0u;
        } else if (V->done) {
            ok = 0;
        } else if (atomicCAS(&F.lock, 0u, 1u) == 0u) {
            // this wave fetches; the others go on with the seeds they have
            r = V->range;
            if ((uint32_t)r >= (uint32_t)(r >> 32) && !V->done) {
                r = next_chunk(grab, F.deal);
                if (r == 0ull) {
                    atomicExch(&F.done, 1u);
                    ok = 0;
                } else {
                    s = (uint32_t)r;
                    m = min(step, (uint32_t)(r >> 32) - s);
                    atomicExch(&F.range, r + step);
                }
            }
            __threadfence_block();
            atomicExch(&F.lock, 0u);
        }
    }
    next = (uint32_t)__builtin_amdgcn_readfirstlane((int)s);
    n = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
    return __builtin_amdgcn_readfirstlane((int)ok) != 0;
}

// Waves per SIMD the counting kernel is compiled for (the compiler then keeps
// it within 512 / kCountOccupancy VGPRs).
constexpr int kCountOccupancy = EMT_COUNT_OCCUPANCY;

// What the lines of one class walk and test, in scalar registers.
struct LineClass {
    const uint2 *recs, *ent;
    const float4 *sorted;
    uint32_t nu, nv, bu, plane, goff;
    int face, packed, c8, c4;  // packed words: u = word + c8 column, v = word + c4 row
};

// Uniform offsets are added to the kernel's own pointers: a pointer put
// together from two words would be of no known address space, and its loads
// flat ones, which also wait for and hold up the LDS.
__device__ __forceinline__ LineClass line_class_of(const DevPtrs &d, uint32_t v, uint32_t cls) {
    const LineGrid *L = line_grid_of(d, v);
    LineClass K;
    const uint32_t n_sub = (uint32_t)(L->sub * L->sub), a = uniform(cls / n_sub);
    const uint32_t sub = cls - a * n_sub, n = d.grids[v].n;
    K.goff = uniform(d.grids[v].grain_off);
    K.nu = uniform((uint32_t)L->nu[a]);
    K.nv = uniform((uint32_t)L->nv[a]);
    K.bu = uniform((uint32_t)L->bu[a]);
    K.plane = uniform(L->plane[a]);
    K.recs = d.lrec + uniform(line_recs(d.nc) * (unsigned long long)K.goff + L->face_off[a] +
                              (size_t)sub * (uint32_t)L->ns[a] * K.plane);
    K.ent = d.lent + uniform((unsigned long long)line_pool((uint32_t)d.nc, K.goff, n, cls));
    K.sorted = d.lsg + uniform(3ull * K.goff + (unsigned long long)a * n);
    K.face = (int)a;
    K.packed = uniform(L->packed);
    K.c8 = uniform(8 * L->c);
    K.c4 = uniform(4 * L->c);
    return K;
}

// A 32-bit byte offset from a uniform pointer: the load adds the two itself.
template <class T>
__device__ __forceinline__ const T *at_byte(const T *p, uint32_t offset) {
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) + offset);
}

// A grain's coordinates in the axes of face a: along it, u, v (and its index).
__device__ __forceinline__ int4 line_axes(int4 g, int a) {
    return make_int4(a == 0 ? g.x : a == 1 ? g.y : g.z, a == 0 ? g.y : g.x, a == 2 ? g.y : g.z, g.w);
}

// Takes up to 64 words off the queue's end and tests their grains, one a
// lane. A cell's first word that points to a list, and a list word with more
// behind it, put their successor back. Counting adds a hit to its line's
// count; listing (kEmit) takes that position in the candidate's member list
// (in any order: the merge treats a list as a set and the fit orders it).
// Returns how many grains it tested.
template <bool kFinite, bool kEmit>
__device__ __forceinline__ uint32_t count_test(CountLds<kFinite, kEmit> &Q, uint32_t &qn,
                                               const LineClass &K, int tol_r, const DevPtrs &d,
                                               int lane) {
    const uint32_t m = min(qn, 64u);
    qn -= m;
    const uint2 item = Q.queue[qn + min((uint32_t)lane, m - 1u)];
    const uint32_t at = item.x & ((1u << kItemLane) - 1u), sl = (item.x >> kItemLane) & 63u;
    const uint2 w = *at_byte(K.ent, 8u * at);
    const float4 A = Q.la[sl], C = Q.lc[sl];
    // lane masks rather than flags: they stay in scalar registers
    const unsigned long long on = ~0ull >> (64u - m), flag = ballot((int)w.x < 0);
    const unsigned long long ptrs = flag & ~ballot((int)item.x < 0), more = flag & on;
    const unsigned long long test = on & ~ptrs;
    const bool ptr = __builtin_amdgcn_inverse_ballot_w64(ptrs);
    float3 h;
    uint32_t rel;
    if (K.packed) {
        h.x = (float)(w.x & 0x7ffffu);
        // (bit 31 of w.x is the list flag)
        h.y = (float)(((int)(w.x << 1) >> 20) + __mul24((int)(item.y >> 19), K.c8));
        h.z = (float)(((int)(w.y << 20) >> 20) + __mul24((int)((item.y >> 2) & 0x3fffu), K.c4));
        rel = w.y >> 12;
    } else {
        const float4 g = K.sorted[ptr ? 0u : w.x & ~kLineList];
        h = make_float3(g.x, g.y, g.z);
        rel = w.y;
    }
    if (more) {
        wave_lds_sync();  // the items have been read
        if (__builtin_amdgcn_inverse_ballot_w64(more))
            Q.queue[__builtin_amdgcn_mbcnt_hi((uint32_t)(more >> 32),
                                              __builtin_amdgcn_mbcnt_lo((uint32_t)more, qn))] =
                make_uint2((ptr ? w.y : at + 1u) | (sl << kItemLane) | kItemList, item.y);
        qn += (uint32_t)__popcll(more);
        wave_lds_sync();
    }
    const float c0 = fmaf(h.y, A.z, fmaf(h.z, -A.y, C.x));
    const float c1 = fmaf(h.z, A.x, fmaf(h.x, -A.z, C.y));
    const float c2 = fmaf(h.x, A.y, fmaf(h.y, -A.x, C.z));
    const float fc = fmaf(c0, c0, fmaf(c1, c1, c2 * c2));
    const unsigned long long near = test & ballot(fc <= C.w);
    const unsigned long long band = near & ballot(fc > A.w);
    bool ok = __builtin_amdgcn_inverse_ballot_w64(near);
    if (band && __builtin_amdgcn_inverse_ballot_w64(band)) {
        // inside the band: decide in int64 from the integer grains (rare)
        const int dx = (int)A.x, dy = (int)A.y, dz = (int)A.z;
        const long long D = (long long)dx * dx + (long long)dy * dy + (long long)dz * dz;
        const int4 gi = line_axes(d.sg[Q.lp[sl]], K.face);
        const long long wx = (int)h.x - gi.x, wy = (int)h.y - gi.y, wz = (int)h.z - gi.z;
        const long long e0 = wy * dz - wz * dy, e1 = wz * dx - wx * dz, e2 = wx * dy - wy * dx;
        ok = e0 * e0 + e1 * e1 + e2 * e2 <= (long long)tol_r * tol_r * D;
    }
    if constexpr (kFinite) {
        const int4 hi = make_int4((int)h.x, (int)h.y, (int)h.z, 0);
        const int4 Ai = make_int4((int)A.x, (int)A.y, (int)A.z, 0);
        ok = ok && axial_ok(hi, Ai, Q.pc[sl]);
    }
    if (ok) {
        const uint32_t n = atomicAdd(&Q.cnt[sl], 1u);
        if constexpr (kEmit) {
            const uint2 mo = Q.mo[sl];
            if (n < mo.y) d.members[mo.x + n] = K.goff + rel;
        }
    }
    return (uint32_t)__popcll(test);
}

// kEmit: the members stage. The same walk and test over the candidates
// instead of the seeds, listing each candidate's grains (its count is known:
// the list must come out exactly that long).
template <bool kFinite, bool kEmit>
__global__ void __launch_bounds__(kCountBlock) __attribute__((amdgpu_waves_per_eu(kCountOccupancy)))
k_count(DevPtrs d, Caps c, Params P) {
    __shared__ CountLds<kFinite, kEmit> sQ[kCountWaves];
    __shared__ Feed s_feed;
    const int lane = lane_id();
    CountLds<kFinite, kEmit> &Q = sQ[threadIdx.x >> 6];
    uint32_t n_items = d.cnt->n_seeds_ok;
    if constexpr (kEmit) {
        // nothing to list when the seeds or the entries overflow their buffer
        // (the call is re-run)
        const bool skip = n_items == 0u || d.cnt->err || d.cnt->n_members > c.mem_cap;
        n_items = skip ? 0u : min(d.cnt->n_cand, c.cand_cap);
    }
    unsigned long long tests = 0, hits = 0;
    // The listing instance has range counters of its own: the counting one
    // leaves its counters used up. A wave takes 64 seeds at a time, or fewer
    // when there are too few for every wave (candidates: for eight times each,
    // as they are far apart and take unlike times: 16 c3 views' members stage
    // 247 -> 215 us).
    uint32_t *grab = d.grab + (kEmit ? 8 * 16 : 0);
    const uint32_t step = min(64u, max(16u, n_items / ((grid_threads() >> 6) * (kEmit ? 8u : 1u))));
    if (threadIdx.x == 0) {
        s_feed.deal = make_deal(n_items, step, kCountWaves, gridDim.x, kChunkSeeds,
                                kEmit || n_items >= kApartSeeds);
        s_feed.range = deal_range(s_feed.deal, blockIdx.x % kXcds, blockIdx.x / kXcds);
        s_feed.lock = 0u;
        s_feed.done = 0u;
    }
    __syncthreads();
    for (;;) {
        uint32_t s0, n_here;
        if (!take_seeds(s_feed, grab, step, s0, n_here)) break;
        if (n_here == 0) {
            __builtin_amdgcn_s_sleep(4);  // another wave is fetching a chunk
            continue;
        }
        // one seed a lane: line constants, class and crossing points
        const uint32_t s = s0 + (uint32_t)lane;
        const bool have = (uint32_t)lane < n_here;
        uint32_t key = 0xffffffffu, th = 0, mcap = 0;
        int iu = -1, idu = 0, iv = -1, idv = 0;
        float klo = 1.0e9f, khi = -1.0f;
        if (have) {
            uint2 pq;
            uint32_t vw;
            if constexpr (kEmit) {
                const Cand cd = d.cand[s];
                pq = make_uint2(cd.p, cd.q);
                vw = cd.v;
                const uint32_t off = d.mem_off[s];
                mcap = ((unsigned long long)off + cd.n <= c.mem_cap) ? cd.n : 0u;
                Q.mo[lane] = make_uint2(off, mcap);
            } else {
                pq = d.seeds[s];
                vw = d.view_of[pq.x];
            }
            const int4 gi = d.sg[pq.x], gj = d.sg[pq.y];
            const int dx = gj.x - gi.x, dy = gj.y - gi.y, dz = gj.z - gi.z;
            th = seed_threshold(dx, dy, dz, P);
            if constexpr (kEmit) {
                // the merge's priority key and threshold of the candidate
                d.key[s] = cand_key(d.cand[s].n, (uint32_t)gi.w, (uint32_t)gj.w);
                if (P.thr_num) d.cand_thr[s] = th;
            }
            if constexpr (kFinite) Q.pc[lane] = axial_bounds(gi, dx, dy, dz, P.cyl_ext);
            Q.lp[lane] = pq.x;
            Q.cnt[lane] = 0u;
            const LineGrid *L = line_grid_of(d, vw);
            const int a = line_face(abs(dx), abs(dy), abs(dz));
            // from here in the face's axes: x along it, y = u, z = v
            const int4 ti = line_axes(gi, a), td = line_axes(make_int4(dx, dy, dz, 0), a);
            float4 a4, c4;
            line_consts(ti, td.x, td.y, td.z, P.r, a4, c4);
            Q.la[lane] = a4;
            Q.lc[lane] = c4;
            const float ga = (float)ti.x, da = a4.x;
            const float ida = __builtin_amdgcn_rcpf(da);
            const float su = a4.y * ida, sv = a4.z * ida;
            key = vw * (uint32_t)d.nc +
                  (uint32_t)((a * L->sub + line_bin(su, L->sub)) * L->sub + line_bin(sv, L->sub));
            const int nu = a == 0 ? L->nu[0] : a == 1 ? L->nu[1] : L->nu[2];
            const int nv = a == 0 ? L->nv[0] : a == 1 ? L->nv[1] : L->nv[2];
            const int ns = a == 0 ? L->ns[0] : a == 1 ? L->ns[1] : L->ns[2];
            const LineCross cu = line_cross(*L, su, ga, ti.y), cv = line_cross(*L, sv, ga, ti.z);
            const float u0 = cu.x0, du = cu.step, v0 = cv.x0, dv = cv.step;
            iu = cu.fixed0();
            idu = cu.fixed_step();
            iv = cv.fixed0();
            idv = cv.fixed_step();
            // slabs whose plane the line crosses inside the cells: a bound a
            // slab too wide costs a look, not a result
            klo = 0.0f;
            khi = (float)(ns - 1);
            if (fabsf(du) > 1e-5f) {
                const float id = __builtin_amdgcn_rcpf(du);
                const float t1 = -u0 * id, t2 = ((float)nu - u0) * id;
                klo = fmaxf(klo, fminf(t1, t2) - 1.0f);
                khi = fminf(khi, fmaxf(t1, t2) + 1.0f);
            }
            if (fabsf(dv) > 1e-5f) {
                const float id = __builtin_amdgcn_rcpf(dv);
                const float t1 = -v0 * id, t2 = ((float)nv - v0) * id;
                klo = fmaxf(klo, fminf(t1, t2) - 1.0f);
                khi = fminf(khi, fmaxf(t1, t2) + 1.0f);
            }
            if constexpr (kFinite) {
                // grains of the cylinder lie within cyl_ext along the line
                // and r across it of the seed's stretch of axis a
                const float reach = (float)P.cyl_ext + (float)P.r + kMargin;
                const float iw = __builtin_amdgcn_rcpf((float)L->w);
                klo = fmaxf(klo, (fminf(ga, ga + da) - reach) * iw - 1.0f);
                khi = fminf(khi, (fmaxf(ga, ga + da) + reach) * iw + 1.0f);
            }
        }
        wave_lds_sync();
        // the classes among the lanes, one after another
        for (unsigned long long left = ballot(have); left;) {
            const uint32_t cls_key =
                (uint32_t)__builtin_amdgcn_readlane((int)key, __ffsll((long long)left) - 1);
            const bool mine = key == cls_key;
            left &= ~ballot(mine);
            const uint32_t vw = cls_key / (uint32_t)d.nc;
            const LineClass K = line_class_of(d, vw, cls_key - vw * (uint32_t)d.nc);
            const float kmin = wave_min(mine ? klo : 1.0e9f), kmax = wave_max(mine ? khi : -1.0f);
            if (kmin > kmax) continue;
            const uint32_t k1 =
                (uint32_t)__builtin_amdgcn_readfirstlane((int)kmax);
            // crossing points in cells, kLineBits fractional bits; negative
            // ones and those past the last cell fail one unsigned compare. (A
            // line far outside may wrap into the cells: it then tests grains
            // it need not.) Lanes of other classes stay outside.
            const uint32_t k0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)kmin);
            uint32_t u = mine ? (uint32_t)iu + k0 * (uint32_t)idu : 0xffffffffu;
            uint32_t v = mine ? (uint32_t)iv + k0 * (uint32_t)idv : 0xffffffffu;
            const uint32_t ddu = mine ? (uint32_t)idu : 0u, ddv = mine ? (uint32_t)idv : 0u;
            const uint32_t lim_u = K.nu << kLineBits, lim_v = K.nv << kLineBits;
            // a finite cylinder's own slabs (an empty range has none)
            const uint32_t first = (uint32_t)klo, slabs = khi >= klo ? (uint32_t)khi - first : 0u;
            size_t first_rec = (size_t)k0 * K.plane;  // the slab's, scalar
            const uint32_t lane_tag = (uint32_t)lane << kItemLane;
            uint32_t qn = 0;
            for (uint32_t k = k0; k <= k1; k += kFetch) {
                uint2 rec[kFetch];
                uint32_t cell[kFetch];  // the cell crossed: u << 16 | v
#pragma unroll
                for (int f = 0; f < kFetch; ++f) {
                    const uint32_t lim = k + (uint32_t)f <= k1 ? lim_u : 0u;  // uniform
                    bool ok = u < lim && v < lim_v;
                    if constexpr (kFinite) ok = ok && k + (uint32_t)f - first <= slabs;
                    cell[f] = __builtin_amdgcn_perm(u, v, 0x07060302u);
                    rec[f].x = 0u;
                    if (ok)
                        rec[f] = *at_byte(K.recs + first_rec, 8u * (__umul24((cell[f] >> 2) & 0x3fffu, K.bu) +
                                                      (cell[f] >> 19)));
                    first_rec += K.plane;
                    u += ddu;
                    v += ddv;
                }
#pragma unroll
                for (int f = 0; f < kFetch; ++f) {
                    // cell 8 (v & 3) + (u & 7) of the record, as the top bit
                    const uint32_t bits =
                        rec[f].x << (((cell[f] << 3) | ((cell[f] >> 16) & 7u)) & 31u);
                    const bool in = (int)bits < 0;
                    const unsigned long long m = ballot(in);
                    if (in)
                        Q.queue[__builtin_amdgcn_mbcnt_hi(
                            (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, qn))] =
                            make_uint2((rec[f].y + (uint32_t)__popc(bits)) | lane_tag,
                                       cell[f]);
                    qn += (uint32_t)__popcll(m);
                }
                wave_lds_sync();
                while (qn >= 64u) tests += count_test(Q, qn, K, P.r, d, lane);
            }
            while (qn > 0u) tests += count_test(Q, qn, K, P.r, d, lane);
        }
        wave_lds_sync();
        if (have) {
            const uint32_t n = Q.cnt[lane];
            if constexpr (kEmit) {
                // the same walk and predicate as the count: a list of another
                // length is never expected; keep every entry a valid grain
                // index and flag an internal error
                if (mcap > 0 && n != mcap) {
                    const uint32_t off = Q.mo[lane].x;
                    for (uint32_t t = n; t < mcap; ++t) d.members[off + t] = Q.lp[lane];
                    atomicOr(&d.cnt->err, 2u);
                }
            } else {
                // only counts that reach the threshold are written, with their
                // bit in the candidate mask (a few percent: scattered 4-byte
                // stores of every count would each cost a partial line write)
                hits += n;
                if (n >= th) {
                    d.seed_n[s] = n;
                    atomicOr(&d.pass[s >> 5], 1u << (s & 31u));
                }
            }
        }
        wave_lds_sync();
    }
    if constexpr (!kEmit) {
        add_spread(d.part64, 2, tests);
        add_spread(d.part64, 3, wave_sum(hits));
    }
}

// ----------------------------------------------- count / members, few grains
//
// Counting over the binned cells, for the calls few_grains names. A wave owns a chunk of
// seeds; each lane holds
// two seed slots in LDS. When a lane's walk ends it closes that slot and at
// once takes the next seed of the chunk into its other slot, so the wave's
// time is the sum of its lines' work rather than a multiple of the longest
// one. Hit counts of a closed slot are final after the next queue flush,
// which writes them out and frees the slot.
//
// The queue holds pieces: each run a lane queues is cut into pieces of at
// most kPiece consecutive grains, and the flush gives every lane one piece.
// The lane maps its piece to the run by one popcount, reads the seed's line
// constants once, issues the loads of all kPiece grains together and tests
// them against the one line, so the mapping and the line constants are paid
// once per piece and the grain loads of a piece are in flight together.
constexpr int kWaves = kBlock / 64;
constexpr int kCountSlots = 128;
constexpr int kPiece = 3;        // grains per queued piece
constexpr int kLanePieces = 24;  // pieces a lane queues per step
constexpr int kPencils = 6;      // pencils a lane fetches per step
constexpr int kRefillMin = 32;   // waiting lanes that start a refill
constexpr uint32_t kFewChunk = 128;             // seeds a wave takes at a time
constexpr int kPieceCap = 128 * kLanePieces;    // queued pieces per wave
constexpr int kRunCap = 64 * kPencils;          // queued runs per wave
constexpr int kPieceWords = kPieceCap / 64;
static_assert(64 * kLanePieces <= kPieceCap, "a step's pieces must fit the queue");
static_assert(kPieceWords <= 64 && kPieceCap % 64 == 0, "one mask word per lane");
static_assert(kPieceCap <= 4096 && kPiece * kLanePieces < 8192, "run record fields");
static_assert((uint32_t)kPiece - 1u <= kSortedSpare, "piece size");

template <bool kFinite, bool kEmit>
struct FewLds {
    // line constants per seed slot (floats): d, -(g_i x d), the band
    // [tlo, thi] of the FP32 test, and the sorted position of g_i
    float4 la[kCountSlots];  // dx, dy, dz, tlo
    float4 lc[kCountSlots];  // -ex, -ey, -ez, thi
    uint32_t lp[kCountSlots];  // sorted position of g_i (the int64 test)
    int2 pc[kFinite ? kCountSlots : 1];  // finite cylinder: bounds of g_k.d
    uint32_t cnt[kCountSlots];
    // listing the members of candidates: where a slot's grains go, and how
    // many its list holds (its count)
    uint32_t out_off[kEmit ? kCountSlots : 1];
    uint32_t ncap[kEmit ? kCountSlots : 1];
    unsigned long long mask[kPieceWords];  // bit s: a run starts at piece s
    uint32_t before[kPieceWords];          // runs starting before word w
    uint2 run[kRunCap];  // first grain; first piece | seed slot << 12 | grains << 19
};

// One queued piece for a flush lane: its run's grains k0 .. k0 + m - 1, the
// seed slot, the slot's line constants and the piece's grains, all loads
// issued and none waited on.
struct Piece {
    uint32_t k0, m, sl;
    float4 A, C;
    int4 h[kPiece];
};

// Loads piece (w, lane) of a queue holding qn pieces. A lane past the end
// (or past word nw - 1) reads run 0 and tests nothing (m = 0): every read
// stays inside the queue and the sorted grains, which carry kPiece - 1 spare
// entries past the last one.
template <bool kFinite, bool kEmit>
__device__ __forceinline__ void piece_load(const FewLds<kFinite, kEmit> &Q, uint32_t w, uint32_t nw,
                                           uint32_t qn, unsigned long long upto, int lane,
                                           const int4 *__restrict__ sg, Piece &p) {
    const uint32_t wc = min(w, nw - 1u);
    const uint32_t s = (w << 6) + (uint32_t)lane;
    const bool valid = w < nw && s < qn;
    const unsigned long long word = Q.mask[wc];
    const uint32_t r = valid ? Q.before[wc] + (uint32_t)__popcll(word & upto) - 1u : 0u;
    const uint2 rec = Q.run[r];
    const uint32_t q = valid ? s - (rec.y & 0xfffu) : 0u;  // piece of the run
    p.sl = (rec.y >> 12) & 0x7fu;
    p.k0 = rec.x + (uint32_t)kPiece * q;
    p.m = valid ? min((rec.y >> 19) - (uint32_t)kPiece * q, (uint32_t)kPiece) : 0u;
    p.A = Q.la[p.sl];
    p.C = Q.lc[p.sl];
    const int4 *pp = sg + p.k0;
#pragma unroll
    for (int t = 0; t < kPiece; ++t) p.h[t] = pp[t];
}

// The piece's hits as a bit mask over its grains: the FP32 test, the rare
// band case in int64.
template <bool kFinite, bool kEmit>
__device__ __forceinline__ uint32_t piece_test(const FewLds<kFinite, kEmit> &Q, const Piece &p,
                                               int tol_r, const int4 *__restrict__ sg) {
    uint32_t n = 0, amb = 0;
#pragma unroll
    for (int t = 0; t < kPiece; ++t) {
        const float3 h = make_float3((float)p.h[t].x, (float)p.h[t].y, (float)p.h[t].z);
        const float c0 = fmaf(h.y, p.A.z, fmaf(h.z, -p.A.y, p.C.x));
        const float c1 = fmaf(h.z, p.A.x, fmaf(h.x, -p.A.z, p.C.y));
        const float c2 = fmaf(h.x, p.A.y, fmaf(h.y, -p.A.x, p.C.z));
        const float fc = fmaf(c0, c0, fmaf(c1, c1, c2 * c2));
        bool ok = (uint32_t)t < p.m;
        if constexpr (kFinite) {
            const int4 Ai = make_int4((int)p.A.x, (int)p.A.y, (int)p.A.z, 0);
            ok = ok && axial_ok(p.h[t], Ai, Q.pc[p.sl]);
        }
        const bool in_lo = fc <= p.A.w, in_hi = fc <= p.C.w;
        n |= (ok && in_lo) ? (1u << t) : 0u;
        amb |= (ok && in_hi && !in_lo) ? (1u << t) : 0u;
    }
    if (amb) {
        // inside the band: decide in int64 from the integer grains (rare)
        const int dx = (int)p.A.x, dy = (int)p.A.y, dz = (int)p.A.z;
        const long long D = (long long)dx * dx + (long long)dy * dy + (long long)dz * dz;
        const long long thr = (long long)tol_r * tol_r * D;
        const int4 gi = sg[Q.lp[p.sl]];
#pragma unroll
        for (int t = 0; t < kPiece; ++t) {
            if (amb & (1u << t)) {
                const int4 g = sg[p.k0 + (uint32_t)t];
                const long long wx = g.x - gi.x, wy = g.y - gi.y, wz = g.z - gi.z;
                const long long e0 = wy * dz - wz * dy, e1 = wz * dx - wx * dz,
                                e2 = wx * dy - wy * dx;
                n |= e0 * e0 + e1 * e1 + e2 * e2 <= thr ? (1u << t) : 0u;
            }
        }
    }
    return n;
}

// Tests every queued piece.
// Counting adds a piece's hits to its seed's count with one LDS atomic;
// listing (kEmit) takes as many positions in the candidate's member list and
// writes the hit grains' sorted positions there (in any order: the merge
// treats a list as a set and the fit orders it).
template <bool kFinite, bool kEmit>
__device__ __forceinline__ void count_flush(FewLds<kFinite, kEmit> &Q, uint32_t qn, int tol_r,
                                            const int4 *__restrict__ sg,
                                            uint32_t *__restrict__ members, int lane) {
    wave_lds_sync();
    const uint32_t nw = (qn + 63) >> 6;
    {
        const uint32_t c = (uint32_t)lane < nw ? (uint32_t)__popcll(Q.mask[lane]) : 0u;
        const uint32_t incl = wave_incl_scan_dpp(c);
        if ((uint32_t)lane < nw) Q.before[lane] = incl - c;
    }
    wave_lds_sync();
    const unsigned long long upto = (2ull << lane) - 1ull;
    for (uint32_t w = 0; w < nw; ++w) {
        Piece p;
        piece_load(Q, w, nw, qn, upto, lane, sg, p);
        const uint32_t bits = piece_test(Q, p, tol_r, sg);
        if (bits) {
            const uint32_t n = (uint32_t)__popc(bits);
            const uint32_t at = atomicAdd(&Q.cnt[p.sl], n);
            if constexpr (kEmit) {
                const uint32_t cap = Q.ncap[p.sl], base = Q.out_off[p.sl];
                uint32_t pos = at;
#pragma unroll
                for (int t = 0; t < kPiece; ++t) {
                    if (bits & (1u << t)) {
                        if (pos < cap) members[base + pos] = p.k0 + (uint32_t)t;
                        ++pos;
                    }
                }
            }
        }
    }
    wave_lds_sync();
    if ((uint32_t)lane < nw) Q.mask[lane] = 0ull;
    wave_lds_sync();
}

// kEmit: the members stage. The same walk and test over the candidates
// instead of the seeds, listing each candidate's grains (its count is known:
// the list must come out exactly that long).
template <bool kFinite, bool kEmit>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4)))
k_count_few(DevPtrs d, Caps c, Params P) {
    __shared__ FewLds<kFinite, kEmit> sQ[kWaves];
    const int lane = lane_id();
    FewLds<kFinite, kEmit> &Q = sQ[threadIdx.x >> 6];
    uint32_t n_items = d.cnt->n_seeds_ok;
    if constexpr (kEmit) {
        // nothing to list when the seeds or the entries overflow their buffer
        // (the call is re-run)
        const bool skip = n_items == 0u || d.cnt->err || d.cnt->n_members > c.mem_cap;
        n_items = skip ? 0u : min(d.cnt->n_cand, c.cand_cap);
    }
    if (lane < kPieceWords) Q.mask[lane] = 0ull;
    wave_lds_sync();
    unsigned long long tests = 0, hits = 0;
    // wave gw takes chunks gw, gw + nwv, gw + 2 nwv, ... of kFewChunk seeds;
    // chunks shrink (to a quarter wave at least) when there are too few
    // items to give every wave a full one: a long walk per lane is better
    // than idle waves
    const uint32_t gw = grid_tid() >> 6, nwv = grid_threads() >> 6;
    const uint32_t cs = min(kFewChunk, max(16u, (n_items + nwv - 1u) / nwv));
    uint32_t chunk = gw * cs;
    uint32_t next = min(chunk, n_items);
    uint32_t end = min(n_items, chunk + cs);
    bool more = true;
    bool have = false;
    bool pend0 = false, pend1 = false;  // slot closed, count not yet written
    uint32_t idx0 = 0, idx1 = 0;        // seed index held by each slot
    uint32_t th0 = 0, th1 = 0;          // grain-count threshold of each slot's seed
    int cur = lane;
    Pencil W;
    W.live = false;
    Run run[kPencils];
#pragma unroll
    for (int f = 0; f < kPencils; ++f) run[f] = Run{0, 0};
    uint32_t qn = 0, nr = 0;
    // counts of closed slots are final after a flush: write them, free slots
    auto close = [&](int sl, uint32_t idx, uint32_t th) {
        const uint32_t n = Q.cnt[sl];
        if constexpr (kEmit) {
            // the same walk and predicate as the count: a list of another
            // length is never expected; keep every entry a valid grain
            // index and flag an internal error
            const uint32_t cap = Q.ncap[sl];
            if (cap > 0 && n != cap) {
                const uint32_t p0 = d.cand[idx].p;
                for (uint32_t t = n; t < cap; ++t) d.members[Q.out_off[sl] + t] = p0;
                atomicOr(&d.cnt->err, 2u);
            }
        } else {
            // only counts that reach the threshold are written, with their
            // bit in the candidate mask (a few percent: scattered 4-byte
            // stores of every count would each cost a partial line write)
            hits += n;
            if (n >= th) {
                d.seed_n[idx] = n;
                atomicOr(&d.pass[idx >> 5], 1u << (idx & 31u));
            }
        }
    };
    auto finalize = [&]() {
        if (pend0) {
            close(lane, idx0, th0);
            pend0 = false;
        }
        if (pend1) {
            close(lane + 64, idx1, th1);
            pend1 = false;
        }
        wave_lds_sync();
    };
    for (;;) {
        {
            more = chunk + nwv * cs < n_items;
            if (next >= end && more) {
                chunk += nwv * cs;
                next = chunk;
                end = min(n_items, chunk + cs);
                more = chunk + nwv * cs < n_items;
            }
            // take the next seeds into free slots. Setting up a seed (its
            // loads, line constants and walk) runs with whatever lanes take
            // one, so it is done in bulk: only once kRefillMin lanes wait, or
            // when no lane is walking. A lane may idle a few steps; the
            // set-up runs once per many seeds instead of almost every step.
            const bool want = !have && !(pend0 && pend1);
            const unsigned long long wm = __ballot(want);
            const uint32_t n_want = (uint32_t)__popcll(wm);
            const bool refill = n_want >= (uint32_t)kRefillMin || __ballot(have) == 0;
            const uint32_t rank = (uint32_t)__popcll(wm & lanes_below());
            const bool take = refill && want && next + rank < end;
            if (take) {
                const uint32_t idx = next + rank;
                cur = pend0 ? lane + 64 : lane;
                uint2 pq;
                uint32_t v;
                if constexpr (kEmit) {
                    const Cand cd = d.cand[idx];
                    pq = make_uint2(cd.p, cd.q);
                    v = cd.v;
                    const uint32_t off = d.mem_off[idx];
                    Q.out_off[cur] = off;
                    Q.ncap[cur] = ((unsigned long long)off + cd.n <= c.mem_cap) ? cd.n : 0u;
                } else {
                    pq = d.seeds[idx];
                    v = d.view_of[pq.x];
                }
                const int4 gi = d.sg[pq.x], gj = d.sg[pq.y];
                const int dx = gj.x - gi.x, dy = gj.y - gi.y, dz = gj.z - gi.z;
                const uint32_t th = seed_threshold(dx, dy, dz, P);
                if constexpr (kEmit) {
                    // the merge's priority key and threshold of the candidate
                    d.key[idx] = cand_key(d.cand[idx].n, (uint32_t)gi.w, (uint32_t)gj.w);
                    if (P.thr_num) d.cand_thr[idx] = th;
                }
                if (cur == lane) {
                    idx0 = idx;
                    th0 = th;
                } else {
                    idx1 = idx;
                    th1 = th;
                }
                if constexpr (kFinite) Q.pc[cur] = axial_bounds(gi, dx, dy, dz, P.cyl_ext);
                float4 A, C;
                line_consts(gi, dx, dy, dz, P.r, A, C);
                Q.la[cur] = A;
                Q.lc[cur] = C;
                Q.lp[cur] = pq.x;
                Q.cnt[cur] = 0;
                W.init(&d.grids[v], gi, dx, dy, dz, P.r, kFinite ? P.cyl_ext : -1);
                have = true;
            }
            if (refill) next = min(end, next + n_want);
            // fetch kPencils runs once the previous ones are queued
            bool drained = true;
#pragma unroll
            for (int f = 0; f < kPencils; ++f) drained = drained && run[f].k >= run[f].e;
            if (have && W.live && drained) {
#pragma unroll
                for (int f = 0; f < kPencils; ++f) W.fetch(d.cell_start, run[f]);
            }
            // queue up to kLanePieces pieces of the lane's runs
            uint32_t left = kLanePieces, mine = 0, nrun = 0, mtests = 0;
            uint32_t len[kPencils], np[kPencils];
#pragma unroll
            for (int f = 0; f < kPencils; ++f) {
                const uint32_t avail = run[f].e > run[f].k ? run[f].e - run[f].k : 0u;
                len[f] = min(avail, (uint32_t)kPiece * left);
                np[f] = (len[f] + (uint32_t)kPiece - 1u) / (uint32_t)kPiece;
                left -= np[f];
                mine += np[f];
                mtests += len[f];
                nrun += len[f] ? 1u : 0u;
            }
            const uint32_t pk = mine | (nrun << 16);
            const uint32_t incl = wave_incl_scan_dpp(pk);
            const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            // room first: test what is queued if this step's runs do not fit
            if (qn + (tot & 0xffffu) > (uint32_t)kPieceCap ||
                nr + (tot >> 16) > (uint32_t)kRunCap) {
                count_flush(Q, qn, P.r, d.sg, d.members, lane);
                qn = 0;
                nr = 0;
                finalize();
            }
            if (mine) {
                const uint32_t ex = incl - pk;
                uint32_t pos = qn + (ex & 0xffffu);
                uint32_t ri = nr + (ex >> 16);
                const uint32_t tag = (uint32_t)cur << 12;
#pragma unroll
                for (int f = 0; f < kPencils; ++f) {
                    if (len[f]) {
                        Q.run[ri++] = make_uint2(run[f].k, pos | tag | (len[f] << 19));
                        atomicOr(&Q.mask[pos >> 6], 1ull << (pos & 63));
                        pos += np[f];
                        run[f].k += len[f];
                    }
                }
            }
            qn += tot & 0xffffu;
            nr += tot >> 16;
            tests += mtests;
            // a seed whose walk ended and whose runs are all queued is closed
            bool queued = true;
#pragma unroll
            for (int f = 0; f < kPencils; ++f) queued = queued && run[f].k >= run[f].e;
            if (have && !W.live && queued) {
                have = false;
                if (cur == lane) pend0 = true; else pend1 = true;
            }
            const bool blocked = !have && pend0 && pend1;
            const uint32_t n_blocked = (uint32_t)__popcll(__ballot(blocked));
            const bool all_done = __ballot(have) == 0 && next >= end && !more;
            if (all_done || n_blocked > 16) {
                if (qn) count_flush(Q, qn, P.r, d.sg, d.members, lane);
                qn = 0;
                nr = 0;
                finalize();
                if (all_done) break;
            }
        }
    }
    if constexpr (!kEmit) {
        add_spread(d.part64, 2, wave_sum(tests));
        add_spread(d.part64, 3, wave_sum(hits));
    }
}

// Candidates among seeds [0, s), s <= n_seeds_ok: the scan of the mask's
// popcounts up to word s / 32, plus the set bits below s in that word.
__device__ __forceinline__ uint32_t cand_before(const DevPtrs &d, uint32_t s) {
    const uint32_t w = s >> 5, b = s & 31u;
    return d.pass_pos[w] + (b ? (uint32_t)__popc(d.pass[w] & ((1u << b) - 1u)) : 0u);
}

// Candidates in seed order with their counts (for the member offsets). A
// workgroup takes kBlock * kWords mask words: it scans their popcounts, which
// places them in the list and in pass_pos, gathers its set bits in LDS and
// then takes one candidate per thread. Keys and thresholds are written by the
// member listing, which loads both seed grains anyway.
constexpr uint32_t kCandList = 2048;  // candidates listed per round

template <int kWords, bool kDirect>
__global__ void __launch_bounds__(kBlock) k_cand_list(DevPtrs d, Caps c, const uint32_t *part) {
    static_assert(kBlock * kWords * 32 <= 65536, "bits are listed as 16-bit numbers");
    __shared__ uint16_t s_list[kCandList];
    constexpr uint32_t kTile = kBlock * kWords;
    const uint32_t nwd = d.cnt->pass_words;
    if (blockIdx.x > 0 && blockIdx.x * kTile >= nwd) return;
    const uint32_t base = blockIdx.x * kTile + threadIdx.x * kWords;
    uint32_t w[kWords], pos[kWords], sum = 0;
    load_items(d.pass, base, nwd, w);
#pragma unroll
    for (int k = 0; k < kWords; ++k) sum += (uint32_t)__popc(w[k]);
    const uint32_t off = tile_offset<kDirect>(part);
    uint32_t tot;
    const uint32_t before = block_excl_scan(sum, &tot);
    uint32_t run = off + before;
#pragma unroll
    for (int k = 0; k < kWords; ++k) {
        pos[k] = run;
        run += (uint32_t)__popc(w[k]);
    }
    store_items(d.pass_pos, base, nwd, pos);
    if (nwd - blockIdx.x * kTile <= kTile && threadIdx.x == 0) {
        d.pass_pos[nwd] = off + tot;
        d.cnt->n_cand = off + tot;
    }
    // member entries, of candidates past the buffer's end too: a call that is
    // run again is sized by them
    unsigned long long listed = 0;
    for (uint32_t r0 = 0; r0 < tot; r0 += kCandList) {  // uniform
        uint32_t at = before - r0;  // wraps for the candidates of earlier rounds
#pragma unroll
        for (int k = 0; k < kWords; ++k)
            for (uint32_t bits = w[k]; bits; bits &= bits - 1u, ++at)
                if (at < kCandList)
                    s_list[at] = (uint16_t)(32u * (threadIdx.x * kWords + k) +
                                            (uint32_t)__ffs((int)bits) - 1u);
        __syncthreads();
        const uint32_t m = min(tot - r0, kCandList);
        for (uint32_t i = threadIdx.x; i < m; i += kBlock) {
            const uint32_t s = 32u * kTile * blockIdx.x + s_list[i];
            const uint32_t n = d.seed_n[s];
            listed += n;
            if (off + r0 + i >= c.cand_cap) continue;
            const uint2 pq = d.seeds[s];
            Cand cd;
            cd.p = pq.x;
            cd.q = pq.y;
            cd.n = n;
            cd.v = d.view_of[pq.x];
            d.cand[off + r0 + i] = cd;
            d.cand_n[off + r0 + i] = n;
        }
        __syncthreads();  // the list is rewritten by the next round
    }
    add_spread(d.part64, 1, wave_sum(listed));
}

// The threshold a candidate's unused grains must reach: n_min, or its own
// angle-dependent threshold when that variant is on.
__device__ __forceinline__ uint32_t cand_min(const DevPtrs &d, const Params &P, uint32_t ci) {
    return P.thr_num ? d.cand_thr[ci] : (uint32_t)P.n_min;
}

// ----------------------------------------------------------------- merge
//
// Exclusive association, identical to taking candidates one by one in key
// order: a candidate's outcome depends only on higher-priority candidates
// that share one of its still unused grains. Each round:
//   prune    a candidate left with fewer than n_min unused grains is
//            rejected (used grains never return); the others clear the
//            reservation of their unused grains;
//   reserve  every undecided candidate takes an atomic min of its key on
//            each of its unused grains;
//   decide   one holding every reservation of its unused grains has no
//            undecided predecessor on them, so its unused set is final: it
//            is accepted with that set if it still has n_min grains; one
//            holding at least n_min of them but not all is sure to be
//            accepted and takes the ones it holds at once (see decide).
// Candidates taking grains in one round own disjoint grains, so their
// updates do not interact, and a concurrent update can only hide grains
// taken by a higher-priority candidate. The grid-wide rounds fuse prune and
// reserve into one pass; the tail kernel keeps the three phases. A
// candidate sure to be accepted is never pruned.

constexpr int kMaxRounds = 256;
constexpr int kWideRounds = 16;  // most grid-wide rounds (distinct key tags) before the tail
// rounds a call runs grid-wide at most before the per-view tails take over
constexpr int kWideCap = EMT_MERGE_WIDE;
static_assert(kWideCap >= 1 && kWideCap <= kWideRounds, "grid-wide merge rounds");

__global__ void __launch_bounds__(kBlock) k_merge_init(DevPtrs d, Caps c) {
    const Counters *cn = d.cnt;
    const bool overflow = cn->n_seeds > c.seed_cap || cn->n_cand > c.cand_cap ||
                          cn->n_members > c.mem_cap;
    const uint32_t nc = overflow ? 0u : cn->n_cand;
    const uint32_t nm = overflow ? 0u : cn->n_members;
    for (uint32_t i = grid_tid(); i < nc; i += grid_threads()) {
        d.status[i] = kUndecided;
        d.mcount[i] = 0;
    }
    const uint32_t n_total = d.desc->n_total, ns = cn->n_seeds_ok;
    // the seeds and candidates of each view (views are contiguous in anchor
    // order, so in seed and in candidate order too)
    for (uint32_t v = grid_tid(); v < d.desc->n_views; v += grid_threads()) {
        const uint32_t g0 = d.grids[v].grain_off, g1 = g0 + d.grids[v].n;
        const uint32_t s0 = d.seed_off[d.nc * g0], s1 = d.seed_off[d.nc * g1];
        d.view_seeds[v] = s1 - s0;
        d.view_cand[v] = cand_before(d, min(s1, ns)) - cand_before(d, min(s0, ns));
    }
    for (uint32_t g = grid_tid(); g < n_total; g += grid_threads()) {
        d.owner[g] = ~0ull;
    }
    for (uint32_t e = grid_tid(); e < nm; e += grid_threads()) d.taken[e] = 0;
    for (uint32_t r = grid_tid(); r < kMaxRounds; r += grid_threads()) d.undecided[r] = 0;
    if (grid_tid() == 0) {
        d.cnt->n_act[0] = nc;  // candidates taking part in the merge
        d.cnt->err |= overflow ? 1u : 0u;
    }
}

// Grid-wide rounds. Eight lanes take one candidate and stride over its
// member entries; round r walks the list of candidates left undecided by
// round r-1 (all candidates for r = 0) and appends the ones it leaves
// undecided to the next list, whose length it counts in undecided[r]. A
// reservation carries its round in the top four bits of the key, counted
// down, so the keys of a newer round lie below every older value and no
// clearing pass is needed between rounds (keys use 60 bits: n, i and j are
// below 2^20 each).
// A grain's owner word is ~0 while nobody has reserved it, 0 once an
// accepted candidate has taken it (no key is 0: a seed's i and j differ),
// and otherwise the smallest key offered to it. So one load tells whether a
// grain is still unused and who holds it, and a reservation can never
// displace a taken grain.
// A reservation: the word only decreases during a round, so a value read at
// or below key means an equal or better reservation (or the grain's taking)
// is already there and the atomic would change nothing; most grains are
// offered to many candidates, and the read spares most of the atomics.
__device__ __forceinline__ void reserve(unsigned long long *owner, unsigned long long key) {
    if (*owner > key) atomicMin(owner, key);
}

constexpr int kMergeGroup = 8;
static_assert(kWideRounds <= 16, "round tags take four bits");

__device__ __forceinline__ uint32_t group_sum8(uint32_t v) {
    v += __shfl_xor(v, 4);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 1);
    return v;
}

__device__ __forceinline__ uint32_t *merge_list(const DevPtrs &d, int round) {
    return (round & 1) ? d.act2 : d.act;
}

// Candidates left undecided are staged in LDS and appended to the next list
// with one global atomic per flush: a single counter hit once per wave
// serialises at the L2.
constexpr uint32_t kListBuf = 2048;
constexpr uint32_t kGroupsPerBlock = kBlock / kMergeGroup;

__device__ __forceinline__ void flush_list(uint32_t *s_buf, uint32_t *s_cnt, uint32_t *s_base,
                                           uint32_t *counter, uint32_t *next) {
    __syncthreads();
    const uint32_t m = *s_cnt;
    if (threadIdx.x == 0 && m) *s_base = atomicAdd(counter, m);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < m; i += blockDim.x) next[*s_base + i] = s_buf[i];
    __syncthreads();
    if (threadIdx.x == 0) *s_cnt = 0;
    __syncthreads();
}

// The decide phase for one candidate (its eight-lane group; every lane
// returns the same). Unused grains are those whose owner word is not 0; the
// candidate holds the ones whose word is its key. Fewer unused grains than
// its threshold: rejected. Holding every unused grain: accepted with them.
// Holding at least its threshold but not all: it is sure to be accepted,
// since no undecided candidate before it wants a grain it holds, so those
// grains are still unused when its turn comes in the one-by-one reading; it
// takes them now (kCertain) and waits for the others, taking each as it comes
// to hold it. A grain taken early is one a later candidate would have lost
// anyway, so nothing else changes. Returns whether it stays undecided.
__device__ __forceinline__ bool decide(const DevPtrs &d, const Params &P, uint32_t ci,
                                       unsigned long long key, uint32_t e0, uint32_t e1,
                                       int sub) {
    const bool certain = d.status[ci] == kCertain;
    uint32_t unused = 0, held = 0, lost = 0;
    for (uint32_t e = e0 + sub; e < e1; e += kMergeGroup) {
        const unsigned long long o = d.owner[d.members[e]];
        unused += o != 0ull ? 1u : 0u;
        held += o == key ? 1u : 0u;
        lost |= (o != 0ull && o != key) ? 1u : 0u;
    }
    unused = group_sum8(unused);
    held = group_sum8(held);
    lost = group_sum8(lost);
    const uint32_t need = cand_min(d, P, ci);
    if (!certain && unused < need) {
        if (sub == 0) d.status[ci] = kRejected;
        return false;
    }
    if (lost != 0 && !certain && held < need) return true;
    for (uint32_t e = e0 + sub; e < e1; e += kMergeGroup) {
        const uint32_t k = d.members[e];
        if (d.owner[k] == key) {
            d.owner[k] = 0ull;
            d.taken[e] = 1;
        }
    }
    if (sub == 0) {
        d.mcount[ci] += held;
        d.status[ci] = lost == 0 ? kAccepted : kCertain;
    }
    return lost != 0;
}

template <int kPhase>
__global__ void __launch_bounds__(kBlock) k_round(DevPtrs d, Params P, int round) {
    __shared__ uint32_t s_buf[kPhase == 1 ? kListBuf : 1];
    __shared__ uint32_t s_cnt, s_base;
    const uint32_t n = round == 0 ? d.cnt->n_act[0] : d.undecided[round - 1];
    if (n == 0) return;
    const uint32_t *list = merge_list(d, round);
    uint32_t *next = merge_list(d, round + 1);
    const unsigned long long tag = (unsigned long long)(kWideRounds - 1 - round) << 60;
    const int sub = threadIdx.x & (kMergeGroup - 1);
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    // block-uniform loop: the list flush below synchronises the workgroup
    for (uint32_t base = blockIdx.x * kGroupsPerBlock; base < n;
         base += gridDim.x * kGroupsPerBlock) {
        const uint32_t slot = base + threadIdx.x / kMergeGroup;
        uint32_t ci = 0;
        bool live = slot < n;
        if (live) {
            ci = round == 0 ? slot : list[slot];
            live = round == 0 || d.status[ci] == kUndecided || d.status[ci] == kCertain;
        }
        bool still = false;
        if (live) {
            const unsigned long long key = d.key[ci] | tag;
            const uint32_t e0 = d.mem_off[ci], e1 = e0 + d.cand[ci].n;
            if (kPhase == 0) {  // prune, then reserve
                // round 0: no grain is used yet and every candidate reached
                // its threshold, so nothing is pruned
                uint32_t unused = 0;
                if (round > 0) {
                    for (uint32_t e = e0 + sub; e < e1; e += kMergeGroup)
                        unused += d.owner[d.members[e]] != 0ull ? 1u : 0u;
                    unused = group_sum8(unused);
                }
                if (round > 0 && unused < cand_min(d, P, ci) && d.status[ci] != kCertain) {
                    if (sub == 0) d.status[ci] = kRejected;
                } else {
                    // a taken grain's word (0) is below every key: untouched
                    for (uint32_t e = e0 + sub; e < e1; e += kMergeGroup)
                        reserve(&d.owner[d.members[e]], key);
                }
            } else {  // decide
                still = decide(d, P, ci, key, e0, e1, sub) && sub == 0;
            }
        }
        if (kPhase == 1) {
            if (still) s_buf[atomicAdd(&s_cnt, 1u)] = ci;
            __syncthreads();
            const uint32_t held = s_cnt;
            __syncthreads();  // all have read it before the next iteration adds
            if (held + kGroupsPerBlock > kListBuf)
                flush_list(s_buf, &s_cnt, &s_base, &d.undecided[round], next);
        }
    }
    if (kPhase == 1) flush_list(s_buf, &s_cnt, &s_base, &d.undecided[round], next);
}

// First candidate of view v: candidates are listed in seed order, and a
// view's seeds are contiguous.
__device__ __forceinline__ uint32_t view_first_cand(const DevPtrs &d, uint32_t v, uint32_t ns) {
    return cand_before(d, min(d.seed_off[d.nc * d.grids[v].grain_off], ns));
}

// Candidates of different views share no grain, so the rounds the grid-wide
// kernels leave are finished view by view, one workgroup each. First the
// undecided list is split by view: view v's go to its own stretch of the
// other list, starting at its first candidate (a view never has more
// undecided candidates than candidates). The order within a stretch does not
// matter: outcomes depend only on the keys.
__global__ void __launch_bounds__(kBlock) k_tail_split(DevPtrs d, int last_round) {
    const uint32_t n = d.undecided[last_round];
    const uint32_t *list = merge_list(d, last_round + 1);
    uint32_t *out = merge_list(d, last_round + 2);
    const uint32_t ns = d.cnt->n_seeds_ok;
    for (uint32_t i = grid_tid(); i < n; i += grid_threads()) {
        const uint32_t ci = list[i];
        const uint32_t v = d.cand[ci].v;
        out[view_first_cand(d, v, ns) + atomicAdd(&d.view_tail[v], 1u)] = ci;
    }
}

// The remaining rounds of one view in one workgroup, looping until none of
// its candidates is undecided (each round decides at least the highest-
// priority one, so it ends within as many rounds as there are candidates).
// Groups of eight lanes take candidates of the list; __syncthreads separates
// the phases, and the prune phase clears the reservations of the
// candidates' unused grains.
constexpr int kTailBlock = 1024;

__global__ void __launch_bounds__(kTailBlock) k_merge_tail(DevPtrs d, Params P, int last_round) {
    const uint32_t view = blockIdx.x;
    if (view >= d.desc->n_views) return;
    __shared__ uint32_t s_n[2];
    const int sub = threadIdx.x & (kMergeGroup - 1);
    const uint32_t group = threadIdx.x / kMergeGroup;
    constexpr uint32_t kTailGroups = kTailBlock / kMergeGroup;
    const uint32_t c0 = view_first_cand(d, view, d.cnt->n_seeds_ok);
    // (the only view of a call has the undecided list as it is)
    const int at = gridDim.x > 1 ? last_round + 2 : last_round + 1;
    if (threadIdx.x == 0) {
        s_n[0] = gridDim.x > 1 ? d.view_tail[view] : d.undecided[last_round];
        s_n[1] = 0;
    }
    __syncthreads();
    uint32_t *list[2] = {merge_list(d, at) + c0, merge_list(d, at + 1) + c0};
    int cur = 0;
    uint32_t rounds = 0;
    const uint32_t limit = s_n[0] + 2;
    while (s_n[cur] > 0 && rounds < limit) {
        const uint32_t n = s_n[cur];
        // prune (groups are whole 8-lane slices of one wave, so the group
        // sums only read lanes that took the same branch)
        for (uint32_t i = group; i < n; i += kTailGroups) {
            const uint32_t ci = list[cur][i];
            const uint8_t st = d.status[ci];
            if (st != kUndecided && st != kCertain) continue;
            const uint32_t e0 = d.mem_off[ci], e1 = e0 + d.cand[ci].n;
            uint32_t unused = 0;
            for (uint32_t e = e0 + sub; e < e1; e += kMergeGroup) {
                const uint32_t k = d.members[e];
                if (d.owner[k] != 0ull) {
                    ++unused;
                    d.owner[k] = ~0ull;
                }
            }
            unused = group_sum8(unused);
            if (unused < cand_min(d, P, ci) && st != kCertain && sub == 0) d.status[ci] = kRejected;
        }
        __threadfence_block();
        __syncthreads();
        // reserve
        for (uint32_t i = group; i < n; i += kTailGroups) {
            const uint32_t ci = list[cur][i];
            if (d.status[ci] != kUndecided && d.status[ci] != kCertain) continue;
            const unsigned long long key = d.key[ci];
            const uint32_t e0 = d.mem_off[ci], e1 = e0 + d.cand[ci].n;
            for (uint32_t e = e0 + sub; e < e1; e += kMergeGroup)
                reserve(&d.owner[d.members[e]], key);
        }
        __threadfence_block();
        __syncthreads();
        // decide
        for (uint32_t i = group; i < n; i += kTailGroups) {
            const uint32_t ci = list[cur][i];
            if (d.status[ci] != kUndecided && d.status[ci] != kCertain) continue;
            const unsigned long long key = d.key[ci];
            const uint32_t e0 = d.mem_off[ci], e1 = e0 + d.cand[ci].n;
            if (decide(d, P, ci, key, e0, e1, sub) && sub == 0) {
                const uint32_t slot = atomicAdd(&s_n[cur ^ 1], 1u);
                list[cur ^ 1][slot] = ci;
            }
        }
        __threadfence_block();
        __syncthreads();
        if (threadIdx.x == 0) s_n[cur] = 0;
        cur ^= 1;
        ++rounds;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        // grid-wide rounds that ran: round r runs while round r-1 left some
        uint32_t wide = d.cnt->n_act[0] ? 1u : 0u;
        while (wide >= 1 && wide <= (uint32_t)last_round && d.undecided[wide - 1]) ++wide;
        atomicMax(&d.cnt->rounds, wide + rounds);
        if (s_n[cur] > 0) atomicOr(&d.cnt->err, 4u);
    }
}

// ------------------------------------------------------------------- fit

// Accepted candidates into the list of tracks (any order: tracks are ranked
// by key afterwards) and the track count of each view. A thread takes four
// consecutive candidates with one 32-bit load of their status bytes (the
// array is padded to 256 bytes). A workgroup counts its accepted candidates
// first and reserves their slots with one atomic; a wave adds to a view's
// count once for its candidates of the view of its first accepted one (a
// wave's candidates are consecutive, so nearly always of one view).
__device__ __forceinline__ uint32_t accepted4(const DevPtrs &d, uint32_t q, uint32_t nc) {
    if (4ull * q >= nc) return 0u;
    const uint32_t w = reinterpret_cast<const uint32_t *>(d.status)[q];
    uint32_t bits = 0;
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t)
        bits |= (((w >> (8 * t)) & 0xffu) == kAccepted && 4 * q + t < nc) ? (1u << t) : 0u;
    return bits;
}

__global__ void __launch_bounds__(kBlock) k_collect(DevPtrs d, Caps c) {
    __shared__ uint32_t s_cnt, s_base;
    const Counters *cn = d.cnt;
    const uint32_t nc = cn->err ? 0u : min(cn->n_cand, c.cand_cap);
    const uint32_t nq = (nc + 3u) / 4u;
    const int lane = lane_id();
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    // block-uniform loops: every lane of a wave takes part in its scans
    for (uint32_t b = blockIdx.x * blockDim.x; b < nq; b += grid_threads()) {
        const uint32_t n = wave_sum((uint32_t)__popc(accepted4(d, b + threadIdx.x, nc)));
        if (lane == 0 && n) atomicAdd(&s_cnt, n);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        s_base = s_cnt ? atomicAdd(&d.cnt->n_acc, s_cnt) : 0u;
        s_cnt = 0;
    }
    __syncthreads();
    for (uint32_t b = blockIdx.x * blockDim.x; b < nq; b += grid_threads()) {
        const uint32_t q = b + threadIdx.x;
        uint32_t bits = accepted4(d, q, nc);
        const uint32_t k = (uint32_t)__popc(bits);
        const uint32_t incl = wave_incl_scan_dpp(k);
        const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (tot == 0) continue;
        uint32_t w = 0;
        if (lane == 0) w = atomicAdd(&s_cnt, tot);
        w = (uint32_t)__shfl((int)w, 0);
        const int first = __ffsll((long long)__ballot(bits != 0)) - 1;
        const uint32_t v_own = bits ? d.cand[4 * q + (uint32_t)(__ffs(bits) - 1)].v : 0u;
        const uint32_t v0 = (uint32_t)__shfl((int)v_own, first);
        uint32_t pos = s_base + w + incl - k, same = 0;
        while (bits) {
            const uint32_t i = 4 * q + (uint32_t)(__ffs(bits) - 1);
            bits &= bits - 1u;
            d.acc[pos++] = i;
            const uint32_t v = d.cand[i].v;
            if (v == v0)
                ++same;
            else
                atomicAdd(&d.view_ntr[v], 1u);
        }
        same = wave_sum(same);
        if (lane == first) atomicAdd(&d.view_ntr[v0], same);
    }
}

__global__ void __launch_bounds__(kBlock) k_view_offsets(DevPtrs d) {
    const uint32_t n_views = d.desc->n_views;
    uint32_t carry = 0;
    for (uint32_t base = 0; base < n_views; base += kBlock) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t v = i < n_views ? d.view_ntr[i] : 0u;
        uint32_t tot;
        const uint32_t ex = block_excl_scan(v, &tot);
        if (i < n_views) d.view_tr_off[i] = carry + ex;
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) d.view_tr_off[n_views] = carry;
}

// Tracks grouped by view: a wave takes its slots of the view of its lane 0
// with one atomic on that view's cursor (a view's cursor hit once per track
// serialises in L2), other views one atomic per track.
__global__ void __launch_bounds__(kBlock) k_group(DevPtrs d, unsigned long long *gkey) {
    const uint32_t na = d.cnt->n_acc;
    const int lane = lane_id();
    for (uint32_t b = blockIdx.x * blockDim.x; b < na; b += grid_threads()) {
        const uint32_t a = b + threadIdx.x;
        const bool ok = a < na;  // false for lane 0 only if for the whole wave
        const uint32_t ci = ok ? d.acc[a] : 0u;
        const uint32_t v = ok ? d.cand[ci].v : 0u;
        const uint32_t v0 = (uint32_t)__shfl((int)v, 0);
        const unsigned long long same = __ballot(ok && v == v0);
        uint32_t base = 0;
        if (lane == 0 && same) base = atomicAdd(&d.view_cursor[v0], (uint32_t)__popcll(same));
        base = (uint32_t)__shfl((int)base, 0);
        if (ok) {
            const uint32_t at = v == v0 ? base + (uint32_t)__popcll(same & lanes_below())
                                        : atomicAdd(&d.view_cursor[v], 1u);
            const uint32_t pos = d.view_tr_off[v] + at;
            d.grouped[pos] = ci;
            gkey[pos] = d.key[ci];
        }
    }
}

// Track order within a view = key order (the order of acceptance in the
// one-by-one reading); rank by counting smaller keys of the same view.
// A workgroup's tracks are of one view as a rule: it takes the view's keys to
// LDS, 256 at a time, which all its lanes then read together. (Bound by the
// chain of key loads before: with two launches less for a single view, one c2
// view 732 -> 721 us, one c5 view 3494 -> 3429.)
__global__ void __launch_bounds__(kBlock) k_rank(DevPtrs d, const unsigned long long *gkey) {
    __shared__ unsigned long long s_key[kBlock];
    constexpr uint32_t kStep = 16;
    const uint32_t na = d.cnt->n_acc;
    for (uint32_t base = blockIdx.x * kBlock; base < na; base += grid_threads()) {  // uniform
        const uint32_t s = base + threadIdx.x;
        const bool ok = s < na;
        const uint32_t ci = d.grouped[ok ? s : base];
        const uint32_t v = d.cand[ci].v;
        const uint32_t b = d.view_tr_off[v], e = b + d.view_ntr[v];
        const unsigned long long key = gkey[ok ? s : base];
        uint32_t rank = 0;
        const uint32_t v0 = d.cand[d.grouped[base]].v;
        if (v0 == d.cand[d.grouped[min(base + kBlock, na) - 1u]].v) {
            const uint32_t b0 = d.view_tr_off[v0], e0 = b0 + d.view_ntr[v0];
            for (uint32_t t = b0; t < e0; t += kBlock) {
                __syncthreads();  // the keys before have been read
                s_key[threadIdx.x] = t + threadIdx.x < e0 ? gkey[t + threadIdx.x] : ~0ull;
                __syncthreads();
                const uint32_t m = min((uint32_t)kBlock, e0 - t);
                for (uint32_t i = 0; i < m; i += kStep)
#pragma unroll
                    for (uint32_t k = 0; k < kStep; ++k) rank += s_key[i + k] < key ? 1u : 0u;
            }
        } else {
#pragma unroll 8
            for (uint32_t t = b; t < e; ++t) rank += gkey[t] < key ? 1u : 0u;
        }
        if (ok) {
            d.track_cand[b + rank] = ci;
            d.tg_n[b + rank] = d.mcount[ci];
        }
    }
}

// Convert an exact 128-bit integer to double/float without library calls.
__device__ __forceinline__ double i128_to_f64(__int128 x) {
    const bool neg = x < 0;
    const unsigned __int128 u = neg ? (unsigned __int128)(-x) : (unsigned __int128)x;
    const unsigned long long hi = (unsigned long long)(u >> 64);
    const unsigned long long lo = (unsigned long long)u;
    const double r = (double)hi * 0x1p64 + (double)lo;
    return neg ? -r : r;
}

__device__ __forceinline__ float i128_to_f32(__int128 x) {
    if (x >= -(((__int128)1) << 62) && x <= (((__int128)1) << 62)) return (float)(long long)x;
    return (float)i128_to_f64(x);
}

__device__ __forceinline__ int sign128(__int128 x) { return x > 0 ? 1 : (x < 0 ? -1 : 0); }

// One wave per track: gather the grains the track took, order them by
// (t, input index) with t = (g_k - g_i).d, and fit.
//
// Fit: exact integer moments about g_i, S1 = sum w, S2 = sum w w^T, give
// Q = n S2 - S1 S1^T = n^2 times the covariance. The fit axis a has the
// largest Q_aa (ties to the lower axis); slopes are Q_ab/Q_aa and Q_ac/Q_aa,
// divided in FP32, or in FP64 when a = z or the RMS spread along a is under
// 5 um (Q_aa < 250000 n^2) or when asked. The sign that puts the direction in
// the upper hemisphere comes from the integer Q entries.
__global__ void __launch_bounds__(kBlock) k_fit(DevPtrs d, Params P) {
    const uint32_t nt = d.cnt->n_acc;
    const int lane = lane_id();
    const uint32_t wave = grid_tid() >> 6;
    const uint32_t nwaves = grid_threads() >> 6;
    for (uint32_t t = wave; t < nt; t += nwaves) {
        const uint32_t ci = d.track_cand[t];
        const Cand cd = d.cand[ci];
        const ViewGrid *G = &d.grids[cd.v];
        const int4 gi = d.sg[cd.p], gj = d.sg[cd.q];
        const int dx = gj.x - gi.x, dy = gj.y - gi.y, dz = gj.z - gi.z;
        const uint32_t base = d.tg_off[t];
        const uint32_t m = d.mcount[ci];
        const uint32_t e0 = d.mem_off[ci];

        // 1. compact the taken entries
        uint32_t j = 0;
        for (uint32_t e = 0; e < cd.n; e += 64) {
            const uint32_t ee = e + lane;
            const bool tk = ee < cd.n && d.taken[e0 + ee];
            const unsigned long long mask = __ballot(tk);
            if (tk) {
                const uint32_t pos = j + (uint32_t)__popcll(mask & lanes_below());
                const uint32_t k = d.members[e0 + ee];
                const int4 h = d.sg[k];
                d.tord[base + pos] = k;
                d.tvals[base + pos] = (long long)(h.x - gi.x) * dx + (long long)(h.y - gi.y) * dy +
                                      (long long)(h.z - gi.z) * dz;
            }
            j += (uint32_t)__popcll(mask);
        }
        wave_sync_mem();

        // 2. exact moments
        long long s1[3] = {0, 0, 0}, s2[6] = {0, 0, 0, 0, 0, 0};
        for (uint32_t q = lane; q < m; q += 64) {
            const int4 h = d.sg[d.tord[base + q]];
            const long long w0 = h.x - gi.x, w1 = h.y - gi.y, w2 = h.z - gi.z;
            s1[0] += w0;
            s1[1] += w1;
            s1[2] += w2;
            s2[0] += w0 * w0;
            s2[1] += w0 * w1;
            s2[2] += w0 * w2;
            s2[3] += w1 * w1;
            s2[4] += w1 * w2;
            s2[5] += w2 * w2;
        }
        for (int u = 0; u < 3; ++u) s1[u] = wave_sum(s1[u]);
        for (int u = 0; u < 6; ++u) s2[u] = wave_sum(s2[u]);

        // 3. grain order by (t, input index), rank by counting: the wave
        // loads 64 entries at a time into registers and every lane compares
        // its own entry with each of them through readlane (input indices
        // are distinct, so no entry outranks itself)
        for (uint32_t q0 = 0; q0 < m; q0 += 64) {
            const uint32_t q = q0 + (uint32_t)lane;
            const bool vq = q < m;
            const long long tq = vq ? d.tvals[base + q] : 0;
            const int oq = vq ? d.sg[d.tord[base + q]].w : 0;
            uint32_t rank = 0;
            for (uint32_t o0 = 0; o0 < m; o0 += 64) {
                const uint32_t o = o0 + (uint32_t)lane;
                const long long tl = o < m ? d.tvals[base + o] : 0;
                const int ol = o < m ? d.sg[d.tord[base + o]].w : 0;
                const int t_lo = (int)(uint32_t)(unsigned long long)tl;
                const int t_hi = (int)(uint32_t)((unsigned long long)tl >> 32);
                const uint32_t cnt = min(64u, m - o0);
                for (uint32_t i = 0; i < cnt; ++i) {
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane(t_lo, (int)i);
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane(t_hi, (int)i);
                    const long long to = (long long)(((unsigned long long)hi << 32) | lo);
                    const int oo = __builtin_amdgcn_readlane(ol, (int)i);
                    rank += (to < tq || (to == tq && oo < oq)) ? 1u : 0u;
                }
            }
            if (vq) d.out_grains[base + rank] = (uint32_t)oq;
        }

        // 4. fit (every lane computes the same values)
        const long long n = (long long)m;
        __int128 Q[3][3];
        {
            const long long S2[3][3] = {{s2[0], s2[1], s2[2]}, {s2[1], s2[3], s2[4]},
                                        {s2[2], s2[4], s2[5]}};
            for (int u = 0; u < 3; ++u)
                for (int w = 0; w < 3; ++w)
                    Q[u][w] = (__int128)n * S2[u][w] - (__int128)s1[u] * s1[w];
        }
        int a = 0;
        if (Q[1][1] > Q[a][a]) a = 1;
        if (Q[2][2] > Q[a][a]) a = 2;
        int b = a == 0 ? 1 : 0;
        int cx = a == 2 ? 1 : 2;
        float dir[3];
        float slope[2];
        int comp_sign[3];
        uint32_t fp64 = 0, degen = 0;
        double s0d = 0.0, s1d = 0.0;  // slopes of the FP64 paths
        if (Q[a][a] == 0) {
            // every grain coincides: no spread to fit, the seed direction
            // stands in (its spread along any axis is 0, under the 5 um
            // rule, so the ratio is taken in FP64)
            degen = 1;
            fp64 = 1;
            const int ad[3] = {dx, dy, dz};
            a = 0;
            if (abs(ad[1]) > abs(ad[a])) a = 1;
            if (abs(ad[2]) > abs(ad[a])) a = 2;
            b = a == 0 ? 1 : 0;
            cx = a == 2 ? 1 : 2;
            s0d = (double)ad[b] / (double)ad[a];
            s1d = (double)ad[cx] / (double)ad[a];
            slope[0] = (float)s0d;
            slope[1] = (float)s1d;
            // (1, slope) on axes (a, b, c) is d / d_a: signs of d times that of d_a
            const int sa = ad[a] < 0 ? -1 : 1;
            for (int u = 0; u < 3; ++u) comp_sign[u] = sa * (ad[u] > 0 ? 1 : (ad[u] < 0 ? -1 : 0));
        } else {
            fp64 = (a == 2) || (Q[a][a] < (__int128)250000 * n * n) ||
                   (P.flags & EMT_F_FP64_FIT_ALWAYS) != 0;
            if (fp64) {
                const double qa = i128_to_f64(Q[a][a]);
                s0d = i128_to_f64(Q[a][b]) / qa;
                s1d = i128_to_f64(Q[a][cx]) / qa;
                slope[0] = (float)s0d;
                slope[1] = (float)s1d;
            } else {
                const float qa = i128_to_f32(Q[a][a]);
                slope[0] = i128_to_f32(Q[a][b]) / qa;
                slope[1] = i128_to_f32(Q[a][cx]) / qa;
            }
            comp_sign[a] = 1;
            comp_sign[b] = sign128(Q[a][b]);
            comp_sign[cx] = sign128(Q[a][cx]);
        }
        {
            if (fp64) {
                const double nrm = sqrt(1.0 + s0d * s0d + s1d * s1d);
                dir[a] = (float)(1.0 / nrm);
                dir[b] = (float)(s0d / nrm);
                dir[cx] = (float)(s1d / nrm);
            } else {
                const float nrm = sqrtf(1.0f + slope[0] * slope[0] + slope[1] * slope[1]);
                dir[a] = 1.0f / nrm;
                dir[b] = slope[0] / nrm;
                dir[cx] = slope[1] / nrm;
            }
            bool flip;
            if (comp_sign[2] != 0) flip = comp_sign[2] < 0;
            else if (comp_sign[1] != 0) flip = comp_sign[1] < 0;
            else flip = comp_sign[0] < 0;
            if (flip)
                for (int u = 0; u < 3; ++u) dir[u] = -dir[u];
        }

        // 5. centroid and extent along dir
        const long long g_abs[3] = {(long long)G->lo[0] + gi.x, (long long)G->lo[1] + gi.y,
                                    (long long)G->lo[2] + gi.z};
        float cen[3];
        for (int u = 0; u < 3; ++u) cen[u] = (float)(g_abs[u] * n + s1[u]) / (float)n * 0.01f;
        float tmin = 3.0e38f, tmax = -3.0e38f;
        for (uint32_t q = lane; q < m; q += 64) {
            const int4 h = d.sg[d.tord[base + q]];
            const long long w[3] = {h.x - gi.x, h.y - gi.y, h.z - gi.z};
            float pr = 0.0f;
            for (int u = 0; u < 3; ++u) pr = fmaf((float)(n * w[u] - s1[u]), dir[u], pr);
            pr = pr / (float)n * 0.01f;
            tmin = fminf(tmin, pr);
            tmax = fmaxf(tmax, pr);
        }
        tmin = wave_min(tmin);
        tmax = wave_max(tmax);
        if (lane == 0) {
            emt_track tr;
            tr.seed[0] = (uint32_t)gi.w;
            tr.seed[1] = (uint32_t)gj.w;
            tr.grain_offset = base;
            tr.n_grains = m;
            tr.axis = (uint32_t)a;
            tr.fit_fp64 = fp64;
            tr.degenerate = degen;
            tr.slope[0] = slope[0];
            tr.slope[1] = slope[1];
            for (int u = 0; u < 3; ++u) {
                tr.dir[u] = dir[u];
                tr.centroid[u] = cen[u];
            }
            tr.t_begin = tmin;
            tr.t_end = tmax;
            d.tracks[t] = tr;
            if (fp64) atomicAdd(&d.cnt->n_fp64, 1u);
        }
    }
}

// Results to the host: counters, per-view tables, tracks and grains, at the
// sizes the device knows, into mapped pinned host memory.
__global__ void __launch_bounds__(kBlock) k_copy_out(DevPtrs d, Caps c) {
    const uint32_t tid = grid_tid(), nt = grid_threads();
    const uint32_t nv = d.desc->n_views;
    const Counters cn = *d.cnt;
    if (tid == 0) *d.out.cnt = cn;
    for (uint32_t v = tid; v < nv; v += nt) {
        d.out.view_seeds[v] = d.view_seeds[v];
        d.out.view_cand[v] = d.view_cand[v];
        d.out.view_ntr[v] = d.view_ntr[v];
        d.out.view_err[v] = d.grids[v].err;
    }
    for (uint32_t v = tid; v <= nv; v += nt) d.out.view_tr_off[v] = d.view_tr_off[v];
    const uint32_t ntr = cn.n_acc <= c.cand_cap ? cn.n_acc : 0u;
    const uint32_t words = ntr * (uint32_t)(sizeof(emt_track) / 4);
    const uint32_t *src = reinterpret_cast<const uint32_t *>(d.tracks);
    uint32_t *dst = reinterpret_cast<uint32_t *>(d.out.tracks);
    for (uint32_t i = tid; i < words; i += nt) dst[i] = src[i];
    const uint32_t ng = cn.n_track_grains <= c.mem_cap ? cn.n_track_grains : 0u;
    for (uint32_t i = tid; i < ng; i += nt) d.out.grains[i] = d.out_grains[i];
    if (d.out.cands) {
        // candidates as input-index pairs with their counts, in list order
        const uint32_t nc = cn.n_cand <= c.cand_cap ? cn.n_cand : 0u;
        for (uint32_t i = tid; i < nc; i += nt) {
            const Cand cd = d.cand[i];
            d.out.cands[3 * i] = (uint32_t)d.sg[cd.p].w;
            d.out.cands[3 * i + 1] = (uint32_t)d.sg[cd.q].w;
            d.out.cands[3 * i + 2] = cd.n;
        }
    }
}

// ---------------------------------------------------- grain recognition
//
// 3D grain recognition on a filtered 8-bit stack (frames z, rows y, columns
// x, x fastest): a pixel above the threshold that no in-stack 3 x 3 x 3
// neighbour outranks (higher, or equal and earlier in frame, row, column
// order) defines a grain, placed at the pulse-height centre of mass of its
// block in 0.01 um units (pitch of each axis num/den units, rounded to the
// nearest unit, halves up, from exact integer sums).
//
// The stack is streamed once. A wave owns a tile of 1024 or 4096 consecutive
// pixels (the stack is one flat byte array, so a tile runs across row ends):
// each lane reads them as one or four 16-byte vectors and marks those above
// threshold; the wave lists its candidates in LDS in pixel order and tests
// them one per lane, which keeps the neighbourhood tests dense although few
// pixels pass the threshold. Waves never wait for one another: a workgroup
// that listed and tested together spent most of its life in barriers behind
// the neighbour loads of its few candidates. The grains' offsets in
// the tile go, in pixel order, to the tile's staging slots. Two pixels next
// to each other in a row cannot both be grains (one outranks the other), and
// tile and row boundaries fall on multiples of four pixels, so a tile holds
// at most half as many grains as pixels: the staging area is bounded. A second,
// small kernel (one workgroup per group of tiles) takes its place in the
// output from the counts of the tiles before it, finds each staged grain's
// tile by a search over the group's tile offsets, and writes the centre of
// mass: grains come out in frame, row, column order without a separate scan
// or a second stream. The grains found go straight to the host's word.
// 52 M pixels with 1400 grains stream in 16.3 us (27.7 with the workgroup's
// lists), 3.2 TB/s, and place in 5.8; with 20000 grains both take 26.9 us
// (52.9 before), and 1.3 M pixels with 10000 grains 13.1 (49.4).

// q = n / d for n < 2^32, d >= 1: double-precision reciprocal, then an
// exact integer correction of the +-1 it may be off by.
__device__ __forceinline__ uint32_t div_rcp(uint32_t n, uint32_t d, double inv) {
    uint32_t q = (uint32_t)((double)n * inv);
    if ((unsigned long long)q * d > n) --q;
    if ((unsigned long long)(q + 1) * d <= n) ++q;
    return q;
}

constexpr uint32_t kCandCap = 256;  // candidates listed per round
// 16-pixel vectors a lane reads. Four keep enough bytes in flight to stream a
// large stack (52 M pixels: 20.0 us with four, 24.4 with two, 42 with one);
// below about 4 M pixels such tiles leave most of the 1024 SIMDs without a
// wave, and a tile of many grains is a long serial chain (1.3 M pixels with
// 10000 grains: 25.2 us with four, 16.2 with two, 13.1 with one; 6.6 M pixels
// with 700: 11.6, 11.9, 13.4).
constexpr uint64_t kSmallStack = 4000000;
constexpr uint32_t kLargeLoads = 4, kSmallLoads = 1;
constexpr uint32_t tile_pix(uint32_t loads) { return 64 * 16 * loads; }
static_assert(tile_pix(kLargeLoads) <= 65536u, "tile offsets are staged as 16 bits");
// the tiles a placing workgroup takes, as a power of two
constexpr uint32_t kLargeGroup = 6, kSmallGroup = 3;
// a placing workgroup reads 2 bytes for every tile before it: up to 64 KB,
// from L2, up to this many tiles (134 M pixels)
constexpr size_t kDirectTiles = 32768;
static_assert(kSmallStack / tile_pix(kSmallLoads) < kDirectTiles, "sums are of large groups");

bool small_stack(const StackGeom &G) { return (uint64_t)G.nx * G.ny * G.nz < kSmallStack; }
uint32_t stack_tile(const StackGeom &G) { return tile_pix(small_stack(G) ? kSmallLoads : kLargeLoads); }

// The 3 x 3 x 3 block around pixel p (flat index): pulse heights w[i]
// (0 outside the stack) with i = 9 (dz+1) + 3 (dy+1) + (dx+1), so
// neighbours 0..12 come before p in frame, row, column order.
struct Block27 {
    uint32_t x, y, z;
    uint32_t w[27];
    uint32_t inside;

    __device__ __forceinline__ void load(const uint8_t *__restrict__ img, const StackGeom &G,
                                         uint32_t p) {
        const uint32_t row = div_rcp(p, G.nx, G.inv_nx);
        x = p - row * G.nx;
        z = div_rcp(row, G.ny, G.inv_ny);
        y = row - z * G.ny;
        const uint32_t plane = G.nx * G.ny;  // at most 2^31 pixels: offsets fit 32 bits
        // bit d + 1: the frame / row / column at offset d exists
        const uint32_t zok = (z > 0 ? 1u : 0u) | 2u | (z + 1 < G.nz ? 4u : 0u);
        const uint32_t yok = (y > 0 ? 1u : 0u) | 2u | (y + 1 < G.ny ? 4u : 0u);
        const uint32_t xok = (x > 0 ? 1u : 0u) | 2u | (x + 1 < G.nx ? 4u : 0u);
        inside = 0;
        // all 27 loads are issued unconditionally (a missing neighbour reads
        // pixel p itself, so every address is inside the stack) and masked
        // afterwards: no branch or wait separates them
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            const int dz = i / 9 - 1, dy = (i / 3) % 3 - 1, dx = i % 3 - 1;
            const bool ok = ((zok >> (dz + 1)) & (yok >> (dy + 1)) & (xok >> (dx + 1)) & 1u) != 0;
            inside |= ok ? 1u << i : 0u;
            // unsigned arithmetic wraps modulo 2^32 to the exact offset
            const uint32_t q =
                ok ? p + (uint32_t)dz * plane + (uint32_t)dy * G.nx + (uint32_t)dx : p;
            // the mask is opaque to the compiler, which would otherwise
            // turn "ok ? load : 0" back into a branch around the load
            uint32_t mask = ok ? 0xffu : 0u;
            asm("" : "+v"(mask));
            w[i] = (uint32_t)img[q] & mask;
        }
    }
    // No neighbour outranks the centre: higher, or equal and earlier. A
    // missing neighbour reads 0 and the centre is above the threshold, so it
    // never outranks. Bitwise, without short-circuits, so that every load is
    // needed and none is moved into a branch.
    __device__ __forceinline__ bool is_top() const {
        const uint32_t v = w[13];
        uint32_t beaten = 0;
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            if (i < 13) beaten |= (uint32_t)(w[i] >= v);
            if (i > 13) beaten |= (uint32_t)(w[i] > v);
        }
        return beaten == 0;
    }
    __device__ __forceinline__ void centre(const StackGeom &G, int32_t *out) const {
        int sw = 0, sx = 0, sy = 0, sz = 0;
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            const int wi = (int)w[i];
            sw += wi;
            sx += wi * ((int)x + i % 3 - 1);
            sy += wi * ((int)y + (i / 3) % 3 - 1);
            sz += wi * ((int)z + i / 9 - 1);
        }
        const int sums[3] = {sx, sy, sz};
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            // floor(num / den), num < 2^47 and 0 < den < 2^31: a double
            // quotient is within one of it, and integer products fix that
            const long long num = 2ll * sums[m] * G.pnum[m] + (long long)sw * G.pden[m];
            const long long den = 2ll * sw * G.pden[m];
            long long q = (long long)((double)num / (double)den);
            if (q * den > num) --q;
            if ((q + 1) * den <= num) ++q;
            out[m] = (int32_t)q;
        }
    }
};

// Bit 7 of every byte of w above thr. The lower seven bits are compared by
// the carry of an addition into bit 7, which stays in its byte.
__device__ __forceinline__ uint32_t above(uint32_t w, uint32_t add, bool upper) {
    const uint32_t t = (w & 0x7f7f7f7fu) + add;
    return (upper ? t & w : t | w) & 0x80808080u;
}

template <uint32_t kLoads>
__global__ void __launch_bounds__(kBlock) k_grain_find(const uint8_t *__restrict__ img,
                                                       StackGeom G, uint32_t n_tiles,
                                                       uint16_t *tile_cnt, uint16_t *stage) {
    constexpr uint32_t kTile = tile_pix(kLoads);
    __shared__ uint32_t s_list[kBlock / 64][kCandCap];
    const int lane = lane_id();
    uint32_t *list = s_list[threadIdx.x >> 6];
    const uint32_t tile = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (tile >= n_tiles) return;
    const uint32_t n_pix = G.nx * G.ny * G.nz;  // a multiple of 4, at most 2^31
    const uint32_t tile0 = tile * kTile, mine = tile0 + 16u * (uint32_t)lane;
    uint4 q[kLoads];
    if (n_pix - tile0 >= kTile) {
#pragma unroll
        for (uint32_t h = 0; h < kLoads; ++h)
            q[h] = *reinterpret_cast<const uint4 *>(img + mine + 1024u * h);
    } else {
#pragma unroll
        for (uint32_t h = 0; h < kLoads; ++h) {
            uint32_t w[4];
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                const uint32_t at = mine + 1024u * h + 4u * k;
                w[k] = at < n_pix ? *reinterpret_cast<const uint32_t *>(img + at) : 0u;
            }
            q[h] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    // bit p of cand[h]: pixel mine + 1024 h + p is above the threshold
    const bool upper = G.thr >= 128u;
    const uint32_t add = (127u - (G.thr & 127u)) * 0x01010101u;
    uint32_t cand[kLoads];
#pragma unroll
    for (uint32_t h = 0; h < kLoads; ++h) {
        // word k's four bytes at bits k, 8 + k, 16 + k, 24 + k
        uint32_t m = (above(q[h].x, add, upper) >> 7) | (above(q[h].y, add, upper) >> 6) |
                     (above(q[h].z, add, upper) >> 5) | (above(q[h].w, add, upper) >> 4);
        uint32_t c = 0;
        for (; m; m &= m - 1u) {
            const uint32_t i = (uint32_t)__ffs((int)m) - 1u;
            c |= 1u << (4u * (i & 7u) + (i >> 3));
        }
        cand[h] = c;
    }
    // the candidates' places in pixel order: vector by vector, lane by lane
    uint32_t before[kLoads], c_total = 0;
#pragma unroll
    for (uint32_t h = 0; h < kLoads; h += 2) {  // two counts a scan
        const uint32_t n = (uint32_t)__popc(cand[h]) |
                           (h + 1 < kLoads ? (uint32_t)__popc(cand[h + 1 < kLoads ? h + 1 : h]) << 16 : 0u);
        const uint32_t incl = wave_incl_scan_dpp(n), excl = incl - n;
        const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        before[h] = c_total + (excl & 0xffffu);
        c_total += tot & 0xffffu;
        if (h + 1 < kLoads) before[h + 1 < kLoads ? h + 1 : h] = c_total + (excl >> 16);
        c_total += tot >> 16;
    }
    uint16_t *st = stage + (size_t)tile * (kTile / 2u);
    uint32_t found = 0;
    for (uint32_t base = 0; base < c_total; base += kCandCap) {  // uniform
        // list this round's candidates
#pragma unroll
        for (uint32_t h = 0; h < kLoads; ++h) {
            uint32_t idx = before[h];
            for (uint32_t bits = cand[h]; bits; bits &= bits - 1u, ++idx)
                if (idx >= base && idx < base + kCandCap)
                    list[idx - base] = mine + 1024u * h + (uint32_t)__ffs((int)bits) - 1u;
        }
        wave_lds_sync();
        const uint32_t m = min(kCandCap, c_total - base);
        for (uint32_t c0 = 0; c0 < m; c0 += 64) {  // uniform
            const uint32_t c = c0 + (uint32_t)lane;
            const uint32_t pix = list[min(c, m - 1u)];
            bool top = false;
            if (c < m) {
                Block27 B;
                B.load(img, G, pix);
                top = B.is_top();
            }
            const unsigned long long tops = __ballot(top);
            const uint32_t slot = found + (uint32_t)__popcll(tops & lanes_below());
            if (top && slot < (kTile / 2u))  // always true: see the bound above
                st[slot] = (uint16_t)(pix - tile0);
            found += (uint32_t)__popcll(tops);
        }
        wave_lds_sync();  // the list is rewritten by the next round
    }
    if (lane == 0) tile_cnt[tile] = (uint16_t)min(found, (kTile / 2u));
}

// Grains of each group of tiles, for stacks of too many tiles for every
// placing workgroup to add up those before it.
__global__ void __launch_bounds__(kBlock) k_grain_sums(const uint16_t *__restrict__ tile_cnt,
                                                       uint32_t n_tiles, uint32_t *group_cnt,
                                                       uint32_t n_groups) {
    const uint32_t g = blockIdx.x * kBlock + threadIdx.x;
    if (g >= n_groups) return;
    uint32_t sum = 0;
    for (uint32_t t = g << kLargeGroup; t < min(n_tiles, (g + 1u) << kLargeGroup); ++t)
        sum += tile_cnt[t];
    group_cnt[g] = sum;
}

// One workgroup per group of 2^lg tiles (8 to 64): its grains' place in the
// output is the sum of the earlier tiles' counts (kSums: of the earlier
// groups' sums) plus the offset of the tile within the group.
template <bool kSums>
__global__ void __launch_bounds__(kBlock) k_grain_place(
    const uint8_t *__restrict__ img, StackGeom G, const uint16_t *__restrict__ tile_cnt,
    const uint32_t *__restrict__ group_cnt, uint32_t n_tiles,
    const uint16_t *__restrict__ stage, uint32_t tile_px, uint32_t lg, int32_t *out,
    uint32_t max_out, uint32_t *total) {
    __shared__ uint32_t s_off[65];
    const uint32_t grp = blockIdx.x, t0 = grp << lg, in_group = 1u << lg;
    uint32_t acc = 0;
    if constexpr (kSums) {
        for (uint32_t i = threadIdx.x; i < grp; i += kBlock) acc += group_cnt[i];
    } else {
        // eight counts a load (a group is a multiple of eight)
        const uint4 *cnt = reinterpret_cast<const uint4 *>(tile_cnt);
        for (uint32_t i = threadIdx.x; i < t0 / 8u; i += kBlock) {
            const uint4 v = cnt[i];
            acc += (v.x & 0xffffu) + (v.x >> 16) + (v.y & 0xffffu) + (v.y >> 16) +
                   (v.z & 0xffffu) + (v.z >> 16) + (v.w & 0xffffu) + (v.w >> 16);
        }
    }
    if (threadIdx.x < 64) {
        const uint32_t t = t0 + threadIdx.x;
        s_off[threadIdx.x + 1] = wave_incl_scan_dpp(threadIdx.x < in_group && t < n_tiles ? tile_cnt[t] : 0u);
        if (threadIdx.x == 0) s_off[0] = 0;
    }
    const uint32_t prefix = block_sum(acc);  // synchronises: s_off is written
    const uint32_t n_here = s_off[in_group];
    if (grp + 1 == gridDim.x && threadIdx.x == 0) *total = prefix + n_here;
    for (uint32_t g = threadIdx.x; g < n_here; g += kBlock) {
        // the tile holding grain g: s_off[lo] <= g < s_off[lo + 1]
        uint32_t lo = 0, hi = in_group;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (s_off[mid] <= g) lo = mid;
            else hi = mid;
        }
        const uint32_t t = t0 + lo;
        const uint32_t p = t * tile_px + stage[(size_t)t * (tile_px / 2u) + (g - s_off[lo])];
        const uint32_t q = prefix + g;
        if (q < max_out) {
            Block27 B;
            B.load(img, G, p);
            B.centre(G, out + 3ull * q);
        }
    }
}

}  // namespace

size_t grain_tile_count(const StackGeom &G) {
    const uint64_t px = (uint64_t)G.nx * G.ny * G.nz, tile = stack_tile(G);
    return (size_t)((px + tile - 1) / tile);
}

size_t grain_group_count(const StackGeom &G) {
    const size_t nt = grain_tile_count(G);
    return nt <= kDirectTiles ? 0 : (nt + (1u << kLargeGroup) - 1) >> kLargeGroup;
}

size_t grain_stage_slots(const StackGeom &G) {
    return grain_tile_count(G) * (stack_tile(G) / 2u);
}

void launch_find_grains(const uint8_t *img, const StackGeom &G, const GrainBufs &b,
                        hipStream_t s) {
    const uint32_t nt = (uint32_t)grain_tile_count(G), sums = (uint32_t)grain_group_count(G);
    const bool small = small_stack(G);
    const uint32_t lg = small ? kSmallGroup : kLargeGroup, px = stack_tile(G);
    const uint32_t ng = (nt + (1u << lg) - 1) >> lg, nb = (nt + kBlock / 64 - 1) / (kBlock / 64);
    if (small)
        k_grain_find<kSmallLoads><<<nb, kBlock, 0, s>>>(img, G, nt, b.tile_cnt, b.stage);
    else
        k_grain_find<kLargeLoads><<<nb, kBlock, 0, s>>>(img, G, nt, b.tile_cnt, b.stage);
    if (sums) {
        k_grain_sums<<<(ng + kBlock - 1) / kBlock, kBlock, 0, s>>>(b.tile_cnt, nt, b.group_cnt, ng);
        k_grain_place<true><<<ng, kBlock, 0, s>>>(img, G, b.tile_cnt, b.group_cnt, nt, b.stage, px,
                                                  lg, b.out, b.max_out, b.total);
    } else {
        k_grain_place<false><<<ng, kBlock, 0, s>>>(img, G, b.tile_cnt, nullptr, nt, b.stage, px, lg,
                                                   b.out, b.max_out, b.total);
    }
}

// ---------------------------------------------------------- filtering
//
// Image filtering: every camera pixel (x, y) has its own gain correction
// (unsigned, 1/256 units) and its own threshold, the same in every frame.
// Per pixel: t = min(255, raw * gain / 256 rounded half up); u = 255 - t
// (inversion: grains become bright); out = u - thr if u > thr, else 0.
// A thread owns kPix consecutive pixels of the frame, keeps their gains and
// thresholds in registers and walks kFilterFrames frames, loading all of
// them before it computes, so the maps are read once per frame group and
// raw and filtered pixels stream through once.
//
// With x = (raw * gain + 128) / 256 < 2^16 all that is max(0, (255 - thr) - x):
// from x = 255 on both are 0. So a pixel is one 24-bit multiply-add, and two
// pixels share a saturating 16-bit subtraction and a byte permutation to pack
// them: 14 instructions for four pixels. The output goes past the caches, which
// the next frames' pixels can use. Calls on 52 M pixels 38.2 -> 31.5 us (kernel
// 20.3 -> 18.2; a copy of as many bytes 13.2), on 210 M pixels 95.5 -> 86.5.

namespace {

constexpr uint32_t kFilterFrames = 8;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

typedef unsigned short us2 __attribute__((ext_vector_type(2)));

// Pixels 2 h and 2 h + 1 of word r in the halves; g: their gains, room: their
// 255 - thr.
__device__ __forceinline__ uint32_t filter_pair(uint32_t r, int h, uint32_t g, uint32_t room) {
    const uint32_t a = __umul24((r >> (16 * h)) & 0xffu, g & 0xffffu) + 128u;
    const uint32_t b = __umul24((r >> (16 * h + 8)) & 0xffu, g >> 16) + 128u;
    const uint32_t x = __builtin_amdgcn_perm(b, a, 0x06050201u);  // a >> 8 | b >> 8 << 16
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(us2, room),
                                                                      __builtin_bit_cast(us2, x)));
}

__device__ __forceinline__ uint32_t filter_word(uint32_t r, uint32_t g01, uint32_t g23,
                                                uint32_t room01, uint32_t room23) {
    return __builtin_amdgcn_perm(filter_pair(r, 1, g23, room23), filter_pair(r, 0, g01, room01),
                                 0x06040200u);
}

template <int kPix>  // pixels a thread owns in each frame: 4 or 16
__global__ void __launch_bounds__(kBlock) k_filter(const uint8_t *__restrict__ raw,
                                                   const uint16_t *__restrict__ gain,
                                                   const uint8_t *__restrict__ thr,
                                                   uint8_t *__restrict__ out, uint32_t chunks,
                                                   uint32_t plane, uint32_t nz) {
    static_assert(kPix == 4 || kPix == 16, "one or four words a frame");
    constexpr int kW = kPix / 4;  // four-pixel words
    const uint32_t c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= chunks) return;
    const uint32_t z0 = blockIdx.y * kFilterFrames;
    const uint32_t nf = min(kFilterFrames, nz - z0);  // uniform
    uint32_t g[2 * kW], t[kW];
    if constexpr (kPix == 16) {
        const uint4 ga = reinterpret_cast<const uint4 *>(gain)[2 * c];
        const uint4 gb = reinterpret_cast<const uint4 *>(gain)[2 * c + 1];
        const uint4 ta = reinterpret_cast<const uint4 *>(thr)[c];
        g[0] = ga.x; g[1] = ga.y; g[2] = ga.z; g[3] = ga.w;
        g[4] = gb.x; g[5] = gb.y; g[6] = gb.z; g[7] = gb.w;
        t[0] = ta.x; t[1] = ta.y; t[2] = ta.z; t[3] = ta.w;
    } else {
        const uint2 ga = reinterpret_cast<const uint2 *>(gain)[c];
        g[0] = ga.x;
        g[1] = ga.y;
        t[0] = reinterpret_cast<const uint32_t *>(thr)[c];
    }
    // 255 - thr in the same halves as the gains
    uint32_t room[2 * kW];
#pragma unroll
    for (int k = 0; k < kW; ++k) {
        room[2 * k] = 0x00ff00ffu - __builtin_amdgcn_perm(0u, t[k], 0x0c010c00u);
        room[2 * k + 1] = 0x00ff00ffu - __builtin_amdgcn_perm(0u, t[k], 0x0c030c02u);
    }
    uint32_t r[kFilterFrames][kW];
#pragma unroll
    for (int f = 0; f < (int)kFilterFrames; ++f) {
        if ((uint32_t)f >= nf) break;
        const size_t off = (size_t)(z0 + f) * plane + (size_t)c * kPix;
        if constexpr (kPix == 16) {
            const uint4 v = *reinterpret_cast<const uint4 *>(raw + off);
            r[f][0] = v.x; r[f][1] = v.y; r[f][2] = v.z; r[f][3] = v.w;
        } else {
            r[f][0] = *reinterpret_cast<const uint32_t *>(raw + off);
        }
    }
#pragma unroll
    for (int f = 0; f < (int)kFilterFrames; ++f) {
        if ((uint32_t)f >= nf) break;
        uint32_t o[kW];
#pragma unroll
        for (int k = 0; k < kW; ++k) 
            o[k] = filter_word(r[f][k], g[2 * k], g[2 * k + 1], room[2 * k], room[2 * k + 1]);
        const size_t off = (size_t)(z0 + f) * plane + (size_t)c * kPix;
        if constexpr (kPix == 16)
            __builtin_nontemporal_store(u32x4{o[0], o[1], o[2], o[3]},
                                        reinterpret_cast<u32x4 *>(out + off));
        else
            *reinterpret_cast<uint32_t *>(out + off) = o[0];
    }
}

}  // namespace

bool launch_filter(const uint8_t *raw, const uint16_t *gain, const uint8_t *thr, uint8_t *out,
                   uint32_t nx, uint32_t ny, uint32_t nz, bool vec16, hipStream_t s) {
    const uint32_t plane = nx * ny;
    if (plane % 4u) return false;
    if (vec16 && plane % 16u) vec16 = false;
    const uint32_t pix = vec16 ? 16u : 4u, chunks = plane / pix;
    const dim3 grid((chunks + kBlock - 1) / kBlock, (nz + kFilterFrames - 1) / kFilterFrames);
    if (vec16)
        k_filter<16><<<grid, kBlock, 0, s>>>(raw, gain, thr, out, chunks, plane, nz);
    else
        k_filter<4><<<grid, kBlock, 0, s>>>(raw, gain, thr, out, chunks, plane, nz);
    return true;
}

namespace {

uint32_t blocks_for(unsigned long long n, uint32_t max_blocks) {
    unsigned long long b = (n + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    return (uint32_t)(b < max_blocks ? b : max_blocks);
}

#ifndef EMT_PERSISTENT_BLOCKS
#define EMT_PERSISTENT_BLOCKS 2048
#endif
constexpr uint32_t kPersistentBlocks = EMT_PERSISTENT_BLOCKS;  // 8 blocks of 4 waves per CU
// the counting kernel's grid: one resident generation (two workgroups of
// twelve waves per CU, bound by registers and LDS), so none waits for a slot
constexpr uint32_t kCountBlocks = EMT_COUNT_BLOCKS;
static_assert(kCountBlocks % kXcds == 0, "whole workgroups per XCD");
constexpr uint32_t kFewBlocks = 1024;  // one resident generation of k_count_few

}  // namespace

// tile sums of a scan of n_cap items, or of the mask words of n_seeds seeds
// (launch_candidates)
size_t scan_scratch_words(uint32_t n_cap, unsigned long long n_seeds) {
    const size_t words = n_seeds / 32 + 1, tiles = words / kBlock + 1;
    return std::max((size_t)n_cap / kScanTile + 1,
                    tiles <= kScanDirect ? tiles : words / (4 * kBlock) + 1) + 1;
}

void launch_prepare(const DevPtrs &d, const Caps &c, const Params &, hipStream_t s) {
    k_zero<<<blocks_for(c.n_cells, 256), kBlock, 0, s>>>(d);
}

void launch_bin(const DevPtrs &d, const Caps &c, const Params &P, hipStream_t s) {
    const uint32_t bx = blocks_for(c.max_view_n, 64);
    dim3 grid(bx, c.n_views);
    k_bbox<<<grid, kBlock, 0, s>>>(d.xyz, d.in_src, d.grids, d.view_of, d.desc);
    k_grid<<<(c.n_views + 63) / 64, 64, 0, s>>>(d.grids, d.lines, d.lpool, d.lcoarse, d.nc,
                                                   d.desc, P);
    k_hist<<<grid, kBlock, 0, s>>>(d.xyz, d.grids, d.cell_of, d.rank, d.cell_count, d.desc);
    scan_excl<kEndTotal>(d.cell_count, &d.desc->n_cells_m1, c.n_cells, d.scan_part,
                         {d.cell_start}, s);
    k_scatter<<<grid, kBlock, 0, s>>>(d.xyz, d.grids, d.cell_of, d.rank, d.cell_start, d.sg,
                                      d.desc);
}

void launch_seeds(const DevPtrs &d, const Caps &c, const Params &P, hipStream_t s) {
    // whole runs for every XCD
    const uint32_t nb = (blocks_for(64ull * c.n_total, 4 * kPersistentBlocks) + 8u * kSeedRun - 1u) /
                        (8u * kSeedRun) * (8u * kSeedRun);
    if (d.nc > 1) k_line_order<<<dim3(3 + d.nc, c.n_views), kOrderBlock, 0, s>>>(d);
    k_seeds<false><<<nb, kBlock, 0, s>>>(d, c, P);
    // offsets in uint32: exact whenever the total fits, which the scan's end checks
    scan_excl<kEndSeeds>(d.seed_cnt, &d.desc->n_anchor, (uint32_t)d.nc * c.n_total, d.scan_part,
                         {d.seed_off, nullptr, d.cnt, d.part64, c.seed_cap}, s);
    k_seeds<true><<<nb, kBlock, 0, s>>>(d, c, P);
}

void launch_count(const DevPtrs &d, const Caps &c, const Params &P, hipStream_t s) {
    if (d.nc == 1) {
        if (P.cyl_ext >= 0)
            k_count_few<true, false><<<kFewBlocks, kBlock, 0, s>>>(d, c, P);
        else
            k_count_few<false, false><<<kFewBlocks, kBlock, 0, s>>>(d, c, P);
        return;
    }
    // workgroups sharing a class's planes: about 4096 in all, at least four
    const uint32_t parts = std::max(4u, std::min(128u, 4096u / ((uint32_t)d.nc * c.n_views)));
    const dim3 grid(parts, d.nc, c.n_views);
    k_line_fill<0><<<grid, kLineBlock, 0, s>>>(d, P);
    k_line_fill<1><<<grid, kLineBlock, 0, s>>>(d, P);
    if (P.cyl_ext >= 0)
        k_count<true, false><<<kCountBlocks, kCountBlock, 0, s>>>(d, c, P);
    else
        k_count<false, false><<<kCountBlocks, kCountBlock, 0, s>>>(d, c, P);
}

void launch_candidates(const DevPtrs &d, const Caps &c, const Params &P, hipStream_t s) {
    const uint32_t words = (uint32_t)(c.seed_cap / 32 + 1);
    const uint32_t nb = words / kBlock + 1;
    if (nb <= kScanDirect) {
        k_scan_part<true, 1><<<nb, kBlock, 0, s>>>(d.pass, &d.cnt->pass_words, words, d.scan_part);
        k_cand_list<1, true><<<nb, kBlock, 0, s>>>(d, c, d.scan_part);
    } else {
        constexpr int kWords = 4;
        constexpr uint32_t kTile = kBlock * kWords;
        const uint32_t nt = words / kTile + 1;
        k_scan_part<true, kWords><<<nt, kBlock, 0, s>>>(d.pass, &d.cnt->pass_words, words, d.scan_part);
        k_scan_parts<<<1, kScanBlock, 0, s>>>(d.scan_part, kTile, &d.cnt->pass_words, words);
        k_cand_list<kWords, false><<<nt, kBlock, 0, s>>>(d, c, d.scan_part);
    }
}

void launch_members(const DevPtrs &d, const Caps &c, const Params &P, hipStream_t s) {
    scan_excl<kEndMembers>(d.cand_n, &d.cnt->n_cand, c.cand_cap, d.scan_part,
                           {d.mem_off, nullptr, d.cnt, d.part64}, s);
    // the counting kernel's walk and test, listing the grains of each candidate
    if (d.nc == 1) {
        if (P.cyl_ext >= 0)
            k_count_few<true, true><<<kFewBlocks, kBlock, 0, s>>>(d, c, P);
        else
            k_count_few<false, true><<<kFewBlocks, kBlock, 0, s>>>(d, c, P);
        return;
    }
    if (P.cyl_ext >= 0)
        k_count<true, true><<<kCountBlocks, kCountBlock, 0, s>>>(d, c, P);
    else
        k_count<false, true><<<kCountBlocks, kCountBlock, 0, s>>>(d, c, P);
}

void launch_merge_init(const DevPtrs &d, const Caps &c, const Params &, hipStream_t s) {
    unsigned long long n = c.cand_cap;
    if (c.n_total > n) n = c.n_total;
    if (c.mem_cap > n) n = c.mem_cap;
    k_merge_init<<<blocks_for(n, kPersistentBlocks), kBlock, 0, s>>>(d, c);
}

void launch_merge(const DevPtrs &d, const Caps &c, const Params &P, hipStream_t s) {
    // Later rounds see a fraction of the candidates: their grids shrink by
    // half per round down to a floor (the loops stride, so any grid is correct).
    // The number of grid-wide rounds comes with the capacities (the host
    // sizes it from the rounds earlier calls needed); the tail finishes
    // whatever they leave.
    const int wide = c.wide_rounds < 1 ? 1 : (c.wide_rounds > kWideRounds ? kWideRounds : c.wide_rounds);
    uint32_t nb = blocks_for((unsigned long long)kMergeGroup * c.cand_cap, 2 * kPersistentBlocks);
    for (int round = 0; round < wide; ++round) {
        k_round<0><<<nb, kBlock, 0, s>>>(d, P, round);
        k_round<1><<<nb, kBlock, 0, s>>>(d, P, round);
        if (round >= 1 && nb > 1024) nb = nb / 2 > 1024 ? nb / 2 : 1024;
    }
    if (c.n_views > 1) k_tail_split<<<64, kBlock, 0, s>>>(d, wide - 1);
    k_merge_tail<<<c.n_views, kTailBlock, 0, s>>>(d, P, wide - 1);
}

int max_merge_rounds() { return kMaxRounds; }
int max_wide_rounds() { return kWideCap; }

void launch_copy_out(const DevPtrs &d, const Caps &c, const Params &, hipStream_t s) {
    k_copy_out<<<64, kBlock, 0, s>>>(d, c);
}

void launch_fit(const DevPtrs &d, const Caps &c, const Params &P, hipStream_t s) {
    const uint32_t nb = blocks_for(c.cand_cap, kPersistentBlocks);
    k_collect<<<nb, kBlock, 0, s>>>(d, c);
    if (c.n_views > 1) k_view_offsets<<<1, kBlock, 0, s>>>(d);  // one view's is 0
    // keys of the grouped tracks reuse the owner array (merge is over)
    unsigned long long *gkey = d.owner;
    k_group<<<nb, kBlock, 0, s>>>(d, gkey);
    k_rank<<<nb, kBlock, 0, s>>>(d, gkey);
    scan_excl<kEndTotal>(d.tg_n, &d.cnt->n_acc, c.cand_cap, d.scan_part,
                         {d.tg_off, &d.cnt->n_track_grains}, s);
    k_fit<<<nb, kBlock, 0, s>>>(d, P);
}

}  // namespace emt
