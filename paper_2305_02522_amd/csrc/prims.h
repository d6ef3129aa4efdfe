// Device-wide primitives of the adjacency builders: exclusive scan and LSD radix
// sort of 64-bit keys (hand-written; one workgroup per sort tile, stable ranks
// from wave votes).  Included by the builder translation units only.
#pragma once

#include "common.h"

namespace {

// ---------------------------------------------------------------- helpers
struct DevBuf {
    void *p = nullptr;
    ~DevBuf() { reset(); }
    void reset()
    {
        if (p)
            (void)hipFree(p);
        p = nullptr;
    }
    hipError_t alloc(size_t bytes) { return hipMalloc(&p, bytes ? bytes : 8); }
    template <typename T> T *as() { return (T *)p; }
    void *release()
    {
        void *q = p;
        p = nullptr;
        return q;
    }
};

static inline unsigned blocks_for(int64_t n, int per_block)
{
    return (unsigned)((n + per_block - 1) / per_block);
}

// ---------------------------------------------------------------- scan
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

// Exclusive scan of `v` across the THREADS threads of a block; returns the
// exclusive prefix of this thread and the block total through `total`.
template <int THREADS = kScanThreads>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *total)
{
    __shared__ uint32_t wave_sum[THREADS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(inc, d, 64);
        if (lane >= d)
            inc += o;
    }
    __syncthreads(); // protects wave_sum against the previous call
    if (lane == 63)
        wave_sum[wave] = inc;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        const uint32_t s = wave_sum[w];
        if (w < wave)
            before += s;
        all += s;
    }
    *total = all;
    return before + inc - v;
}

__global__ __launch_bounds__(kScanThreads) void scan_reduce_kernel(const uint32_t *__restrict__ in,
                                                                   uint32_t n,
                                                                   uint32_t *__restrict__ sums)
{
    const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const uint32_t v = in[min(base + k, n - 1)];
        s += base + k < n ? v : 0;
    }
    uint32_t total;
    (void)block_exclusive_scan(s, &total);
    if (threadIdx.x == 0)
        sums[blockIdx.x] = total;
}

// In-place exclusive scan of one tile, plus the tile's offset (0 if null).
__global__ __launch_bounds__(kScanThreads) void scan_apply_kernel(uint32_t *__restrict__ data,
                                                                  uint32_t n,
                                                                  const uint32_t *__restrict__ offs)
{
    const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        v[k] = data[min(base + k, n - 1)]; // unconditional: eight loads in flight
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < n) ? v[k] : 0;
        s += v[k];
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan(s, &total) + (offs ? offs[blockIdx.x] : 0);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n)
            data[base + k] = run;
        run += v[k];
    }
}

// The whole scan as one workgroup, 8,192 words a turn: a sort pass over a small graph is a chain
// of launches of a few microseconds each, and the three launches of the general scan were
// three of its five.
constexpr int kScanSmallThreads = 1024;
constexpr uint32_t kScanSmallMax = 32768; // four turns

// One CU reads and writes it all: 16-byte accesses, or issuing them is what takes the time
// (13,000 words: 13 us with 4-byte ones, 4 us so).
__global__ __launch_bounds__(kScanSmallThreads) void scan_small_kernel(uint32_t *__restrict__ data,
                                                                       uint32_t n)
{
    uint32_t before = 0;
    for (uint32_t b = 0; b < n; b += kScanSmallThreads * kScanItems) {
        const uint32_t base = b + threadIdx.x * kScanItems;
        const bool whole = base + kScanItems <= n;
        uint32_t v[kScanItems];
        if (whole) {
            const uint4 p = *(const uint4 *)(data + base), q = *(const uint4 *)(data + base + 4);
            v[0] = p.x, v[1] = p.y, v[2] = p.z, v[3] = p.w;
            v[4] = q.x, v[5] = q.y, v[6] = q.z, v[7] = q.w;
        } else {
#pragma unroll
            for (int k = 0; k < kScanItems; ++k)
                v[k] = base + k < n ? data[base + k] : 0;
        }
        uint32_t s = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k)
            s += v[k];
        uint32_t total;
        uint32_t run = block_exclusive_scan<kScanSmallThreads>(s, &total) + before;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const uint32_t x = v[k];
            v[k] = run;
            run += x;
        }
        if (whole) {
            *(uint4 *)(data + base) = make_uint4(v[0], v[1], v[2], v[3]);
            *(uint4 *)(data + base + 4) = make_uint4(v[4], v[5], v[6], v[7]);
        } else {
#pragma unroll
            for (int k = 0; k < kScanItems; ++k)
                if (base + k < n)
                    data[base + k] = v[k];
        }
        before += total;
    }
}

// Exclusive scan of data[0..n) in place.  `ws` must hold scan_ws_words(n) words.
static size_t scan_ws_words(uint64_t n)
{
    size_t w = 0;
    while (n > (uint64_t)kScanTile) {
        n = (n + kScanTile - 1) / kScanTile;
        w += n;
    }
    return w + 1;
}

static void scan_inplace(uint32_t *data, uint32_t n, uint32_t *ws, hipStream_t s)
{
    const uint32_t tiles = (n + kScanTile - 1) / kScanTile;
    if (tiles <= 1) {
        scan_apply_kernel<<<1, kScanThreads, 0, s>>>(data, n, nullptr);
        return;
    }
    if (n <= kScanSmallMax && bg_aligned(data, 16)) {
        scan_small_kernel<<<1, kScanSmallThreads, 0, s>>>(data, n);
        return;
    }
    scan_reduce_kernel<<<tiles, kScanThreads, 0, s>>>(data, n, ws);
    scan_inplace(ws, tiles, ws + tiles, s);
    scan_apply_kernel<<<tiles, kScanThreads, 0, s>>>(data, n, ws);
}

// ---------------------------------------------------------------- radix sort
// One pass: digit histogram per tile, scan, scatter.  Bound by memory (a pass reads the keys
// twice and writes them once), so what counts is that the writes are whole lines: a workgroup of
// eight wavefronts first puts its tile in digit order in LDS, then writes runs of ~32 keys
// (256 bytes) per digit.  Writing each key straight to its place from one wavefront's tile of
// 2,048 keys, the form before this one, left runs of 64 bytes spread over 32 instructions.
// 115 M keys, one pass: 246 us for the histogram and 478 us for the scatter, 3.8 TB/s both; the
// build they are most of went from 37.5 to 21.5 ms with them (and with fewer passes).
// Sorts of fewer than kSortSmall keys take tiles of 2,048 keys: with 8,192 there are too few
// workgroups for 256 CUs.
constexpr int kSortThreads = 512;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortItems = 16;     // keys per thread
constexpr int kSortItemsSmall = 4; // the same, fewer than kSortSmall keys
constexpr uint32_t kSortTile = kSortThreads * kSortItems;
constexpr uint32_t kSortTileSmall = kSortThreads * kSortItemsSmall;
constexpr uint32_t kSortSmall = 1u << 20;

// Orders a wavefront's own LDS accesses (the hardware keeps them in program order).
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int ITEMS>
__global__ __launch_bounds__(kSortThreads) void radix_hist_kernel(const uint64_t *__restrict__ keys,
                                                                  uint32_t n, int shift,
                                                                  uint32_t *__restrict__ hist,
                                                                  uint32_t tiles)
{
    __shared__ uint32_t h[256];
    if (threadIdx.x < 256)
        h[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t base = blockIdx.x * (uint32_t)(kSortThreads * ITEMS) + threadIdx.x;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const uint32_t idx = base + it * kSortThreads;
        if (idx < n)
            atomicAdd(&h[(uint32_t)(keys[idx] >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 256)
        hist[(uint64_t)threadIdx.x * tiles + blockIdx.x] = h[threadIdx.x];
}

template <int ITEMS>
__global__ __launch_bounds__(kSortThreads) void radix_scatter_kernel(
    const uint64_t *__restrict__ in, uint64_t *__restrict__ out, uint32_t n, int shift,
    const uint32_t *__restrict__ offsets, uint32_t tiles)
{
    constexpr uint32_t kTile = kSortThreads * ITEMS;
    __shared__ uint64_t sorted[kTile];
    __shared__ uint32_t count[kSortWaves][256]; // keys seen of each digit, then first place in tile
    __shared__ uint32_t place[256];             // output index of a digit's keys, less place in tile
    __shared__ uint32_t wave_sum[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t tile0 = blockIdx.x * kTile;
    const uint32_t base = tile0 + wave * (64 * ITEMS) + lane;
    uint64_t key[ITEMS];
    uint32_t rank[ITEMS];
    // places past the end hold the largest digit and come last, so they end up behind every key
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        key[it] = base + it * 64 < n ? in[base + it * 64] : ~0ull;
    uint32_t *mine = count[wave];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        mine[lane + 64 * q] = 0;
    wave_lds_order();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const uint32_t d = (uint32_t)(key[it] >> shift) & 255u;
        // lanes holding the same digit: intersect the 8 vote masks
        uint64_t peers = ~0ull;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t r = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
        const uint32_t seen = mine[d];
        wave_lds_order(); // every lane has read before a leader writes
        if (r == 0)
            mine[d] = seen + (uint32_t)__popcll(peers);
        wave_lds_order();
        rank[it] = seen + r;
    }
    __syncthreads();
    uint32_t total = 0, inc = 0;
    if (threadIdx.x < 256) {
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
            const uint32_t c = count[w][threadIdx.x];
            count[w][threadIdx.x] = total;
            total += c;
        }
        inc = total;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(inc, d, 64);
            if (lane >= d)
                inc += o;
        }
        if (lane == 63)
            wave_sum[wave] = inc;
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        uint32_t first = inc - total;
        for (int w = 0; w < wave; ++w)
            first += wave_sum[w];
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w)
            count[w][threadIdx.x] += first;
        place[threadIdx.x] = offsets[(uint64_t)threadIdx.x * tiles + blockIdx.x] - first;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        sorted[count[wave][(uint32_t)(key[it] >> shift) & 255u] + rank[it]] = key[it];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const uint32_t i = it * kSortThreads + threadIdx.x;
        if (tile0 + i < n) {
            const uint64_t k = sorted[i];
            out[place[(uint32_t)(k >> shift) & 255u] + i] = k;
        }
    }
}

// Histogram words of any sort of at most n keys.
static size_t sort_hist_words(uint32_t n)
{
    const uint32_t small = ((n < kSortSmall ? n : kSortSmall) + kSortTileSmall - 1) / kSortTileSmall;
    const uint32_t large = (n + kSortTile - 1) / kSortTile;
    return (size_t)256 * (small > large ? small : large);
}

// Sorts keys[0..n) on bits [lo, hi), keys equal there staying in order (LSD, 8 bits a pass; the
// last pass may look at bits above hi).  Returns the buffer that holds the result (a or b).
static uint64_t *radix_sort(uint64_t *a, uint64_t *b, uint32_t n, int lo, int hi, uint32_t *hist,
                            uint32_t *scan_ws, hipStream_t s)
{
    const bool small = n < kSortSmall;
    const uint32_t tile = small ? kSortTileSmall : kSortTile;
    const uint32_t tiles = (n + tile - 1) / tile;
    for (int shift = lo; shift < hi; shift += 8) {
        if (small)
            radix_hist_kernel<kSortItemsSmall><<<tiles, kSortThreads, 0, s>>>(a, n, shift, hist,
                                                                             tiles);
        else
            radix_hist_kernel<kSortItems><<<tiles, kSortThreads, 0, s>>>(a, n, shift, hist, tiles);
        scan_inplace(hist, 256u * tiles, scan_ws, s);
        if (small)
            radix_scatter_kernel<kSortItemsSmall><<<tiles, kSortThreads, 0, s>>>(a, b, n, shift,
                                                                                hist, tiles);
        else
            radix_scatter_kernel<kSortItems><<<tiles, kSortThreads, 0, s>>>(a, b, n, shift, hist,
                                                                           tiles);
        uint64_t *t = a;
        a = b;
        b = t;
    }
    return a;
}

} // namespace
