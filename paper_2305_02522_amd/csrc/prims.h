// Device-wide primitives of the adjacency builders: exclusive scans and LSD radix
// sorts of 64-bit keys, over all of memory or inside one workgroup (hand-written; stable
// ranks from wave votes).  Included by the builder translation units only.
#pragma once

#include "common.h"

namespace {

// ---------------------------------------------------------------- helpers
// A block of the context's pool.  Given back when it goes out of scope: the stream must be idle
// by then, or the next user of the block must be work on the same stream.
struct DevBuf {
    bg_pool *pool;
    bg_block b{};
    explicit DevBuf(bitgnn_ctx *ctx) : pool(ctx->pool) {}
    DevBuf(const DevBuf &) = delete;
    DevBuf &operator=(const DevBuf &) = delete;
    ~DevBuf() { reset(); }
    void reset()
    {
        bg_pool_give(pool, b);
        b = bg_block{};
    }
    hipError_t alloc(size_t bytes) { return bg_pool_take(pool, bytes, &b); }
    template <typename T> T *as() { return (T *)b.p; }
    // the handle owns the block from now on
    template <typename T> T *give(bitgnn_adj *adj)
    {
        T *q = (T *)b.p;
        adj->owned[adj->n_owned++] = b;
        b = bg_block{};
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

// Tile sums of array blockIdx.y (the arrays are `stride` words apart, their sums gridDim.x).
__global__ __launch_bounds__(kScanThreads) void scan_reduce_kernel(const uint32_t *__restrict__ in,
                                                                   uint32_t n, uint32_t stride,
                                                                   uint32_t *__restrict__ sums)
{
    in += (uint64_t)blockIdx.y * stride;
    const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const uint32_t v = in[min(base + k, n - 1)]; // unconditional: eight loads in flight
        s += base + k < n ? v : 0;
    }
    uint32_t total;
    (void)block_exclusive_scan(s, &total);
    if (threadIdx.x == 0)
        sums[blockIdx.y * gridDim.x + blockIdx.x] = total;
}

// In-place exclusive scan of one tile of array blockIdx.y, plus the tile's offset (0 if null).
__global__ __launch_bounds__(kScanThreads) void scan_apply_kernel(uint32_t *__restrict__ data,
                                                                  uint32_t n, uint32_t stride,
                                                                  const uint32_t *__restrict__ offs)
{
    data += (uint64_t)blockIdx.y * stride;
    const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        v[k] = data[min(base + k, n - 1)];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = base + k < n ? v[k] : 0;
        s += v[k];
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan(s, &total) +
                   (offs ? offs[blockIdx.y * gridDim.x + blockIdx.x] : 0);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n)
            data[base + k] = run;
        run += v[k];
    }
}

// Words of workspace for the exclusive scans of `arrays` arrays of n words.
static size_t scan_ws_words(uint64_t n, int arrays = 1)
{
    size_t w = 0;
    while (n > (uint64_t)kScanTile) {
        n = (n + kScanTile - 1) / kScanTile;
        w += n;
    }
    return (w + 1) * arrays;
}

// Exclusive scans, in place, of `arrays` arrays of n >= 1 words that are `stride` words apart.
static void scan_inplace(uint32_t *data, uint32_t n, uint32_t *ws, hipStream_t s, int arrays = 1,
                         uint32_t stride = 0)
{
    const uint32_t tiles = (n + kScanTile - 1) / kScanTile;
    const dim3 grid(tiles, arrays);
    if (tiles <= 1) {
        scan_apply_kernel<<<grid, kScanThreads, 0, s>>>(data, n, stride, nullptr);
        return;
    }
    scan_reduce_kernel<<<grid, kScanThreads, 0, s>>>(data, n, stride, ws);
    scan_inplace(ws, tiles, ws + (size_t)tiles * arrays, s, arrays, tiles);
    scan_apply_kernel<<<grid, kScanThreads, 0, s>>>(data, n, stride, ws);
}

// ---------------------------------------------------------------- ranks by digit
// Orders a wavefront's own LDS accesses (the hardware keeps them in program order).
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Stable ranks of a wavefront's keys by one digit of `width` <= BITS bits.  Key `it` of lane l is
// number 64 * it + l; rank[it] becomes the number of its predecessors with the same digit, and
// count[2^BITS], zeroed here, the keys of each digit.  Lanes with the same digit find each other
// through a wave vote per bit.
template <typename K, int ITEMS, int BITS = 8>
__device__ __forceinline__ void wave_digit_ranks(const K (&key)[ITEMS], uint32_t (&rank)[ITEMS],
                                                 int items, int shift, uint32_t *count,
                                                 int width = BITS)
{
    const int lane = threadIdx.x & 63;
    const uint32_t mask = (1u << width) - 1;
#pragma unroll
    for (int q = 0; q < (1 << BITS) / 64; ++q)
        count[lane + 64 * q] = 0;
    wave_lds_order();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if (it < items) {
            const uint32_t d = (uint32_t)(key[it] >> shift) & mask;
            uint64_t peers = ~0ull;
#pragma unroll
            for (int b = 0; b < BITS; ++b) {
                if (b < width) {
                    const bool bit = (d >> b) & 1u;
                    const uint64_t m = __ballot(bit);
                    peers &= bit ? m : ~m;
                }
            }
            const uint32_t r = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
            const uint32_t seen = count[d];
            wave_lds_order(); // every lane has read before a leader writes
            if (r == 0)
                count[d] = seen + (uint32_t)__popcll(peers);
            wave_lds_order();
            rank[it] = seen + r;
        }
    }
}

// Turns the wavefronts' digit counts, count[w][digit], into the first place of each wavefront's
// keys of a digit when the block's keys are in digit order.  Returns, for threads below 2^BITS,
// the first place of digit threadIdx.x in the block.  Barriers before and after.
template <int WAVES, int BITS = 8>
__device__ __forceinline__ uint32_t block_digit_places(uint32_t (*count)[1 << BITS],
                                                       uint32_t *wave_sum)
{
    constexpr int kDigits = 1 << BITS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    uint32_t c[WAVES], total = 0, inc = 0;
    if (threadIdx.x < kDigits) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            c[w] = count[w][threadIdx.x];
            total += c[w];
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
    uint32_t first = inc - total;
    if (threadIdx.x < kDigits) {
        for (int w = 0; w < wave; ++w)
            first += wave_sum[w];
        uint32_t at = first;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            count[w][threadIdx.x] = at;
            at += c[w];
        }
    }
    __syncthreads();
    return first;
}

// Sorts, in LDS, up to 1024 * ITEMS keys of a block of 1,024 threads on bits [lo, hi), equal ones
// staying in order.  Key 64 * items * wave + 64 * it + lane comes in key[it] (places past the end
// hold ~0 and end up last); the sorted keys are in `stage` afterwards (1024 * items of them).
constexpr int kLdsSortThreads = 1024;
template <typename K, int ITEMS>
__device__ __forceinline__ void lds_sort(K (&key)[ITEMS], int items, int lo, int hi, K *stage,
                                         uint32_t (*count)[256], uint32_t *wave_sum)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int base = wave * 64 * items + lane;
    for (int shift = lo; shift < hi || shift == lo; shift += 8) {
        uint32_t rank[ITEMS];
        if (shift > lo) {
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
                if (it < items)
                    key[it] = stage[base + it * 64];
        }
        wave_digit_ranks<K, ITEMS>(key, rank, items, shift, count[wave]);
        (void)block_digit_places<kLdsSortThreads / 64>(count, wave_sum);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            if (it < items)
                stage[count[wave][(uint32_t)(key[it] >> shift) & 255u] + rank[it]] = key[it];
        __syncthreads();
    }
}

// ---------------------------------------------------------------- radix sort
// One pass: digit histogram per tile, scan, scatter.  Bound by memory (a pass reads the keys
// twice and writes them once), so what counts is that the writes are whole lines: a workgroup of
// eight wavefronts first puts its tile in digit order in LDS, then writes runs of ~32 keys
// (256 bytes) per digit.  Writing each key straight to its place from one wavefront's tile of
// 2,048 keys left runs of 64 bytes spread over 32 instructions: 115 M keys, one pass, 2.1 ms that
// way, 245 us for the histogram and 487 us for the scatter so.
// Sorts of fewer than kSortSmall keys take tiles of 2,048 keys: with 8,192 there are too few
// workgroups for 256 CUs.
constexpr int kSortThreads = 512;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortItems = 16;     // keys per thread
constexpr int kSortItemsSmall = 4; // the same, fewer than kSortSmall keys
constexpr uint32_t kSortTile = kSortThreads * kSortItems;
constexpr uint32_t kSortTileSmall = kSortThreads * kSortItemsSmall;
constexpr uint32_t kSortSmall = 1u << 20;

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
    __shared__ uint32_t count[kSortWaves][256];
    __shared__ uint32_t place[256]; // output index of a digit's keys, less place in tile
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
    wave_digit_ranks<uint64_t, ITEMS>(key, rank, ITEMS, shift, count[wave]);
    const uint32_t first = block_digit_places<kSortWaves>(count, wave_sum);
    if (threadIdx.x < 256)
        place[threadIdx.x] = offsets[(uint64_t)threadIdx.x * tiles + blockIdx.x] - first;
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

// Bits that hold the values 0 .. v.
static int bits_of(uint32_t v) { return v ? 32 - __builtin_clz(v) : 0; }

// A sort small enough for one workgroup: one launch instead of three a pass.
constexpr int kOneWgItems = 16;
constexpr uint32_t kOneWgKeys = kLdsSortThreads * kOneWgItems;
constexpr size_t kOneWgLds = kOneWgKeys * 8 + 16 * 256 * 4 + 64;

__global__ __launch_bounds__(kLdsSortThreads) void one_wg_sort_kernel(uint64_t *__restrict__ keys,
                                                                      uint32_t n, int lo, int hi)
{
    extern __shared__ uint64_t lds64[];
    uint32_t(*count)[256] = (uint32_t(*)[256])(lds64 + kOneWgKeys);
    uint32_t *wave_sum = (uint32_t *)(count + 16);
    const int items = (int)((n + kLdsSortThreads - 1) / kLdsSortThreads);
    const uint32_t base = (threadIdx.x >> 6) * 64 * items + (threadIdx.x & 63);
    uint64_t key[kOneWgItems];
#pragma unroll
    for (int it = 0; it < kOneWgItems; ++it)
        if (it < items)
            key[it] = base + it * 64 < n ? keys[base + it * 64] : ~0ull;
    lds_sort<uint64_t, kOneWgItems>(key, items, lo, hi, lds64, count, wave_sum);
    for (uint32_t i = threadIdx.x; i < n; i += kLdsSortThreads)
        keys[i] = lds64[i];
}

} // namespace
