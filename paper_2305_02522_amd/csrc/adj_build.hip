// Adjacency builder: edge list -> 0/1 aggregation matrix A_hat as a set of
// (row, col) pairs (Section 2.1: A_hat = A + I; Section 3.2.1: the sparse bit
// matrix only stores which entries are 1).
//
// Everything runs on the GPU with hand-written kernels.  The pairs are sorted in two ways:
//   - by buckets of consecutive rows: the pairs are dealt out to the buckets in one or two passes
//     over memory, in no order, and each bucket (4 to 8 thousand pairs on average) is sorted,
//     rid of its duplicates and counted by one workgroup in LDS;
//   - where a bucket holds more pairs than LDS (a row of tens of thousands of neighbours), or a
//     pair does not fit 32 bits inside its bucket: one 64-bit key (row << cb | col) per pair, LSD
//     radix sort, flag-scan-compact, row pointers by binary search.
// Then the degrees give the row pointers and everything the host needs to know in one copy, and
// a degree-sorted row order (rows of similar length share a wavefront in the aggregation kernel).
// The paper's 4x4 bit tiles are not used: at the densities of these graphs a
// tile holds one non-zero (Section 4.2 says the same of its own data), so the
// fine-grained format here is the sorted column list itself.
#include "prims.h"

#include <stdlib.h>

namespace {

// What the build tells the host, in one copy once the degrees are known.
struct BuildInfo {
    int32_t err;         // an endpoint is out of range
    uint32_t overflow;   // a bucket does not fit in LDS: nothing behind it has run
    uint32_t nnz;
    uint32_t max_degree;
    uint32_t bits[33];   // rows whose degree has that many bits
    uint32_t parts;      // row parts of the column-blocked form, and rows with more than one
    uint32_t multi;
    uint32_t n_long[2];  // rows longer than kSegLenSmall / kSegLenLarge, and their segments
    uint32_t n_segs[2];
};

// ---------------------------------------------------------------- buckets
// A bucket is 2^shift rows.  What bounds the passes is memory: the pairs are read three times and
// written twice (once where 512 buckets suffice), 4 bytes each inside the buckets.  Dealing out
// needs whole lines: a workgroup puts 16,384 pairs in bucket order in LDS, takes its places in
// every bucket with one atomic add, and writes runs; hence at most 256 buckets (or 512, in one
// pass) at a time, and a second pass for the buckets inside those.
// 57 M edges on 232,965 nodes, symmetric, to CSR: 12.3 ms as an LSD sort of 64-bit keys with
// tiles of 2,048 keys, 5.4 with tiles of 8,192, 2.1 so.
constexpr uint32_t kBucketThreads = 1024;
constexpr uint32_t kBucketItems = 32;
constexpr uint32_t kBucketCap = kBucketThreads * kBucketItems; // pairs that fit in LDS
// A larger bucket is sorted through memory by its workgroup, at ~3 ns a pair; all the pairs as
// 64-bit keys take ~0.1 ns each and a third of a millisecond.
constexpr uint32_t kBucketMost = 131072;                       // plus a 32nd of all pairs
constexpr uint32_t kMaxBuckets = 16384;                        // 64 KB of LDS counters
constexpr uint32_t kDealEdges = 8;                             // per thread
constexpr uint32_t kDealTile = 2 * kDealEdges * kBucketThreads; // pairs a workgroup deals out
constexpr uint32_t kDealMax = 512;                             // buckets dealt out in one pass
constexpr size_t kBucketLds = kBucketCap * 4 + 16 * 256 * 4 + 64;

struct BucketPlan {
    uint32_t n, rows_shift, buckets; // nodes; 2^rows_shift of them a bucket
    uint32_t cb;                     // bits of a column
    uint32_t deal_shift, deals;      // 2^deal_shift buckets a deal of the first pass (0: one pass)
    uint32_t loops;
    __host__ __device__ uint32_t rows_of(uint32_t b, uint32_t shift) const
    {
        const uint32_t r0 = b << shift, left = n - r0;
        return left < (1u << shift) ? left : 1u << shift;
    }
};

// An edge's endpoints; out of range ones are noted and count as (0, 0).
__device__ __forceinline__ bool edge_of(const int32_t *src, const int32_t *dst, uint32_t t,
                                        uint32_t n, uint32_t &i, uint32_t &j)
{
    i = (uint32_t)src[t];
    j = (uint32_t)dst[t];
    const bool ok = i < n && j < n; // negative values wrap to >= 2^31 > n
    if (!ok)
        i = j = 0;
    return ok;
}

__global__ __launch_bounds__(kBucketThreads) void bucket_count_kernel(
    const int32_t *__restrict__ src, const int32_t *__restrict__ dst, uint32_t E, int symmetrize,
    BucketPlan p, uint32_t *__restrict__ partial, BuildInfo *__restrict__ info)
{
    extern __shared__ uint32_t h[];
    for (uint32_t b = threadIdx.x; b < p.buckets; b += kBucketThreads)
        h[b] = 0;
    __syncthreads();
    bool bad = false;
    const uint32_t step = gridDim.x * kBucketThreads * 4;
    for (uint32_t t0 = blockIdx.x * kBucketThreads * 4; t0 < E; t0 += step) {
        uint32_t i[4], j[4];
        bool in[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t t = t0 + k * kBucketThreads + threadIdx.x;
            in[k] = t < E;
            bad |= !edge_of(src, dst, in[k] ? t : E - 1, p.n, i[k], j[k]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (in[k]) {
                atomicAdd(&h[i[k] >> p.rows_shift], 1u);
                if (symmetrize)
                    atomicAdd(&h[j[k] >> p.rows_shift], 1u);
            }
    }
    if (bad)
        atomicOr(&info->err, 1);
    __syncthreads();
    uint32_t *out = partial + (uint64_t)blockIdx.x * p.buckets;
    for (uint32_t b = threadIdx.x; b < p.buckets; b += kBucketThreads)
        out[b] = h[b];
}

// Sums the partial counts into the first of them: 32 buckets by 8 shares of the counts a workgroup.
__global__ __launch_bounds__(256) void bucket_reduce_kernel(uint32_t *__restrict__ partial,
                                                            uint32_t buckets, uint32_t g)
{
    __shared__ uint32_t sum[8][32];
    const uint32_t b = blockIdx.x * 32 + (threadIdx.x & 31), q = threadIdx.x >> 5;
    uint32_t s = 0;
    if (b < buckets)
#pragma unroll 8
        for (uint32_t k = q; k < g; k += 8)
            s += partial[(uint64_t)k * buckets + b];
    sum[q][threadIdx.x & 31] = s;
    __syncthreads();
    if (q == 0 && b < buckets) {
        for (int k = 1; k < 8; ++k)
            s += sum[k][threadIdx.x];
        partial[b] = s;
    }
}

// Places of the buckets (self loops included), where each of the two passes goes on writing, and
// the first tile of each deal in the second pass.
__global__ __launch_bounds__(kBucketThreads) void bucket_place_kernel(
    const uint32_t *__restrict__ partial, uint32_t g, BucketPlan p, uint32_t largest_allowed,
    uint32_t *__restrict__ place, uint32_t *__restrict__ next, uint32_t *__restrict__ deal_next,
    uint32_t *__restrict__ deal_tile, BuildInfo *__restrict__ info)
{
    constexpr uint32_t kPer = kMaxBuckets / kBucketThreads;
    const uint32_t per = (p.buckets + kBucketThreads - 1) / kBucketThreads; // <= kPer
    uint32_t c[kPer], sum = 0, largest = 0;
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t b = threadIdx.x * per + k;
        c[k] = 0;
        if (k < per && b < p.buckets) {
            for (uint32_t q = 0; q < g; ++q)
                c[k] += partial[(uint64_t)q * p.buckets + b];
            if (p.loops)
                c[k] += p.rows_of(b, p.rows_shift);
        }
        sum += c[k];
        largest = max(largest, c[k]);
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan<kBucketThreads>(sum, &total);
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t b = threadIdx.x * per + k;
        if (k < per && b < p.buckets) {
            place[b] = run;
            next[b] = run;
            if ((b & ((1u << p.deal_shift) - 1)) == 0)
                deal_next[b >> p.deal_shift] = run;
        }
        run += c[k];
    }
    if (threadIdx.x == 0)
        place[p.buckets] = total;
    if (largest > largest_allowed)
        atomicOr(&info->overflow, 1u);
    __syncthreads();
    // pairs of deal t without the self loops, which the bucket sort adds
    uint32_t tiles = 0;
    if (threadIdx.x < p.deals) {
        const uint32_t b0 = threadIdx.x << p.deal_shift;
        const uint32_t b1 = min(b0 + (1u << p.deal_shift), p.buckets);
        uint32_t pairs = place[b1] - place[b0];
        if (p.loops)
            pairs -= p.rows_of(threadIdx.x, p.rows_shift + p.deal_shift);
        tiles = (pairs + kDealTile - 1) / kDealTile;
    }
    const uint32_t first = block_exclusive_scan<kBucketThreads>(tiles, &total);
    if (threadIdx.x < p.deals)
        deal_tile[threadIdx.x] = first;
    if (threadIdx.x == 0)
        deal_tile[p.deals] = total;
}

// Deals out one tile: pair k of this thread goes to digit[k] (>= D: no pair).
template <typename K, int ITEMS>
__device__ __forceinline__ void deal_tile_out(const K (&key)[ITEMS], uint32_t (&digit)[ITEMS],
                                              uint32_t D, uint32_t *__restrict__ next,
                                              K *__restrict__ out)
{
    extern __shared__ uint64_t lds64[];
    __shared__ uint32_t count[kDealMax], first[kDealMax], dest[kDealMax];
    K *stage = (K *)lds64;
    if (threadIdx.x < kDealMax)
        count[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
        if (digit[k] < D)
            digit[k] |= atomicAdd(&count[digit[k]], 1u) << 16; // at most 16,383
        else
            digit[k] = ~0u;
    __syncthreads();
    const uint32_t c = threadIdx.x < D ? count[threadIdx.x] : 0;
    uint32_t total;
    const uint32_t f = block_exclusive_scan<kBucketThreads>(c, &total);
    if (threadIdx.x < D) {
        first[threadIdx.x] = f;
        dest[threadIdx.x] = c ? atomicAdd(&next[threadIdx.x], c) : 0;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
        if (digit[k] != ~0u)
            stage[first[digit[k] & 0xFFFFu] + (digit[k] >> 16)] = key[k];
    __syncthreads();
    for (uint32_t d = threadIdx.x >> 5; d < D; d += kBucketThreads / 32) {
        const uint32_t n = count[d], f0 = first[d], o = dest[d];
        for (uint32_t i = threadIdx.x & 31; i < n; i += 32)
            out[o + i] = stage[f0 + i];
    }
}

// First pass: a row's deal is row >> deal_rows; the pair keeps the rest of the row and the column.
template <typename K>
__global__ __launch_bounds__(kBucketThreads) void deal_edges_kernel(
    const int32_t *__restrict__ src, const int32_t *__restrict__ dst, uint32_t E, int symmetrize,
    BucketPlan p, uint32_t *__restrict__ deal_next, K *__restrict__ out,
    const BuildInfo *__restrict__ info)
{
    if (info->overflow)
        return;
    const uint32_t deal_rows = p.rows_shift + p.deal_shift;
    const uint32_t low = deal_rows < 32 ? (1u << deal_rows) - 1 : ~0u;
    K key[2 * kDealEdges];
    uint32_t digit[2 * kDealEdges];
    const uint32_t t0 = blockIdx.x * (kDealEdges * kBucketThreads) + threadIdx.x;
#pragma unroll
    for (uint32_t k = 0; k < kDealEdges; ++k) {
        const uint32_t t = t0 + k * kBucketThreads;
        uint32_t i, j;
        (void)edge_of(src, dst, t < E ? t : E - 1, p.n, i, j);
        key[2 * k] = ((K)(i & low) << p.cb) | j;
        key[2 * k + 1] = ((K)(j & low) << p.cb) | i;
        digit[2 * k] = t < E ? i >> deal_rows : ~0u;
        digit[2 * k + 1] = t < E && symmetrize ? j >> deal_rows : ~0u;
    }
    deal_tile_out<K, 2 * kDealEdges>(key, digit, p.deals, deal_next, out);
}

// Second pass: the pairs of each deal into its 2^deal_shift buckets.
template <typename K>
__global__ __launch_bounds__(kBucketThreads) void deal_buckets_kernel(
    const K *__restrict__ in, BucketPlan p, const uint32_t *__restrict__ place,
    const uint32_t *__restrict__ deal_tile, uint32_t *__restrict__ next, uint32_t *__restrict__ out,
    const BuildInfo *__restrict__ info)
{
    __shared__ uint32_t mine;
    if (info->overflow || blockIdx.x >= deal_tile[p.deals])
        return;
    if (threadIdx.x < p.deals && deal_tile[threadIdx.x] <= blockIdx.x &&
        blockIdx.x < deal_tile[threadIdx.x + 1])
        mine = threadIdx.x;
    __syncthreads();
    const uint32_t deal = mine, b0 = deal << p.deal_shift;
    const uint32_t b1 = min(b0 + (1u << p.deal_shift), p.buckets);
    uint32_t end = place[b1];
    if (p.loops)
        end -= p.rows_of(deal, p.rows_shift + p.deal_shift);
    const uint32_t t0 = place[b0] + (blockIdx.x - deal_tile[deal]) * kDealTile + threadIdx.x;
    const int bits = (int)(p.rows_shift + p.cb);
    const K low = ((K)1 << bits) - 1; // bits < 32 where K is 32 bits wide
    uint32_t key[2 * kDealEdges], digit[2 * kDealEdges];
#pragma unroll
    for (uint32_t k = 0; k < 2 * kDealEdges; ++k) {
        const uint32_t t = t0 + k * kBucketThreads;
        const K v = in[t < end ? t : end - 1];
        key[k] = (uint32_t)(v & low);
        digit[k] = t < end ? (uint32_t)(v >> bits) : ~0u;
    }
    deal_tile_out<uint32_t, 2 * kDealEdges>(key, digit, b1 - b0, next + b0, out);
}

// Drops the duplicates of a tile of n <= kBucketCap sorted pairs in LDS, which `prev` precedes
// (unless it is the first tile) and `next` follows (unless it is the last): distinct columns go
// to out[at ..), and cnt[row] grows by the distinct pairs up to a row's last pair and shrinks by
// those before its first.  Returns `at` behind the last one.
__device__ __forceinline__ uint32_t distinct_pairs(const uint32_t *stage, uint32_t n, bool first,
                                                   uint32_t prev, bool last, uint32_t next,
                                                   uint32_t cb, uint32_t at, uint32_t *out,
                                                   uint32_t *cnt, uint32_t *wave_sum)
{
    const int items = (int)((n + kBucketThreads - 1) / kBucketThreads);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t base = wave * 64 * items + lane, mask = (1u << cb) - 1; // cb <= 31
    uint32_t firsts = 0, mine = 0; // this lane's first pairs of their kind, by item
    for (int it = 0; it < items; ++it) {
        const uint32_t i = base + it * 64;
        const bool f = i < n && (i ? stage[i] != stage[i - 1] : first || stage[0] != prev);
        firsts |= (uint32_t)f << it;
        mine += (uint32_t)__popcll(__ballot(f));
    }
    __syncthreads();
    if (lane == 0)
        wave_sum[wave] = mine;
    __syncthreads();
    uint32_t all = 0, run = at;
    for (int w = 0; w < (int)kBucketThreads / 64; ++w) {
        if (w == wave)
            run += all;
        all += wave_sum[w];
    }
    for (int it = 0; it < items; ++it) {
        const uint32_t i = base + it * 64;
        const bool f = (firsts >> it) & 1u;
        const uint64_t m = __ballot(f);
        const uint32_t to = run + __builtin_amdgcn_mbcnt_hi(
                                      (uint32_t)(m >> 32),
                                      __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        run += (uint32_t)__popcll(m);
        if (i < n) {
            const uint32_t key = stage[i], row = key >> cb;
            if (f)
                out[to] = key & mask;
            if (i ? stage[i - 1] >> cb != row : first || prev >> cb != row)
                atomicSub(&cnt[row], to);
            if (i + 1 < n ? stage[i + 1] >> cb != row : last || next >> cb != row)
                atomicAdd(&cnt[row], to + f);
        }
    }
    return at + all;
}

// Sorts each bucket of up to kBucketSmall pairs on (row, column) and drops duplicates, in place:
// the columns of its rows follow each other from the bucket's place on, and the rows' degrees are
// known.  Bound by instruction issue, so the passes are the cheapest that sort: the first one, on
// the 12 low bits, needs no order among equal digits and gives places with one LDS atomic each;
// the stable ones behind it take at most 7 bits, a vote per bit.  Two workgroups a CU (80 KB of
// LDS, 64 registers), so that one computes at the other's barriers.  115 M pairs of 22 bits:
// 824 us, and 455 for the 12 % of the buckets that are larger; 1,947 with three stable passes of 8 bits and one workgroup of twice the pairs a CU.
constexpr int kSmallItems = 15;
constexpr uint32_t kBucketSmall = kBucketThreads * kSmallItems;
constexpr uint32_t kFirstBits = 12;
constexpr uint32_t kSmallDigit = 128;
constexpr size_t kSmallLds = kBucketSmall * 4 + (4u << kFirstBits) + 64;

__global__ __launch_bounds__(kBucketThreads) __attribute__((amdgpu_waves_per_eu(8))) void
bucket_sort_small_kernel(uint32_t *__restrict__ pairs, BucketPlan p,
                         const uint32_t *__restrict__ place, int32_t *__restrict__ deg,
                         const BuildInfo *__restrict__ info)
{
    extern __shared__ uint64_t lds64[];
    uint32_t *stage = (uint32_t *)lds64, *cnt = stage + kBucketSmall;
    uint32_t *wave_sum = cnt + (1u << kFirstBits);
    const uint32_t b = blockIdx.x, o = place[b], n = place[b + 1] - o;
    if (info->overflow || n > kBucketSmall)
        return;
    const uint32_t row0 = b << p.rows_shift, rows = p.rows_of(b, p.rows_shift);
    const uint32_t drawn = n - (p.loops ? rows : 0);
    const int items = (int)((n + kBucketThreads - 1) / kBucketThreads);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t base = wave * 64 * items + lane;
    uint32_t *io = pairs + o;
    uint32_t key[kSmallItems], rank[kSmallItems];
    for (uint32_t d = threadIdx.x; d < 1u << kFirstBits; d += kBucketThreads)
        cnt[d] = 0;
#pragma unroll
    for (int it = 0; it < kSmallItems; ++it)
        if (it < items) {
            const uint32_t i = base + it * 64, r = i - drawn; // self loop of row r, i >= drawn
            key[it] = i < drawn ? io[i] : i < n ? (r << p.cb) | (row0 + r) : ~0u;
        }
    __syncthreads();
    constexpr uint32_t low = (1u << kFirstBits) - 1;
#pragma unroll
    for (int it = 0; it < kSmallItems; ++it)
        if (it < items && base + it * 64 < n)
            rank[it] = atomicAdd(&cnt[key[it] & low], 1u);
    __syncthreads();
    {
        static_assert((1u << kFirstBits) == 4 * kBucketThreads, "four counters a thread");
        uint4 c = *(const uint4 *)(cnt + 4 * threadIdx.x);
        uint32_t total;
        const uint32_t run = block_exclusive_scan<kBucketThreads>(c.x + c.y + c.z + c.w, &total);
        c = make_uint4(run, run + c.x, run + c.x + c.y, run + c.x + c.y + c.z);
        *(uint4 *)(cnt + 4 * threadIdx.x) = c;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kSmallItems; ++it)
        if (it < items) { // places past the end keep ~0 and stay behind every pair
            const uint32_t i = base + it * 64;
            stage[i < n ? cnt[key[it] & low] + rank[it] : i] = key[it];
        }
    __syncthreads();
    const int bits = (int)(p.rows_shift + p.cb), rest = bits - (int)kFirstBits;
    const int passes = rest > 0 ? (rest + 6) / 7 : 0;
    uint32_t(*count)[kSmallDigit] = (uint32_t(*)[kSmallDigit])cnt;
    int shift = kFirstBits;
    for (int q = passes; q > 0; --q) {
        const int width = (bits - shift + q - 1) / q; // the same for all, rounded up first
#pragma unroll
        for (int it = 0; it < kSmallItems; ++it)
            if (it < items)
                key[it] = stage[base + it * 64];
        wave_digit_ranks<uint32_t, kSmallItems, 7>(key, rank, items, shift, count[wave], width);
        block_digit_places<kBucketThreads / 64, 7>(count, wave_sum);
        const uint32_t mask = (1u << width) - 1;
#pragma unroll
        for (int it = 0; it < kSmallItems; ++it)
            if (it < items)
                stage[count[wave][(key[it] >> shift) & mask] + rank[it]] = key[it];
        __syncthreads();
        shift += width;
    }
    for (uint32_t r = threadIdx.x; r < rows; r += kBucketThreads)
        cnt[r] = 0;
    __syncthreads();
    (void)distinct_pairs(stage, n, true, 0, true, 0, p.cb, 0, io, cnt, wave_sum);
    __syncthreads();
    for (uint32_t r = threadIdx.x; r < rows; r += kBucketThreads)
        deg[row0 + r] = (int32_t)cnt[r];
}

// The same for larger buckets (rows of thousands of neighbours next to each other): up to
// kBucketCap pairs in LDS, more through memory, in tiles of that size, to and fro between `pairs`
// and `other`.
__global__ __launch_bounds__(kBucketThreads) void bucket_sort_large_kernel(
    uint32_t *__restrict__ pairs, uint32_t *__restrict__ other, BucketPlan p,
    const uint32_t *__restrict__ place, int32_t *__restrict__ deg,
    const BuildInfo *__restrict__ info)
{
    extern __shared__ uint64_t lds64[];
    __shared__ uint32_t digit_place[256];
    uint32_t *stage = (uint32_t *)lds64;
    uint32_t(*count)[256] = (uint32_t(*)[256])(stage + kBucketCap);
    uint32_t *wave_sum = (uint32_t *)(count + 16);
    if (info->overflow)
        return;
    const uint32_t b = blockIdx.x, row0 = b << p.rows_shift, rows = p.rows_of(b, p.rows_shift);
    const uint32_t o = place[b], n = place[b + 1] - o, drawn = n - (p.loops ? rows : 0);
    if (n <= kBucketSmall)
        return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int bits = (int)(p.rows_shift + p.cb);
    uint32_t *cnt = &count[0][0]; // 4,096 words of row counts, once sorted (rows_shift <= 12)
    uint32_t *in = pairs + o, *out = other + o;
    uint32_t key[kBucketItems];
    if (n <= kBucketCap) {
        const int items = (int)((n + kBucketThreads - 1) / kBucketThreads);
        const uint32_t base = wave * 64 * items + lane;
#pragma unroll
        for (int it = 0; it < (int)kBucketItems; ++it)
            if (it < items) {
                const uint32_t i = base + it * 64;
                const uint32_t r = i - drawn; // self loop of row r, where i >= drawn
                key[it] = i < drawn ? in[i] : i < n ? (r << p.cb) | (row0 + r) : ~0u;
            }
        lds_sort<uint32_t, kBucketItems>(key, items, 0, bits, stage, count, wave_sum);
        for (uint32_t r = threadIdx.x; r < rows; r += kBucketThreads)
            cnt[r] = 0;
        __syncthreads();
        (void)distinct_pairs(stage, n, true, 0, true, 0, p.cb, 0, in, cnt, wave_sum);
    } else {
        for (uint32_t r = threadIdx.x; r < n - drawn; r += kBucketThreads)
            in[drawn + r] = (r << p.cb) | (row0 + r);
        const uint32_t base = wave * (64 * kBucketItems) + lane;
        for (int shift = 0; shift < bits; shift += 8) {
            __syncthreads();
            if (threadIdx.x < 256)
                digit_place[threadIdx.x] = 0;
            __syncthreads();
            for (uint32_t i = threadIdx.x; i < n; i += kBucketThreads)
                atomicAdd(&digit_place[(in[i] >> shift) & 255u], 1u);
            __syncthreads();
            uint32_t total, c = threadIdx.x < 256 ? digit_place[threadIdx.x] : 0;
            c = block_exclusive_scan<kBucketThreads>(c, &total);
            if (threadIdx.x < 256)
                digit_place[threadIdx.x] = c;
            for (uint32_t t0 = 0; t0 < n; t0 += kBucketCap) {
                const uint32_t m = min(n - t0, kBucketCap);
                uint32_t rank[kBucketItems];
#pragma unroll
                for (int it = 0; it < (int)kBucketItems; ++it)
                    key[it] = base + it * 64 < m ? in[t0 + base + it * 64] : ~0u;
                wave_digit_ranks<uint32_t, kBucketItems>(key, rank, kBucketItems, shift,
                                                         count[wave]);
                const uint32_t first =
                    block_digit_places<kBucketThreads / 64>(count, wave_sum);
#pragma unroll
                for (int it = 0; it < (int)kBucketItems; ++it)
                    stage[count[wave][(key[it] >> shift) & 255u] + rank[it]] = key[it];
                // a digit's pairs go to digit_place on, from `first` of the tile on
                __syncthreads();
                uint32_t *from = count[0]; // first place in the tile
                if (threadIdx.x < 256)
                    from[threadIdx.x] = first;
                __syncthreads();
                for (uint32_t i = threadIdx.x; i < m; i += kBucketThreads) {
                    const uint32_t v = stage[i], d = (v >> shift) & 255u;
                    out[digit_place[d] + i - from[d]] = v;
                }
                __syncthreads();
                if (threadIdx.x < 256) {
                    const uint32_t end = threadIdx.x < 255 ? from[threadIdx.x + 1] : kBucketCap;
                    digit_place[threadIdx.x] += min(end, m) - min(from[threadIdx.x], m);
                }
                __syncthreads();
            }
            uint32_t *t = in;
            in = out;
            out = t;
        }
        __syncthreads();
        for (uint32_t r = threadIdx.x; r < rows; r += kBucketThreads)
            cnt[r] = 0;
        __syncthreads();
        uint32_t at = 0, prev = 0;
        for (uint32_t t0 = 0; t0 < n; t0 += kBucketCap) {
            const uint32_t m = min(n - t0, kBucketCap);
            for (uint32_t i = threadIdx.x; i < m; i += kBucketThreads)
                stage[i] = in[t0 + i];
            const uint32_t next = t0 + m < n ? in[t0 + m] : 0;
            __syncthreads();
            // columns never pass the pairs that have been read
            at = distinct_pairs(stage, m, t0 == 0, prev, t0 + m == n, next, p.cb, at, pairs + o, cnt,
                                wave_sum);
            prev = stage[m - 1];
            __syncthreads();
        }
    }
    __syncthreads();
    for (uint32_t r = threadIdx.x; r < rows; r += kBucketThreads)
        deg[row0 + r] = (int32_t)cnt[r];
}

// The buckets' columns without the gaps that duplicates left.
__global__ __launch_bounds__(256) void bucket_columns_kernel(const uint32_t *__restrict__ pairs,
                                                             BucketPlan p,
                                                             const uint32_t *__restrict__ place,
                                                             const uint32_t *__restrict__ rowptr,
                                                             int32_t *__restrict__ col)
{
    const uint32_t b = blockIdx.x, row0 = b << p.rows_shift;
    const uint32_t to = rowptr[row0], n = rowptr[row0 + p.rows_of(b, p.rows_shift)] - to;
    const uint32_t *from = pairs + place[b];
    col += to;
#pragma unroll 8
    for (uint32_t i = threadIdx.x; i < n; i += 256)
        col[i] = (int32_t)from[i];
}

// ---------------------------------------------------------------- 64-bit keys
__global__ void make_keys_kernel(const int32_t *__restrict__ src, const int32_t *__restrict__ dst,
                                 uint32_t E, uint32_t N, int symmetrize, int self_loops, int cb,
                                 uint64_t *__restrict__ keys, BuildInfo *__restrict__ info)
{
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < E) {
        uint32_t i, j;
        if (!edge_of(src, dst, t, N, i, j))
            atomicOr(&info->err, 1);
        keys[t] = ((uint64_t)i << cb) | j;
        if (symmetrize)
            keys[(uint64_t)E + t] = ((uint64_t)j << cb) | i;
    }
    if (self_loops && t < N)
        keys[(uint64_t)E * (symmetrize ? 2 : 1) + t] = ((uint64_t)t << cb) | t;
}

__global__ __launch_bounds__(kScanThreads) void uniq_count_kernel(const uint64_t *__restrict__ keys,
                                                                  uint32_t n,
                                                                  uint32_t *__restrict__ counts)
{
    const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const uint32_t i = base + k;
        if (i < n && (i == 0 || keys[i] != keys[i - 1]))
            ++s;
    }
    uint32_t total;
    (void)block_exclusive_scan(s, &total);
    if (threadIdx.x == 0)
        counts[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void uniq_compact_kernel(
    const uint64_t *__restrict__ keys, uint32_t n, const uint32_t *__restrict__ offs,
    uint64_t *__restrict__ out)
{
    const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    bool f[kScanItems];
    uint64_t kv[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const uint32_t i = base + k;
        kv[k] = (i < n) ? keys[i] : 0;
        f[k] = i < n && (i == 0 || kv[k] != keys[i - 1]);
        s += f[k];
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan(s, &total) + offs[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        if (f[k])
            out[run++] = kv[k];
}

__global__ void split_keys_kernel(const uint64_t *__restrict__ ukeys, uint32_t nnz, int cb,
                                  int32_t *__restrict__ col)
{
    const uint32_t u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u < nnz)
        col[u] = (int32_t)(ukeys[u] & ((1ull << cb) - 1));
}

// index of the first key whose row is >= r
__device__ __forceinline__ uint32_t first_of_row(const uint64_t *ukeys, uint32_t nnz, int cb,
                                                 uint32_t r)
{
    const uint64_t want = (uint64_t)r << cb;
    uint32_t lo = 0, hi = nnz;
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (ukeys[mid] < want)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

__global__ void key_degrees_kernel(const uint64_t *__restrict__ ukeys,
                                   const uint32_t *__restrict__ nnz, int cb, uint32_t N,
                                   int32_t *__restrict__ deg)
{
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < N)
        deg[r] = (int32_t)(first_of_row(ukeys, *nnz, cb, r + 1) - first_of_row(ukeys, *nnz, cb, r));
}

// ---------------------------------------------------------------- degrees
// Copies the degrees to where the row pointers are scanned, and counts what the host asks of them.
__global__ __launch_bounds__(kScanThreads) void degree_info_kernel(const int32_t *__restrict__ deg,
                                                                   uint32_t N, uint32_t part_len,
                                                                   uint32_t *__restrict__ rowptr,
                                                                   BuildInfo *__restrict__ info)
{
    __shared__ uint32_t bits[33], sums[7], top;
    if (threadIdx.x < 33)
        bits[threadIdx.x] = 0;
    if (threadIdx.x < 7)
        sums[threadIdx.x] = 0;
    if (threadIdx.x == 0)
        top = 0;
    __syncthreads();
    uint32_t most = 0;
    uint32_t v[7] = {}; // entries, parts, rows with several, long rows and segments of both lengths
    const uint32_t seg_len[2] = {kSegLenSmall, kSegLenLarge};
    for (int k = 0; k < kScanItems; ++k) {
        const uint32_t i = blockIdx.x * kScanTile + k * kScanThreads + threadIdx.x;
        if (i > N)
            continue;
        const uint32_t d = i < N ? (uint32_t)deg[i] : 0;
        rowptr[i] = d;
        if (i == N)
            continue;
        // one add per distinct number of bits in the wavefront: most rows have the same few
        const uint32_t len = 32 - __clz((int)d);
        uint64_t same = __ballot(true);
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const uint64_t m = __ballot((len >> q) & 1u);
            same &= (len >> q) & 1u ? m : ~m;
        }
        if (__builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32),
                                      __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u)) == 0)
            atomicAdd(&bits[len], (uint32_t)__popcll(same));
        most = max(most, d);
        v[0] += d;
        v[1] += d > part_len ? (d + part_len - 1) / part_len : 1;
        v[2] += d > part_len;
        for (int q = 0; q < 2; ++q)
            if (d > seg_len[q]) {
                v[3 + q] += 1;
                v[5 + q] += (d + seg_len[q] - 1) / seg_len[q];
            }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
#pragma unroll
        for (int q = 0; q < 7; ++q)
            v[q] += __shfl_xor(v[q], d, 64);
        most = max(most, (uint32_t)__shfl_xor(most, d, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        for (int q = 0; q < 7; ++q)
            atomicAdd(&sums[q], v[q]);
        atomicMax(&top, most);
    }
    __syncthreads();
    if (threadIdx.x == 0)
        atomicMax(&info->max_degree, top);
    if (threadIdx.x < 33 && bits[threadIdx.x])
        atomicAdd(&info->bits[threadIdx.x], bits[threadIdx.x]);
    if (threadIdx.x < 7 && sums[threadIdx.x]) {
        uint32_t *to[7] = {&info->nnz,       &info->parts,     &info->multi,    &info->n_long[0],
                           &info->n_long[1], &info->n_segs[0], &info->n_segs[1]};
        atomicAdd(to[threadIdx.x], sums[threadIdx.x]);
    }
}

// ---------------------------------------------------------------- row order
// What the degree order brings: by slot (position in the order) the exclusive prefix sums of the
// degrees, of the row parts and of the row segments, N + 1 words each; by node its slot, and the
// slot as {column block, position inside}.
struct OrderArrays {
    int32_t *order, *rank;
    uint32_t *block_rank;
    uint32_t *sums; // [3][N + 1]
};

struct OrderRules {
    uint32_t part_len, cbn;
    const BuildInfo *info;
};

__device__ __forceinline__ void slot_counts(uint32_t d, const OrderRules &r, uint32_t (&c)[3])
{
    const uint32_t seg_len = r.info->nnz >= kSegLargeNnz ? kSegLenLarge : kSegLenSmall;
    c[0] = d;
    c[1] = d > r.part_len ? (d + r.part_len - 1) / r.part_len : 1;
    c[2] = d > seg_len ? (d + seg_len - 1) / seg_len : 1;
}

__device__ __forceinline__ void place_slot(uint32_t slot, uint32_t node, const OrderRules &r,
                                           const OrderArrays &a)
{
    a.order[slot] = (int32_t)node;
    a.rank[node] = (int32_t)slot;
    const uint32_t block = slot / r.cbn;
    a.block_rank[node] = (block << 16) | (slot - block * r.cbn);
}

// ascending sort of this key = decreasing degree, ties by row id
__device__ __forceinline__ uint64_t order_key(uint32_t d, uint32_t node)
{
    return ((uint64_t)(0xFFFFFFFFu - d) << 32) | node;
}

// The order keys of up to kOneWgKeys nodes, sorted by one workgroup.
__global__ __launch_bounds__(kLdsSortThreads) void order_one_wg_kernel(
    const int32_t *__restrict__ deg, uint32_t N, const BuildInfo *__restrict__ info,
    uint64_t *__restrict__ keys)
{
    extern __shared__ uint64_t lds64[];
    uint32_t(*count)[256] = (uint32_t(*)[256])(lds64 + kOneWgKeys);
    uint32_t *wave_sum = (uint32_t *)(count + 16);
    const int items = (int)((N + kLdsSortThreads - 1) / kLdsSortThreads);
    const uint32_t base = (threadIdx.x >> 6) * 64 * items + (threadIdx.x & 63);
    uint64_t key[kOneWgItems];
#pragma unroll
    for (int it = 0; it < kOneWgItems; ++it)
        if (it < items) {
            const uint32_t i = base + it * 64;
            key[it] = i < N ? order_key((uint32_t)deg[i], i) : ~0ull;
        }
    lds_sort<uint64_t, kOneWgItems>(key, items, 32, 64 - __clz((int)info->max_degree), lds64, count,
                                    wave_sum);
    for (uint32_t i = threadIdx.x; i < N; i += kLdsSortThreads)
        keys[i] = lds64[i];
}

// Their places and prefix sums: every workgroup adds up what lies before its 1,024 slots itself
// (two launches fewer than a scan on a chain of launches of a few microseconds each).
__global__ __launch_bounds__(kLdsSortThreads) void order_small_kernel(
    const uint64_t *__restrict__ keys, uint32_t N, OrderRules r, OrderArrays a)
{
    uint32_t c[3], sum[3] = {}, total;
    for (uint32_t i = threadIdx.x; i < blockIdx.x * kLdsSortThreads; i += kLdsSortThreads) {
        slot_counts(0xFFFFFFFFu - (uint32_t)(keys[i] >> 32), r, c);
        for (int q = 0; q < 3; ++q)
            sum[q] += c[q];
    }
    const uint32_t slot = blockIdx.x * kLdsSortThreads + threadIdx.x;
    const uint64_t key = slot < N ? keys[slot] : ~0ull;
    slot_counts(0xFFFFFFFFu - (uint32_t)(key >> 32), r, c);
    if (slot < N)
        place_slot(slot, (uint32_t)key, r, a);
    for (int q = 0; q < 3; ++q) {
        (void)block_exclusive_scan<kLdsSortThreads>(sum[q], &total);
        const uint32_t before = total;
        const uint32_t in = block_exclusive_scan<kLdsSortThreads>(slot < N ? c[q] : 0, &total);
        if (slot <= N)
            a.sums[(uint64_t)q * (N + 1) + slot] = before + in;
    }
}

__global__ void order_keys_kernel(const int32_t *__restrict__ deg, uint32_t N,
                                  uint64_t *__restrict__ keys)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N)
        keys[i] = order_key((uint32_t)deg[i], i);
}

// Counts of each slot, to be scanned (entry N is 0: the scans end with the totals).
__global__ void order_from_keys_kernel(const uint64_t *__restrict__ keys, uint32_t N, OrderRules r,
                                       OrderArrays a)
{
    const uint32_t slot = blockIdx.x * blockDim.x + threadIdx.x;
    if (slot > N)
        return;
    uint32_t c[3] = {};
    if (slot < N) {
        place_slot(slot, (uint32_t)keys[slot], r, a);
        slot_counts(0xFFFFFFFFu - (uint32_t)(keys[slot] >> 32), r, c);
    }
    for (int q = 0; q < 3; ++q)
        a.sums[(uint64_t)q * (N + 1) + slot] = c[q];
}

__global__ void seg_slot_kernel(const uint32_t *__restrict__ seg_ptr, uint32_t n_long,
                                uint32_t *__restrict__ seg_slot)
{
    const uint32_t slot = blockIdx.x * blockDim.x + threadIdx.x;
    if (slot >= n_long)
        return;
    for (uint32_t v = seg_ptr[slot]; v < seg_ptr[slot + 1]; ++v)
        seg_slot[v] = slot;
}

__global__ void col_slot_kernel(const int32_t *__restrict__ col, uint32_t nnz,
                                const int32_t *__restrict__ rank, int32_t *__restrict__ col_slot)
{
    const uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < nnz)
        col_slot[e] = rank[col[e]];
}

} // namespace

// The buckets of a graph of N nodes and `pairs` pairs (duplicates included), or false where the
// 64-bit keys are the way.  Buckets of 4 to 8 thousand pairs leave room for uneven ones in
// half of a CU's LDS (15,360); small graphs take as few as give every CU a bucket.
static bool plan_buckets(uint32_t N, uint32_t pairs, bool loops, BucketPlan *plan)
{
    BucketPlan p{};
    p.n = N;
    p.loops = loops;
    p.cb = 1;
    while ((1ull << p.cb) < N)
        ++p.cb;
    const uint32_t avg = pairs / N + 1;
    uint32_t want = pairs / 256;
    want = want < 256 ? 256 : want > 4096 ? 4096 : want;
    const auto buckets_of = [&] { return ((uint64_t)N + (1u << p.rows_shift) - 1) >> p.rows_shift; };
    while (p.rows_shift < 12 && p.rows_shift + p.cb < 32 &&
           (((uint64_t)avg << p.rows_shift) < want ||
            (buckets_of() > kMaxBuckets && ((uint64_t)avg << p.rows_shift) <= kBucketSmall / 2)))
        ++p.rows_shift;
    const uint64_t buckets = buckets_of();
    if (buckets > kMaxBuckets || p.cb > 31)
        return false;
    p.buckets = (uint32_t)buckets;
    if (p.buckets > kDealMax)
        while (((p.buckets - 1) >> p.deal_shift) >= 256)
            ++p.deal_shift;
    p.deals = ((p.buckets - 1) >> p.deal_shift) + 1;
    *plan = p;
    return true;
}

template <typename K>
static void launch_deals(hipStream_t s, const int32_t *src, const int32_t *dst, uint32_t E, bool sym,
                         const BucketPlan &p, K *between, uint32_t *out, uint32_t *next,
                         uint32_t *deal_next, const uint32_t *place, const uint32_t *deal_tile,
                         const BuildInfo *info)
{
    const unsigned tiles = blocks_for(E, kDealEdges * kBucketThreads);
    (void)hipFuncSetAttribute((const void *)deal_edges_kernel<K>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, kDealTile * sizeof(K));
    deal_edges_kernel<K><<<tiles, kBucketThreads, kDealTile * sizeof(K), s>>>(
        src, dst, E, sym, p, deal_next, p.deal_shift ? between : (K *)out, info);
    if (!p.deal_shift)
        return;
    (void)hipFuncSetAttribute((const void *)deal_buckets_kernel<K>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, kDealTile * 4);
    const unsigned most = (unsigned)((uint64_t)E * (sym ? 2 : 1) / kDealTile) + p.deals;
    deal_buckets_kernel<K><<<most, kBucketThreads, kDealTile * 4, s>>>(between, p, place, deal_tile,
                                                                      next, out, info);
}

// Sorted sets of pairs, by the buckets or by the 64-bit keys: degrees, and the columns still in
// `pairs` (bucket places) or `keys`.
struct SortedPairs {
    bool bucketed;
    BucketPlan plan;
    DevBuf pairs, place; // buckets
    DevBuf keys;         // 64-bit keys
    explicit SortedPairs(bitgnn_ctx *ctx) : bucketed(false), plan{}, pairs(ctx), place(ctx), keys(ctx) {}
};

static int sort_by_buckets(bitgnn_ctx *ctx, hipStream_t s, const int32_t *src, const int32_t *dst,
                           uint32_t E, bool sym, SortedPairs &o, int32_t *deg, BuildInfo *info)
{
    const BucketPlan &p = o.plan;
    const uint64_t npairs = (uint64_t)E * (sym ? 2 : 1) + (p.loops ? p.n : 0);
    const bool wide = p.rows_shift + p.deal_shift + p.cb > 32;
    // workgroups that count: at least 4,096 edges each, two of them a CU at most
    uint32_t g = (uint32_t)blocks_for(E, 4 * kBucketThreads);
    g = g > 512 ? 512 : g;
    DevBuf partial(ctx), next(ctx), deals(ctx), between(ctx);
    BG_HIP(ctx, o.pairs.alloc(npairs * 4));
    BG_HIP(ctx, o.place.alloc(((size_t)p.buckets + 1) * 4));
    BG_HIP(ctx, partial.alloc((size_t)g * p.buckets * 4));
    BG_HIP(ctx, next.alloc((size_t)p.buckets * 4));
    BG_HIP(ctx, deals.alloc(2 * ((size_t)p.deals + 1) * 4));
    BG_HIP(ctx, between.alloc(npairs * (wide && p.deal_shift ? 8 : 4)));
    uint32_t *deal_next = deals.as<uint32_t>(), *deal_tile = deal_next + p.deals + 1;
    if (E > 0) {
        (void)hipFuncSetAttribute((const void *)bucket_count_kernel,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, kMaxBuckets * 4);
        bucket_count_kernel<<<g, kBucketThreads, (size_t)p.buckets * 4, s>>>(
            src, dst, E, sym, p, partial.as<uint32_t>(), info);
        BG_LAUNCH_CHECK(ctx, "bucket_count");
        if (g > 4) {
            bucket_reduce_kernel<<<blocks_for(p.buckets, 32), 256, 0, s>>>(partial.as<uint32_t>(),
                                                                          p.buckets, g);
            g = 1;
        }
    }
    bucket_place_kernel<<<1, kBucketThreads, 0, s>>>(
        partial.as<uint32_t>(), g, p, kBucketMost + (uint32_t)(npairs / 32),
        o.place.as<uint32_t>(), next.as<uint32_t>(), deal_next, deal_tile, info);
    BG_LAUNCH_CHECK(ctx, "bucket_place");
    if (E > 0) {
        if (wide && p.deal_shift)
            launch_deals(s, src, dst, E, sym, p, between.as<uint64_t>(), o.pairs.as<uint32_t>(),
                         next.as<uint32_t>(), deal_next, o.place.as<uint32_t>(), deal_tile, info);
        else
            launch_deals(s, src, dst, E, sym, p, between.as<uint32_t>(), o.pairs.as<uint32_t>(),
                         next.as<uint32_t>(), deal_next, o.place.as<uint32_t>(), deal_tile, info);
        BG_LAUNCH_CHECK(ctx, "deal");
    }
    (void)hipFuncSetAttribute((const void *)bucket_sort_small_kernel,
                              hipFuncAttributeMaxDynamicSharedMemorySize, kSmallLds);
    bucket_sort_small_kernel<<<p.buckets, kBucketThreads, kSmallLds, s>>>(
        o.pairs.as<uint32_t>(), p, o.place.as<uint32_t>(), deg, info);
    if (npairs > kBucketSmall) { // else no bucket can be larger
        (void)hipFuncSetAttribute((const void *)bucket_sort_large_kernel,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, kBucketLds);
        bucket_sort_large_kernel<<<p.buckets, kBucketThreads, kBucketLds, s>>>(
            o.pairs.as<uint32_t>(), between.as<uint32_t>(), p, o.place.as<uint32_t>(), deg, info);
    }
    BG_LAUNCH_CHECK(ctx, "bucket_sort");
    o.bucketed = true;
    return BITGNN_OK;
}

static int sort_by_keys(bitgnn_ctx *ctx, hipStream_t s, const int32_t *src, const int32_t *dst,
                        uint32_t E, uint32_t N, bool sym, bool loops, SortedPairs &o, int32_t *deg,
                        BuildInfo *info)
{
    const uint32_t nkeys = E * (sym ? 2 : 1) + (loops ? N : 0); // > 0: buckets take the others
    int cb = 1;
    while ((1ll << cb) < N)
        ++cb;
    const uint32_t tiles = (nkeys + kScanTile - 1) / kScanTile;
    DevBuf other(ctx), hist(ctx), scan_ws(ctx), counts(ctx);
    const size_t hist_words = sort_hist_words(nkeys);
    const size_t most = hist_words > (size_t)tiles + 1 ? hist_words : (size_t)tiles + 1;
    BG_HIP(ctx, o.keys.alloc((size_t)nkeys * 8));
    BG_HIP(ctx, other.alloc((size_t)nkeys * 8));
    BG_HIP(ctx, hist.alloc(hist_words * 4));
    BG_HIP(ctx, scan_ws.alloc(scan_ws_words(most) * 4));
    BG_HIP(ctx, counts.alloc(((size_t)tiles + 1) * 4));
    make_keys_kernel<<<blocks_for(E > N ? E : N, 256), 256, 0, s>>>(
        src, dst, E, N, sym, loops, cb, o.keys.as<uint64_t>(), info);
    BG_LAUNCH_CHECK(ctx, "make_keys");
    uint64_t *sorted = radix_sort(o.keys.as<uint64_t>(), other.as<uint64_t>(), nkeys, 0, 2 * cb,
                                  hist.as<uint32_t>(), scan_ws.as<uint32_t>(), s);
    BG_LAUNCH_CHECK(ctx, "radix_sort");
    if (sorted == o.keys.as<uint64_t>()) { // the distinct keys go to the other buffer: keep that
        const bg_block b = o.keys.b;
        o.keys.b = other.b;
        other.b = b;
    }
    uniq_count_kernel<<<tiles, kScanThreads, 0, s>>>(sorted, nkeys, counts.as<uint32_t>());
    BG_HIP(ctx, hipMemsetAsync(counts.as<uint32_t>() + tiles, 0, 4, s));
    scan_inplace(counts.as<uint32_t>(), tiles + 1, scan_ws.as<uint32_t>(), s);
    uniq_compact_kernel<<<tiles, kScanThreads, 0, s>>>(sorted, nkeys, counts.as<uint32_t>(),
                                                       o.keys.as<uint64_t>());
    key_degrees_kernel<<<blocks_for(N, 256), 256, 0, s>>>(
        o.keys.as<uint64_t>(), counts.as<uint32_t>() + tiles, cb, N, deg);
    BG_LAUNCH_CHECK(ctx, "unique");
    o.bucketed = false;
    return BITGNN_OK;
}

static int adj_build(bitgnn_ctx *ctx, hipStream_t s, const int32_t *src, const int32_t *dst,
                     int64_t E64, int64_t N64, uint32_t flags, bitgnn_adj **out)
{
    BG_REQUIRE(ctx, out, BITGNN_ERR_INVALID_ARG, "bitgnn_adj_build: out is null");
    BG_REQUIRE(ctx, E64 >= 0 && N64 >= 1, BITGNN_ERR_INVALID_ARG,
               "bitgnn_adj_build: E=%lld N=%lld", (long long)E64, (long long)N64);
    BG_REQUIRE(ctx, (flags & ~3u) == 0, BITGNN_ERR_INVALID_ARG, "bitgnn_adj_build: flags=%u",
               flags);
    BG_REQUIRE(ctx, E64 == 0 || (src && dst), BITGNN_ERR_INVALID_ARG,
               "bitgnn_adj_build: null edge arrays");
    BG_REQUIRE(ctx, bg_aligned(src, 4) && bg_aligned(dst, 4), BITGNN_ERR_ALIGNMENT,
               "bitgnn_adj_build: misaligned edge arrays");
    const bool sym = flags & BITGNN_ADJ_SYMMETRIZE;
    const bool loops = flags & BITGNN_ADJ_ADD_SELF_LOOPS;
    const int64_t nkeys64 = E64 * (sym ? 2 : 1) + (loops ? N64 : 0);
    BG_REQUIRE(ctx, nkeys64 + N64 < (1ll << 31), BITGNN_ERR_RANGE,
               "bitgnn_adj_build: %lld stored pairs + N exceed 32-bit offsets", (long long)nkeys64);
    BG_NEED_DEVICE(ctx);

    BG_HIP(ctx, hipSetDevice(ctx->device));
    const uint32_t E = (uint32_t)E64, N = (uint32_t)N64;
    DevBuf rowptr(ctx), col(ctx), deg(ctx), order(ctx), rank(ctx), block_rank(ctx), sums(ctx);
    DevBuf info_buf(ctx), scan_ws(ctx);
    BG_HIP(ctx, rowptr.alloc(((size_t)N + 1) * 4));
    BG_HIP(ctx, deg.alloc((size_t)N * 4));
    BG_HIP(ctx, order.alloc((size_t)N * 4));
    BG_HIP(ctx, rank.alloc((size_t)N * 4));
    BG_HIP(ctx, block_rank.alloc((size_t)N * 4));
    BG_HIP(ctx, sums.alloc(((size_t)N + 1) * 3 * 4));
    BG_HIP(ctx, scan_ws.alloc(scan_ws_words((uint64_t)N + 1, 3) * 4));
    BG_HIP(ctx, info_buf.alloc(sizeof(BuildInfo)));
    BuildInfo *d_info = info_buf.as<BuildInfo>();
    const OrderRules rules{(uint32_t)ctx->part_len, (uint32_t)ctx->cb_nodes, d_info};
    const OrderArrays arrays{order.as<int32_t>(), rank.as<int32_t>(), block_rank.as<uint32_t>(),
                             sums.as<uint32_t>()};

    SortedPairs sorted(ctx);
    bool buckets = plan_buckets(N, (uint32_t)nkeys64, loops, &sorted.plan) || nkeys64 == 0;
    BuildInfo info;
    for (;;) {
        BG_HIP(ctx, hipMemsetAsync(d_info, 0, sizeof(BuildInfo), s));
        if (nkeys64 == 0)
            BG_HIP(ctx, hipMemsetAsync(deg.as<void>(), 0, (size_t)N * 4, s));
        else {
            const int rc = buckets ? sort_by_buckets(ctx, s, src, dst, E, sym, sorted,
                                                     deg.as<int32_t>(), d_info)
                                   : sort_by_keys(ctx, s, src, dst, E, N, sym, loops, sorted,
                                                  deg.as<int32_t>(), d_info);
            if (rc != BITGNN_OK)
                return rc;
        }
        degree_info_kernel<<<blocks_for((int64_t)N + 1, kScanTile), kScanThreads, 0, s>>>(
            deg.as<int32_t>(), N, (uint32_t)ctx->part_len, rowptr.as<uint32_t>(), d_info);
        BG_LAUNCH_CHECK(ctx, "degree_info");
        scan_inplace(rowptr.as<uint32_t>(), N + 1, scan_ws.as<uint32_t>(), s);
        BG_HIP(ctx, hipMemcpyAsync(&info, d_info, sizeof(info), hipMemcpyDeviceToHost, s));
        BG_HIP(ctx, hipStreamSynchronize(s));
        BG_REQUIRE(ctx, info.err == 0, BITGNN_ERR_INDEX_RANGE,
                   "bitgnn_adj_build: an edge endpoint is outside [0, %lld)", (long long)N64);
        if (!info.overflow)
            break;
        buckets = false; // a row too long for LDS: once more with 64-bit keys
        sorted.pairs.reset();
    }
    const uint32_t nnz = info.nnz;

    // columns, and the degree order
    BG_HIP(ctx, col.alloc((size_t)nnz * 4));
    if (nnz == 0) // kernels may read (not use) the first column of an empty graph
        BG_HIP(ctx, hipMemsetAsync(col.as<void>(), 0, 4, s));
    else if (sorted.bucketed)
        bucket_columns_kernel<<<sorted.plan.buckets, 256, 0, s>>>(
            sorted.pairs.as<uint32_t>(), sorted.plan, sorted.place.as<uint32_t>(),
            rowptr.as<uint32_t>(), col.as<int32_t>());
    else {
        int cb = 1;
        while ((1ll << cb) < N64)
            ++cb;
        split_keys_kernel<<<blocks_for(nnz, 256), 256, 0, s>>>(sorted.keys.as<uint64_t>(), nnz, cb,
                                                               col.as<int32_t>());
    }
    BG_LAUNCH_CHECK(ctx, "columns");
    if (N <= kOneWgKeys) {
        (void)hipFuncSetAttribute((const void *)order_one_wg_kernel,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, kOneWgLds);
        DevBuf keys(ctx);
        BG_HIP(ctx, keys.alloc((size_t)N * 8));
        order_one_wg_kernel<<<1, kLdsSortThreads, kOneWgLds, s>>>(deg.as<int32_t>(), N, d_info,
                                                                  keys.as<uint64_t>());
        order_small_kernel<<<N / kLdsSortThreads + 1, kLdsSortThreads, 0, s>>>(
            keys.as<uint64_t>(), N, rules, arrays);
    } else {
        DevBuf a(ctx), b(ctx), hist(ctx), ws(ctx);
        BG_HIP(ctx, a.alloc((size_t)N * 8));
        BG_HIP(ctx, b.alloc((size_t)N * 8));
        BG_HIP(ctx, hist.alloc(sort_hist_words(N) * 4));
        BG_HIP(ctx, ws.alloc(scan_ws_words(sort_hist_words(N)) * 4));
        order_keys_kernel<<<blocks_for(N, 256), 256, 0, s>>>(deg.as<int32_t>(), N,
                                                             a.as<uint64_t>());
        const uint64_t *k = radix_sort(a.as<uint64_t>(), b.as<uint64_t>(), N, 32,
                                       32 + bits_of(info.max_degree), hist.as<uint32_t>(),
                                       ws.as<uint32_t>(), s);
        order_from_keys_kernel<<<blocks_for((int64_t)N + 1, 256), 256, 0, s>>>(k, N, rules, arrays);
        scan_inplace(arrays.sums, N + 1, scan_ws.as<uint32_t>(), s, 3, N + 1);
    }
    BG_LAUNCH_CHECK(ctx, "order");
    sorted.pairs.reset(); // later work on this stream may take the memory
    sorted.keys.reset();

    bitgnn_adj *adj = (bitgnn_adj *)calloc(1, sizeof(bitgnn_adj));
    BG_REQUIRE(ctx, adj, BITGNN_ERR_INVALID_ARG, "bitgnn_adj_build: out of host memory");
    adj->device = ctx->device;
    adj->pool = ctx->pool;
    bg_pool_hold(adj->pool);
    adj->n = N64;
    adj->nnz = nnz;
    adj->max_degree = info.max_degree;
    for (int k = 31; k >= 0; --k)
        adj->n_ge[k] = (k < 31 ? adj->n_ge[k + 1] : 0) + info.bits[k + 1];
    adj->device_bytes = ((size_t)N + 1) * 4 + (size_t)nnz * 4 + (size_t)N * 8;
    adj->rowptr = rowptr.give<uint32_t>(adj);
    adj->col = col.give<int32_t>(adj);
    adj->deg = deg.give<int32_t>(adj);
    adj->order = order.give<int32_t>(adj);
    // dense enough: also build the column-blocked form for the LDS-staged bit-SpMM
    int rc = BITGNN_OK;
    if ((int64_t)nnz >= (int64_t)ctx->min_avg_degree * N64)
        rc = bg_build_blocked(ctx, s, adj,
                              bg_slots{block_rank.as<uint32_t>(), arrays.sums,
                                       arrays.sums + N + 1, info.parts, info.multi});
    // CSR-only and larger than a cache: column ids in degree-order slots.  On a power-law
    // graph a few percent of the nodes take half of all gathers; in a degree-ordered copy of
    // the activations their rows are adjacent and stay in L2.
    if (rc == BITGNN_OK && !adj->blk && nnz > 0 && N >= 65536)
        rc = [&]() -> int {
            DevBuf col_slot(ctx);
            BG_HIP(ctx, col_slot.alloc((size_t)nnz * 4));
            col_slot_kernel<<<blocks_for(nnz, 256), 256, 0, s>>>(
                adj->col, nnz, rank.as<int32_t>(), col_slot.as<int32_t>());
            BG_LAUNCH_CHECK(ctx, "col_slot");
            adj->col_slot = col_slot.give<int32_t>(adj);
            adj->device_bytes += (size_t)nnz * 4;
            return BITGNN_OK;
        }();
    // segments of the long rows for the CSR bit-SpMM
    const int large = (int64_t)nnz >= kSegLargeNnz;
    adj->seg_len = large ? kSegLenLarge : kSegLenSmall;
    adj->n_long = info.n_long[large];
    adj->n_long_segs = adj->n_long ? info.n_segs[large] : 0;
    if (rc == BITGNN_OK && adj->n_long)
        rc = [&]() -> int {
            DevBuf seg_ptr(ctx), seg_slot(ctx);
            BG_HIP(ctx, seg_ptr.alloc(((size_t)adj->n_long + 1) * 4));
            BG_HIP(ctx, seg_slot.alloc((size_t)adj->n_long_segs * 4));
            BG_HIP(ctx, hipMemcpyAsync(seg_ptr.as<void>(), arrays.sums + 2 * ((size_t)N + 1),
                                       ((size_t)adj->n_long + 1) * 4, hipMemcpyDeviceToDevice, s));
            seg_slot_kernel<<<blocks_for(adj->n_long, 256), 256, 0, s>>>(
                seg_ptr.as<uint32_t>(), adj->n_long, seg_slot.as<uint32_t>());
            BG_LAUNCH_CHECK(ctx, "seg_slot");
            adj->seg_slot = seg_slot.give<uint32_t>(adj);
            adj->seg_ptr = seg_ptr.give<uint32_t>(adj);
            adj->device_bytes += ((size_t)N + 1) * 4 + (size_t)adj->n_long_segs * 4;
            return BITGNN_OK;
        }();
    // the aggregation workspace for the default widths: compute calls never allocate
    if (rc == BITGNN_OK)
        rc = bitgnn_ctx_reserve(ctx, bg_adj_workspace_bytes(adj, kDefaultWsChannels,
                                                            kDefaultWsClasses));
    if (rc == BITGNN_OK)
        rc = [&]() -> int {
            BG_HIP(ctx, hipStreamSynchronize(s)); // the temporaries go back
            return BITGNN_OK;
        }();
    if (rc != BITGNN_OK) {
        bitgnn_adj_destroy(adj);
        return rc;
    }
    *out = adj;
    return BITGNN_OK;
}

extern "C" int bitgnn_adj_build(bitgnn_ctx *ctx, void *stream, const int32_t *src,
                                const int32_t *dst, int64_t E, int64_t N, uint32_t flags,
                                bitgnn_adj **out)
{
    if (!ctx)
        return BITGNN_ERR_INVALID_ARG;
    const int rc = adj_build(ctx, (hipStream_t)stream, src, dst, E, N, flags, out);
    // the temporaries are back in the pool: nothing may still run on them, also after an error
    if (ctx->device >= 0 && rc != BITGNN_OK)
        (void)hipStreamSynchronize((hipStream_t)stream);
    return rc;
}

extern "C" int bitgnn_adj_workspace_bytes(const bitgnn_adj *adj, int32_t C_max, int32_t M_max,
                                          size_t *bytes)
{
    if (!adj || !bytes || C_max < 1 || C_max > 2048 || M_max < 1)
        return BITGNN_ERR_INVALID_ARG;
    *bytes = bg_adj_workspace_bytes(adj, C_max, M_max);
    return BITGNN_OK;
}

extern "C" int bitgnn_adj_info(const bitgnn_adj *adj, int64_t *N, int64_t *nnz,
                               int64_t *max_degree, size_t *device_bytes)
{
    if (!adj)
        return BITGNN_ERR_INVALID_ARG;
    if (N)
        *N = adj->n;
    if (nnz)
        *nnz = adj->nnz;
    if (max_degree)
        *max_degree = adj->max_degree;
    if (device_bytes)
        *device_bytes = adj->device_bytes;
    return BITGNN_OK;
}

extern "C" int bitgnn_adj_csr(const bitgnn_adj *adj, const uint32_t **rowptr, const int32_t **col,
                              const int32_t **deg)
{
    if (!adj)
        return BITGNN_ERR_INVALID_ARG;
    if (rowptr)
        *rowptr = adj->rowptr;
    if (col)
        *col = adj->col;
    if (deg)
        *deg = adj->deg;
    return BITGNN_OK;
}

extern "C" int bitgnn_adj_blocked_info(const bitgnn_adj *adj, int64_t *parts, int64_t *slices,
                                       int64_t *workgroups, int64_t *tiles, int64_t *stored_ids,
                                       int64_t *cb_nodes)
{
    if (!adj)
        return BITGNN_ERR_INVALID_ARG;
    const bitgnn_blocked *b = adj->blk;
    if (parts)
        *parts = b ? b->n_vrows : 0;
    if (slices)
        *slices = b ? b->n_slices : 0;
    if (workgroups)
        *workgroups = b ? b->n_wgs : 0;
    if (tiles)
        *tiles = b ? b->n_tiles : 0;
    if (stored_ids)
        *stored_ids = b ? (int64_t)b->n_groups * 64 * kGroupSteps : 0;
    if (cb_nodes)
        *cb_nodes = b ? b->cbn : 0;
    return BITGNN_OK;
}

// Waits for the device, as freeing memory would: the arrays go back to the pool, where another
// build on any stream may take them.  Where waiting is refused (a stream is being recorded) they
// are freed instead.
extern "C" void bitgnn_adj_destroy(bitgnn_adj *adj)
{
    if (!adj)
        return;
    int device = -1;
    (void)hipGetDevice(&device);
    const bool idle = (device == adj->device || hipSetDevice(adj->device) == hipSuccess) &&
                      hipDeviceSynchronize() == hipSuccess;
    for (int i = 0; i < adj->n_owned; ++i) {
        if (idle)
            bg_pool_give(adj->pool, adj->owned[i]);
        else
            (void)hipFree(adj->owned[i].p);
    }
    if (device >= 0 && device != adj->device)
        (void)hipSetDevice(device);
    bg_pool_drop(adj->pool);
    free(adj->blk);
    free(adj);
}
