// Column-blocked, length-balanced form of the adjacency for the LDS-staged
// bit-SpMM (the role of the paper's fine-representing / dynamic-coarsening
// scheme, Section 3.2.1: store the sparse bit matrix finely, coarsen on chip).
//
// Why: a 16-byte activation row gathered from global memory costs a whole
// 128-byte cache line (measured ~0.33 gathers/clock/CU on MI355X), while the
// same gather from LDS runs ~11x faster.  So the activation matrix is cut into
// column blocks of `cbn` nodes that fit the 160 KB LDS, and the adjacency is
// stored so that a workgroup streams, per column block, only 16-bit column ids
// local to the block.
//
// Layout decisions
//  - nodes are renumbered by decreasing degree ("slot"), so that hub columns
//    share the first blocks and rows of similar length sit together;
//  - a row's neighbour list (grouped by column block) is cut into parts of at
//    most `part_len` entries ("virtual rows"): a hub row becomes many parts,
//    each touching one or two column blocks; partial counts are merged later.
//    This bounds the work of one lane, which balances wavefronts on a
//    power-law graph;
//  - parts are ordered by (first block, last block, entries in the first block,
//    entries in the second block), so that the lanes of a tile have similar
//    step counts; 64 consecutive parts form a slice (one wavefront, one part per
//    lane), 16 slices a workgroup.  For every (slice, block) tile the ids are stored lane-
//    interleaved in groups of kGroupSteps steps: group g holds
//    idx16[(g*64+lane)*kGroupSteps+k], padded with ids cbn .. cbn+15, which address
//    all-zero LDS rows.  The groups of a slice are consecutive, so a wavefront
//    reads one contiguous stream; one padding group closes the array so that
//    reading one group ahead is always in bounds.
#include "prims.h"

#include <stdlib.h>

namespace {

constexpr uint32_t kMaxParts = (1u << 30) - 1;

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t o = __shfl_xor(v, d, 64);
        v = o < v ? o : v;
    }
    return v;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t o = __shfl_xor(v, d, 64);
        v = o > v ? o : v;
    }
    return v;
}

// ---------------------------------------------------------------- entries by column block
// Every row's entries in slot order, grouped by column block, as {block << 16 | position inside}:
// a counting sort of each row by a group of WAVES wavefronts.  Inside a block any order serves
// (the tiles choose their own), so one LDS atomic per entry gives its place.  Entries stay in
// registers between counting and placing up to 8 per lane; longer rows are read twice.
// Bound by the gathers of block_rank (one word per entry out of an L2-resident table).
// This took the place of a radix sort of the (row slot, column slot) pairs: 110.6 M entries
// 10.5 ms -> 472 us for the rows of 512 entries and more, 253 us for the others.
template <int WAVES>
__global__ __launch_bounds__(256) void group_rows_kernel(
    const uint32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
    const int32_t *__restrict__ order, bg_slots slots, uint32_t first, uint32_t last, uint32_t ncb,
    uint32_t *__restrict__ entries)
{
    extern __shared__ uint32_t lds[]; // [4 / WAVES][ncb]
    constexpr int kHeld = 8;
    constexpr uint32_t kThreads = 64 * WAVES;
    const uint32_t group = threadIdx.x / kThreads, t = threadIdx.x % kThreads;
    const uint32_t s = first + blockIdx.x * (4 / WAVES) + group;
    uint32_t *count = lds + group * ncb;
    const bool in = s < last;
    const uint32_t row = in ? (uint32_t)order[s] : 0;
    const uint32_t beg = in ? rowptr[row] : 0, d = in ? rowptr[row + 1] - beg : 0;
    const int32_t *c = col + beg;
    uint32_t *out = entries + (in ? slots.entry_ptr[s] : 0);
    auto sync = [] {
        if (WAVES > 1)
            __syncthreads();
        else
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    for (uint32_t b = t; b < ncb; b += kThreads)
        count[b] = 0;
    sync();
    uint32_t v[kHeld], at[kHeld];
#pragma unroll
    for (int k = 0; k < kHeld; ++k)
        v[k] = k * kThreads + t < d ? (uint32_t)c[k * kThreads + t] : 0;
#pragma unroll
    for (int k = 0; k < kHeld; ++k)
        if (k * kThreads < d)
            v[k] = slots.block_rank[v[k]];
#pragma unroll
    for (int k = 0; k < kHeld; ++k)
        if (k * kThreads + t < d)
            at[k] = atomicAdd(&count[v[k] >> 16], 1u);
    if (d > kHeld * kThreads) {
        sync(); // the held entries' places come first in their blocks
        for (uint32_t k = kHeld * kThreads + t; k < d; k += kThreads)
            atomicAdd(&count[slots.block_rank[c[k]] >> 16], 1u);
    }
    sync();
    if (t < 64) { // exclusive prefix of the counts
        uint32_t run = 0;
        for (uint32_t b0 = 0; b0 < ncb; b0 += 64) {
            const uint32_t n = b0 + t < ncb ? count[b0 + t] : 0;
            uint32_t inc = n;
#pragma unroll
            for (int q = 1; q < 64; q <<= 1) {
                const uint32_t o = __shfl_up(inc, q, 64);
                if ((int)t >= q)
                    inc += o;
            }
            if (b0 + t < ncb)
                count[b0 + t] = run + inc - n;
            run += __shfl(inc, 63, 64);
        }
    }
    sync();
#pragma unroll
    for (int k = 0; k < kHeld; ++k)
        if (k * kThreads + t < d)
            out[count[v[k] >> 16] + at[k]] = v[k];
    if (d > kHeld * kThreads) {
        // a held entry's place was taken relative to the block's first: the others follow it
        sync();
#pragma unroll
        for (int k = 0; k < kHeld; ++k)
            atomicAdd(&count[v[k] >> 16], 1u);
        sync();
        for (uint32_t k = kHeld * kThreads + t; k < d; k += kThreads) {
            const uint32_t e = slots.block_rank[c[k]];
            out[atomicAdd(&count[e >> 16], 1u)] = e;
        }
    }
}

// ---------------------------------------------------------------- parts
struct PartArrays {
    uint2 *range;   // [V] by part: its entries {first, one past the last}
    uint32_t *slot; // [V] row slot | bit 31: the row's only part
    uint64_t *key;  // [V] {first block, last block, shape} << 32 | part
};

// first of the entries [a, z) in a block >= `block`
__device__ __forceinline__ uint32_t block_bound(const uint32_t *entries, uint32_t a, uint32_t z,
                                                uint32_t block)
{
    while (a < z) {
        const uint32_t m = (a + z) >> 1;
        if (entries[m] >> 16 < block)
            a = m + 1;
        else
            z = m;
    }
    return a;
}

// part descriptors and their sort keys (blocks take `nb` bits)
__global__ void parts_kernel(const uint32_t *__restrict__ entries, bg_slots slots, int nb,
                             PartArrays p)
{
    const uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= slots.parts)
        return;
    // the rows with several parts come first; behind them there is one part a row
    const uint32_t lead = slots.part_ptr[slots.multi];
    uint32_t s = slots.multi + (v - lead), part = 0, np = 1;
    if (v < lead) {
        uint32_t a = 0, z = slots.multi; // last slot with part_ptr <= v
        while (z - a > 1) {
            const uint32_t m = (a + z) >> 1;
            if (slots.part_ptr[m] <= v)
                a = m;
            else
                z = m;
        }
        s = a;
        part = v - slots.part_ptr[s];
        np = slots.part_ptr[s + 1] - slots.part_ptr[s];
    }
    const uint32_t r0 = slots.entry_ptr[s], d = slots.entry_ptr[s + 1] - r0;
    const uint32_t plen = (d + np - 1) / np;
    const uint32_t b = r0 + min(d, part * plen), e = r0 + min(d, (part + 1) * plen);
    const uint32_t lo = e > b ? entries[b] >> 16 : 0, hi = e > b ? entries[e - 1] >> 16 : 0;
    p.range[v] = make_uint2(b, e);
    p.slot[v] = s | (np == 1 ? 0x80000000u : 0u);
    // Entries in the part's first two blocks (its heaviest: columns are in degree
    // order).  The parts of a slice share their tiles' step counts (the longest lane's),
    // so within a block range they are ordered by these two counts rather than by
    // length: on a Reddit-shaped graph 12 % fewer stored ids than ordering by length.
    const uint32_t e0 = block_bound(entries, b, e, lo + 1);
    const uint32_t e1 = block_bound(entries, e0, e, lo + 2);
    const uint32_t c0 = e0 - b, c1 = e1 - e0;
    const uint32_t shape = ((31u - min(c0 >> 3, 31u)) << 5) | (31u - min(c1 >> 2, 31u));
    const uint64_t order = ((((uint64_t)lo << nb) | hi) << 10) | shape; // at most 34 bits
    p.key[v] = (order << 30) | v;
}

// per slice: range of column blocks its parts touch
__global__ __launch_bounds__(256) void slice_range_kernel(const uint64_t *__restrict__ keys,
                                                          uint32_t V, uint32_t S, int nb,
                                                          uint32_t *__restrict__ sl_cb,
                                                          uint32_t *__restrict__ sl_ntiles)
{
    const uint32_t slice = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (slice >= S) { // scan terminator
        if (slice == S && lane == 0)
            sl_ntiles[S] = 0;
        return;
    }
    const uint32_t pos = slice * 64 + lane;
    const bool valid = pos < V;
    const uint64_t blocks = valid ? keys[pos] >> 40 : 0;
    const uint32_t mask = (1u << nb) - 1;
    const uint32_t lo = wave_min_u32(valid ? (uint32_t)(blocks >> nb) : 0xFFFFu);
    const uint32_t hi = wave_max_u32((uint32_t)blocks & mask);
    if (lane == 0) {
        sl_cb[slice] = lo | (hi << 16);
        sl_ntiles[slice] = hi - lo + 1;
    }
}

// ---------------------------------------------------------------- tiles
// The ids of a slice's parts come into LDS in whole lines, a part per wavefront at a time,
// together with the first entry of every (part, column block) of a window of 64 blocks; the
// tiles of the window are then counted or filled by the wavefronts in turn.  With the lanes
// walking their parts in global memory instead, one 8-byte key at a time, counting 160 M
// stored ids took 1,556 us; 140 so.
constexpr uint32_t kTileWindow = 64;
constexpr uint32_t kBoundStride = kTileWindow + 2; // 16-bit words, 33 banks apart

struct SliceArrays {
    const uint64_t *keys; // sorted part keys
    const uint2 *range;
    const uint32_t *entries;
    const uint32_t *sl_cb;
    const uint32_t *tile_base;
    uint32_t V;
};

__host__ __device__ constexpr uint32_t round_up_16(uint32_t n) { return (n + 15u) & ~15u; }

// A vote among the 16 lanes of one of a wavefront's four teams.
__device__ __forceinline__ uint32_t team_vote(bool v, uint32_t team)
{
    return (uint32_t)(__ballot(v) >> (team * 16)) & 0xFFFFu;
}

// Loads the bounds of the blocks [w0, w0 + nb) and, with IDS, the positions inside the blocks.
template <bool IDS>
__device__ __forceinline__ void load_slice(const SliceArrays &a, const uint2 *part, uint32_t w0,
                                           uint32_t nb, uint32_t id_stride, uint16_t *bound,
                                           uint16_t *ids)
{
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    constexpr int kAhead = 4; // 256 entries: a whole part of the default length
    uint32_t next[kAhead];
    auto request = [&](uint32_t p) {
        const uint2 r = part[p];
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
            next[k] = r.x + k * 64 + lane < r.y ? a.entries[r.x + k * 64 + lane] : ~0u;
    };
    request(wave);
    for (uint32_t p = wave; p < 64; p += waves) {
        uint32_t v[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
            v[k] = next[k];
        if (p + waves < 64)
            request(p + waves);
        const uint2 r = part[p];
        const uint32_t len = r.y - r.x;
        uint16_t *bp = bound + p * kBoundStride;
        uint32_t before = w0; // blocks of the window up to here have their bound
        for (uint32_t k0 = 0; k0 <= len; k0 += 64) { // one place past the end closes the last block
            const uint32_t k = k0 + lane;
            uint32_t e = ~0u;
#pragma unroll
            for (int q = 0; q < kAhead; ++q)
                if (k0 == q * 64u)
                    e = v[q];
            if (k0 >= kAhead * 64u && k < len)
                e = a.entries[r.x + k];
            const uint32_t block = e >> 16; // past the end: 65,535
            uint32_t from = __shfl_up(block, 1, 64);
            from = lane == 0 ? before : max(from + 1, w0);
            // entries of a part are in block order: bounds of the blocks behind the previous entry's
            const uint32_t to = min(block + 1, w0 + nb + 1);
            for (uint32_t b = from; b < to; ++b)
                bp[b - w0] = (uint16_t)min(k, len);
            before = max(before, min(__shfl(block, 63, 64) + 1, w0 + nb + 1));
            if (IDS && k < len)
                ids[p * id_stride + k] = (uint16_t)e;
        }
    }
    __syncthreads();
}

// steps of every (slice, block) tile = its longest lane; in groups
__global__ __launch_bounds__(256) void tile_count_kernel(SliceArrays a,
                                                         uint32_t *__restrict__ tile_group)
{
    __shared__ uint2 part[64];
    __shared__ uint16_t bound[64 * kBoundStride];
    const uint32_t slice = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t lo = a.sl_cb[slice] & 0xFFFFu, hi = a.sl_cb[slice] >> 16;
    if (threadIdx.x < 64) {
        const uint32_t pos = slice * 64 + lane;
        part[lane] = pos < a.V ? a.range[(uint32_t)a.keys[pos] & kMaxParts] : make_uint2(0, 0);
    }
    __syncthreads();
    for (uint32_t w0 = lo; w0 <= hi; w0 += kTileWindow) {
        const uint32_t nb = min(kTileWindow, hi + 1 - w0);
        load_slice<false>(a, part, w0, nb, 0, bound, nullptr);
        const uint16_t *b = bound + lane * kBoundStride;
        for (uint32_t t = wave; t < nb; t += 4) {
            const uint32_t m = wave_max_u32((uint32_t)b[t + 1] - b[t]);
            if (lane == 0)
                tile_group[a.tile_base[slice] + w0 - lo + t] = (m + kGroupSteps - 1) / kGroupSteps;
        }
        __syncthreads();
    }
}

// Writes the lane-interleaved ids.
//
// Order of a lane's ids inside a tile (free: the sum does not depend on it).  The LDS
// serves a 16-byte gather of 16 consecutive lanes in one pass when the 16 rows fall into
// different 16-byte bank groups, i.e. differ in (row mod 16).  So lane L wants, at step k,
// a row of class (L + k) mod 16: an id goes to the first free step of its class, ids whose
// class has no step left take any free step, and padding steps address the all-zero row
// of the wanted class (rows cbn .. cbn + 15 of the staged block are zero).
//
// A team of 16 lanes places the ids of one (part, tile), 16 at a time: votes give an id its
// number inside its class and with it its step; the ids left over wait in LDS and are dealt out
// to the free steps, in order, when all have been placed.  A team takes a fixed ~100 instructions
// per 16 ids; one lane per part, the form before, ~60 per id and more where the search for free
// steps diverged: 160 M stored ids 5,597 -> 800 us.
constexpr int kFillThreads = 512;

__global__ __launch_bounds__(kFillThreads) void tile_fill_kernel(
    SliceArrays a, uint32_t cbn, uint32_t part_len, uint32_t id_stride,
    const uint32_t *__restrict__ tile_group, uint16_t *__restrict__ idx16)
{
    extern __shared__ uint64_t lds64[];
    __shared__ uint2 part[64];
    __shared__ uint16_t bound[64 * kBoundStride];
    // [64][id_stride] ids, then per team the steps and the ids left over
    uint16_t *ids = (uint16_t *)lds64;
    const uint32_t team_words = 2 * round_up_16(part_len);
    const uint32_t slice = blockIdx.x, lane = threadIdx.x & 63;
    const uint32_t q = threadIdx.x & 15, team = (threadIdx.x >> 4) & 3, wave = threadIdx.x >> 6;
    uint16_t *step_id = ids + 64 * id_stride + (threadIdx.x >> 4) * team_words;
    uint16_t *left = step_id + round_up_16(part_len);
    const uint32_t lo = a.sl_cb[slice] & 0xFFFFu, hi = a.sl_cb[slice] >> 16;
    if (threadIdx.x < 64) {
        const uint32_t pos = slice * 64 + lane;
        part[lane] = pos < a.V ? a.range[(uint32_t)a.keys[pos] & kMaxParts] : make_uint2(0, 0);
    }
    __syncthreads();
    for (uint32_t w0 = lo; w0 <= hi; w0 += kTileWindow) {
        const uint32_t nb = min(kTileWindow, hi + 1 - w0);
        load_slice<true>(a, part, w0, nb, id_stride, bound, ids);
        for (uint32_t job = wave; job < nb * 16; job += blockDim.x >> 6) {
            const uint32_t t = job >> 4, L = (job & 15) * 4 + team;
            const uint32_t tile = a.tile_base[slice] + w0 - lo + t;
            const uint32_t g0 = tile_group[tile], g1 = tile_group[tile + 1];
            const uint32_t steps = (g1 - g0) * kGroupSteps;
            const uint32_t first = bound[L * kBoundStride + t];
            const uint32_t cnt = bound[L * kBoundStride + t + 1] - first;
            const uint16_t *src = ids + L * id_stride + first;
            for (uint32_t k = q; k < steps; k += 16)
                step_id[k] = 0xFFFFu;
            wave_lds_order();
            uint32_t seen = 0, n_left = 0; // ids of class q so far; ids left over
            for (uint32_t i0 = 0; __any(i0 < cnt); i0 += 16) {
                const bool in = i0 + q < cnt;
                const uint32_t id = in ? src[i0 + q] : 0;
                const uint32_t c = (id - L) & 15u; // steps c, c + 16, ... are of the id's class
                uint32_t same = team_vote(in, team), class_q = same;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const uint32_t m = team_vote((c >> b) & 1u, team);
                    same &= (c >> b) & 1u ? m : ~m;
                    class_q &= (q >> b) & 1u ? m : ~m;
                }
                const uint32_t before = (1u << q) - 1;
                const uint32_t number = __shfl(seen, (int)(team * 16 + c), 64) +
                                        (uint32_t)__popc(same & before);
                seen += (uint32_t)__popc(class_q);
                const uint32_t k = c + 16 * number;
                const uint32_t over = team_vote(in && k >= steps, team);
                if (in && k < steps)
                    step_id[k] = (uint16_t)id;
                else if (in)
                    left[n_left + (uint32_t)__popc(over & before)] = (uint16_t)id;
                n_left += (uint32_t)__popc(over);
            }
            wave_lds_order();
            uint32_t taken = 0;
            for (uint32_t k0 = 0; k0 < steps; k0 += 16) {
                const uint32_t k = k0 + q; // steps is a multiple of 8
                const bool open = k < steps && step_id[k] == 0xFFFFu;
                const uint32_t m = team_vote(open, team);
                const uint32_t f = taken + (uint32_t)__popc(m & ((1u << q) - 1));
                if (open)
                    step_id[k] = f < n_left ? left[f] : (uint16_t)(cbn + ((L + k) & 15u));
                taken += (uint32_t)__popc(m);
            }
            wave_lds_order();
            for (uint32_t k = q * 8; k < steps; k += 128) {
                uint4 v;
                __builtin_memcpy(&v, __builtin_assume_aligned(step_id + k, 16), 16);
                uint16_t *out = idx16 + ((uint64_t)(g0 + k / kGroupSteps) * 64 + L) * kGroupSteps +
                                k % kGroupSteps;
                __builtin_memcpy(__builtin_assume_aligned(out, 16), &v, 16);
            }
            wave_lds_order();
        }
        __syncthreads();
    }
}

// the padding group behind the last tile
__global__ void tail_group_kernel(uint16_t *__restrict__ idx16, uint32_t G, int cbn)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 64u * kGroupSteps)
        idx16[(uint64_t)G * 64 * kGroupSteps + i] = (uint16_t)cbn;
}

// per processing position: {part id (row-major: the parts of a row are consecutive ids)
// | bit 31 if it is the row's only part, node id of the row}
__global__ void part_info_kernel(const uint64_t *__restrict__ svkeys, uint32_t V,
                                 const uint32_t *__restrict__ v_slot,
                                 const int32_t *__restrict__ order, uint2 *__restrict__ part_info)
{
    const uint32_t pos = blockIdx.x * blockDim.x + threadIdx.x;
    if (pos < V) {
        const uint32_t v = (uint32_t)svkeys[pos] & kMaxParts;
        const uint32_t sl = v_slot[v];
        part_info[pos] = make_uint2(v | (sl & 0x80000000u), (uint32_t)order[sl & 0x7FFFFFFFu]);
    }
}

// Sort key of a workgroup: estimated time, complemented so that an ascending sort lists
// the heaviest first.  The wavefronts of a workgroup meet at every column block, so a
// block costs its refill plus the longest tile among the slices (measured on MI355X:
// about 1.56 us per refill of 8192 rows, 0.51 us per group of 8 steps on the critical
// path, 10 us per work item); the unit below is 10 ns.  One wavefront a workgroup.
__global__ __launch_bounds__(256) void wg_cost_kernel(const uint32_t *__restrict__ sl_cb,
                                                      const uint32_t *__restrict__ sl_tile_base,
                                                      const uint32_t *__restrict__ tile_group,
                                                      uint32_t S, uint32_t W, uint32_t spw, int cbn,
                                                      uint32_t tiles, uint32_t *__restrict__ wg_cb,
                                                      uint64_t *__restrict__ keys,
                                                      uint32_t *__restrict__ mail)
{
    const uint32_t w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (blockIdx.x == 0 && threadIdx.x == 0) { // what the host waits for
        mail[0] = sl_tile_base[S];
        mail[1] = tile_group[tiles];
    }
    if (w >= W)
        return;
    const uint32_t s0 = w * spw, s1 = min(s0 + spw, S);
    uint32_t wlo = 0xFFFFu, whi = 0;
    for (uint32_t sl = s0; sl < s1; ++sl) {
        wlo = min(wlo, sl_cb[sl] & 0xFFFFu);
        whi = max(whi, sl_cb[sl] >> 16);
    }
    uint32_t crit = 0; // groups: at most 2^22 (G has 32-bit byte offsets)
    for (uint32_t cb = wlo + lane; cb <= whi; cb += 64) {
        uint32_t longest = 0;
        for (uint32_t sl = s0; sl < s1; ++sl) {
            const uint32_t lo = sl_cb[sl] & 0xFFFFu, hi = sl_cb[sl] >> 16;
            if (cb >= lo && cb <= hi) {
                const uint32_t t = sl_tile_base[sl] + cb - lo;
                longest = max(longest, tile_group[t + 1] - tile_group[t]);
            }
        }
        crit += longest;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
        crit += __shfl_xor(crit, d, 64);
    const uint64_t fills = whi - wlo + 1;
    const uint64_t cost =
        (uint64_t)crit * (51 * kGroupSteps / 8) + fills * (156ull * cbn / 8192) + 1000;
    if (lane == 0) {
        wg_cb[w] = wlo | (whi << 16);
        keys[w] = ((0xFFFFFFFFull - min(cost, (uint64_t)0xFFFFFFFFull)) << 32) | w;
    }
}

// What the aggregation kernel reads at its start, flattened so that it takes two
// dependent loads instead of five: per dispatch position {workgroup, its block range},
// per slice {its block range, first tile, first group}.
__global__ void wg_item_kernel(const uint64_t *__restrict__ keys, uint32_t W,
                               const uint32_t *__restrict__ wg_cb, uint2 *__restrict__ wg_item)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < W) {
        const uint32_t w = (uint32_t)keys[i];
        wg_item[i] = make_uint2(w, wg_cb[w]);
    }
}

__global__ void slice_desc_kernel(const uint32_t *__restrict__ sl_cb,
                                  const uint32_t *__restrict__ sl_tile_base,
                                  const uint32_t *__restrict__ tile_group, uint32_t S,
                                  uint4 *__restrict__ sl_desc)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < S)
        sl_desc[i] = make_uint4(sl_cb[i], sl_tile_base[i], tile_group[sl_tile_base[i]], 0u);
}

} // namespace

// Builds adj->blk from the CSR arrays of `adj` and its degree order (already on the device).
int bg_build_blocked(bitgnn_ctx *ctx, hipStream_t s, bitgnn_adj *adj, const bg_slots &slots)
{
    const uint32_t n = (uint32_t)adj->n, nnz = (uint32_t)adj->nnz, V = slots.parts;
    const int cbn = ctx->cb_nodes, part_len = ctx->part_len;
    const int64_t ncb = (adj->n + cbn - 1) / cbn;
    if (ncb > 4095 || nnz == 0 || cbn > kMaxCbNodes || V >= kMaxParts)
        return BITGNN_OK; // stays on the CSR path

    // entries by column block: rows of more than 8 entries a lane of one wavefront come first
    DevBuf entries(ctx);
    BG_HIP(ctx, entries.alloc((size_t)nnz * 4));
    const uint32_t n_wide = adj->n_ge[9]; // rows of 512 entries and more
    if (n_wide > 0)
        group_rows_kernel<4><<<n_wide, 256, (size_t)ncb * 4, s>>>(
            adj->rowptr, adj->col, adj->order, slots, 0, n_wide, (uint32_t)ncb,
            entries.as<uint32_t>());
    if (n > n_wide)
        group_rows_kernel<1><<<blocks_for(n - n_wide, 4), 256, (size_t)ncb * 16, s>>>(
            adj->rowptr, adj->col, adj->order, slots, n_wide, n, (uint32_t)ncb,
            entries.as<uint32_t>());
    BG_LAUNCH_CHECK(ctx, "group_rows");

    // parts, sorted by (first block, last block, shape)
    const int nb = bits_of((uint32_t)ncb - 1);
    const uint32_t S = (V + 63) / 64;
    // work items of 16 slices, or of 8 or 4 on graphs with too few slices to give every
    // compute unit an item of 16 (measured on the 131 K-node R-MAT graph: 126 us per
    // aggregation with 135 items of 16 slices, 107 us with 270 items of 8)
    uint32_t spw = kSlicesPerWg;
    const uint32_t want = (uint32_t)(ctx->n_cus > 0 ? ctx->n_cus : 256);
    while (spw > 4 && (S + spw - 1) / spw < want)
        spw /= 2;
    const uint32_t W = (S + spw - 1) / spw;
    DevBuf range(ctx), v_slot(ctx), vk_a(ctx), vk_b(ctx), hist(ctx), scan_ws(ctx);
    BG_HIP(ctx, range.alloc((size_t)V * 8));
    BG_HIP(ctx, v_slot.alloc((size_t)V * 4));
    BG_HIP(ctx, vk_a.alloc((size_t)V * 8));
    BG_HIP(ctx, vk_b.alloc((size_t)V * 8));
    BG_HIP(ctx, hist.alloc(sort_hist_words(V) * 4)); // W <= V
    const size_t scans = sort_hist_words(V) > (size_t)S + 1 ? sort_hist_words(V) : (size_t)S + 1;
    BG_HIP(ctx, scan_ws.alloc(scan_ws_words(scans) * 4));
    (void)hipFuncSetAttribute((const void *)one_wg_sort_kernel,
                              hipFuncAttributeMaxDynamicSharedMemorySize, kOneWgLds);
    auto sort = [&](uint64_t *a, uint64_t *b, uint32_t count, int lo, int hi) -> uint64_t * {
        if (count > kOneWgKeys)
            return radix_sort(a, b, count, lo, hi, hist.as<uint32_t>(), scan_ws.as<uint32_t>(), s);
        one_wg_sort_kernel<<<1, kLdsSortThreads, kOneWgLds, s>>>(a, count, lo, hi);
        return a;
    };
    parts_kernel<<<blocks_for(V, 256), 256, 0, s>>>(
        entries.as<uint32_t>(), slots, nb,
        PartArrays{range.as<uint2>(), v_slot.as<uint32_t>(), vk_a.as<uint64_t>()});
    BG_LAUNCH_CHECK(ctx, "parts");
    const uint64_t *svkeys =
        sort(vk_a.as<uint64_t>(), vk_b.as<uint64_t>(), V, 30, 40 + 2 * nb);

    // Tiles.  Their number is known to the device alone; where every slice spanning every block
    // is no great waste of memory, that bound is used instead of waiting for it.
    DevBuf sl_cb(ctx), sl_tile_base(ctx), wg_cb(ctx), part_info(ctx);
    BG_HIP(ctx, sl_cb.alloc((size_t)S * 4));
    BG_HIP(ctx, sl_tile_base.alloc(((size_t)S + 1) * 4));
    BG_HIP(ctx, wg_cb.alloc((size_t)W * 4));
    BG_HIP(ctx, part_info.alloc((size_t)V * 8));
    slice_range_kernel<<<blocks_for((int64_t)S + 1, 4), 256, 0, s>>>(
        svkeys, V, S, nb, sl_cb.as<uint32_t>(), sl_tile_base.as<uint32_t>());
    scan_inplace(sl_tile_base.as<uint32_t>(), S + 1, scan_ws.as<uint32_t>(), s);
    uint32_t T = 0;
    uint64_t tiles = (uint64_t)S * ncb;
    if (tiles > (1u << 20)) {
        BG_HIP(ctx, hipMemcpyAsync(&T, sl_tile_base.as<uint32_t>() + S, 4, hipMemcpyDeviceToHost, s));
        BG_HIP(ctx, hipStreamSynchronize(s));
        tiles = T;
    }
    DevBuf tile_group(ctx), tile_scan_ws(ctx);
    BG_HIP(ctx, tile_group.alloc((tiles + 1) * 4));
    BG_HIP(ctx, tile_scan_ws.alloc(scan_ws_words(tiles + 1) * 4));
    BG_HIP(ctx, hipMemsetAsync(tile_group.as<uint32_t>() + T, 0, (tiles + 1 - T) * 4, s));
    const SliceArrays slice{svkeys, range.as<uint2>(), entries.as<uint32_t>(),
                            sl_cb.as<uint32_t>(), sl_tile_base.as<uint32_t>(), V};
    tile_count_kernel<<<S, 256, 0, s>>>(slice, tile_group.as<uint32_t>());
    BG_LAUNCH_CHECK(ctx, "tile count");
    // behind the last tile the counts are 0, so entry T (and every one behind it) is the total
    scan_inplace(tile_group.as<uint32_t>(), (uint32_t)tiles + 1, tile_scan_ws.as<uint32_t>(), s);
    volatile uint32_t *mail = (volatile uint32_t *)ctx->mail; // {tiles, groups}
    // meanwhile: dispatch order, heaviest workgroups first, and the descriptors
    DevBuf wg_item(ctx), sl_desc(ctx), wk_a(ctx), wk_b(ctx);
    BG_HIP(ctx, wg_item.alloc((size_t)W * 8));
    BG_HIP(ctx, sl_desc.alloc((size_t)S * 16));
    BG_HIP(ctx, wk_a.alloc((size_t)W * 8));
    BG_HIP(ctx, wk_b.alloc((size_t)W * 8));
    wg_cost_kernel<<<blocks_for(W, 4), 256, 0, s>>>(
        sl_cb.as<uint32_t>(), sl_tile_base.as<uint32_t>(), tile_group.as<uint32_t>(), S, W, spw,
        cbn, (uint32_t)tiles, wg_cb.as<uint32_t>(), wk_a.as<uint64_t>(), (uint32_t *)ctx->mail);
    const uint64_t *wsorted = sort(wk_a.as<uint64_t>(), wk_b.as<uint64_t>(), W, 32, 64);
    wg_item_kernel<<<blocks_for(W, 256), 256, 0, s>>>(wsorted, W, wg_cb.as<uint32_t>(),
                                                     wg_item.as<uint2>());
    slice_desc_kernel<<<blocks_for(S, 256), 256, 0, s>>>(sl_cb.as<uint32_t>(),
                                                        sl_tile_base.as<uint32_t>(),
                                                        tile_group.as<uint32_t>(), S,
                                                        sl_desc.as<uint4>());
    part_info_kernel<<<blocks_for(V, 256), 256, 0, s>>>(svkeys, V, v_slot.as<uint32_t>(),
                                                       adj->order, part_info.as<uint2>());
    BG_LAUNCH_CHECK(ctx, "wg_item / slice_desc");
    BG_HIP(ctx, hipStreamSynchronize(s));
    T = mail[0];
    const uint32_t G = mail[1];
    constexpr uint64_t kGroupIds = 64ull * kGroupSteps;
    if (((uint64_t)G + 1) * kGroupIds * 2 >= (1ull << 32)) // the kernel uses 32-bit byte offsets
        return BITGNN_OK;
    // Many column blocks with few neighbours each pad the tiles heavily: beyond 6 stored
    // ids per non-zero the plain CSR kernel is the better choice (a threshold of 0 stored
    // non-zeros per node forces the blocked form whatever the padding).
    if (ctx->min_avg_degree > 0 && (uint64_t)G * kGroupIds > 6ull * nnz)
        return BITGNN_OK;

    DevBuf idx16(ctx), row_vptr(ctx);
    BG_HIP(ctx, idx16.alloc(((size_t)G + 1) * kGroupIds * 2));
    BG_HIP(ctx, row_vptr.alloc(((size_t)n + 1) * 4));
    BG_HIP(ctx, hipMemcpyAsync(row_vptr.as<void>(), slots.part_ptr, ((size_t)n + 1) * 4,
                               hipMemcpyDeviceToDevice, s));
    tail_group_kernel<<<blocks_for((int64_t)kGroupIds, 256), 256, 0, s>>>(idx16.as<uint16_t>(), G,
                                                                         cbn);
    // 16-bit words between two parts in LDS: an odd number of 32-bit words.  Long parts leave room
    // for fewer wavefronts (1,023 entries: 140 KB of ids and bounds, 16 KB a wavefront).
    const uint32_t id_stride = (((uint32_t)part_len + 1) / 2 | 1u) * 2;
    const size_t ids_lds = (size_t)64 * id_stride * 2;
    const size_t wave_lds = (size_t)4 * 2 * round_up_16((uint32_t)part_len) * 2;
    int waves = kFillThreads / 64;
    while (waves > 1 && ids_lds + waves * wave_lds + 9216 > (size_t)160 * 1024)
        waves /= 2;
    const size_t fill_lds = ids_lds + waves * wave_lds;
    (void)hipFuncSetAttribute((const void *)tile_fill_kernel,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)fill_lds);
    tile_fill_kernel<<<S, 64 * waves, fill_lds, s>>>(slice, (uint32_t)cbn, (uint32_t)part_len,
                                                     id_stride, tile_group.as<uint32_t>(),
                                                     idx16.as<uint16_t>());
    BG_LAUNCH_CHECK(ctx, "tile fill");

    bitgnn_blocked *b = (bitgnn_blocked *)calloc(1, sizeof(bitgnn_blocked));
    BG_REQUIRE(ctx, b, BITGNN_ERR_INVALID_ARG, "bitgnn_adj_build: out of host memory");
    b->cbn = cbn;
    b->n_multi = slots.multi;
    b->ncb = (int32_t)ncb;
    b->part_len = part_len;
    b->forced = ctx->min_avg_degree == 0;
    b->n_vrows = V;
    b->n_slices = S;
    b->spw = (int32_t)spw;
    b->n_wgs = W;
    b->n_tiles = T;
    b->n_groups = G;
    b->device_bytes = ((size_t)G + 1) * kGroupIds * 2 + ((size_t)T + 1) * 4 + (size_t)S * 16 +
                      (size_t)W * 8 + ((size_t)n + 1) * 4 + (size_t)V * 8;
    b->wg_item = wg_item.give<uint2>(adj);
    b->sl_desc = sl_desc.give<uint4>(adj);
    b->tile_group = tile_group.give<uint32_t>(adj);
    b->idx16 = idx16.give<uint16_t>(adj);
    b->row_vptr = row_vptr.give<uint32_t>(adj);
    b->part_info = part_info.give<uint2>(adj);
    adj->blk = b;
    adj->device_bytes += b->device_bytes;
    return BITGNN_OK;
}
