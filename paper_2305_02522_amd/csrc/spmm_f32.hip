// Weighted / full-precision aggregation: the BSpMM variants of Section 3.1.1 whose
// activation operand or output is full precision, and the weighted adjacency written as
// the 0/1 matrix times its factorisation vectors,
//   Y[i][c] = r[i] * sum_{j in N(i)} f[j] * x[j][c],
// with x in float or as packed +-1 bits, and Y stored as float or binarized again.
// D^-1/2 A D^-1/2 is r = f = deg^-1/2, the mean aggregator r = 1/deg.
//
// Arithmetic: fp32, one rounded multiply and one rounded add per neighbour in the stored
// (ascending column) order, then one multiply by r[i]; no fused multiply-add, no
// re-association.  A value is therefore reproducible bit for bit, which matters where it
// decides an output bit.
//
// Two forms:
//  * teams: 16 lanes walk one row for a window of 16 V channels, V per lane, so a gather
//    instruction serves four rows.  A team's 16 lanes hold the ids (as byte offsets) and
//    factors of 16 neighbours and hand them out with DPP row broadcasts, which the address
//    add and the multiply take as an operand: no scalar work per neighbour.
//  * hubs: the sum of a row has a fixed order, so its adds are a serial chain, and on a
//    power-law graph the longest row's chain is longer than everything else together.  Hub
//    rows get a workgroup per 64 channels in which seven wavefronts gather and multiply (that
//    has no order) and leave the products in LDS, and one wavefront does nothing but read and
//    add them.  choose_plan() prices which rows are hubs.
#include "common.h"

#include <cmath>
#include <type_traits>

namespace {

constexpr int kSpBlock = 256;          // threads of a workgroup; of a launch with hubs:
constexpr int kHubBlock = 512;
constexpr int kTeam = 16;              // lanes of a team: one DPP row
constexpr int kHubProd = 7;            // producer wavefronts of a hub workgroup
constexpr int kHubPer = 16;            // neighbours a producer takes per stage (4 per team)
constexpr int kHubStage = kHubProd * kHubPer;
constexpr uint32_t kFactorAt = 60;     // where a 64-byte row of bytes holds its factor
constexpr size_t kHubLds = 2ull * kHubStage * 64 * sizeof(float); // two stages of products

// One rounded multiply, one rounded add: contraction is off, so the pair is never fused.
__device__ __forceinline__ float mul_rounded(float a, float b)
{
#pragma clang fp contract(off)
    return a * b;
}
__device__ __forceinline__ float add_rounded(float a, float b)
{
#pragma clang fp contract(off)
    return a + b;
}

// Lane K of the caller's row of 16 lanes, to all 16 of them.
template <int K> __device__ __forceinline__ uint32_t row_bcast(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + K, 0xF, 0xF, true);
}
template <int K> __device__ __forceinline__ float row_bcast_f(float v)
{
    return __int_as_float((int)row_bcast<K>((uint32_t)__float_as_int(v)));
}

template <int I> struct const_int {
    static constexpr int value = I;
};
template <int B, int E, class F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (B < E) {
        f(const_int<B>{});
        static_for<B + 1, E>(f);
    }
}

// V consecutive values of a row of x as a lane loads them.
// XKIND: 0 float rows, 1 packed +-1 rows, 2 int16 rows with a per-channel scale (the raw
// integers of a BMM and its SCL: the value alpha_c * (float)z is formed here, with the same
// single rounding as the BMM's own scale epilogue, from half the gathered bytes), 3 the same in
// bytes (z / 2 + 128: the integers of a product of even length are even), 4 byte rows of 64 bytes
// whose last four are the row's factor
template <int XKIND, int V> struct x_piece;
template <int V> struct x_piece<0, V> {
    float v[V];
};
template <int V> struct x_piece<1, V> {
    uint32_t v;
};
template <int V> struct x_piece<2, V> {
    int16_t v[V];
};

template <int V> struct x_piece<3, V> {
    uint32_t v; // V <= 4
};
template <int V> struct x_piece<4, V> : x_piece<3, V> {};

// alpha * z, rounded once, for the integer z in the low or high half of `h`: the half is converted
// on the way in.  (-0 is what leaves every product, and the sign of a zero, as it is.)
template <int HI> __device__ __forceinline__ float mul_half(float alpha, uint32_t h)
{
    float p;
    if (HI)
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,1,0] op_sel_hi:[0,1,0]"
            : "=v"(p)
            : "v"(alpha), "v"(h), "s"(0x80000000u));
    else
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[0,1,0]"
            : "=v"(p)
            : "v"(alpha), "v"(h), "s"(0x80000000u));
    return p;
}
// Bytes 2 HI and 2 HI + 1 of a word as a pair of halves holding z = 2 (byte - 128): behind 0x64 a
// byte is the half 1024 + byte.
template <int HI> __device__ __forceinline__ uint32_t even_pair(uint32_t w)
{
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    const uint32_t biased =
        __builtin_amdgcn_perm(0x64646464u, w, HI ? 0x04030402u : 0x04010400u);
    const h2 z = __builtin_elementwise_fma(__builtin_bit_cast(h2, biased), (h2)(_Float16)2,
                                           (h2)(_Float16)-2304);
    return __builtin_bit_cast(uint32_t, z);
}

struct SpmmArgs {
    const uint32_t *rowptr;
    const int32_t *col;
    const int32_t *order;
    const void *x;
    int64_t row_bytes; // bytes from one row of x to the next
    const float *xscale;
    int32_t C;
    const float *r, *f, *tau;
    void *out;
    int64_t ldo;
    uint32_t n_hub;       // rows (the first of the degree order) that take the hub form
    uint32_t hub_tiles;   // 64-channel tiles of a hub row
    uint32_t slot0, slot_end; // rows of the teams, in degree order
    uint32_t windows;      // channel windows of a row
    uint32_t group;        // windows of a row that are taken side by side
    uint32_t group_blocks; // workgroups per group of windows
    // byte rows: where *wide is set some value has no byte, and these int16 rows are taken
    const uint32_t *wide;
    const void *x16;
    int64_t row_bytes16;
};

// The sign a packed bit gives f: bit set -> +f, clear -> -f.  `inv` holds the inverted bit at
// position 31 - sh.
__device__ __forceinline__ float signed_f(uint32_t inv, uint32_t sh, float f)
{
    return __int_as_float((int)(((inv << sh) & 0x80000000u) ^ (uint32_t)__float_as_int(f)));
}

// What a lane reads of a row of x: V channels, nominally from c on.  At the end of a float or
// integer row the lane is moved back to end with the row (it then shares channels with its
// neighbour lane, which computes the same values); of a packed row it reads the 32-bit word
// that holds its V bits.
template <int XKIND, int V> struct x_lane {
    int32_t cs;       // first channel read
    uint32_t off;     // byte offset in the row
    uint32_t bsh;     // packed rows: bit position of channel c in the word
    static __device__ __forceinline__ int32_t first(const SpmmArgs &a, int32_t c)
    {
        return XKIND == 1 ? c : (c < a.C - V ? c : a.C - V);
    }
    __device__ __forceinline__ x_lane(const SpmmArgs &a, int32_t c) : cs(first(a, c)), bsh(0)
    {
        if (XKIND == 1) {
            const int32_t dw = c >> 5, last = 2 * ((a.C + 63) / 64) - 1;
            off = (uint32_t)(dw < last ? dw : last) * 4u;
            bsh = (uint32_t)(c & 31);
        } else {
            off = (uint32_t)cs * (XKIND == 2 ? 2u : XKIND >= 3 ? 1u : 4u);
            if (XKIND == 4 && c == 15 * V)
                off = kFactorAt; // the team's last lane brings the factor
        }
    }
    // the piece of neighbour number K of the 16 whose ids the team's lanes hold
    template <int K, bool BIG>
    __device__ __forceinline__ x_piece<XKIND, V> load(const SpmmArgs &a, uint32_t id) const
    {
        typedef typename std::conditional<BIG, uint64_t, uint32_t>::type ofs_t;
        const ofs_t rofs = (ofs_t)id * (ofs_t)a.row_bytes;
        ofs_t o;
        if constexpr (BIG)
            o = ((uint64_t)row_bcast<K>((uint32_t)((uint64_t)rofs >> 32)) << 32) |
                row_bcast<K>((uint32_t)rofs);
        else
            o = row_bcast<K>((uint32_t)rofs);
        x_piece<XKIND, V> x;
        __builtin_memcpy(&x, (const char *)a.x + (ofs_t)(o + off), sizeof(x));
        return x;
    }
    template <bool HASF>
    __device__ __forceinline__ void products(const x_piece<XKIND, V> &x, const float (&sc)[V],
                                             float f, float (&p)[V]) const
    {
        if constexpr (XKIND == 1) {
            const uint32_t inv = ~x.v >> bsh;
#pragma unroll
            for (int v = 0; v < V; ++v)
                p[v] = signed_f(inv, 31u - (uint32_t)v, f);
        } else if constexpr (XKIND >= 3) {
            static_for<0, (V + 1) / 2>([&](auto ii) {
                constexpr int I = decltype(ii)::value;
                const uint32_t z = even_pair<I>(x.v);
                p[2 * I] = mul_half<0>(sc[2 * I], z);
                if constexpr (2 * I + 1 < V)
                    p[2 * I + 1] = mul_half<1>(sc[2 * I + 1], z);
            });
            if (HASF)
#pragma unroll
                for (int v = 0; v < V; ++v)
                    p[v] = mul_rounded(f, p[v]);
        } else {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                p[v] = (float)x.v[v];
                if (XKIND == 2)
                    p[v] = mul_rounded(sc[v], p[v]);
                if (HASF)
                    p[v] = mul_rounded(f, p[v]);
            }
        }
    }
};

// One hub row, one 64-channel tile.  Wavefront 0 adds; the others produce, each the products
// of kHubPer neighbours per stage: a team of 16 lanes takes one neighbour at a time, V
// channels per lane, as in the team form, so an instruction serves four neighbours.  LDS holds
// two stages as [neighbour][64 channels].
template <int XKIND, bool BITS_OUT, bool HASF, int V, bool BIG>
__device__ __forceinline__ void spmm_hub_row(const SpmmArgs &a, uint32_t slot, uint32_t tile,
                                             float *prod)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t i = (uint32_t)a.order[slot];
    const uint32_t beg = a.rowptr[i], end = a.rowptr[i + 1], deg = end - beg; // deg > 0
    // Stages come in blocks of four, whatever is left of the row: a loop exit in between would
    // make the compiler wait there for every load in flight.
    const uint32_t blocks = (deg + 4 * kHubStage - 1) / (4 * kHubStage);
    const int32_t c0 = (int32_t)(tile * 64);
    // (nothing is scheduled across: arithmetic hoisted over it would wait for its loads there)
    auto barrier = [] {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    if (wave > 0) {
        typedef x_piece<XKIND, V> piece;
        const uint32_t p = (uint32_t)wave - 1, q = (uint32_t)lane >> 4, sub = (uint32_t)lane & 15;
        const x_lane<XKIND, V> xl(a, c0 + (int32_t)sub * V);
        float sc[V];
#pragma unroll
        for (int v = 0; v < V; ++v)
            sc[v] = XKIND >= 2 ? a.xscale[xl.cs + v] : 1.0f;
        // A team's 16 lanes hold the ids of its neighbours of four stages (four per stage).
        auto ids_of = [&](uint32_t b) -> uint32_t {
            const uint32_t k =
                (4 * b + (sub >> 2)) * kHubStage + p * kHubPer + 4 * (sub & 3) + q;
            return (uint32_t)a.col[beg + (k < deg ? k : deg - 1)];
        };
        auto load = [&](uint32_t id, auto jj, piece (&x)[4]) {
            constexpr int J = decltype(jj)::value;
            static_for<0, 4>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                x[K] = xl.template load<4 * J + K, BIG>(a, id);
            });
        };
        auto products = [&](auto jj, const piece (&x)[4], float fl) {
            constexpr int J = decltype(jj)::value;
            float *dst = prod + (J & 1) * (kHubStage * 64) + (p * kHubPer + q) * 64 + sub * V;
            static_for<0, 4>([&](auto kk) {
                constexpr int K = decltype(kk)::value;
                const float fk = HASF ? row_bcast_f<4 * J + K>(fl) : 1.0f;
                float v[V];
                xl.template products<HASF>(x[K], sc, fk, v);
                __builtin_memcpy(__builtin_assume_aligned(dst + 4 * K * 64, 4 * V), v, sizeof(v));
            });
        };
        // Rows are requested three stages ahead, ids and factors a block of four stages ahead.
        piece x[4][4];
        uint32_t ida = ids_of(0), idb = ids_of(1);
        float fa = HASF ? a.f[ida] : 1.0f;
        __builtin_amdgcn_sched_barrier(0); // ids and factors stay older than the rows
        load(ida, const_int<0>{}, x[0]);
        load(ida, const_int<1>{}, x[1]);
        load(ida, const_int<2>{}, x[2]);
        for (uint32_t b = 0; b < blocks; ++b) {
            const uint32_t idc = ids_of(b + 2);
            const float fb = HASF ? a.f[idb] : 1.0f;
            load(ida, const_int<3>{}, x[3]);
            __builtin_amdgcn_sched_barrier(0);
            products(const_int<0>{}, x[0], fa);
            barrier();
            load(idb, const_int<0>{}, x[0]);
            __builtin_amdgcn_sched_barrier(0);
            products(const_int<1>{}, x[1], fa);
            barrier();
            load(idb, const_int<1>{}, x[1]);
            __builtin_amdgcn_sched_barrier(0);
            products(const_int<2>{}, x[2], fa);
            barrier();
            load(idb, const_int<2>{}, x[2]);
            __builtin_amdgcn_sched_barrier(0);
            products(const_int<3>{}, x[3], fa);
            barrier();
            ida = idb;
            idb = idc;
            fa = fb;
        }
        return;
    }
    // the consumer: lane = channel, one add per neighbour in stored order
    const int32_t c = c0 + lane;
    const bool live = c < a.C;
    const int32_t cc = live ? c : a.C - 1;
    // the lane's place in a neighbour's 64 products (a producer lane at the end of the row
    // holds V channels that end with the row)
    const int32_t piece0 = (cc - c0) / V * V;
    const int32_t at = piece0 + (cc - x_lane<XKIND, V>::first(a, c0 + piece0));
    float acc = 0.0f;
    for (uint32_t s = 0; s < 4 * blocks; ++s) {
        barrier(); // the products of stage s are in LDS
        const float *src = prod + (s & 1u) * (kHubStage * 64) + at;
        const uint32_t done = s * kHubStage, left = deg > done ? deg - done : 0u;
        if (left >= (uint32_t)kHubStage) {
            // (three batches ahead: the adds of one batch take half of an LDS latency)
            constexpr int kBatch = 16, kBatches = kHubStage / kBatch, kDeep = 3;
            static_assert(kHubStage % kBatch == 0 && kBatches > kDeep, "whole batches");
            float v[kDeep + 1][kBatch];
#pragma unroll
            for (int b = 0; b < kDeep; ++b)
#pragma unroll
                for (int k = 0; k < kBatch; ++k)
                    v[b][k] = src[(b * kBatch + k) * 64];
#pragma unroll
            for (int b = 0; b < kBatches; ++b) {
                if (b + kDeep < kBatches)
#pragma unroll
                    for (int k = 0; k < kBatch; ++k)
                        v[(b + kDeep) % (kDeep + 1)][k] = src[((b + kDeep) * kBatch + k) * 64];
#pragma unroll
                for (int k = 0; k < kBatch; ++k)
                    acc = add_rounded(acc, v[b % (kDeep + 1)][k]);
            }
        } else {
            for (uint32_t k = 0; k < left; ++k)
                acc = add_rounded(acc, src[k * 64]);
        }
    }
    const float y = mul_rounded(a.r ? a.r[i] : 1.0f, acc);
    if (BITS_OUT) {
        const uint64_t word = __ballot(live && y >= a.tau[cc]);
        if (lane == 0)
            ((uint64_t *)a.out)[(int64_t)i * a.ldo + tile] = word;
    } else if (live) {
        ((float *)a.out)[(int64_t)i * a.ldo + c] = y;
    }
}

// A team per row and channel window; tb: number of the workgroup among those of the teams.
template <int XKIND, bool BITS_OUT, bool HASF, int V, bool BIG, int kThreads>
__device__ __forceinline__ void spmm_team_rows(const SpmmArgs &a, uint32_t tb)
{
    // window and row of this team: a group of windows of a row side by side (one instruction then
    // covers adjacent pieces of a row), one group of all rows after the other
    // (the divisions are latency that every row waits for, so what needs none goes without)
    constexpr bool GATHERF = HASF && XKIND != 4; // else the rows bring their factors
    const uint32_t grp = a.group < a.windows ? tb / a.group_blocks : 0u;
    const uint32_t team = (tb - grp * a.group_blocks) * (kThreads / kTeam) + threadIdx.x / kTeam;
    const uint32_t team_row = a.group == 1 ? team : team / a.group;
    const uint32_t window = grp * a.group + (team - team_row * a.group);
    const uint32_t sub = threadIdx.x & 15;
    const uint32_t slot = a.slot0 + team_row;
    const bool has = slot < a.slot_end && window < a.windows;
    const uint32_t i = has ? (uint32_t)a.order[slot] : 0u;
    const uint32_t beg = has ? a.rowptr[i] : 0u, deg = has ? a.rowptr[i + 1] - beg : 0u;
    // row lengths of the wavefront's four teams (scalar)
    uint32_t dmin = (uint32_t)__builtin_amdgcn_readlane((int)deg, 0), dmax = dmin;
#pragma unroll
    for (int q = 1; q < 4; ++q) {
        const uint32_t d = (uint32_t)__builtin_amdgcn_readlane((int)deg, 16 * q);
        dmin = d < dmin ? d : dmin;
        dmax = d > dmax ? d : dmax;
    }
    const int32_t c = (int32_t)(window * (kTeam * V) + sub * V); // this lane's first channel
    const x_lane<XKIND, V> xl(a, c);
    float sc[V], acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        acc[v] = 0.0f;
        sc[v] = XKIND >= 2 ? a.xscale[xl.cs + v] : 1.0f;
    }
    typedef x_piece<XKIND, V> piece;
    // rows in flight: two sets of 8 (4 where a piece is 16 bytes: two sets of 8 spill)
    constexpr int kAhead = sizeof(piece) >= 16 ? 4 : 8;

    // The lane's neighbour of the block at t; past the row's end its last one, of an empty row
    // any (the first entry of the column array is always a valid node).
    auto ids_of = [&](uint32_t t) -> uint32_t {
        const uint32_t k = t + sub;
        return (uint32_t)a.col[k < deg ? beg + k : deg ? beg + deg - 1 : 0u];
    };
    // the neighbours from the first'th on of the block whose ids the team holds, as many as the
    // array takes
    auto load = [&](uint32_t id, auto first, auto &x) {
        constexpr int K0 = decltype(first)::value;
        static_for<0, (int)(sizeof(x) / sizeof(x[0]))>([&](auto kk) {
            constexpr int K = decltype(kk)::value;
            x[K] = xl.template load<K0 + K, BIG>(a, id);
        });
    };
    auto consume = [&](float fl, auto first, const auto &x, uint32_t t, auto full) {
        constexpr int K0 = decltype(first)::value;
        static_for<0, (int)(sizeof(x) / sizeof(x[0]))>([&](auto kk) {
            constexpr int K = decltype(kk)::value;
            float fk = 1.0f;
            if constexpr (HASF && XKIND == 4)
                fk = row_bcast_f<15>(__int_as_float((int)x[K].v));
            else if constexpr (HASF)
                fk = row_bcast_f<K0 + K>(fl);
            if (decltype(full)::value || t + K0 + K < deg) {
                float p[V];
                xl.template products<HASF>(x[K], sc, fk, p);
#pragma unroll
                for (int v = 0; v < V; ++v)
                    acc[v] = add_rounded(acc[v], p[v]);
            }
        });
    };
    // Four rows of at most 4 or 8 neighbours request just those; the loop below asks for 24 (20)
    // (54,198 nodes, 265 K non-zeros, int16 rows of 192 channels 36 us with the loop alone, 23 so).
    auto short_rows = [&](auto count) {
        const uint32_t id = ids_of(0);
        const float fl = GATHERF ? a.f[id] : 1.0f;
        piece x[decltype(count)::value];
        load(id, const_int<0>{}, x);
        consume(fl, const_int<0>{}, x, 0, std::false_type{});
    };
    if (dmax <= 4) {
        short_rows(const_int<4>{});
    } else if (dmax <= 8) {
        short_rows(const_int<8>{});
    } else {
        // The ids of a block of 16 neighbours are requested two blocks ahead, the factors one
        // block ahead, the rows kAhead neighbours ahead.
        uint32_t id0 = ids_of(0), id1 = ids_of(16);
        float f0 = GATHERF ? a.f[id0] : 1.0f;
        piece x[2][kAhead];
        __builtin_amdgcn_sched_barrier(0); // ids and factors stay older than the rows
        load(id0, const_int<0>{}, x[0]);
        auto step = [&](uint32_t t, auto full) {
            const float f1 = GATHERF ? a.f[id1] : 1.0f;
            const uint32_t id2 = ids_of(t + 32);
            static_for<0, 16 / kAhead>([&](auto qq) {
                constexpr int Q = decltype(qq)::value;
                if constexpr (Q + 1 < 16 / kAhead)
                    load(id0, const_int<(Q + 1) * kAhead>{}, x[(Q + 1) & 1]);
                else
                    load(id1, const_int<0>{}, x[0]);
                __builtin_amdgcn_sched_barrier(0); // the requests go out before the sums wait
                consume(f0, const_int<Q * kAhead>{}, x[Q & 1], t, full);
                __builtin_amdgcn_sched_barrier(0);
            });
            id0 = id1;
            id1 = id2;
            f0 = f1;
        };
        // First the blocks that are whole for all four teams.  No load stands behind a branch: the
        // waits after it would have to be for every load in flight.
        uint32_t t = 0;
        for (; t + 16 <= dmin; t += 16)
            step(t, std::true_type{});
        for (; t < dmax; t += 16)
            step(t, std::false_type{});
    }
    const float ri = (a.r && has) ? a.r[i] : 1.0f;
    if (BITS_OUT) {
        // the lane's V bits at their nominal positions (channels past C fall off), OR-ed over
        // the lanes that share a 32-bit word
        uint32_t bits = 0;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int32_t cv = xl.cs + v;
            const bool bit =
                cv < a.C && mul_rounded(ri, acc[v]) >= a.tau[cv < a.C ? cv : a.C - 1];
            bits |= bit ? (1u << v) : 0u;
        }
        const uint32_t back = (uint32_t)(c - xl.cs);
        bits = back < (uint32_t)V ? bits >> back : 0u;
        uint32_t w = bits << (c & 31);
        w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xF, 0xF, false);
        w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x4E, 0xF, 0xF, false);
        if (V <= 4)
            w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x141, 0xF, 0xF, false);
        if (V == 1)
            w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x140, 0xF, 0xF, false);
        // one lane per 32-bit word; V = 1 covers half a word, its team also clears the rest
        const int32_t words32 = 2 * ((a.C + 63) / 64);
        uint32_t *o = (uint32_t *)a.out + (int64_t)i * a.ldo * 2;
        if (has && (c & 31) == 0 && (c >> 5) < words32)
            o[c >> 5] = w;
        if (V == 1 && has && sub == 1)
            o[1] = 0u;
    } else if (has) {
        float y[V];
#pragma unroll
        for (int v = 0; v < V; ++v)
            y[v] = mul_rounded(ri, acc[v]);
        float *o = (float *)a.out + (int64_t)i * a.ldo;
        // A packed row's lane at the end of the row is not moved back: it stores what is there, one
        // by one.  (Every lane did, with a store instruction per channel: 54,198 nodes, 265 K
        // non-zeros, 256 channels with factors 39 us; in 16-byte stores 18.)
        if (XKIND != 1 ? c < a.C : c + V <= a.C) {
            __builtin_memcpy(o + xl.cs, y, sizeof(y));
        } else if (XKIND == 1) {
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (c + v < a.C)
                    o[c + v] = y[v];
        }
    }
}

// V: channels per lane of a team.  BIG: the rows of x span 4 GiB or more (64-bit offsets).
// HUBS: the launch starts with hub workgroups; their registers and LDS halve the wavefronts of the other rows,
// so launches without hubs take a kernel of their own.
template <int XKIND, bool BITS_OUT, bool HASF, int V, bool BIG, bool HUBS>
__device__ __forceinline__ void spmm_f32_rows(const SpmmArgs &a, float *prod)
{
    constexpr int kThreads = HUBS ? kHubBlock : kSpBlock;
    uint32_t tb = blockIdx.x;
    if constexpr (HUBS) {
        const uint32_t hub_blocks = a.n_hub * a.hub_tiles;
        if (tb < hub_blocks) { // workgroup-uniform; the longest rows start first
            spmm_hub_row<XKIND == 4 ? 3 : XKIND, BITS_OUT, HASF, V == 1 ? 1 : 4, BIG>(
                a, tb / a.hub_tiles, tb % a.hub_tiles, prod);
            return;
        }
        tb -= hub_blocks;
    }
    spmm_team_rows<XKIND, BITS_OUT, HASF, V, BIG, kThreads>(a, tb);
}
template <int XKIND, bool BITS_OUT, bool HASF, int V, bool BIG, bool HUBS>
__global__ __launch_bounds__(HUBS ? kHubBlock : kSpBlock, 4) void spmm_f32_kernel(
    const SpmmArgs a)
{
    extern __shared__ float prod[];
    if constexpr (XKIND >= 3) {
        if (a.wide && *a.wide) { // (the same for the whole launch)
            SpmmArgs b = a;
            b.x = a.x16;
            b.row_bytes = a.row_bytes16;
            spmm_f32_rows<2, BITS_OUT, HASF, V, BIG, HUBS>(b, prod);
            return;
        }
    }
    spmm_f32_rows<XKIND, BITS_OUT, HASF, V, BIG, HUBS>(a, prod);
}

} // namespace

int bg_check_spmm_f32(bitgnn_ctx *ctx, const bitgnn_adj *adj, const void *x, int x_is_bits,
                      int32_t C, int64_t ldx, const float *r, const float *f, int epilogue,
                      const float *tau, const void *out, int64_t ldo)
{
    if (!ctx)
        return BITGNN_ERR_INVALID_ARG;
    BG_REQUIRE(ctx, adj, BITGNN_ERR_INVALID_ARG, "bitgnn_spmm_f32: adj is null");
    BG_REQUIRE(ctx, epilogue == BITGNN_EPI_SCALE_F32 || epilogue == BITGNN_EPI_THRESH_BITS,
               BITGNN_ERR_INVALID_ARG, "bitgnn_spmm_f32: epilogue %d (SCALE_F32 or THRESH_BITS)",
               epilogue);
    const int64_t cw = ((int64_t)C + 63) / 64;
    const bool bits_out = epilogue == BITGNN_EPI_THRESH_BITS;
    BG_REQUIRE(ctx,
               C >= 1 && ldx >= (x_is_bits ? cw : (int64_t)C) &&
                   ldo >= (bits_out ? cw : (int64_t)C),
               BITGNN_ERR_INVALID_ARG, "bitgnn_spmm_f32: C=%d ldx=%lld ldo=%lld", C, (long long)ldx,
               (long long)ldo);
    BG_REQUIRE(ctx, x && out && (!bits_out || tau), BITGNN_ERR_INVALID_ARG,
               "bitgnn_spmm_f32: null pointer");
    BG_REQUIRE(ctx,
               bg_aligned(x, x_is_bits ? 8 : 4) && bg_aligned(out, bits_out ? 8 : 4) &&
                   bg_aligned(r, 4) && bg_aligned(f, 4) && bg_aligned(tau, 4),
               BITGNN_ERR_ALIGNMENT, "bitgnn_spmm_f32: misaligned pointer");
    BG_REQUIRE(ctx, adj->n < (1ll << 31) && C <= (1 << 29), BITGNN_ERR_UNSUPPORTED,
               "bitgnn_spmm_f32: N or C too large");
    return BITGNN_OK;
}

namespace {

uint32_t windows_of(int32_t C, int V) { return ((uint32_t)C + kTeam * V - 1) / (kTeam * V); }

// What a launch without the fixed part of a call (about 5 us) is expected to take in
// microseconds, with the rows of at least 2^k neighbours as hub rows (k < 0: none).  Two things
// take time side by side: the longest row that a team walks, and everybody's gathers.  Fitted on
// 201 graphs (R-MAT, Chung-Lu, block model; 2,000 to 370,000 nodes, mean degree 3 to 400), 3,500
// operands of 3 to 500 channels, each k timed in turn; the k chosen here is on average 1 to 2 %
// slower than the best of them.
double team_us(const bitgnn_adj *adj, int xkind, int32_t C, bool bits_out, bool large, int V,
               int k)
{
    // ns per neighbour of a row; per gather of a team; per row and window (order, row pointers,
    // store; the thresholds of 8 channels per lane cost most).  `large`: x is larger than an L2.
    double chain, gather, row;
    if (V == 1)
        chain = large ? 30 : 18, gather = large ? 0.0052 : 0.0025, row = 0.07;
    else if (xkind == 1)
        chain = V == 8 ? 54 : 33, gather = V == 4 || large ? 0.005 : 0.0075,
        row = V == 8 && bits_out ? 0.2 : 0.09;
    else if (xkind >= 2)
        chain = 42, gather = 0.0085, row = 0.14;
    else
        chain = large ? 65 : 35, gather = large ? 0.0075 : 0.0095, row = 0.13;
    const double windows = windows_of(C, V), nnz = (double)adj->nnz, n = (double)adj->n;
    if (k < 0)
        return std::hypot(chain * (double)adj->max_degree,
                          windows * (nnz * gather + n * row)) * 1e-3;
    // Non-zeros of the hub rows, from the counts (a row between two powers of two counts as their
    // mean).  A hub workgroup takes 4 ns of the chip and 0.017 per neighbour, and its LDS and
    // registers leave fewer wavefronts to the other rows.
    double hub = 0;
    for (int j = k; j < 31 && adj->n_ge[j]; ++j) {
        const double lo = (double)(1u << j), hi = std::fmin(2 * lo, (double)adj->max_degree + 1);
        hub += (double)(adj->n_ge[j] - adj->n_ge[j + 1]) * 0.5 * (lo + hi);
    }
    hub = std::fmin(hub, nnz);
    const double rows = adj->n_ge[k], tiles = (double)((C + 63) / 64);
    const double walk = (V == 1 || xkind == 1 ? 1.1 : 1.2) *
                        std::fmin((double)adj->max_degree, (double)(1u << k));
    const double teams =
        windows * ((nnz - hub) * gather * 1.2 + (n - rows) * row * (V == 8 ? 1.0 : 1.5));
    return std::hypot(chain * walk, teams + tiles * (rows * 4 + hub * 0.017)) * 1e-3 + 1.2;
}

struct Plan {
    int V;          // channels per lane of a team
    uint32_t n_hub; // hub rows
    double us;      // its price
};

// Channels per lane: 16 bytes of a float row, 8 of an integer row; narrow rows spread over all
// lanes of a team.  Packed rows take 4 or 8 bits per lane: 8 halve the gathers, 4 walk a row
// faster (34 against 54 ns a neighbour) and store it faster, so both are priced.  Hub rows are
// those of at least 2^k neighbours, k >= 7, for the k that is priced lowest; R-MAT graph of 8,192
// nodes, 111 K non-zeros, longest row 1,526, packed rows of 100 channels with factors: 104 us
// without hubs, 13 at 2^7; Chung-Lu graph of 22,106 nodes, 7.7 M, 2,538, 256 floats: 498 without,
// 845 at 2^7, 563 at 2^10.
Plan choose_plan(const bitgnn_adj *adj, int xkind, int32_t C, bool bits_out, bool large, int V)
{
    Plan best{0, 0, 0};
    const int Vs[2] = {V ? V : xkind != 1 && C <= 16 ? 1 : 4, 8};
    for (int q = 0; q < (xkind == 1 && C > 64 ? 2 : 1); ++q)
        for (int k = 6; k < 31; ++k) {
            const int kk = k == 6 ? -1 : k; // 6: no hubs
            const uint32_t n_hub = kk < 0 ? 0 : adj->n_ge[kk];
            // (no hubs left; or more workgroups than a launch takes: fewer than 2^32 threads)
            if (kk >= 0 && n_hub == 0)
                break;
            if ((uint64_t)n_hub * (((uint32_t)C + 63) / 64) * kHubBlock > 1u << 30)
                continue;
            // (of float and integer rows 2^9 is the best most often, and within a few per cent
            // where it is not: it wins what the prices do not tell apart)
            const double us = team_us(adj, xkind, C, bits_out, large, Vs[q], kk) *
                              (kk == 9 && xkind != 1 ? 0.93 : 1.0);
            if (best.V == 0 || us < best.us)
                best = Plan{Vs[q], n_hub, us};
        }
    return best;
}

} // namespace

// `xscale` non-null: x holds int16 rows (ldx in int16 units) and a value is
// xscale[c] * (float)x; otherwise x_is_bits selects packed +-1 or float rows.
int bg_launch_spmm_f32(bitgnn_ctx *ctx, hipStream_t s, const bitgnn_adj *adj, const void *x,
                       int x_is_bits, int32_t C, int64_t ldx, const float *r, const float *f,
                       int epilogue, const float *tau, void *out, int64_t ldo,
                       const float *xscale, const bg_byte_rows *bytes)
{
    if (adj->n == 0)
        return BITGNN_OK;
    const bool bits_out = epilogue == BITGNN_EPI_THRESH_BITS;
    SpmmArgs a;
    a.rowptr = adj->rowptr;
    a.col = adj->col;
    a.order = adj->order;
    a.x = x;
    a.row_bytes = ldx * (xscale ? 2 : x_is_bits ? 8 : 4);
    a.wide = nullptr;
    a.x16 = x;
    a.row_bytes16 = a.row_bytes;
    // Channels per lane of byte rows: 3 where 15 lanes then hold all of them, a fifth less
    // arithmetic (their bits would straddle words, so bits take 4, like wider rows: with 8 a row's
    // walk is longer; 30,000 nodes, 5.7 M non-zeros, 128 channels to bits: int16 rows 133 us, bytes
    // with 8 per lane 173, with 4 123; 150,000 nodes, 43.5 M: 950, 659 and 680).
    int byte_v = 0;
    if (bytes) {
        a.wide = bytes->wide;
        a.x = bytes->z;
        a.row_bytes = bytes->row_bytes;
        byte_v = f && C > 32 && C <= 45 && !bits_out ? 3 : 4;
    }
    a.xscale = xscale;
    a.C = C;
    a.r = r;
    a.f = f;
    a.tau = tau;
    a.out = out;
    a.ldo = ldo;
    a.hub_tiles = ((uint32_t)C + 63) / 64;
    const uint64_t table = (uint64_t)adj->n * (uint64_t)a.row_bytes;
    const bool large = table > (4u << 20); // than an L2
    const Plan plan =
        choose_plan(adj, xscale ? 2 : x_is_bits ? 1 : 0, C, bits_out, large, byte_v);
    // +-1 rows without factors: the float sum of a row is its integer sum, exact while partial
    // sums stay below 2^24, so the bit aggregation's counters give it.  It needs the workspace
    // (without it the floats are added here) and is taken where it is priced lower; which is
    // better has no simple line: 23,507 nodes, 2.2 M non-zeros, 256 channels to bits 19 us against
    // 45 added as floats, 8,920 nodes, 788 K, 64 channels 23 against 10.  On 958 operands the
    // choice costs 1.5 % more than always knowing the faster one.
    if (x_is_bits && !xscale && !f && C <= 2048 && adj->max_degree < (1ll << 24) &&
        adj->n * (int64_t)((C + 31) / 32) < (1ll << 31) &&
        bg_adj_workspace_bytes(adj, C, 1) <= ctx->sc->ws_bytes &&
        bg_bspmm_scaled_us(adj, C, bits_out) < plan.us)
        return bg_launch_bspmm_scaled(ctx, s, adj, (const uint64_t *)x, C, ldx, r,
                                      bits_out ? tau : nullptr, out, ldo);
    const uint32_t n_hub = plan.n_hub;
    const int V = plan.V;
    a.windows = windows_of(C, V);
    // All windows of a row side by side; two other orders keep a smaller part of the table hot
    // where it is larger than an L2 and its rows are gathered often (24 times on average).
    //  * Four windows (1 KB of a float row) of all rows after the other, where the gathers take
    //    several times as long as the longest row's walk, which is then paid once per group.
    //    500 floats with factors: 4,643 nodes, 296 K non-zeros, longest row 90: 49 us side by
    //    side, 38 in fours; but 3,111 nodes, 305 K, longest row 536: 40 and 53.  500 int16
    //    channels: 48,545 nodes, 9.1 M, 2,856: 907 and 823; but 8,911 nodes, 2.5 M, 1,442: 170
    //    and 202.
    //  * One window after the other, where the windows are whole cache lines and nothing but the
    //    rows is gathered (300,001 nodes, 14.7 M non-zeros, 128 floats: 769 and 683 us; with
    //    factors, which are gathered once per window, it loses; of 256 floats at a mean degree
    //    below 10 it takes 1.1, of 192 1.2 times the time).
    // Packed rows are short.
    a.group = a.windows;
    if (!x_is_bits && adj->nnz >= 24 * adj->n) {
        if (!f && a.row_bytes % 128 == 0 && bg_aligned(a.x, 128) && table > (8u << 20))
            a.group = 1;
        else if (large && a.windows > 4 &&
                 adj->nnz * (int64_t)a.windows >= 16000 * adj->max_degree)
            a.group = 4;
    }
    const uint32_t groups = (a.windows + a.group - 1) / a.group;
    const bool big = table >= (1ull << 32);
    uint32_t threads, grid;
    auto launch = [&](auto xk, auto v) {
        constexpr int XK = decltype(xk)::value, VV = decltype(v)::value;
        auto go = [&](auto bo, auto hf, auto bg) {
            // (forms that are not launched are not built: bits of 3 channels per lane, offsets
            // of byte rows beyond 32 bits, factors in rows without them)
            constexpr bool BO = decltype(bo)::value && VV != 3,
                           HF = decltype(hf)::value || XK == 4,
                           BG = decltype(bg)::value && XK < 3;
            if (a.n_hub)
                spmm_f32_kernel<XK, BO, HF, VV, BG, true>
                    <<<grid, threads, kHubLds, s>>>(a);
            else
                spmm_f32_kernel<XK, BO, HF, VV, BG, false><<<grid, threads, 0, s>>>(a);
        };
        auto go2 = [&](auto bo, auto hf) {
            big ? go(bo, hf, std::true_type{}) : go(bo, hf, std::false_type{});
        };
        auto go3 = [&](auto bo) { f ? go2(bo, std::true_type{}) : go2(bo, std::false_type{}); };
        bits_out ? go3(std::true_type{}) : go3(std::false_type{});
    };
    // One launch, unless there are more than 2^26 teams.
    const int64_t rows_max = (1ll << 26) / (groups * a.group);
    bg_time_begin(ctx, s);
    for (int64_t slot = n_hub; slot == n_hub || slot < adj->n; slot += rows_max) {
        const int64_t rows = adj->n - slot < rows_max ? adj->n - slot : rows_max;
        a.slot0 = (uint32_t)slot;
        a.slot_end = (uint32_t)(slot + rows);
        a.n_hub = slot == n_hub ? n_hub : 0; // the hub rows start first
        threads = a.n_hub ? kHubBlock : kSpBlock;
        const uint32_t teams = threads / kTeam; // of a workgroup
        a.group_blocks = ((uint32_t)rows * a.group + teams - 1) / teams;
        grid = a.n_hub * a.hub_tiles + groups * a.group_blocks;
        if (bytes) {
            if (V == 3)
                launch(const_int<4>{}, const_int<3>{});
            else if (bytes->has_factor)
                launch(const_int<4>{}, const_int<4>{});
            else
                launch(const_int<3>{}, const_int<4>{});
        } else if (xscale) {
            if (V == 1)
                launch(const_int<2>{}, const_int<1>{});
            else
                launch(const_int<2>{}, const_int<4>{});
        } else if (x_is_bits) {
            if (V == 4)
                launch(const_int<1>{}, const_int<4>{});
            else
                launch(const_int<1>{}, const_int<8>{});
        } else {
            if (V == 1)
                launch(const_int<0>{}, const_int<1>{});
            else
                launch(const_int<0>{}, const_int<4>{});
        }
    }
    bg_time_end(ctx, s);
    BG_LAUNCH_CHECK(ctx, "bitgnn_spmm_f32");
    return BITGNN_OK;
}

extern "C" int bitgnn_spmm_f32(bitgnn_ctx *ctx, void *stream, const bitgnn_adj *adj, const void *x,
                               int x_is_bits, int32_t C, int64_t ldx, const float *r,
                               const float *f, int epilogue, const float *tau, void *out,
                               int64_t ldo)
{
    int rc = bg_check_spmm_f32(ctx, adj, x, x_is_bits, C, ldx, r, f, epilogue, tau, out, ldo);
    if (rc != BITGNN_OK)
        return rc;
    BG_NEED_DEVICE(ctx);
    return bg_launch_spmm_f32(ctx, (hipStream_t)stream, adj, x, x_is_bits, C, ldx, r, f, epilogue,
                              tau, out, ldo, nullptr, nullptr);
}

int bg_check_spmm_i16(bitgnn_ctx *ctx, const bitgnn_adj *adj, const int16_t *z, int32_t C,
                      int64_t ldz, const float *alpha, const float *r, const float *f,
                      int epilogue, const float *tau, const void *out, int64_t ldo)
{
    // same shape rules as float rows (ldz counts int16 elements; z is 4-byte aligned)
    int rc = bg_check_spmm_f32(ctx, adj, z, 0, C, ldz, r, f, epilogue, tau, out, ldo);
    if (rc != BITGNN_OK)
        return rc;
    BG_REQUIRE(ctx, alpha, BITGNN_ERR_INVALID_ARG, "bitgnn_spmm_i16: alpha is null");
    BG_REQUIRE(ctx, bg_aligned(alpha, 4), BITGNN_ERR_ALIGNMENT,
               "bitgnn_spmm_i16: misaligned alpha");
    return BITGNN_OK;
}

extern "C" int bitgnn_spmm_i16(bitgnn_ctx *ctx, void *stream, const bitgnn_adj *adj,
                               const int16_t *z, int32_t C, int64_t ldz, const float *alpha,
                               const float *r, const float *f, int epilogue, const float *tau,
                               void *out, int64_t ldo)
{
    int rc = bg_check_spmm_i16(ctx, adj, z, C, ldz, alpha, r, f, epilogue, tau, out, ldo);
    if (rc != BITGNN_OK)
        return rc;
    BG_NEED_DEVICE(ctx);
    return bg_launch_spmm_f32(ctx, (hipStream_t)stream, adj, z, 0, C, ldz, r, f, epilogue, tau,
                              out, ldo, alpha, nullptr);
}

namespace {

// int16 rows -> byte rows z / 2 + 128, eight channels per thread; of rows that bring their factor
// a thread behind the channels writes it.  Sets *wide (if there is one) where a value has no byte.
// Bound by the 2 + 1 bytes per channel that it moves (232,965 rows of 128: 16 us).
__global__ __launch_bounds__(256) void byte_rows_kernel(const int16_t *z, int64_t n, int32_t C,
                                                        int64_t ld, int groups_log2, uint8_t *out,
                                                        const float *f, uint32_t *wide)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, i = t >> groups_log2;
    if (i >= n)
        return;
    const int32_t g = (int32_t)(t & ((1 << groups_log2) - 1)), c0 = 8 * g;
    uint32_t w[2] = {0, 0};
    bool out_of_range = false;
    if (c0 < C) {
        typedef int16_t i16x8 __attribute__((ext_vector_type(8)));
        const i16x8 v = *(const i16x8 *)(z + i * ld + c0); // rows are padded to 16 bytes
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int32_t b = (v[k] >> 1) + 128;
            out_of_range |= c0 + k < C && (uint32_t)b > 255u;
            w[k / 4] |= (uint32_t)(b & 255) << (8 * (k % 4));
        }
    } else if (f && c0 + 4 == (int32_t)kFactorAt) {
        w[1] = (uint32_t)__float_as_int(f[i]);
    }
    *(uint2 *)(out + (i << (groups_log2 + 3)) + c0) = make_uint2(w[0], w[1]);
    if (out_of_range && wide)
        *wide = 1u;
}

__global__ void clear_word_kernel(uint32_t *p) { *p = 0u; }

} // namespace

// Whether byte rows pay: microseconds that the aggregation is expected to save against those of
// writing them and, where a value may have no byte (K > 254), of clearing the word that says so.
// Rows of up to 32 channels are a line or less either way.  With a factor in the row (up to 56
// channels) the factors' gathers go too: 41 channels, 89,250 nodes, 1 M non-zeros 46 -> 40 us,
// 300,000 and 23.8 M 386 -> 263, 8,192 and 0.4 M 26.5 either way.  Wider rows gain where the table
// is larger than an L2: 128 channels, 300,000 nodes, 23.8 M 663 -> 435; 5,000 and 1.7 M 43 -> 46.
bool bg_byte_rows_pay(const bitgnn_adj *adj, int32_t C, int32_t K, bool has_f)
{
    // (products of random bits have a deviation of sqrt(K): above 1,800 the range of a byte is
    // less than six of them, and some value of a large table has none)
    if (K % 2 != 0 || K > 1800 || C <= 32 || C > 256)
        return false;
    const double nnz = (double)adj->nnz, n = (double)adj->n;
    const double cost = 4.5 + (K > 254 ? 10.0 : 0.0) + n * C * 0.5e-6;
    double gain = 4.5e-6 * nnz + 4.0;
    if (!has_f || C > 56)
        gain = (C > 64 ? 6e-6 * ((C + 63) / 64) : 2.5e-6) * nnz *
               (n * 2 * C > (double)(4 << 20) ? 1.0 : 0.2);
    return gain > 1.3 * cost;
}

int bg_launch_byte_rows(bitgnn_ctx *ctx, hipStream_t s, const int16_t *z, int64_t n, int32_t C,
                        int64_t ld, const float *f, uint32_t *wide, bg_byte_rows *b)
{
    b->has_factor = f && C <= 56;
    b->wide = wide;
    int groups_log2 = 3;
    while ((8 << groups_log2) < b->row_bytes)
        ++groups_log2;
    if (wide)
        clear_word_kernel<<<1, 1, 0, s>>>(wide);
    byte_rows_kernel<<<(unsigned)(((n << groups_log2) + 255) / 256), 256, 0, s>>>(
        z, n, C, ld, groups_log2, (uint8_t *)b->z, b->has_factor ? f : nullptr, wide);
    BG_LAUNCH_CHECK(ctx, "byte_rows_kernel");
    return BITGNN_OK;
}

namespace {

// int32 rows -> int16 rows in place (the int16 row starts where the int32 row did): one
// wavefront per row reads a 64-channel tile, then writes it; the bytes a tile's write
// covers belong to this tile's first half or to tiles already read.  The two views of the
// row alias on purpose: the destination type says so, and compiler barriers keep every
// tile's load in front of its store and the store in front of the next tile's load.
typedef int16_t __attribute__((may_alias)) i16_alias;
__global__ __launch_bounds__(256) void narrow_rows_kernel(int32_t *z, int64_t n, int32_t M,
                                                          int64_t ld32)
{
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= n)
        return;
    const volatile int32_t *src = z + row * ld32;
    i16_alias *dst = (i16_alias *)(z + row * ld32);
    for (int32_t c0 = 0; c0 < M; c0 += 64) {
        const int32_t c = c0 + lane;
        const int32_t v = c < M ? src[c] : 0;
        asm volatile("" ::: "memory"); // the whole tile is loaded (one instruction) ...
        if (c < M)
            dst[c] = (int16_t)v; // ... before any lane stores (the store waits for the load)
        asm volatile("" ::: "memory");
    }
}

} // namespace

// Raw BMM integers (|z| <= 32767) in int32 rows of stride ld32 -> int16 rows of stride
// 2 * ld32 (in int16 units) at the same addresses.
int bg_launch_narrow_rows(bitgnn_ctx *ctx, hipStream_t s, int32_t *z, int64_t n, int32_t M,
                          int64_t ld32)
{
    if (n == 0)
        return BITGNN_OK;
    narrow_rows_kernel<<<(unsigned)((n + 3) / 4), 256, 0, s>>>(z, n, M, ld32);
    BG_LAUNCH_CHECK(ctx, "narrow_rows_kernel");
    return BITGNN_OK;
}
