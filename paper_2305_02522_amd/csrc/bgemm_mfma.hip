// BMM on the matrix cores (Section 2.2: c = n - 2 popc(a xor b); the paper runs it on
// 1-bit tensor cores, which CDNA4 does not have).  The narrowest format there is 4-bit floating
// point (E2M1), which holds +-1 exactly: a stored bit becomes the nibble +1 (0x2) or -1 (0xA)
// and v_mfma_scale_f32_16x16x128_f8f6f4, with unit scales, adds products of +-1 in float32.
// Every partial sum is an integer (plus one half, see below) far below 2^23, so the result is
// the exact integer whatever the order of the additions.  Positions that hold no element (pad
// bits inside a row and behind it) are zero in both operands, so each adds (-1)(-1) = 1, and a
// constant takes them off again:
//   Z[i][c] = sum_k (+-1)(+-1) - (stored positions - K).
//
// gfx950 mapping
//  - a lane's operand is 32 elements = one 32-bit word of a packed row, widened to four
//    registers with two VALU ops each.  Nibble j of register q is bit 4 j + q of the word: the
//    elements of a row may be taken in any order that both operands share;
//  - the weights are widened once per workgroup and stay in LDS for its life, in the order in
//    which lanes read them (16 consecutive bytes a lane: no bank conflicts).  64 x K / 2 bytes a
//    64 columns: 256 columns of 1,024 bits fill 128 KB; wider outputs run as column chunks;
//  - a wavefront owns 16 R node rows and walks column groups of CT tiles of 16: R x CT
//    accumulators of 16 x 16, every weight operand read from LDS feeds R MFMAs, every widened
//    row word CT;
//  - the weights are the MFMA's first operand, so a lane ends up with 4 columns (4 g + j of
//    every tile) of ONE node row: integers and logits leave as runs of 4.  For thresholded bits
//    the tiles' columns are dealt so that the 16 values of four tiles are 16 consecutive bits of
//    an output word: column 16 g + 4 t + j in row 4 g + j of tile t.  The accumulators start at
//    1/2 - T - (pad positions), so a bit is the complement of the result's sign, one
//    v_alignbit each;
//  - row words are requested two K steps ahead, across column groups and panels.
// Against the bits widened to bytes for the int8 cores (the form before) a MFMA takes twice the
// elements in half the time, an operand 8 VALU ops per 32 elements instead of 24, and there is no
// launch that widens the weights: 2.4 M x 512 x 256 to bits 432 -> 177 us, 2.4 M x 200 x 256
// 291 -> 115, 233 K x 128 x 128 25 -> 9.3, and shapes that the VALU kernel used to win, 89 K x
// 1000 x 256 79 -> 25, 10 K x 1433 x 64 28 -> 8.5.  What bounds it: 2.4 M x 512 x 256 is 0.64
// Pop in 177 us, 36 % of the peak; the epilogue's and the widening's VALU ops take about as long
// as the MFMAs.  Wide integers and logits are bound by writing them (2.4 M x 256: 4.3 TB/s).
#include "common.h"

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr size_t kMfLdsLimit = 140 * 1024; // weights; up to 18 KB of staged outputs beside them

// 32 bits -> 32 elements of +-1 in four bits each
__device__ __forceinline__ v8i widen32(uint32_t w)
{
    v8i r = {};
    const uint32_t m = ~w; // sign bits
#pragma unroll
    for (int q = 0; q < 4; ++q)
        r[q] = (int)(((m << (3 - q)) & 0x88888888u) | 0x22222222u);
    return r;
}

__device__ __forceinline__ v4f mfma_pm1(const v8i &a, const v8i &b, const v4f &c)
{
    // formats 4: E2M1; scales 2^(127 - 127)
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 4, 4, 0, 0x7F7F7F7F, 0,
                                                            0x7F7F7F7F);
}

struct MfArgs {
    const uint32_t *x;
    int64_t n, x_stride;   // rows; 32-bit words between them
    int32_t K, kw32;       // elements and stored 32-bit words of a row
    const uint32_t *w;
    int64_t w_stride;
    int32_t M, tiles;      // columns, tiles of 16 of them
    int32_t steps;         // of 128 positions
    const int32_t *T;
    const float *alpha;
    void *out;
    int64_t out_stride;
};

// Column of row `a` (0..15) of a tile.
template <int EPI> __device__ __forceinline__ int mf_column(int tile, int a)
{
    if (EPI == BITGNN_EPI_THRESH_BITS)
        return 64 * (tile >> 2) + 16 * (a >> 2) + 4 * (tile & 3) + (a & 3);
    return 16 * tile + a;
}

// The widened weights, in the order in which lanes read them, and the column constants behind.
template <int EPI>
__device__ __forceinline__ void mf_load_weights(const MfArgs &p, uint4 *wl, float *colk, float *colf)
{
    const int tid = threadIdx.x, all = p.steps * p.tiles * 64;
#pragma unroll 8
    for (int i = tid; i < all; i += blockDim.x) {
        const int s = (i >> 6) / p.tiles, t = (i >> 6) - s * p.tiles;
        const int c = mf_column<EPI>(t, i & 15), k = 4 * s + ((i >> 4) & 3);
        const bool in = c < p.M && k < p.kw32;
        const uint32_t word = p.w[in ? (int64_t)c * p.w_stride + k : 0];
        const v8i v = widen32(in ? word : 0u);
        wl[i] = make_uint4(v[0], v[1], v[2], v[3]);
    }
    for (int i = tid; i < p.tiles * 16; i += blockDim.x) {
        const int c = mf_column<EPI>(i >> 4, i & 15);
        const int pad = 128 * p.steps - p.K;
        float k = (float)-pad;
        if (EPI == BITGNN_EPI_THRESH_BITS) {
            // |Z| <= K, so thresholds beyond +-(K + 1) decide nothing more; a column beyond M
            // never passes
            const int32_t lim = p.K + 1;
            int32_t t = c < p.M ? p.T[c] : lim;
            t = t > lim ? lim : (t < -lim ? -lim : t);
            k = 0.5f + (float)(-t - pad);
        }
        colk[i] = k;
        colf[i] = EPI == BITGNN_EPI_SCALE_F32 && c < p.M ? p.alpha[c] : 0.0f;
    }
}

template <int R, int CT>
__device__ __forceinline__ void mf_start(v4f (&acc)[R][CT], const float *colk, int t0, int g)
{
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        const v4f k = *(const v4f *)(colk + (t0 + t) * 16 + 4 * g);
#pragma unroll
        for (int h = 0; h < R; ++h)
            acc[h][t] = k;
    }
}

// One K step: the weights' operands at wk, the rows' words in x.
template <int R, int CT>
__device__ __forceinline__ void mf_step(v4f (&acc)[R][CT], const uint4 *wk, const uint32_t (&x)[R])
{
    v8i b[R];
#pragma unroll
    for (int h = 0; h < R; ++h)
        b[h] = widen32(x[h]);
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        const uint4 u = wk[t * 64];
        const v8i a = {(int)u.x, (int)u.y, (int)u.z, (int)u.w, 0, 0, 0, 0};
#pragma unroll
        for (int h = 0; h < R; ++h)
            acc[h][t] = mfma_pm1(a, b[h], acc[h][t]);
    }
}

// Orders a wavefront's own LDS accesses (the hardware keeps them in program order).
__device__ __forceinline__ void mf_wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Integers and logits leave through LDS, two tiles at a time, so that a store instruction writes
// whole 128-byte lines of eight rows; straight from the accumulators it would write 64 bytes of
// sixteen (233 K x 512 x 256 to floats: 76 us that way, 56 so).
constexpr int kMfStageRow = 36; // 32 columns, 16-byte rows that start four banks apart
constexpr size_t kMfStage = 16 * kMfStageRow * 4;

template <int EPI> __host__ __device__ constexpr size_t mf_stage_bytes(int waves)
{
    return EPI == BITGNN_EPI_THRESH_BITS ? 0 : waves * kMfStage;
}

template <int EPI, int R, int CT>
__device__ __forceinline__ void mf_store(const MfArgs &p, const v4f (&acc)[R][CT],
                                         const float *colf, uint32_t *stage, int64_t row0, int t0,
                                         int lane)
{
    const int r = lane & 15, g = lane >> 4;
    if (EPI == BITGNN_EPI_THRESH_BITS) {
#pragma unroll
        for (int h = 0; h < R; ++h) {
            const int64_t i = row0 + 16 * h + r;
#pragma unroll
            for (int w = 0; w < CT / 4; ++w) {
                uint32_t neg = 0;
#pragma unroll
                for (int q = 15; q >= 0; --q)
                    neg = __builtin_amdgcn_alignbit(
                        neg, __float_as_uint(acc[h][4 * w + q / 4][q % 4]), 31);
                if (i < p.n)
                    ((uint16_t *)((uint64_t *)p.out + i * p.out_stride + t0 / 4 + w))[g] =
                        (uint16_t)~neg;
            }
        }
        return;
    }
    if (EPI == kEpiRawI16) { // four tiles are 128 bytes of a row
#pragma unroll
        for (int t = 0; t < CT; t += 4) {
            if (16 * (t0 + t) >= p.M) // wave-uniform
                break;
#pragma unroll
            for (int h = 0; h < R; ++h) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    int16_t v[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        v[j] = (int16_t)(int32_t)acc[h][t + q][j];
                    __builtin_memcpy(stage + r * kMfStageRow + 8 * q + 2 * g, v, 8);
                }
                mf_wave_order();
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int row = (lane >> 3) + 8 * q, c = 16 * (t0 + t) + 8 * (lane & 7);
                    const int64_t i = row0 + 16 * h + row;
                    const uint4 v = *(const uint4 *)(stage + row * kMfStageRow + 4 * (lane & 7));
                    if (i < p.n && c < p.M) // rows are padded to 16 bytes
                        *(uint4 *)((int16_t *)p.out + i * p.out_stride + c) = v;
                }
                mf_wave_order();
            }
        }
        return;
    }
#pragma unroll
    for (int t = 0; t < CT; t += 2) {
        const int c0 = 16 * (t0 + t);
        if (c0 >= p.M) // wave-uniform
            break;
#pragma unroll
        for (int h = 0; h < R; ++h) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const v4f f = *(const v4f *)(colf + c0 + 16 * q + 4 * g);
                uint32_t v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    v[j] = EPI == BITGNN_EPI_RAW_I32
                               ? (uint32_t)(int32_t)acc[h][t + q][j]
                               // + 0: a sum of 0 is +0, whatever its sign here
                               : __float_as_uint(f[j] * (acc[h][t + q][j] + 0.0f));
                *(uint4 *)(stage + r * kMfStageRow + 16 * q + 4 * g) =
                    make_uint4(v[0], v[1], v[2], v[3]);
            }
            mf_wave_order();
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int row = (lane >> 3) + 8 * q, c = c0 + 4 * (lane & 7);
                const int64_t i = row0 + 16 * h + row;
                const uint4 v = *(const uint4 *)(stage + row * kMfStageRow + 4 * (lane & 7));
                uint32_t *o = (uint32_t *)p.out + i * p.out_stride + c;
                if (i < p.n && c + 4 <= p.M)
                    __builtin_memcpy(o, &v, 16);
                else if (i < p.n && c < p.M) {
                    o[0] = v.x;
                    if (c + 1 < p.M)
                        o[1] = v.y;
                    if (c + 2 < p.M)
                        o[2] = v.z;
                }
            }
            mf_wave_order();
        }
    }
}

template <int EPI, int R, int CT>
__global__ __launch_bounds__(512) void bgemm_mfma_kernel(MfArgs p)
{
    extern __shared__ uint4 wl[]; // [steps][tiles][64 lanes], then the column constants
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    float *colk = (float *)(wl + p.steps * p.tiles * 64), *colf = colk + p.tiles * 16;
    uint32_t *stage = (uint32_t *)(colf + p.tiles * 16) + wave * (kMfStage / 4);
    mf_load_weights<EPI>(p, wl, colk, colf);
    __syncthreads(); // the last barrier: weights and constants are read-only from here on

    const int64_t rows = (int64_t)waves * 16 * R, last = p.n - 1;
    // requests, two steps ahead of the products: position in the sequence panel, group, step
    int64_t q_panel = blockIdx.x;
    int q_t0 = 0, q_s = 0;
    const uint32_t *row[R];
    auto at_panel = [&] {
#pragma unroll
        for (int h = 0; h < R; ++h) {
            const int64_t i = q_panel * rows + wave * (16 * R) + 16 * h + r;
            row[h] = p.x + (i < last ? i : last) * p.x_stride; // clamped: no load is conditional
        }
    };
    auto request = [&](uint32_t (&x)[R]) {
        const int k = 4 * q_s + g, kc = k < p.kw32 ? k : p.kw32 - 1;
#pragma unroll
        for (int h = 0; h < R; ++h)
            x[h] = row[h][kc];
        if (++q_s == p.steps) {
            q_s = 0;
            q_t0 += CT;
            if (q_t0 >= p.tiles) {
                q_t0 = 0;
                q_panel += gridDim.x;
                at_panel();
            }
        }
    };
    uint32_t x0[R], x1[R];
    at_panel();
    request(x0);
    request(x1);
    for (int64_t panel = blockIdx.x; panel * rows < p.n; panel += gridDim.x) {
        const int64_t row0 = panel * rows + wave * (16 * R);
        for (int t0 = 0; t0 < p.tiles; t0 += CT) {
            v4f acc[R][CT];
            mf_start<R, CT>(acc, colk, t0, g);
            const uint4 *wk = wl + t0 * 64 + lane;
            for (int s = 0; s < p.steps; ++s) {
                uint32_t x[R];
#pragma unroll
                for (int h = 0; h < R; ++h) {
                    x[h] = 4 * s + g < p.kw32 ? x0[h] : 0u;
                    x0[h] = x1[h];
                }
                request(x1);
                mf_step<R, CT>(acc, wk, x);
                wk += p.tiles * 64;
            }
            mf_store<EPI, R, CT>(p, acc, colf, stage, row0, t0, lane);
        }
    }
}

// Full-precision activations (BMM.FBB / BMM.FBF, Section 3.1.2: BIN folded into the product).  A
// wavefront reads 16 R rows, 64 floats a load: the wave-wide compare mask is 64 bits of the packed
// row, put into lanes of two registers and, GROUP masks at a time, into LDS, where the products
// take their words from.  Three VALU ops per 64 floats against 2 x 2 per 64 channels of output
// when every lane adds popcounts for its own channel: bound by the stream of the features for any
// width.  Four groups of loads are in flight, across rows and panels.  131 K x 512 x 256: 83 us
// with popcounts, 58 so (268 MB); 233 K x 128 x 128 65 and 35.
struct MfFloats {
    const float *x;
    int64_t ldx;
    const float *tau;
    int32_t votes, row_words; // of 64 floats; 32-bit words between rows in LDS
};

template <int EPI, int R, int CT, int GROUP, bool TAU>
__global__ __launch_bounds__(512) void bgemm_f32_mfma_kernel(MfArgs p, MfFloats f)
{
    // [steps][tiles][64 lanes], column constants, rows of every wavefront, thresholds
    extern __shared__ uint4 wl[];
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    float *colk = (float *)(wl + p.steps * p.tiles * 64), *colf = colk + p.tiles * 16;
    uint32_t *stage = (uint32_t *)(colf + p.tiles * 16) + wave * (kMfStage / 4);
    uint32_t *words = (uint32_t *)(colf + p.tiles * 16) + mf_stage_bytes<EPI>(waves) / 4;
    float *tl = (float *)(words + waves * (16 * R) * f.row_words);
    words += wave * (16 * R) * f.row_words;
    constexpr int kRows = 16 * R;
    const int64_t rows = (int64_t)waves * kRows, last = p.n - 1;
    const int groups = (f.votes + GROUP - 1) / GROUP;
    const uint64_t tail = p.K % 64 ? (1ull << (p.K % 64)) - 1 : ~0ull;
    int64_t q_panel = blockIdx.x;
    int q_row = 0, q_group = 0;
    const float *qx = nullptr;
    auto at_row = [&] {
        const int64_t i = q_panel * rows + wave * kRows + q_row;
        qx = f.x + (i < last ? i : last) * f.ldx;
    };
    auto request = [&](float (&v)[GROUP]) {
#pragma unroll
        for (int b = 0; b < GROUP; ++b) {
            const int k = (q_group * GROUP + b) * 64 + lane;
            v[b] = qx[k < p.K ? k : p.K - 1];
        }
        if (++q_group == groups) {
            q_group = 0;
            if (++q_row == kRows) {
                q_row = 0;
                q_panel += gridDim.x;
            }
            at_row();
        }
    };
    constexpr int kAhead = 4;
    float v[kAhead][GROUP];
    at_row();
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
        request(v[q]);
    int c_row = 0, c_group = 0; // what is consumed
    auto consume = [&](const float (&v)[GROUP]) {
        uint32_t lo = 0, hi = 0;
#pragma unroll
        for (int b = 0; b < GROUP; ++b) {
            const int vote = c_group * GROUP + b; // at most 9 past the last one
            const float t = TAU ? tl[vote < f.votes ? vote * 64 + lane : lane] : 0.0f;
            uint64_t m = __ballot(v[b] >= t);
            m = vote == f.votes - 1 ? m & tail : m;
            asm("v_writelane_b32 %0, %1, %2" : "+v"(lo) : "s"((uint32_t)m), "n"(b));
            asm("v_writelane_b32 %0, %1, %2" : "+v"(hi) : "s"((uint32_t)(m >> 32)), "n"(b));
        }
        const int vote = c_group * GROUP + lane;
        if (lane < GROUP && vote < f.votes)
            *(uint2 *)(words + c_row * f.row_words + 2 * vote) = make_uint2(lo, hi);
        if (++c_group == groups) {
            c_group = 0;
            ++c_row;
        }
    };
    mf_load_weights<EPI>(p, wl, colk, colf);
    for (int i = lane; i < 16 * R * f.row_words; i += 64) // the words behind a row stay zero
        words[i] = 0u;
    if (TAU)
        for (int i = threadIdx.x; i < f.votes * 64; i += blockDim.x)
            tl[i] = f.tau[i < p.K ? i : p.K - 1];
    __syncthreads(); // the last barrier
    for (int64_t panel = blockIdx.x; panel * rows < p.n; panel += gridDim.x) {
        const int64_t row0 = panel * rows + wave * kRows;
        c_row = 0;
        for (int i = 0; i < kRows * groups; i += kAhead) // a multiple of 16 groups
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                consume(v[q]);
                request(v[q]);
            }
        mf_wave_order();
        for (int t0 = 0; t0 < p.tiles; t0 += CT) {
            v4f acc[R][CT];
            mf_start<R, CT>(acc, colk, t0, g);
            const uint4 *wk = wl + t0 * 64 + lane;
            for (int s = 0; s < p.steps; ++s) {
                uint32_t x[R];
#pragma unroll
                for (int h = 0; h < R; ++h)
                    x[h] = words[(16 * h + r) * f.row_words + 4 * s + g];
                mf_step<R, CT>(acc, wk, x);
                wk += p.tiles * 64;
            }
            mf_store<EPI, R, CT>(p, acc, colf, stage, row0, t0, lane);
        }
        mf_wave_order();
    }
}

// Tiles of the M columns: the kernel takes them in groups of four or eight.
int32_t mf_tiles(int32_t M) { return (M + 63) / 64 * 4; }

// Output columns per launch: all of them when the widened weights fit in LDS, else the largest
// multiple of 64 (whole output words) that does; 0 = the shape does not fit at all.
int32_t mf_chunk(int32_t kwords, int32_t M)
{
    const int64_t steps = ((int64_t)kwords + 1) / 2, tile = steps * 1024 + 128;
    if (mf_tiles(M) * tile <= (int64_t)kMfLdsLimit)
        return M;
    return (int32_t)((int64_t)kMfLdsLimit / (4 * tile) * 64);
}

template <int EPI, int R, int CT>
int mf_launch(bitgnn_ctx *ctx, hipStream_t s, const MfArgs &p, unsigned grid, int threads,
              size_t lds)
{
    BG_HIP(ctx, hipFuncSetAttribute((const void *)bgemm_mfma_kernel<EPI, R, CT>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    bgemm_mfma_kernel<EPI, R, CT><<<grid, threads, lds, s>>>(p);
    BG_LAUNCH_CHECK(ctx, "bgemm_mfma");
    return BITGNN_OK;
}

template <int EPI>
int mf_launch_epi(bitgnn_ctx *ctx, hipStream_t s, MfArgs p)
{
    p.tiles = mf_tiles(p.M);
    const size_t weights = (size_t)p.tiles * ((size_t)p.steps * 1024 + 128);
    const int64_t cus = ctx->n_cus > 0 ? ctx->n_cus : 256;
    // 64 rows a wavefront where that still gives every CU rows, else 16
    const bool wide = p.n >= cus * 256;
    // two workgroups a CU where they fit
    const int threads = weights + mf_stage_bytes<EPI>(4) > 78 * 1024 ? 512 : 256;
    const size_t lds = weights + mf_stage_bytes<EPI>(threads / 64);
    const int64_t rows = (int64_t)(threads / 64) * (wide ? 64 : 16);
    const int64_t panels = (p.n + rows - 1) / rows, fit = cus * ((160 * 1024) / (lds + 1024));
    const int64_t most = cus * 8 < fit ? cus * 8 : fit;
    const unsigned grid = (unsigned)(panels < most ? panels : most);
    if (p.tiles % 8 == 0)
        return wide ? mf_launch<EPI, 4, 8>(ctx, s, p, grid, threads, lds)
                    : mf_launch<EPI, 1, 8>(ctx, s, p, grid, threads, lds);
    return wide ? mf_launch<EPI, 4, 4>(ctx, s, p, grid, threads, lds)
                : mf_launch<EPI, 1, 4>(ctx, s, p, grid, threads, lds);
}

template <int EPI, int GROUP, bool TAU>
int mf_launch_f32_group(bitgnn_ctx *ctx, hipStream_t s, const MfArgs &p, const MfFloats &f)
{
    // 16 rows a wavefront: with 32, the last of two or three turns was a fifth of the time
    constexpr int R = 1, CT = 4;
    auto lds_of = [&](int threads) {
        return (size_t)p.tiles * ((size_t)p.steps * 1024 + 128) +
               mf_stage_bytes<EPI>(threads / 64) +
               (size_t)(threads / 64) * 16 * R * f.row_words * 4 + (TAU ? (size_t)f.votes * 256 : 0);
    };
    const int threads = lds_of(256) > 52 * 1024 ? 512 : 256;
    const size_t lds = lds_of(threads);
    const int64_t cus = ctx->n_cus > 0 ? ctx->n_cus : 256, rows = threads / 64 * 16 * R;
    const int64_t panels = (p.n + rows - 1) / rows, most = cus * ((160 * 1024) / (lds + 1024));
    BG_HIP(ctx, hipFuncSetAttribute((const void *)bgemm_f32_mfma_kernel<EPI, R, CT, GROUP, TAU>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    bgemm_f32_mfma_kernel<EPI, R, CT, GROUP, TAU>
        <<<(unsigned)(panels < most ? panels : most), threads, lds, s>>>(p, f);
    BG_LAUNCH_CHECK(ctx, "bgemm_f32_mfma");
    return BITGNN_OK;
}

template <int EPI>
int mf_launch_f32_epi(bitgnn_ctx *ctx, hipStream_t s, const MfArgs &p, const MfFloats &f)
{
    // loads of 64 floats in flight at a time: the size that fits the row with the fewest to spare
    const int sizes[6] = {10, 8, 6, 5, 4, 2};
    int best = 10;
    for (int k = 1; k < 6; ++k) // large ones first: of equal fits the one with fewer groups
        if ((f.votes + sizes[k] - 1) / sizes[k] * sizes[k] <
                (f.votes + best - 1) / best * best &&
            (sizes[k] >= 8 || f.votes <= sizes[k]))
            best = sizes[k];
#define BG_F32(G)                                                                                 \
    (f.tau ? mf_launch_f32_group<EPI, G, true>(ctx, s, p, f)                                      \
           : mf_launch_f32_group<EPI, G, false>(ctx, s, p, f))
    switch (best) {
    case 2: return BG_F32(2);
    case 4: return BG_F32(4);
    case 5: return BG_F32(5);
    case 6: return BG_F32(6);
    case 8: return BG_F32(8);
    default: return BG_F32(10);
    }
#undef BG_F32
}

} // namespace

// Whether the matrix-core kernel takes float rows of this shape, all its columns at once.
bool bg_bgemm_f32_mfma_applies(const bitgnn_ctx *ctx, int32_t K, int32_t M, int epilogue)
{
    if (ctx->bgemm_path == BITGNN_BGEMM_VALU)
        return false;
    const int64_t steps = ((int64_t)K + 127) / 128, row_words = 4 * (steps | 1);
    if (mf_tiles(M) * (steps * 1024 + 128) + 8 * (int64_t)kMfStage + 8 * 16 * row_words * 4 +
            ((int64_t)K + 64) * 4 > 160 * 1024)
        return false;
    if (ctx->bgemm_path == BITGNN_BGEMM_MFMA)
        return true;
    // Popcounts keep up with the stream of the features up to 128 channels, and lead by a few
    // per cent where a row is one chunk of theirs (K <= 640; 602 x 128, 233 K rows: 107 against
    // 112 us) -- unless rows are short (128 x 128: 65 against 35) or take two chunks (1000 x 100:
    // 211 against 186).  Short rows to wide floats are bound by the stores, theirs are a little
    // better (100 x 256, 233 K rows: 80 against 89).
    if (M > 128)
        return epilogue == BITGNN_EPI_THRESH_BITS || K > 128;
    return K <= 256 || (K > 640 && M > 64);
}

int bg_launch_bgemm_f32_mfma(bitgnn_ctx *ctx, hipStream_t s, const float *x, int64_t n, int32_t K,
                             int64_t ldx, const float *tau, const uint64_t *wbits, int32_t M,
                             int64_t w_stride, int epilogue, const int32_t *T, const float *alpha,
                             void *out, int64_t out_stride)
{
    MfArgs p{};
    p.n = n;
    p.K = K;
    p.kw32 = (K + 63) / 64 * 2;
    p.steps = (K + 127) / 128;
    p.w = (const uint32_t *)wbits;
    p.w_stride = w_stride * 2;
    p.M = M;
    p.tiles = mf_tiles(M);
    p.T = T;
    p.alpha = alpha;
    p.out = out;
    p.out_stride = out_stride;
    const MfFloats f{x, ldx, tau, (K + 63) / 64, 4 * (p.steps | 1)};
    switch (epilogue) {
    case BITGNN_EPI_THRESH_BITS:
        return mf_launch_f32_epi<BITGNN_EPI_THRESH_BITS>(ctx, s, p, f);
    case BITGNN_EPI_RAW_I32: return mf_launch_f32_epi<BITGNN_EPI_RAW_I32>(ctx, s, p, f);
    case kEpiRawI16: return mf_launch_f32_epi<kEpiRawI16>(ctx, s, p, f);
    default: return mf_launch_f32_epi<BITGNN_EPI_SCALE_F32>(ctx, s, p, f);
    }
}

// Whether the matrix-core kernel takes this shape.
bool bg_bgemm_mfma_applies(const bitgnn_ctx *ctx, int64_t n, int32_t kwords, int32_t M)
{
    if (ctx->bgemm_path == BITGNN_BGEMM_VALU)
        return false;
    const int32_t chunk = mf_chunk(kwords, M);
    if (chunk < M && chunk < 64)
        return false;
    if (ctx->bgemm_path == BITGNN_BGEMM_MFMA)
        return true;
    // a context without a GPU launches neither: the sizes it has always named
    if (ctx->device < 0)
        return kwords <= 16 && n >= (kwords > 8 ? 131072 : 65536);
    // every workgroup widens the weights first, about 1 us per 16 KB: with few rows the VALU
    // kernel is done by then (512 x 512, 128 KB: 10.0 against 13.1 us at 2,708 rows, level at 10 K;
    // 1000 x 1000, in seven chunks: 30 against 50 us at 10 K, 70 against 51 at 20 K)
    return n * 24 >= (int64_t)mf_tiles(M) * ((kwords + 1) / 2) * 1024;
}

int bg_launch_bgemm_mfma(bitgnn_ctx *ctx, hipStream_t s, const uint64_t *xbits, int64_t n,
                         int64_t x_stride, int32_t K, int32_t kwords, const uint64_t *wbits,
                         int32_t M, int64_t w_stride, int epilogue, const int32_t *T,
                         const float *alpha, void *out, int64_t out_stride)
{
    const int32_t chunk = mf_chunk(kwords, M);
    BG_REQUIRE(ctx, chunk >= M || chunk >= 64, BITGNN_ERR_UNSUPPORTED,
               "bitgnn_bgemm: shape too large for the matrix-core kernel");
    for (int32_t c0 = 0; c0 < M; c0 += chunk) {
        MfArgs p{};
        p.x = (const uint32_t *)xbits;
        p.n = n;
        p.x_stride = x_stride * 2;
        p.K = K;
        p.kw32 = kwords * 2;
        p.steps = (kwords + 1) / 2;
        p.w = (const uint32_t *)(wbits + (int64_t)c0 * w_stride);
        p.w_stride = w_stride * 2;
        p.M = M - c0 < chunk ? M - c0 : chunk;
        p.T = T ? T + c0 : nullptr;
        p.alpha = alpha ? alpha + c0 : nullptr;
        p.out = epilogue == BITGNN_EPI_THRESH_BITS ? (void *)((uint64_t *)out + c0 / 64)
                : epilogue == kEpiRawI16           ? (void *)((int16_t *)out + c0)
                                                   : (void *)((int32_t *)out + c0);
        p.out_stride = out_stride;
        int rc;
        switch (epilogue) {
        case BITGNN_EPI_THRESH_BITS: rc = mf_launch_epi<BITGNN_EPI_THRESH_BITS>(ctx, s, p); break;
        case BITGNN_EPI_RAW_I32: rc = mf_launch_epi<BITGNN_EPI_RAW_I32>(ctx, s, p); break;
        case kEpiRawI16: rc = mf_launch_epi<kEpiRawI16>(ctx, s, p); break;
        default: rc = mf_launch_epi<BITGNN_EPI_SCALE_F32>(ctx, s, p); break;
        }
        if (rc != BITGNN_OK)
            return rc;
    }
    return BITGNN_OK;
}
