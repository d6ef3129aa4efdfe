// ADD: the auxiliary element-wise merge of two activation tensors (Section 3.1.2: the
// self-connectivity of GraphSAGE is merged with ADD.BBF or ADD.FFF), with the operands in
// packed +-1 bits or in floats, and the result in floats or binarized again (BIN folded in,
// as the other low-level functions do).
//
// gfx950 mapping: 16 lanes take a 64-channel tile of a row, 4 channels each: 16 bytes of a
// float operand, one broadcast 8-byte word of a bit operand.  A wavefront's 64 lanes take four
// adjacent tiles (1 KB of a float operand per load) and go on by four tiles a turn, four turns
// in flight.  The thresholded bits of a lane are a nibble; four DPP OR steps leave the tile's
// word in all 16 lanes, each lane keeps the word of one turn and the wavefront stores all its
// words at once.  Bound by the HBM stream of the operands / result: 300,001 x 100 floats, two
// operands to bits, 62 -> 36 us against one channel per lane and one tile per wavefront and
// turn; 131,072 x 128 floats to floats 31 -> 32, 19,717 x 256 11.3 -> 10.1 (16 consecutive
// tiles per 16 lanes had taken 38 and 13.2 there).
#include "common.h"

namespace {

constexpr int kAddBlock = 256;
constexpr int kAddUnroll = 4;

// Four channels of a row of an operand, from k on (k + 4 <= C for float rows).
template <bool BITS> struct add_piece {
    float v[4];
    __device__ __forceinline__ void load(const void *p, int64_t ofs, int32_t k)
    {
        __builtin_memcpy(v, (const float *)p + ofs + k, sizeof(v));
    }
    __device__ __forceinline__ float at(int j, int32_t) const { return v[j]; }
};
template <> struct add_piece<true> {
    uint64_t w[2]; // the words of channel k and of channel k + 3
    __device__ __forceinline__ void load(const void *p, int64_t ofs, int32_t k)
    {
        w[0] = ((const uint64_t *)p)[ofs + (k >> 6)];
        w[1] = ((const uint64_t *)p)[ofs + ((k + 3) >> 6)];
    }
    __device__ __forceinline__ float at(int j, int32_t k) const
    {
        const uint64_t x = ((k + j) >> 6) == (k >> 6) ? w[0] : w[1];
        return ((x >> ((k + j) & 63)) & 1ull) ? 1.0f : -1.0f;
    }
};

__device__ __forceinline__ uint32_t or_row16(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);  // quad [1,0,3,2]
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);  // quad [2,3,0,1]
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false); // half-row mirror
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false); // row mirror
    return v;
}

// C >= 4: a lane at the end of a row is moved back to end with it (it then shares channels with
// its neighbour lane; its nibble is shifted to match).
template <bool A_BITS, bool B_BITS, bool BITS_OUT>
__global__ __launch_bounds__(kAddBlock) void add4_kernel(const void *__restrict__ a, int64_t lda,
                                                         const void *__restrict__ b, int64_t ldb,
                                                         int64_t n, int32_t C, int32_t tiles,
                                                         int32_t turns,
                                                         const float *__restrict__ tau,
                                                         void *__restrict__ out, int64_t ldo)
{
    const int lane = threadIdx.x & 63, sub = lane & 15, grp = lane >> 4;
    const int64_t wave = (int64_t)blockIdx.x * (kAddBlock / 64) +
                         __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t total = n * (int64_t)tiles;
    const int64_t q0 = wave * (4 * turns); // first tile of this wavefront
    if (q0 >= total)
        return;
    // four tiles a turn, one per 16 lanes; the first row is wave-uniform, the tiles' rows follow in
    // 32 bits
    const int64_t rowb = q0 / tiles;
    const uint32_t offb = (uint32_t)(q0 - rowb * tiles) + (uint32_t)grp;
    uint32_t drow = offb / (uint32_t)tiles;
    int32_t t = (int32_t)(offb - drow * (uint32_t)tiles);
    const uint32_t turn_rows = 4u / (uint32_t)tiles;
    const int32_t turn_tiles = 4 - (int32_t)turn_rows * tiles;
    const int64_t last = n - 1 - rowb;
    const uint32_t dlast = last > 64 ? 64u : (uint32_t)last; // rows past the last are clamped
    uint32_t mine_lo = 0, mine_hi = 0, mine_drow = 0;
    int32_t mine_t = 0;
    for (int i0 = 0; i0 < turns; i0 += kAddUnroll) {
        add_piece<A_BITS> va[kAddUnroll];
        add_piece<B_BITS> vb[kAddUnroll];
        float tv[kAddUnroll][4];
        int32_t kk[kAddUnroll], kn[kAddUnroll];
        int64_t row[kAddUnroll];
        bool ok[kAddUnroll];
#pragma unroll
        for (int u = 0; u < kAddUnroll; ++u) {
            ok[u] = drow <= dlast;
            row[u] = rowb + (ok[u] ? drow : dlast);
            kn[u] = t * 64 + 4 * sub;
            kk[u] = kn[u] < C - 4 ? kn[u] : C - 4;
            va[u].load(a, row[u] * lda, kk[u]);
            vb[u].load(b, row[u] * ldb, kk[u]);
            if (BITS_OUT)
                __builtin_memcpy(tv[u], tau + kk[u], sizeof(tv[u]));
            if (sub == i0 + u) {
                mine_drow = drow;
                mine_t = t;
            }
            drow += turn_rows;
            t += turn_tiles;
            if (t >= tiles) {
                t -= tiles;
                ++drow;
            }
        }
#pragma unroll
        for (int u = 0; u < kAddUnroll; ++u) {
            float y[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                y[j] = va[u].at(j, kk[u]) + vb[u].at(j, kk[u]);
            if (BITS_OUT) {
                uint32_t nib = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    nib |= y[j] >= tv[u][j] ? 1u << j : 0u;
                const uint32_t back = (uint32_t)(kn[u] - kk[u]);
                nib = back < 4u ? nib >> back : 0u;
                const uint32_t placed = nib << (4 * (sub & 7));
                const uint32_t lo = or_row16(sub < 8 ? placed : 0u);
                const uint32_t hi = or_row16(sub < 8 ? 0u : placed);
                if (sub == i0 + u) {
                    mine_lo = lo;
                    mine_hi = hi;
                }
            } else if (ok[u] && kn[u] < C) {
                __builtin_memcpy((float *)out + row[u] * ldo + kk[u], y, sizeof(y));
            }
        }
    }
    if (BITS_OUT && sub < turns && q0 + 4 * sub + grp < total)
        ((uint64_t *)out)[(rowb + mine_drow) * ldo + mine_t] = ((uint64_t)mine_hi << 32) | mine_lo;
}

// Rows of fewer than 4 channels: one row per thread.
template <bool A_BITS, bool B_BITS, bool BITS_OUT>
__global__ __launch_bounds__(kAddBlock) void add_narrow_kernel(const void *__restrict__ a,
                                                               int64_t lda,
                                                               const void *__restrict__ b,
                                                               int64_t ldb, int64_t n, int32_t C,
                                                               const float *__restrict__ tau,
                                                               void *__restrict__ out, int64_t ldo)
{
    const int64_t row = (int64_t)blockIdx.x * kAddBlock + threadIdx.x;
    if (row >= n)
        return;
    uint64_t word = 0;
    for (int32_t c = 0; c < C; ++c) {
        const float va = A_BITS ? ((((const uint64_t *)a)[row * lda] >> c) & 1ull ? 1.0f : -1.0f)
                                : ((const float *)a)[row * lda + c];
        const float vb = B_BITS ? ((((const uint64_t *)b)[row * ldb] >> c) & 1ull ? 1.0f : -1.0f)
                                : ((const float *)b)[row * ldb + c];
        const float y = va + vb;
        if (BITS_OUT)
            word |= (uint64_t)(y >= tau[c]) << c;
        else
            ((float *)out)[row * ldo + c] = y;
    }
    if (BITS_OUT)
        ((uint64_t *)out)[row * ldo] = word;
}

} // namespace

extern "C" int bitgnn_add(bitgnn_ctx *ctx, void *stream, const void *a, int a_is_bits,
                          int64_t lda, const void *b, int b_is_bits, int64_t ldb, int64_t n,
                          int32_t C, int epilogue, const float *tau, void *out, int64_t ldo)
{
    if (!ctx)
        return BITGNN_ERR_INVALID_ARG;
    BG_REQUIRE(ctx, n >= 0 && C >= 1, BITGNN_ERR_INVALID_ARG, "bitgnn_add: n=%lld C=%d",
               (long long)n, C);
    const int64_t words = ((int64_t)C + 63) / 64;
    const bool bits_out = epilogue == BITGNN_EPI_THRESH_BITS;
    BG_REQUIRE(ctx, bits_out || epilogue == BITGNN_EPI_SCALE_F32, BITGNN_ERR_INVALID_ARG,
               "bitgnn_add: epilogue %d (THRESH_BITS or SCALE_F32)", epilogue);
    BG_REQUIRE(ctx, !bits_out || tau, BITGNN_ERR_INVALID_ARG,
               "bitgnn_add: THRESH_BITS needs tau");
    BG_REQUIRE(ctx, lda >= (a_is_bits ? words : C) && ldb >= (b_is_bits ? words : C) &&
                        ldo >= (bits_out ? words : C),
               BITGNN_ERR_INVALID_ARG, "bitgnn_add: lda=%lld ldb=%lld ldo=%lld too small for C=%d",
               (long long)lda, (long long)ldb, (long long)ldo, C);
    if (n == 0)
        return BITGNN_OK;
    BG_REQUIRE(ctx, a && b && out, BITGNN_ERR_INVALID_ARG, "bitgnn_add: null pointer");
    BG_REQUIRE(ctx, bg_aligned(a, a_is_bits ? 8 : 4) && bg_aligned(b, b_is_bits ? 8 : 4) &&
                        bg_aligned(out, bits_out ? 8 : 4) && bg_aligned(tau, 4),
               BITGNN_ERR_ALIGNMENT, "bitgnn_add: misaligned pointer");
    BG_NEED_DEVICE(ctx);
    hipStream_t s = (hipStream_t)stream;
    // A launch takes fewer than 2^32 threads: rows in chunks of at most 2^28 tiles.
    const int64_t chunk = C >= 4 ? (1ll << 28) / words : 1ll << 30;
    for (int64_t r0 = 0; r0 < n; r0 += chunk) {
        const int64_t rows = n - r0 < chunk ? n - r0 : chunk;
        // 16 turns store 64 words at once; below 2^18 tiles (8 wavefronts of 4 turns per SIMD and
        // two rounds) 4 turns, so that more wavefronts share the work: 19,717 x 500, bits and
        // floats to bits 15.4 us with 16 turns, 9.5 with 4.
        const int turns = rows * words < 1 << 18 ? 4 : 16;
        const int64_t threads =
            C >= 4 ? (rows * words + 4 * turns - 1) / (4 * turns) * 64 : rows;
        const unsigned blocks = (unsigned)((threads + kAddBlock - 1) / kAddBlock);
        const void *pa = (const char *)a + r0 * lda * (a_is_bits ? 8 : 4);
        const void *pb = (const char *)b + r0 * ldb * (b_is_bits ? 8 : 4);
        void *po = (char *)out + r0 * ldo * (bits_out ? 8 : 4);
#define BG_ADD(AB, BB, OB)                                                                        \
    do {                                                                                          \
        if (C >= 4)                                                                               \
            add4_kernel<AB, BB, OB><<<blocks, kAddBlock, 0, s>>>(                                 \
                pa, lda, pb, ldb, rows, C, (int32_t)words, turns, tau, po, ldo);                  \
        else                                                                                      \
            add_narrow_kernel<AB, BB, OB><<<blocks, kAddBlock, 0, s>>>(pa, lda, pb, ldb, rows, C, \
                                                                       tau, po, ldo);             \
    } while (0)
        switch ((a_is_bits ? 4 : 0) | (b_is_bits ? 2 : 0) | (bits_out ? 1 : 0)) {
        case 0: BG_ADD(false, false, false); break;
        case 1: BG_ADD(false, false, true); break;
        case 2: BG_ADD(false, true, false); break;
        case 3: BG_ADD(false, true, true); break;
        case 4: BG_ADD(true, false, false); break;
        case 5: BG_ADD(true, false, true); break;
        case 6: BG_ADD(true, true, false); break;
        default: BG_ADD(true, true, true); break;
        }
#undef BG_ADD
    }
    BG_LAUNCH_CHECK(ctx, "add_kernel");
    return BITGNN_OK;
}
