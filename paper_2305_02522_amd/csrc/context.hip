// Context life cycle and error reporting.
#include "common.h"

#include <pthread.h>
#include <stdlib.h>

// ---------------------------------------------------------------- pool
namespace {
struct PoolNode {
    bg_block b;
    PoolNode *next;
};
} // namespace

struct bg_pool {
    pthread_mutex_t lock;
    PoolNode *kept; // newest first
    size_t bytes;
    int owners;
    bool closed;
};

bg_pool *bg_pool_create()
{
    bg_pool *pool = (bg_pool *)calloc(1, sizeof(bg_pool));
    if (pool) {
        pthread_mutex_init(&pool->lock, nullptr);
        pool->owners = 1;
    }
    return pool;
}

// The smallest kept block that wastes at most a quarter (or 64 KB), else a new one.
hipError_t bg_pool_take(bg_pool *pool, size_t bytes, bg_block *out)
{
    const size_t unit = bytes < ((size_t)1 << 20) ? 512 : (size_t)1 << 21;
    bytes = ((bytes ? bytes : 1) + unit - 1) / unit * unit;
    pthread_mutex_lock(&pool->lock);
    PoolNode **best = nullptr;
    for (PoolNode **q = &pool->kept; *q; q = &(*q)->next) {
        const size_t have = (*q)->b.bytes;
        if (have >= bytes && have <= bytes + bytes / 4 + 65536 &&
            (!best || have < (*best)->b.bytes))
            best = q;
    }
    if (best) {
        PoolNode *n = *best;
        *best = n->next;
        *out = n->b;
        pool->bytes -= n->b.bytes;
        free(n);
    }
    pthread_mutex_unlock(&pool->lock);
    if (best)
        return hipSuccess;
    out->bytes = bytes;
    hipError_t e = hipMalloc(&out->p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        bg_pool_trim(pool);
        e = hipMalloc(&out->p, bytes);
    }
    if (e != hipSuccess)
        *out = bg_block{};
    return e;
}

// Keeps the block; the ones kept longest go where that would exceed the bound.
void bg_pool_give(bg_pool *pool, bg_block b)
{
    if (!b.p)
        return;
    PoolNode *n = b.bytes <= kPoolBytes ? (PoolNode *)malloc(sizeof(PoolNode)) : nullptr;
    PoolNode *gone = nullptr;
    pthread_mutex_lock(&pool->lock);
    const bool keep = n && !pool->closed;
    if (keep) {
        *n = PoolNode{b, pool->kept};
        pool->kept = n;
        pool->bytes += b.bytes;
        size_t sum = 0;
        for (PoolNode **q = &pool->kept; *q; q = &(*q)->next) {
            sum += (*q)->b.bytes;
            if (sum > kPoolBytes) {
                gone = *q;
                *q = nullptr;
                pool->bytes = sum - gone->b.bytes;
                break;
            }
        }
    }
    pthread_mutex_unlock(&pool->lock);
    if (!keep) {
        (void)hipFree(b.p);
        free(n);
    }
    while (gone) {
        PoolNode *next = gone->next;
        (void)hipFree(gone->b.p);
        free(gone);
        gone = next;
    }
}

void bg_pool_trim(bg_pool *pool)
{
    pthread_mutex_lock(&pool->lock);
    PoolNode *n = pool->kept;
    pool->kept = nullptr;
    pool->bytes = 0;
    pthread_mutex_unlock(&pool->lock);
    while (n) {
        PoolNode *next = n->next;
        (void)hipFree(n->b.p);
        free(n);
        n = next;
    }
}

void bg_pool_hold(bg_pool *pool)
{
    pthread_mutex_lock(&pool->lock);
    ++pool->owners;
    pthread_mutex_unlock(&pool->lock);
}

void bg_pool_drop(bg_pool *pool)
{
    pthread_mutex_lock(&pool->lock);
    const bool last = --pool->owners == 0;
    pthread_mutex_unlock(&pool->lock);
    if (last) {
        bg_pool_trim(pool);
        pthread_mutex_destroy(&pool->lock);
        free(pool);
    }
}

void bg_pool_close(bg_pool *pool)
{
    pthread_mutex_lock(&pool->lock);
    pool->closed = true;
    pthread_mutex_unlock(&pool->lock);
    bg_pool_trim(pool);
    bg_pool_drop(pool);
}

// ---------------------------------------------------------------- life cycle
extern "C" int bitgnn_ctx_create(bitgnn_ctx **out, int device)
{
    if (!out || device < -1)
        return BITGNN_ERR_INVALID_ARG;
    bitgnn_ctx *ctx = (bitgnn_ctx *)calloc(1, sizeof(bitgnn_ctx));
    if (!ctx)
        return BITGNN_ERR_INVALID_ARG;
    ctx->device = device;
    ctx->cb_nodes = kMaxCbNodes;
    ctx->part_len = 255;
    ctx->min_avg_degree = 8;
    ctx->fused_spin_limit = 1u << 22;
    ctx->sc = &ctx->own;
    if (device >= 0) {
        int count = 0;
        hipError_t e = hipGetDeviceCount(&count);
        if (e != hipSuccess || device >= count) {
            free(ctx);
            return BITGNN_ERR_HIP;
        }
        e = hipSetDevice(device);
        if (e == hipSuccess)
            e = hipDeviceGetAttribute(&ctx->n_cus, hipDeviceAttributeMultiprocessorCount, device);
        if (e == hipSuccess)
            e = hipMalloc((void **)&ctx->own.queue, 256);
        if (e == hipSuccess)
            e = hipMemset(ctx->own.queue, 0, 256);
        if (e == hipSuccess)
            e = hipMalloc((void **)&ctx->own.seed_table, kSeedTableWords * sizeof(uint32_t));
        if (e == hipSuccess)
            e = hipHostMalloc(&ctx->mail, kMailBytes, hipHostMallocDefault);
        if (e == hipSuccess && !(ctx->pool = bg_pool_create()))
            e = hipErrorOutOfMemory;
        if (e != hipSuccess) {
            if (ctx->mail)
                (void)hipHostFree(ctx->mail);
            if (ctx->own.queue)
                (void)hipFree(ctx->own.queue);
            if (ctx->own.seed_table)
                (void)hipFree(ctx->own.seed_table);
            free(ctx);
            return BITGNN_ERR_HIP;
        }
        ctx->own.seed_table_words = kSeedTableWords;
        if (bg_static_scratch_init(ctx) != BITGNN_OK) {
            bitgnn_ctx_destroy(ctx);
            return BITGNN_ERR_HIP;
        }
    }
    *out = ctx;
    return BITGNN_OK;
}

extern "C" void bitgnn_ctx_destroy(bitgnn_ctx *ctx)
{
    if (!ctx)
        return;
    if (ctx->own.seed_table)
        (void)hipFree(ctx->own.seed_table);
    if (ctx->own.queue)
        (void)hipFree(ctx->own.queue);
    if (ctx->own.ws)
        (void)hipFree(ctx->own.ws);
    while (ctx->retired) {
        bg_retired *r = ctx->retired;
        ctx->retired = r->next;
        (void)hipFree(r->p);
        free(r);
    }
    if (ctx->pool)
        bg_pool_close(ctx->pool);
    if (ctx->mail)
        (void)hipHostFree(ctx->mail);
    for (int i = 0; i < 2 * kMaxTimed; ++i)
        if (ctx->tev[i])
            (void)hipEventDestroy(ctx->tev[i]);
    free(ctx);
}

extern "C" const char *bitgnn_last_error(const bitgnn_ctx *ctx) { return ctx ? ctx->err : ""; }

extern "C" int bitgnn_ctx_set_tuning(bitgnn_ctx *ctx, int32_t cb_nodes, int32_t part_len,
                                     int32_t min_avg_degree)
{
    if (!ctx)
        return BITGNN_ERR_INVALID_ARG;
    BG_REQUIRE(ctx, cb_nodes >= 64 && cb_nodes <= kMaxCbNodes && part_len >= 4 && part_len <= 1023 &&
                        min_avg_degree >= 0,
               BITGNN_ERR_INVALID_ARG,
               "bitgnn_ctx_set_tuning: cb_nodes=%d (64..10208) part_len=%d (4..1023) "
               "min_avg_degree=%d (>= 0)",
               cb_nodes, part_len, min_avg_degree);
    ctx->cb_nodes = cb_nodes;
    ctx->part_len = part_len;
    ctx->min_avg_degree = min_avg_degree;
    return BITGNN_OK;
}

extern "C" int bitgnn_ctx_set_bgemm_path(bitgnn_ctx *ctx, int path)
{
    if (!ctx)
        return BITGNN_ERR_INVALID_ARG;
    BG_REQUIRE(ctx, path >= BITGNN_BGEMM_AUTO && path <= BITGNN_BGEMM_MFMA, BITGNN_ERR_INVALID_ARG,
               "bitgnn_ctx_set_bgemm_path: path=%d (0 auto, 1 VALU, 2 matrix cores)", path);
    ctx->bgemm_path = path;
    return BITGNN_OK;
}

extern "C" int bitgnn_ctx_bgemm_kernel(const bitgnn_ctx *ctx, int64_t n, int32_t kwords, int32_t M,
                                       int *kernel)
{
    if (!ctx || !kernel || n < 0 || kwords < 1 || M < 1)
        return BITGNN_ERR_INVALID_ARG;
    *kernel = bg_bgemm_mfma_applies(ctx, n, kwords, M) ? BITGNN_BGEMM_MFMA : BITGNN_BGEMM_VALU;
    return BITGNN_OK;
}

// The aggregation workspace.  Only this set-up call (and bitgnn_adj_build, through it)
// allocates: it may synchronize the device to replace a smaller workspace.  One that a recorded
// call works in is kept until the context is destroyed, because the graph may be replayed.
extern "C" int bitgnn_ctx_reserve(bitgnn_ctx *ctx, size_t bytes)
{
    if (!ctx)
        return BITGNN_ERR_INVALID_ARG;
    BG_NEED_DEVICE(ctx);
    bg_scratch &own = ctx->own;
    if (bytes <= own.ws_bytes)
        return BITGNN_OK;
    bytes = (bytes + (1u << 20)) & ~(size_t)((1u << 20) - 1);
    if (own.ws && own.ws_recorded) {
        bg_retired *r = (bg_retired *)malloc(sizeof(bg_retired));
        BG_REQUIRE(ctx, r, BITGNN_ERR_INVALID_ARG, "bitgnn_ctx_reserve: out of host memory");
        void *ws = nullptr;
        hipError_t e = hipMalloc(&ws, bytes);
        if (e == hipErrorOutOfMemory) { // the builds' kept memory first
            (void)hipGetLastError();
            bg_pool_trim(ctx->pool);
            e = hipMalloc(&ws, bytes);
        }
        if (e != hipSuccess)
            free(r);
        BG_HIP(ctx, e);
        *r = bg_retired{own.ws, ctx->retired};
        ctx->retired = r;
        own.ws = ws;
    } else {
        if (own.ws) {
            BG_HIP(ctx, hipDeviceSynchronize());
            BG_HIP(ctx, hipFree(own.ws));
            own.ws = nullptr;
            own.ws_bytes = 0;
        }
        hipError_t e = hipMalloc(&own.ws, bytes);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            bg_pool_trim(ctx->pool);
            e = hipMalloc(&own.ws, bytes);
        }
        BG_HIP(ctx, e);
    }
    own.ws_bytes = bytes;
    own.ws_recorded = false;
    return BITGNN_OK;
}

extern "C" int bitgnn_ctx_workspace(const bitgnn_ctx *ctx, size_t *bytes)
{
    if (!ctx || !bytes)
        return BITGNN_ERR_INVALID_ARG;
    *bytes = ctx->own.ws_bytes;
    return BITGNN_OK;
}

// Compute calls never allocate: a workspace that is too small is an error.  Notes whether the
// call is being recorded (the null stream cannot be; where the runtime gives no answer, it may).
int bg_ws_need(bitgnn_ctx *ctx, hipStream_t s, size_t bytes, const char *who)
{
    if (bytes > ctx->sc->ws_bytes)
        return bitgnn_fail(ctx, BITGNN_ERR_WORKSPACE,
                           "%s: needs %zu bytes of workspace, %zu available "
                           "(bitgnn_adj_workspace_bytes + bitgnn_ctx_reserve)",
                           who, bytes, ctx->sc->ws_bytes);
    if (s && !ctx->sc->ws_recorded) {
        hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
        const bool known = hipStreamIsCapturing(s, &st) == hipSuccess;
        if (!known)
            (void)hipGetLastError();
        ctx->sc->ws_recorded = !known || st != hipStreamCaptureStatusNone;
    }
    return BITGNN_OK;
}

extern "C" int bitgnn_ctx_kernel_timing(bitgnn_ctx *ctx, int enable)
{
    if (!ctx)
        return BITGNN_ERR_INVALID_ARG;
    BG_NEED_DEVICE(ctx);
    if (enable && !ctx->tev[0])
        for (int i = 0; i < 2 * kMaxTimed; ++i)
            BG_HIP(ctx, hipEventCreate(&ctx->tev[i]));
    ctx->timing = enable ? 1 : 0;
    ctx->n_timed = 0;
    return BITGNN_OK;
}

extern "C" int bitgnn_ctx_kernel_times(bitgnn_ctx *ctx, float *ms, int32_t capacity,
                                       int32_t *count)
{
    if (!ctx)
        return BITGNN_ERR_INVALID_ARG;
    BG_REQUIRE(ctx, ms && count && capacity >= 0, BITGNN_ERR_INVALID_ARG,
               "bitgnn_ctx_kernel_times: null pointer or negative capacity");
    BG_NEED_DEVICE(ctx);
    int k = 0;
    for (; k < ctx->n_timed && k < capacity; ++k) {
        BG_HIP(ctx, hipEventSynchronize(ctx->tev[2 * k + 1]));
        BG_HIP(ctx, hipEventElapsedTime(&ms[k], ctx->tev[2 * k], ctx->tev[2 * k + 1]));
    }
    *count = k;
    ctx->n_timed = 0;
    return BITGNN_OK;
}
