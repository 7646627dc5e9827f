// Embedding synchronisation between the hot tables and the full tables (Sec. 3 (4);
// Sec. 6.2, "Embedding Synchronization"): when training switches between hot and cold
// mini-batches, the hot rows are copied back to their places in the full tables, or
// fetched from there again.  One launch covers all tables.
//
// A pure row copy: per hot row 4 bytes of id, dim*4 bytes read and dim*4 bytes written.
// The hot side is a stream; the full-table side is rows of dim*4 bytes at ascending but
// scattered addresses (hot ids ascend with the slot).  A lane moves 16 bytes, a thread
// has four independent copies in flight.
#include "fae_internal.h"

#define SYNC_THREADS 256
#define SYNC_UNROLL 4

struct SyncArgs {
    float *hotW[FAE_MAX_TABLES];
    float *W[FAE_MAX_TABLES];
    const int32_t *hot_ids[FAE_MAX_TABLES];
    int64_t rows[FAE_MAX_TABLES];
    int64_t n_vec[FAE_MAX_TABLES];         // n_hot_z * (dim / vector width)
    int64_t blk_start[FAE_MAX_TABLES + 1]; // 64-bit: a 64 GiB hot set has more than 2^31 vectors
    int32_t n_tables, dim, to_full;
    uint32_t *status;
};

typedef float sync_v4 __attribute__((ext_vector_type(4)));
template <bool STREAM> __device__ __forceinline__ float4 sync_load(const float4 *p)
{
    if (!STREAM)
        return *p;
    const sync_v4 v = __builtin_nontemporal_load((const sync_v4 *)p);
    return make_float4(v.x, v.y, v.z, v.w);
}
template <bool STREAM> __device__ __forceinline__ float sync_load(const float *p)
{
    return STREAM ? __builtin_nontemporal_load(p) : *p;
}
template <bool STREAM> __device__ __forceinline__ void sync_store(float4 *p, const float4 &v)
{
    const sync_v4 t = {v.x, v.y, v.z, v.w};
    if (STREAM)
        __builtin_nontemporal_store(t, (sync_v4 *)p);
    else
        *p = v;
}
template <bool STREAM> __device__ __forceinline__ void sync_store(float *p, float v)
{
    if (STREAM)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// Bytes of hot rows from which on both sides are streamed past the caches.  Nothing that is copied is
// read again by the launch, but the other direction or a training step comes next, and below, the hot rows
// and their places in the full tables are still in the last-level cache (256 MB) by then.  Both
// directions, microseconds, cached / streamed: 49 MiB 31.8 / 41.7, 98 MiB 59.4 / 76.2, 146 MiB 93.8 / 111.9,
// 159 MiB 118.6 / 121.2, 195 MiB 162.9 / 147.1, 391 MiB 316 / 291; one direction and a forward: 98 MiB
// 44.5 / 50.5, 146 MiB 70.2 / 68.7, 159 MiB 86.9 / 80.9, 195 MiB 95.3 / 84.9 (10 MiB: no difference).
#define SYNC_STREAM_BYTES (144LL << 20)

// A workgroup takes 1024 consecutive vectors; a vector's row comes from one division per workgroup
// and a small offset, which shortens the small copies (a division and a walk over the tables per vector
// before: both directions of 8 x 10 000 rows of 64 41 -> 25 us).  0.92 M rows of 64, streamed, one
// direction: 102 -> 88 us, 4.6 -> 5.4 TB/s.
template <typename V, bool STREAM> __global__ __launch_bounds__(SYNC_THREADS) void sync_rows_kernel(SyncArgs a)
{
    constexpr int VW = sizeof(V) / sizeof(float);
    const int64_t b = blockIdx.x;
    const int z = fae_find_table(a.blk_start, a.n_tables, b);
    const uint32_t ncols = (uint32_t)a.dim / VW;
    const int64_t base = (b - a.blk_start[z]) * (SYNC_THREADS * SYNC_UNROLL);
    const int64_t slot0 = fae_div_small(base, ncols);
    const uint32_t c0 = (uint32_t)(base - slot0 * ncols);
    const int64_t left = a.n_vec[z] - base; // at least one: the grid has no empty workgroup
    const int32_t *ids = a.hot_ids[z] + slot0;
    V *hot = (V *)a.hotW[z];
    V *full = (V *)a.W[z];
    int64_t src[SYNC_UNROLL], dst[SYNC_UNROLL];
    int32_t row[SYNC_UNROLL];
    uint32_t c[SYNC_UNROLL];
    bool bad = false;
#pragma unroll
    for (int k = 0; k < SYNC_UNROLL; ++k) { // every id is asked for before the first is looked at
        const uint32_t i = k * SYNC_THREADS + threadIdx.x;
        const uint32_t q = c0 + i, ds = q / ncols;
        c[k] = q - ds * ncols;
        row[k] = (int64_t)i < left ? ids[ds] : 0;
    }
#pragma unroll
    for (int k = 0; k < SYNC_UNROLL; ++k) {
        const uint32_t i = k * SYNC_THREADS + threadIdx.x;
        src[k] = dst[k] = -1;
        if ((int64_t)i >= left)
            continue;
        if (row[k] < 0 || row[k] >= a.rows[z]) {
            bad = true; // never dereferenced
        } else {
            const int64_t e = base + i, f = (int64_t)row[k] * ncols + c[k];
            src[k] = a.to_full ? e : f;
            dst[k] = a.to_full ? f : e;
        }
    }
    const V *from = a.to_full ? hot : full;
    V *to = a.to_full ? full : hot;
    V v[SYNC_UNROLL];
#pragma unroll
    for (int k = 0; k < SYNC_UNROLL; ++k)
        if (src[k] >= 0)
            v[k] = sync_load<STREAM>(from + src[k]);
#pragma unroll
    for (int k = 0; k < SYNC_UNROLL; ++k)
        if (src[k] >= 0)
            sync_store<STREAM>(to + dst[k], v[k]);
    if (bad)
        fae_flag(a.status, FAE_STATUS_ERANGE);
}

extern "C" int32_t fae_sync_hot_rows(fae_ctx *ctx, const fae_tables *tables, const int64_t *h_n_hot,
                                     const int32_t *const *h_hot_ids, float *const *h_hotW,
                                     float *const *h_W, int32_t direction)
{
    int32_t rc = fae_check_tables(ctx, tables, "fae_sync_hot_rows");
    if (rc != FAE_OK)
        return rc;
    if (!h_n_hot || !h_hot_ids || !h_hotW || !h_W)
        return fae_fail(ctx, FAE_EINVAL, "fae_sync_hot_rows: null argument");
    if (direction != FAE_SYNC_HOT_TO_FULL && direction != FAE_SYNC_FULL_TO_HOT)
        return fae_fail(ctx, FAE_EINVAL, "fae_sync_hot_rows: unknown direction %d", direction);
    const int nt = tables->n_tables, dim = tables->dim;
    bool vec = dim % 4 == 0;
    SyncArgs a;
    memset(&a, 0, sizeof(a));
    for (int z = 0; z < nt; ++z) {
        if (h_n_hot[z] < 0 || h_n_hot[z] > tables->h_rows[z])
            return fae_fail(ctx, FAE_EINVAL, "fae_sync_hot_rows: n_hot[%d]=%lld outside [0, rows]", z,
                            (long long)h_n_hot[z]);
        if (h_n_hot[z] > 0 && (!h_hot_ids[z] || !h_hotW[z] || !h_W[z]))
            return fae_fail(ctx, FAE_EINVAL, "fae_sync_hot_rows: null pointer for table %d", z);
        vec = vec && ((((uintptr_t)h_hotW[z]) | ((uintptr_t)h_W[z])) & 15) == 0;
    }
    const int vw = vec ? 4 : 1;
    int64_t blocks = 0, bytes = 0;
    for (int z = 0; z < nt; ++z) {
        bytes += h_n_hot[z] * dim * 4;
        a.hotW[z] = h_hotW[z];
        a.W[z] = h_W[z];
        a.hot_ids[z] = h_hot_ids[z];
        a.rows[z] = tables->h_rows[z];
        a.n_vec[z] = h_n_hot[z] * (dim / vw);
        a.blk_start[z] = blocks;
        blocks += (a.n_vec[z] + SYNC_THREADS * SYNC_UNROLL - 1) / (SYNC_THREADS * SYNC_UNROLL);
    }
    a.blk_start[nt] = blocks;
    a.n_tables = nt;
    a.dim = dim;
    a.to_full = direction == FAE_SYNC_HOT_TO_FULL;
    a.status = ctx->d_block;
    if (blocks == 0)
        return FAE_OK;
    if (blocks > 2147483647LL)
        return fae_fail(ctx, FAE_EINVAL, "fae_sync_hot_rows: more than 2^31 workgroups; split the call by tables");
    FAE_HIP(ctx, hipSetDevice(ctx->device));
    fae_ktimer kt(ctx, FAE_K_SYNC_ROWS);
    const dim3 grid((unsigned)blocks), block(SYNC_THREADS);
    const bool stream = bytes >= SYNC_STREAM_BYTES;
    if (vec && stream)
        FAE_LAUNCH(ctx, (sync_rows_kernel<float4, true>), grid, block, 0, ctx->stream, a);
    else if (vec)
        FAE_LAUNCH(ctx, (sync_rows_kernel<float4, false>), grid, block, 0, ctx->stream, a);
    else if (stream)
        FAE_LAUNCH(ctx, (sync_rows_kernel<float, true>), grid, block, 0, ctx->stream, a);
    else
        FAE_LAUNCH(ctx, (sync_rows_kernel<float, false>), grid, block, 0, ctx->stream, a);
    FAE_LAUNCH_CHECK(ctx);
    return FAE_OK;
}
