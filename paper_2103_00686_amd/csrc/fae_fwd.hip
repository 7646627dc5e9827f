// Hot mini-batch forward: row gather + sum pooling over HBM-resident hot tables.
//
// One launch covers every table of the batch; each table has the lane mapping of its bags:
//   group-per-bag : LPR adjacent lanes own one bag, each lane one 16-byte column
//                   slice; bags of a wave sit side by side (best for one-hot / short bags);
//   wave-per-bag  : the 64/LPR lane groups of a wave take alternate entries of one
//                   bag and are combined with cross-lane shuffles (best for long,
//                   uneven bags: no lane group idles while its neighbour finishes).
// Bandwidth bound: per lookup one slot (4 B) and one row (dim*4 B) are read, per bag
// one row is written.  No arithmetic beyond one add per loaded float.
#include "fae_internal.h"
#include "fae_device.h"

enum { FWD_ONEHOT, FWD_GROUP, FWD_WAVE };

struct FwdArgs {
    const float *W[FAE_MAX_TABLES];
    const int32_t *slots[FAE_MAX_TABLES];
    const int32_t *offsets[FAE_MAX_TABLES];
    int32_t n_hot[FAE_MAX_TABLES];
    int32_t n_lookups[FAE_MAX_TABLES];
    int32_t blk_start[FAE_MAX_TABLES + 1];
    int32_t kind[FAE_MAX_TABLES]; // FWD_ONEHOT, FWD_GROUP or FWD_WAVE
    int32_t n_tables;
    int32_t dim;
    int32_t n_samples;
    int64_t out_stride;
    float *out;
    uint32_t *status;
    int32_t stream_out; // non-temporal stores for the pooled output
    int32_t mean;       // divide the pooled sum by the bag's length (bags of one lookup are unaffected)
};

// Sums of up to FWD_PLAIN_MAX terms per lane group are plain ones (worst case FWD_PLAIN_MAX * 2^-24
// of the sum of their magnitudes, inside the 1e-5 the result is held to); longer sums carry the
// rounding error along (COMP), so that a bag of thousands of lookups stays as accurate as a short
// one, also when it adds one popular row over and over, which otherwise drifts one way.
#define FWD_PLAIN_MAX 128

// A lane group that owns a bag alone adds the rows it has in flight in pairs, about FWD_PART rows into one
// part and the parts up: for a bag of n rows chains of FWD_PART / 4 and n / FWD_PART additions, about what
// a wave's lane groups have when they share the bag.  Which of the two a table gets goes by its own average
// length, and its rounding error should not (bags of 1-6 and one of 120 in forty, dim 16, against 64 bits:
// one after the other 1.4e-7, shared 6.0e-8, in parts 6.2e-8; dim 64: 1.4e-7, 7.8e-8, 6.2e-8; same time).
// A part ends with the slots at hand (LPR rows), with fewer than eight lanes after FWD_PART rows of the bag.
#define FWD_PART 16
template <typename V, int N> __device__ __forceinline__ void fwd_add_pairs(V &part, V (&v)[N])
{
#pragma unroll
    for (int m = N / 2; m > 0; m /= 2)
#pragma unroll
        for (int i = 0; i < m; ++i) {
            v[i] = v[2 * i];
            vec_ops<V>::add(v[i], v[2 * i + 1]);
        }
    vec_ops<V>::add(part, v[0]);
}
template <typename V> __device__ __forceinline__ void fwd_end_part(V &acc, V &part)
{
    vec_ops<V>::add(acc, part);
    part = vec_ops<V>::zero();
}

// Adds rows of a bag whose next WIDTH slots are held one per lane by the lanes of a lane group of
// WIDTH lanes: this group's rows are numbers first, first + STRIDE, ... below count.  UN rows are in
// flight; the slots are already there, so a row costs one round trip and not two in a row.
template <typename V, int WIDTH, int STRIDE, int UN, bool COMP>
__device__ __forceinline__ void fwd_add_rows(V &acc, V &lost, const V *W, int slot, int first, int count, int ncols, int c, bool active)
{
    for (int j = first; j - first < count; j += STRIDE * UN) { // every lane of the WIDTH stays in: they hold the slots
        V v[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int e = j + u * STRIDE;
            const int sl = __shfl(slot, e, WIDTH); // e wraps inside the group past its end: not used then
            v[u] = (active && e < count && sl >= 0) ? W[(int64_t)sl * ncols + c] : vec_ops<V>::zero();
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            if (!COMP)
                vec_ops<V>::add(acc, v[u]);
            else if (j + u * STRIDE < count) // a zero behind an infinite sum would make it NaN: inf - inf in the carried error
                vec_ops<V>::add_comp(acc, lost, v[u]);
        }
    }
}

// The same for a lane group that owns its bag alone (plain sum); done: rows of the bag that are in already
template <typename V, int LPR>
__device__ __forceinline__ void fwd_add_parts(V &acc, V &part, const V *W, int slot, int count, uint32_t done, int ncols, int c, bool active)
{
    for (int j = 0; j < count; j += 4) {
        V v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int sl = __shfl(slot, j + u, LPR); // LPR is a multiple of 4
            v[u] = (active && j + u < count && sl >= 0) ? W[(int64_t)sl * ncols + c] : vec_ops<V>::zero();
        }
        fwd_add_pairs(part, v);
    }
    if (LPR >= 8 || (done + LPR) % FWD_PART == 0)
        fwd_end_part(acc, part);
}

// lane 0's or lane 1's value of a group of one or two lanes (both are active); from: known at compile time
template <int LPR> __device__ __forceinline__ int fwd_pair_lane(int v, int from)
{
    if (LPR == 1)
        return v;
    return from == 0 ? __builtin_amdgcn_mov_dpp(v, 0xA0, 0xf, 0xf, false)  // lanes 0, 0, 2, 2 of every four
                     : __builtin_amdgcn_mov_dpp(v, 0xF5, 0xf, 0xf, false); // lanes 1, 1, 3, 3
}

// The same for a lane group of one or two lanes, which takes eight lookups at a time, j0 .. j0 + 7:
// a lane reads 8 / LPR consecutive slots at once, lookup e is in register e % PER of lane e / PER, and
// the eight rows are in flight together.  nl: length of the list (entries behind the bag are read, not used).
template <typename V, int LPR, bool COMP>
__device__ __forceinline__ void fwd_add_narrow(V &acc, V &lost, const V *W, const int32_t *slots, uint32_t j0, int count, uint32_t done, uint32_t nl,
                                               int n_hot, int ncols, int c, uint32_t *status)
{
    constexpr int PER = 8 / LPR;
    const int first = threadIdx.x % LPR * PER;
    int slot[PER];
    if (j0 + 8 <= nl) {
        __builtin_memcpy(slot, slots + j0 + first, sizeof(slot)); // one load; the bag may start at any entry
    } else {
#pragma unroll
        for (int k = 0; k < PER; ++k)
            slot[k] = first + k < count ? slots[j0 + first + k] : 0;
    }
    bool bad = false;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if ((unsigned)slot[k] >= (unsigned)n_hot) {
            bad |= first + k < count;
            slot[k] = -1;
        }
    }
    if (bad)
        fae_flag(status, FAE_STATUS_ERANGE);
    V v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int sl = fwd_pair_lane<LPR>(slot[e % PER], e / PER);
        v[e] = (e < count && sl >= 0 && c < ncols) ? W[(int64_t)sl * ncols + c] : vec_ops<V>::zero();
    }
    if constexpr (COMP) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (e < count)
                vec_ops<V>::add_comp(acc, lost, v[e]);
    } else {
        fwd_add_pairs(lost, v); // the part
    }
    if (!COMP && (done + 8) % FWD_PART == 0)
        fwd_end_part(acc, lost);
}

// The lane's slot of a chunk (-1: past the end, or out of range and flagged).  Lookups are numbered
// without a sign here: the last chunk of a bag may step past 2^31.
__device__ __forceinline__ int fwd_slot(const int32_t *slots, uint32_t j, uint32_t end, int n_hot, uint32_t *status)
{
    int sl = j < end ? slots[j] : -1;
    if (j < end && (unsigned)sl >= (unsigned)n_hot) {
        fae_flag(status, FAE_STATUS_ERANGE);
        sl = -1;
    }
    return sl;
}

// One launch for every table; the workgroup's table says which mapping (a.kind):
//   one-hot   256 samples per workgroup, 64 per wave;
//   group     LPR lanes own a bag, 256 / LPR bags per workgroup: short bags;
//   wave      a wave owns a bag, its 64 / LPR lane groups take alternate rows: long bags.
// What bounds it: rows that miss the L2 (large tables), else the chain offsets -> slots -> rows of a
// bag.  So the slots of a bag (64 of them, or LPR for a lane group) come with one load and are handed
// out by lane shuffles, and a row costs one round trip instead of two in a row, with 8 rows per group
// in flight in the wave mapping of LPR >= 32 and 4 elsewhere; the mapping goes by each table's own bags,
// and all tables share the launch:
//   8 x 65 536 bags of about 20, dim 128: 650 -> 521 us (10.3 TB/s of rows out of L2 and beyond)
//   3 tables with bags of up to 100 and a one-hot one, 6007 samples, dim 100: 9 + 28.7 -> 27.2 us
//   3 tables of short bags and 2 one-hot ones, 3001 samples, dim 20: 4.7 + 11.9 -> 9.1 us
// A group of one or two lanes would get one or two rows out of such a load, so it reads eight slots at a
// time (fwd_add_narrow).  One slot per lane / four slots and rows in turn / now, microseconds:
//   five tables, 65 536 bags of 1-100: dim 2 (LPR 2, scalar) 174 / 130 / 92; dim 8 (LPR 2) 228 / 184 / 139
//   three tables, 2048 bags of 1-100: dim 4 (LPR 1) 53 / 31 / 24, dim 1 35.4 / 17.1 / 15.1
// Groups of four keep one slot per lane: with eight rows in flight the kernel takes the wave mapping more
// (84 -> 89 us for five tables of 32 768 bags of 1-100, dim 16) than the group mapping gains (33.3 -> 29.7 us, bags of 1-30).
template <typename V, int LPR> __global__ __launch_bounds__(256, 8) void fwd_kernel(FwdArgs a)
{
    const int z = fae_find_table(a.blk_start, a.n_tables, blockIdx.x);
    const int bl = blockIdx.x - a.blk_start[z];
    const int kind = a.kind[z];
    if (kind == FWD_ONEHOT) {
        const int64_t s0 = ((int64_t)bl * (256 / FAE_WAVE) + threadIdx.x / FAE_WAVE) * FAE_WAVE;
        fwd_onehot_wave<V, LPR, (LPR < 32 ? 8 : 4)>((const V *)a.W[z], a.slots[z], a.n_hot[z], s0, a.n_samples, a.out + (int64_t)z * a.dim,
                                a.out_stride, a.dim, a.status, a.stream_out != 0);
        return;
    }
    constexpr int G = FAE_WAVE / LPR; // lane groups per wave
    const int lane = fae_lane(), g = lane / LPR, l = lane % LPR;
    const bool wave = kind == FWD_WAVE;
    const int64_t s = wave ? (int64_t)bl * (256 / FAE_WAVE) + __builtin_amdgcn_readfirstlane(threadIdx.x / FAE_WAVE)
                           : (int64_t)bl * (256 / LPR) + threadIdx.x / LPR;
    const bool in = s < a.n_samples;
    const int32_t *off = a.offsets[z];
    const int32_t *slots = a.slots[z];
    int beg = in ? (off ? off[s] : (int)s) : 0;
    int end = in ? (off ? off[s + 1] : (int)s + 1) : 0;
    if (beg < 0 || end > a.n_lookups[z] || beg > end) { // malformed CSR: never dereferenced
        fae_flag(a.status, FAE_STATUS_ERANGE);
        end = beg = 0;
    }
    const int ncols = a.dim / (int)(sizeof(V) / sizeof(float));
    const V *W = (const V *)a.W[z];
    const int n_hot = a.n_hot[z];
    V *const o = (V *)(a.out + s * a.out_stride + (int64_t)z * a.dim);
    if (wave) {
        if (!in)
            return;
        for (int c0 = 0; c0 == 0 || (LPR == FAE_WAVE && c0 < ncols); c0 += LPR) { // fewer lanes: the row is no wider than they are
            const int c = c0 + l;
            V acc = vec_ops<V>::zero(), lost = vec_ops<V>::zero();
            for (uint32_t j0 = beg; j0 < (uint32_t)end; j0 += FAE_WAVE) {
                const int slot = fwd_slot(slots, j0 + lane, end, n_hot, a.status);
                const int count = end - j0 < FAE_WAVE ? (int)(end - j0) : FAE_WAVE;
                if (end - beg > FWD_PLAIN_MAX * G) // the same for the whole wave
                    fwd_add_rows<V, FAE_WAVE, G, (LPR < 4 ? LPR : 4), true>(acc, lost, W, slot, g, count, ncols, c, c < ncols);
                else
                    fwd_add_rows<V, FAE_WAVE, G, (LPR < 4 ? LPR : G <= 2 ? 8 : 4), false>(acc, lost, W, slot, g, count, ncols, c, c < ncols);
            }
            // combine the lane groups (all 64 lanes take part in the shuffles)
#pragma unroll
            for (int m = LPR; m < FAE_WAVE; m <<= 1)
                vec_ops<V>::add(acc, vec_ops<V>::shfl_xor(acc, m));
            if (a.mean && end - beg > 1)
                vec_ops<V>::scale(acc, 1.0f / (float)(end - beg));
            if (g == 0 && c < ncols)
                o[c] = acc;
        }
    } else {
        for (int c0 = 0; c0 == 0 || (LPR == FAE_WAVE && c0 < ncols); c0 += LPR) { // fewer lanes: the row is no wider than they are
            const int c = c0 + l;
            V acc = vec_ops<V>::zero(), lost = vec_ops<V>::zero();
            if constexpr (LPR < 4) {
                for (uint32_t j0 = beg; j0 < (uint32_t)end; j0 += 8) { // a lane group leaves as a whole
                    const int count = end - j0 < 8 ? (int)(end - j0) : 8;
                    if (end - beg > FWD_PLAIN_MAX)
                        fwd_add_narrow<V, LPR, true>(acc, lost, W, slots, j0, count, j0 - beg, a.n_lookups[z], n_hot, ncols, c, a.status);
                    else
                        fwd_add_narrow<V, LPR, false>(acc, lost, W, slots, j0, count, j0 - beg, a.n_lookups[z], n_hot, ncols, c, a.status);
                }
            } else {
                for (uint32_t j0 = beg; j0 < (uint32_t)end; j0 += LPR) { // a lane group leaves as a whole
                    const int count = end - j0 < LPR ? (int)(end - j0) : LPR;
                    const int slot = fwd_slot(slots, j0 + l, end, n_hot, a.status);
                    if (end - beg > FWD_PLAIN_MAX)
                        fwd_add_rows<V, LPR, 1, 4, true>(acc, lost, W, slot, 0, count, ncols, c, c < ncols);
                    else
                        fwd_add_parts<V, LPR>(acc, lost, W, slot, count, j0 - beg, ncols, c, c < ncols);
                }
            }
            if (end - beg <= FWD_PLAIN_MAX)
                vec_ops<V>::add(acc, lost); // the last part
            if (a.mean && end - beg > 1)
                vec_ops<V>::scale(acc, 1.0f / (float)(end - beg));
            if (in && c < ncols)
                o[c] = acc;
        }
    }
}

// One-hot tables beside bags: from this many bytes of their pooled rows on they get a launch of their
// own, fwd_onehot_kernel's.  Below, one launch for all is shorter (its bags and rows overlap, and a launch
// is saved), above the deeper copy is worth more.  One launch / two, microseconds:
//   25 one-hot tables and one of bags of 1-10: 26 x 4096 x 64 (100 MiB) 12.6 / 15.2, 50 001 x 64 (305 MiB) 99 / 106,
//   90 000 x 64 (549 MiB) 176 / 173, 131 072 x 64 (800 MiB) 248 / 238, 131 072 x 128 (1.6 GiB) 482 / 465;
//   10 and one: 131 072 x 128 (640 MiB) 214.5 / 217; 13 and three: 65 536 x 256 (832 MiB) 335 / 336
#define FWD_SPLIT_BYTES (768LL << 20)

// Every table one-hot: no bag code beside it, so sixteen rows fit in flight per lane group (26 tables of
// 50 001 samples, dim 64: 68.5 us, against 77.0 us for fwd_kernel with its eight).
template <typename V, int LPR> __global__ __launch_bounds__(256) void fwd_onehot_kernel(FwdArgs a)
{
    const int z = fae_find_table(a.blk_start, a.n_tables, blockIdx.x);
    const int bl = blockIdx.x - a.blk_start[z];
    const int64_t s0 = ((int64_t)bl * (256 / FAE_WAVE) + threadIdx.x / FAE_WAVE) * FAE_WAVE;
    fwd_onehot_wave<V, LPR, 16>((const V *)a.W[z], a.slots[z], a.n_hot[z], s0, a.n_samples, a.out + (int64_t)z * a.dim,
                                a.out_stride, a.dim, a.status, a.stream_out != 0);
}

template <typename V, int LPR> static void fwd_launch(fae_ctx *ctx, const FwdArgs &a, bool bags, int blocks)
{
    if (bags)
        FAE_LAUNCH(ctx, (fwd_kernel<V, LPR>), dim3(blocks), dim3(256), 0, ctx->stream, a);
    else
        FAE_LAUNCH(ctx, (fwd_onehot_kernel<V, LPR>), dim3(blocks), dim3(256), 0, ctx->stream, a);
}

template <typename V> static void fwd_dispatch(fae_ctx *ctx, const FwdArgs &a, int lpr, bool bags, int blocks)
{
    switch (lpr) {
    case 1: fwd_launch<V, 1>(ctx, a, bags, blocks); break;
    case 2: fwd_launch<V, 2>(ctx, a, bags, blocks); break;
    case 4: fwd_launch<V, 4>(ctx, a, bags, blocks); break;
    case 8: fwd_launch<V, 8>(ctx, a, bags, blocks); break;
    case 16: fwd_launch<V, 16>(ctx, a, bags, blocks); break;
    case 32: fwd_launch<V, 32>(ctx, a, bags, blocks); break;
    default: fwd_launch<V, 64>(ctx, a, bags, blocks); break;
    }
}

static int32_t fwd_impl(fae_ctx *ctx, const fae_tables *hot_tables, const float *const *h_hotW,
                        const fae_batch *hot_batch, float *out, int64_t out_row_stride, int pooling);

extern "C" int32_t fae_embbag_fwd(fae_ctx *ctx, const fae_tables *hot_tables, const float *const *h_hotW,
                                  const fae_batch *hot_batch, float *out, int64_t out_row_stride)
{
    return fwd_impl(ctx, hot_tables, h_hotW, hot_batch, out, out_row_stride, FAE_POOL_SUM);
}

extern "C" int32_t fae_embbag_fwd_opts(fae_ctx *ctx, const fae_tables *hot_tables, const float *const *h_hotW,
                                       const fae_batch *hot_batch, float *out, int64_t out_row_stride,
                                       const fae_step_opts *opts)
{
    if (!ctx)
        return FAE_EINVAL;
    if (!opts || (opts->pooling != FAE_POOL_SUM && opts->pooling != FAE_POOL_MEAN))
        return fae_fail(ctx, FAE_EINVAL, "fae_embbag_fwd_opts: null options or unknown pooling");
    return fwd_impl(ctx, hot_tables, h_hotW, hot_batch, out, out_row_stride, opts->pooling);
}

static int32_t fwd_impl(fae_ctx *ctx, const fae_tables *hot_tables, const float *const *h_hotW,
                        const fae_batch *hot_batch, float *out, int64_t out_row_stride, int pooling)
{
    int32_t rc = fae_check_tables(ctx, hot_tables, "fae_embbag_fwd");
    if (rc != FAE_OK)
        return rc;
    rc = fae_check_batch(ctx, hot_tables, hot_batch, "fae_embbag_fwd");
    if (rc != FAE_OK)
        return rc;
    if (hot_batch->index_bits == 64)
        return fae_fail(ctx, FAE_EINVAL, "fae_embbag_fwd: hot slots are int32");
    const int nt = hot_tables->n_tables, dim = hot_tables->dim;
    const int64_t S = hot_batch->n_samples;
    if (S == 0)
        return FAE_OK;
    if (!h_hotW || !out || out_row_stride < (int64_t)nt * dim)
        return fae_fail(ctx, FAE_EINVAL, "fae_embbag_fwd: null output/weights or out_row_stride < n_tables*dim");
    FAE_HIP(ctx, hipSetDevice(ctx->device));

    FwdArgs a;
    memset(&a, 0, sizeof(a));
    bool vec = (dim % 4 == 0) && (out_row_stride % 4 == 0) && (((uintptr_t)out) % 16 == 0);
    for (int z = 0; z < nt; ++z) {
        if (!h_hotW[z] && hot_tables->h_rows[z] > 0)
            return fae_fail(ctx, FAE_EINVAL, "fae_embbag_fwd: null weights for table %d", z);
        a.W[z] = h_hotW[z];
        a.slots[z] = hot_batch->h_indices[z];
        a.offsets[z] = hot_batch->h_offsets ? hot_batch->h_offsets[z] : nullptr;
        a.n_hot[z] = (int32_t)hot_tables->h_rows[z];
        a.n_lookups[z] = (int32_t)hot_batch->h_n_lookups[z];
        if (((uintptr_t)h_hotW[z]) % 16 != 0)
            vec = false;
    }
    const int ncols = vec ? dim / 4 : dim;
    int lpr = 1;
    while (lpr < ncols && lpr < 64)
        lpr <<= 1;
    const int groups = 64 / lpr;
    a.n_tables = nt;
    a.dim = dim;
    a.n_samples = (int32_t)S;
    a.out_stride = out_row_stride;
    a.out = out;
    a.status = ctx->d_block;
    a.stream_out = ctx->opt_fwd_stream != 0;
    a.mean = pooling == FAE_POOL_MEAN;
    int n_bags = 0;
    for (int z = 0; z < nt; ++z)
        n_bags += a.offsets[z] || ctx->opt_fwd != 0;
    // A wave per bag pays once a bag keeps every lane group of the wave busy for two rounds.  Eight groups and
    // more do from one and a half rounds on where a wave for every bag finds room on the chip at once (32 to a
    // CU) or nearly so: there the longest bag's chain is the time.  Three tables of bags of 1-30, dim 20, us by
    // wave | by group: 2048 samples 6.5 | 8.2, 3001 7.2 | 9.1, 6007 11.3 | 11.0, 12000 17.9 | 15.3; of 10-20:
    // 3001 7.1 | 7.5, 4500 8.9 | 8.2; of 1-60, dim 16, 2048: 6.5 | 13.6.  Two groups, bags of 1-5, dim 100,
    // 3001: 6.3 | 6.0; with four no difference.  With one round: bags of 1-20, dim 32, 4500: 8.3 | 7.1.
    const double rounds = groups >= 8 && (double)S * n_bags <= 40.0 * ctx->n_cu ? 1.5 : 2.0;
    for (int z = 0; z < nt; ++z) {
        a.kind[z] = FWD_ONEHOT;
        if (a.offsets[z] || ctx->opt_fwd != 0) {
            bool wave = groups > 1 && (double)hot_batch->h_n_lookups[z] >= rounds * groups * (double)S;
            if (ctx->opt_fwd == 1)
                wave = false;
            if (ctx->opt_fwd == 2)
                wave = groups > 1;
            a.kind[z] = wave ? FWD_WAVE : FWD_GROUP;
        }
    }
    const bool split = n_bags > 0 && (int64_t)(nt - n_bags) * S * dim * 4 >= FWD_SPLIT_BYTES;
    for (int part = split ? 0 : 1; part < 2; ++part) { // the one-hot tables by themselves, then the others (or all)
        int64_t blocks = 0;
        for (int z = 0; z < nt; ++z) {
            a.blk_start[z] = (int32_t)blocks;
            const bool bag = a.kind[z] != FWD_ONEHOT;
            if (split && bag != (part == 1))
                continue;
            const int64_t per_block = !bag ? 256 : (a.kind[z] == FWD_WAVE ? 256 / FAE_WAVE : 256 / lpr);
            blocks += (S + per_block - 1) / per_block;
            if (blocks >= 2147483647LL)
                return fae_fail(ctx, FAE_EINVAL, "fae_embbag_fwd: batch too large for one launch");
        }
        a.blk_start[nt] = (int32_t)blocks;
        fae_ktimer kt(ctx, FAE_K_FWD);
        if (vec)
            fwd_dispatch<float4>(ctx, a, lpr, n_bags > 0 && part == 1, (int)blocks);
        else
            fwd_dispatch<float>(ctx, a, lpr, n_bags > 0 && part == 1, (int)blocks);
        FAE_LAUNCH_CHECK(ctx);
    }
    return FAE_OK;
}
