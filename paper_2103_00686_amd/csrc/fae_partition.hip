// Input Classifier (Sec. 4.2): a sparse input is hot iff every access in every table
// hits a hot row.  Hot and cold inputs keep their original order; for the hot ones
// the hot slots and a rebuilt CSR are emitted so that consecutive slices are the
// hot mini-batches.  Integer-only work: random 4-byte gathers into the remap, an
// AND-reduction per sample, a stable compaction.
#include "fae_internal.h"

#define PT_THREADS 256
#define PT_MIN_TILE 16
#define PT_MAX_TILE PT_THREADS // samples per tile: one sample per thread
#define PT_SCAN_TILE 1024      // what the size of the workspace goes by
#define PT_SUM_MAX 16384       // counters (rows x tiles) up to which every tile adds up those before it by itself

struct PartArgs {
    const void *idx[FAE_MAX_TABLES]; // int32 or int64 row ids
    const int32_t *offsets[FAE_MAX_TABLES];
    const int32_t *remap[FAE_MAX_TABLES];
    int32_t *slots[FAE_MAX_TABLES];
    int32_t *hoffsets[FAE_MAX_TABLES];
    int32_t n_rows[FAE_MAX_TABLES];
    int32_t n_lookups[FAE_MAX_TABLES];
    int32_t one_hot[FAE_MAX_TABLES]; // the n_one tables with one lookup per sample
    int32_t csr[FAE_MAX_TABLES];     // the n_csr tables with offsets
    int32_t wide;                    // the ids are int64
    int32_t n_tables, n_one, n_csr;
    int32_t n_samples;
    int32_t tile_log;     // samples per tile: 1 << tile_log
    int32_t n_tiles;
    int32_t scanned;      // tile_sums holds running totals over row after row (else the tiles' own counts)
    uint32_t *cold;       // [n_samples] 1 = some access is cold
    int32_t *tile_sums;   // [(1 + n_csr) * n_tiles + 1]; row 0 = hot samples, row 1 + c = hot lookups of table csr[c]
    int32_t *hot_samples;
    int32_t *cold_samples;
    uint32_t *status;
    uint32_t *scalars;    // device scalars: [0] = n_hot_samples, [1+z] = hot lookups of table z
};
static_assert(sizeof(PartArgs) <= 4096, "kernel arguments are passed by value");

// lookups of sample s in a table with offsets `off`; a malformed entry sets *bad and counts none
__device__ __forceinline__ int part_len(const int32_t *off, int nl, int n_samples, int s, bool *bad)
{
    const int b = off[s], e = off[s + 1];
    if (b < 0 || e < b || e > nl || (s == 0 && b != 0) || (s == n_samples - 1 && e != nl)) {
        *bad = true;
        return 0;
    }
    return e - b;
}

// the sample (inside the tile of n samples) that owns lookup j: s_off[0..n] holds the tile's offsets
__device__ __forceinline__ int part_owner(const int *s_off, int n, int j)
{
    int lo = 0, hi = n; // the last entry <= j
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (s_off[mid] <= j)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Two kernels, a workgroup per tile of samples in each: the first classifies the tile's samples over
// all tables and leaves the tile's counts, the second adds up the counts of the tiles before it and
// writes the lists, the slots and the offsets.  Bound by the random 4-byte gathers into the remaps
// (a whole sector of a cache line each), so a thread keeps PT_LK of them in flight; a
// tile sees all tables of its samples, so that "some access is cold" needs no cleared array, no
// store per lookup and no pass of its own, and the position among the hot samples never leaves LDS.
// The lookups of a tile of a table with offsets are one range: a lookup finds its sample in the
// tile's offsets in LDS instead of searching all offsets in memory.
//   26 one-hot tables, 262 144 samples: 56 us in two kernels, 140 -> 99 us a call (before: 76 us in
//   seven launches: clear, mark, count, scan, lists, offsets, slots; and two waits instead of one)
#define PT_LK 8

// table of item i (see below); with tiles of whole waves it is the same for every lane, and said so
// its descriptors are scalar loads
template <bool WAVE_TILES> __device__ __forceinline__ int part_table(const PartArgs &a, int i)
{
    const int n = i >> a.tile_log;
    return a.one_hot[WAVE_TILES ? __builtin_amdgcn_readfirstlane(n) : n];
}

template <bool WAVE_TILES> __global__ __launch_bounds__(PT_THREADS) void part_classify_kernel(PartArgs a)
{
    __shared__ uint32_t s_cold[PT_MAX_TILE];
    __shared__ int s_off[PT_MAX_TILE + 1];
    __shared__ int s_bad;
    const int T = 1 << a.tile_log, s0 = blockIdx.x << a.tile_log;
    const int ns = a.n_samples - s0 < T ? a.n_samples - s0 : T;
    const int t = threadIdx.x;
    bool bad = false;
    s_cold[t] = 0u;
    if (t == 0)
        s_bad = 0;
    __syncthreads();
    // tables with one lookup per sample: item i is sample i % T of table i / T
    const int items = a.n_one << a.tile_log;
    for (int i0 = t; i0 < items; i0 += PT_LK * PT_THREADS) {
        int r[PT_LK], m[PT_LK];
#pragma unroll
        for (int k = 0; k < PT_LK; ++k) {
            const int i = i0 + k * PT_THREADS, s = i & (T - 1);
            r[k] = -2;
            if (i < items && s < ns) {
                const int z = part_table<WAVE_TILES>(a, i);
                r[k] = fae_load_row(a.idx[z], (int64_t)s0 + s, a.wide, a.n_rows[z]);
            }
        }
#pragma unroll
        for (int k = 0; k < PT_LK; ++k) {
            const int i = i0 + k * PT_THREADS;
            m[k] = -1;
            if (r[k] >= 0)
                m[k] = a.remap[part_table<WAVE_TILES>(a, i)][r[k]];
        }
#pragma unroll
        for (int k = 0; k < PT_LK; ++k) {
            if (r[k] == -2)
                continue;
            bad = bad || r[k] < 0;
            if (m[k] < 0)
                s_cold[(i0 + k * PT_THREADS) & (T - 1)] = 1u; // every writer stores the same value
        }
    }
    // tables with offsets; a sample is checked whether it is hot or cold
    for (int c = 0; c < a.n_csr; ++c) {
        const int z = a.csr[c];
        const int32_t *off = a.offsets[z];
        bool bad_here = false;
        if (t <= ns)
            s_off[t] = off[s0 + t];
        if (t == 0 && ns == PT_MAX_TILE)
            s_off[PT_MAX_TILE] = off[s0 + PT_MAX_TILE];
        if (t < ns)
            (void)part_len(off, a.n_lookups[z], a.n_samples, s0 + t, &bad_here);
        if (bad_here)
            s_bad = 1;
        __syncthreads();
        if (s_bad == 0) { // a malformed tile is not walked: the call reports it
            const int lo = s_off[0], hi = s_off[ns];
            const int32_t *remap = a.remap[z];
            for (uint32_t j0 = (uint32_t)lo + t; j0 < (uint32_t)hi; j0 += PT_LK * PT_THREADS) { // unsigned: j0 may step past 2^31
                int r[PT_LK], m[PT_LK];
#pragma unroll
                for (int k = 0; k < PT_LK; ++k) {
                    const uint32_t j = j0 + k * PT_THREADS;
                    r[k] = j < (uint32_t)hi ? fae_load_row(a.idx[z], j, a.wide, a.n_rows[z]) : -2;
                }
#pragma unroll
                for (int k = 0; k < PT_LK; ++k)
                    m[k] = r[k] >= 0 ? remap[r[k]] : -1;
#pragma unroll
                for (int k = 0; k < PT_LK; ++k) {
                    if (r[k] == -2)
                        continue;
                    bad = bad || r[k] < 0;
                    if (m[k] < 0)
                        s_cold[part_owner(s_off, ns, (int)(j0 + k * PT_THREADS))] = 1u;
                }
            }
        }
        __syncthreads(); // s_off is filled again for the next table
    }
    __syncthreads();
    if (bad || (t == 0 && s_bad))
        fae_flag(a.status, FAE_STATUS_ERANGE);
    if (t < ns)
        a.cold[s0 + t] = s_cold[t];
    // the tile's counts, a row per wave: hot samples, then the hot lookups of each table with offsets
    for (int row = t / FAE_WAVE; row <= a.n_csr; row += PT_THREADS / FAE_WAVE) {
        int c = 0;
        for (int s = fae_lane(); s < ns; s += FAE_WAVE) {
            bool ignored = false;
            if (!s_cold[s]) {
                const int z = row > 0 ? a.csr[row - 1] : 0;
                c += row > 0 ? part_len(a.offsets[z], a.n_lookups[z], a.n_samples, s0 + s, &ignored) : 1;
            }
        }
        c = __shfl(fae_wave_incl_scan(c), FAE_WAVE - 1, FAE_WAVE);
        if (fae_lane() == 0)
            a.tile_sums[(int64_t)row * a.n_tiles + blockIdx.x] = c;
    }
}

template <bool WAVE_TILES> __global__ __launch_bounds__(PT_THREADS) void part_emit_kernel(PartArgs a)
{
    __shared__ int lds[PT_THREADS / FAE_WAVE + 1];
    __shared__ int s_base[FAE_MAX_TABLES + 1]; // per row: what the tiles before this one hold
    __shared__ int s_hot[PT_MAX_TILE];         // position of the sample among the tile's hot ones, -1 if it is cold
    __shared__ int s_off[PT_MAX_TILE + 1], s_dst[PT_MAX_TILE];
    const int T = 1 << a.tile_log, tile = blockIdx.x, s0 = tile << a.tile_log;
    const int ns = a.n_samples - s0 < T ? a.n_samples - s0 : T;
    const int t = threadIdx.x, lane = fae_lane();
    const bool hot = t < ns && a.cold[s0 + t] == 0u;
    for (int row = t / FAE_WAVE; row <= a.n_csr; row += PT_THREADS / FAE_WAVE) {
        const int32_t *sums = a.tile_sums + (int64_t)row * a.n_tiles;
        int c = 0;
        if (a.scanned) {
            c = sums[tile] - sums[0];
        } else {
#pragma unroll 8
            for (int i = lane; i < tile; i += FAE_WAVE)
                c += sums[i];
            c = __shfl(fae_wave_incl_scan(c), FAE_WAVE - 1, FAE_WAVE);
        }
        if (lane == 0)
            s_base[row] = c;
    }
    int n_here;
    const int pos = fae_block_excl_scan<PT_THREADS>(hot ? 1 : 0, lds, &n_here); // its barriers also publish s_base
    const int h0 = s_base[0];
    if (t < ns) {
        s_hot[t] = hot ? pos : -1;
        if (hot)
            a.hot_samples[h0 + pos] = s0 + t;
        else
            a.cold_samples[s0 + t - h0 - pos] = s0 + t;
    }
    __syncthreads();
    const bool last = tile == a.n_tiles - 1; // it also writes the closing offsets and the totals
    if (last && t == 0)
        a.scalars[0] = (uint32_t)(h0 + n_here);
    if (last && t < a.n_one) {
        const int z = a.one_hot[t];
        a.hoffsets[z][h0 + n_here] = h0 + n_here;
        a.scalars[1 + z] = (uint32_t)(h0 + n_here);
    }
    const int items = n_here > 0 ? a.n_one << a.tile_log : 0;
    for (int i0 = t; i0 < items; i0 += PT_LK * PT_THREADS) {
        int r[PT_LK], h[PT_LK], m[PT_LK];
#pragma unroll
        for (int k = 0; k < PT_LK; ++k) {
            const int i = i0 + k * PT_THREADS, s = i & (T - 1);
            h[k] = i < items && s < ns ? s_hot[s] : -1;
            r[k] = -1;
            if (h[k] >= 0) {
                const int z = part_table<WAVE_TILES>(a, i);
                r[k] = fae_load_row(a.idx[z], (int64_t)s0 + s, a.wide, a.n_rows[z]);
            }
        }
#pragma unroll
        for (int k = 0; k < PT_LK; ++k) {
            m[k] = 0;
            if (r[k] >= 0) // always, for a hot sample: the first kernel has checked every id
                m[k] = a.remap[part_table<WAVE_TILES>(a, i0 + k * PT_THREADS)][r[k]];
        }
#pragma unroll
        for (int k = 0; k < PT_LK; ++k)
            if (h[k] >= 0) {
                const int z = part_table<WAVE_TILES>(a, i0 + k * PT_THREADS);
                a.hoffsets[z][h0 + h[k]] = h0 + h[k]; // one lookup per sample: hot sample h starts at h
                if (r[k] >= 0)
                    a.slots[z][h0 + h[k]] = m[k];
            }
    }
    for (int c = 0; c < a.n_csr; ++c) {
        const int z = a.csr[c];
        const int32_t *off = a.offsets[z];
        const int nl = a.n_lookups[z], base = s_base[1 + c];
        bool bad = false;
        int len = 0;
        if (t < ns)
            len = part_len(off, nl, a.n_samples, s0 + t, &bad);
        len = hot ? len : 0;
        const bool walk = !__syncthreads_or(bad); // (also: s_off and s_dst of the table before are no longer read)
        if (t <= ns)
            s_off[t] = off[s0 + t];
        if (t == 0 && ns == PT_MAX_TILE)
            s_off[PT_MAX_TILE] = off[s0 + PT_MAX_TILE];
        int here;
        const int at = base + fae_block_excl_scan<PT_THREADS>(len, lds, &here);
        if (t < ns)
            s_dst[t] = at;
        if (hot)
            a.hoffsets[z][h0 + pos] = at;
        if (last && t == 0) {
            a.hoffsets[z][h0 + n_here] = base + here;
            a.scalars[1 + z] = (uint32_t)(base + here);
        }
        __syncthreads();
        if (!walk || here == 0)
            continue;
        const int lo = s_off[0], hi = s_off[ns];
        const int32_t *remap = a.remap[z];
        int32_t *slots = a.slots[z];
        for (uint32_t j0 = (uint32_t)lo + t; j0 < (uint32_t)hi; j0 += PT_LK * PT_THREADS) { // unsigned: j0 may step past 2^31
            int r[PT_LK], dst[PT_LK], m[PT_LK];
#pragma unroll
            for (int k = 0; k < PT_LK; ++k) {
                const uint32_t j = j0 + k * PT_THREADS;
                r[k] = dst[k] = -1;
                if (j >= (uint32_t)hi)
                    continue;
                const int s = part_owner(s_off, ns, (int)j);
                const int d = s_dst[s] + ((int)j - s_off[s]);
                if (s_hot[s] >= 0 && d >= 0 && d < nl) {
                    dst[k] = d;
                    r[k] = fae_load_row(a.idx[z], j, a.wide, a.n_rows[z]);
                }
            }
#pragma unroll
            for (int k = 0; k < PT_LK; ++k)
                m[k] = r[k] >= 0 ? remap[r[k]] : -1;
#pragma unroll
            for (int k = 0; k < PT_LK; ++k)
                if (r[k] >= 0)
                    slots[dst[k]] = m[k];
        }
    }
}

static int64_t part_tiles(int64_t S) { return (S + PT_SCAN_TILE - 1) / PT_SCAN_TILE; }

// words behind the cold flags, for the tiles' counts
static size_t part_count_words(int nt, int64_t S)
{
    return (fae_align_up((size_t)S * 4 + 4, 256) + fae_align_up(((size_t)nt + 1) * (size_t)part_tiles(S) * 4 + 8, 256)) / 4;
}

extern "C" size_t fae_partition_workspace_bytes(const fae_tables *tables, int64_t n_samples)
{
    if (!tables || n_samples < 0)
        return 0;
    size_t S = (size_t)n_samples;
    size_t tiles = (size_t)part_tiles(n_samples);
    return fae_align_up(S * 4 + 4, 256) * 2 + fae_align_up(((size_t)tables->n_tables + 1) * tiles * 4 + 8, 256) + 256;
}

extern "C" int32_t fae_partition_batch(fae_ctx *ctx, const fae_tables *tables, const fae_batch *in,
                                       const int32_t *const *h_remap, int32_t *hot_samples,
                                       int32_t *cold_samples, int64_t *h_n_hot_samples,
                                       int32_t *const *h_slots, int32_t *const *h_hoffsets,
                                       int64_t *h_n_hot_lookups, void *ws, size_t ws_bytes)
{
    int32_t rc = fae_check_tables(ctx, tables, "fae_partition_batch");
    if (rc != FAE_OK)
        return rc;
    rc = fae_check_batch(ctx, tables, in, "fae_partition_batch");
    if (rc != FAE_OK)
        return rc;
    if (!h_remap || !h_n_hot_samples || !h_slots || !h_hoffsets || !h_n_hot_lookups)
        return fae_fail(ctx, FAE_EINVAL, "fae_partition_batch: null argument");
    const int nt = tables->n_tables;
    const int64_t S = in->n_samples;
    if (nt + 2 > FAE_BLK_WORDS - FAE_BLK_SCALARS)
        return fae_fail(ctx, FAE_EINVAL, "fae_partition_batch: too many tables");
    if (S == 0) {
        *h_n_hot_samples = 0;
        for (int z = 0; z < nt; ++z)
            h_n_hot_lookups[z] = 0;
        return FAE_OK;
    }
    if (!hot_samples || !cold_samples)
        return fae_fail(ctx, FAE_EINVAL, "fae_partition_batch: null sample lists");
    if (!ws || ws_bytes < fae_partition_workspace_bytes(tables, S))
        return fae_fail(ctx, FAE_ENOSPC, "fae_partition_batch: workspace too small");
    FAE_HIP(ctx, hipSetDevice(ctx->device));

    PartArgs a;
    memset(&a, 0, sizeof(a));
    for (int z = 0; z < nt; ++z) {
        if (!h_remap[z] && tables->h_rows[z] > 0)
            return fae_fail(ctx, FAE_EINVAL, "fae_partition_batch: null remap for table %d", z);
        if (!h_hoffsets[z] || (!h_slots[z] && in->h_n_lookups[z] > 0))
            return fae_fail(ctx, FAE_EINVAL, "fae_partition_batch: null outputs for table %d", z);
        a.idx[z] = in->h_indices[z];
        a.offsets[z] = in->h_offsets ? in->h_offsets[z] : nullptr;
        a.remap[z] = h_remap[z];
        a.slots[z] = h_slots[z];
        a.hoffsets[z] = h_hoffsets[z];
        a.n_rows[z] = (int32_t)tables->h_rows[z];
        a.n_lookups[z] = (int32_t)in->h_n_lookups[z];
        if (a.offsets[z])
            a.csr[a.n_csr++] = z;
        else
            a.one_hot[a.n_one++] = z;
    }
    // Samples per tile: enough tiles for eight workgroups on every compute unit, but no more than
    // the workspace has counters for (256 samples per tile always fit).
    const int rows = 1 + a.n_csr;
    const size_t words = part_count_words(nt, S);
    const auto tiles_of = [&](int log) { return (S + (1LL << log) - 1) >> log; };
    int log = 4;
    while ((1 << log) < PT_MAX_TILE &&
           (tiles_of(log) > 8LL * ctx->n_cu || (size_t)rows * (size_t)tiles_of(log) + 1 > words))
        ++log;
    static_assert(PT_MIN_TILE == 1 << 4, "smallest tile");
    const int64_t tiles = tiles_of(log);
    fae_carver cv(ws, ws_bytes);
    a.cold = cv.take<uint32_t>((size_t)S + 1);
    a.tile_sums = cv.take<int32_t>(words);
    if (!cv.ok || (size_t)rows * (size_t)tiles + 1 > words)
        return fae_fail(ctx, FAE_ENOSPC, "fae_partition_batch: workspace too small");
    a.wide = in->index_bits == 64;
    a.n_tables = nt;
    a.n_samples = (int32_t)S;
    a.tile_log = log;
    a.n_tiles = (int32_t)tiles;
    // Every tile reads the counts in front of it, or one more launch turns them into running totals:
    // the first is the shorter way while the counters are few (their reads grow with the square).
    a.scanned = (int64_t)rows * tiles > PT_SUM_MAX;
    a.hot_samples = hot_samples;
    a.cold_samples = cold_samples;
    a.status = ctx->d_block;
    a.scalars = ctx->d_block + FAE_BLK_SCALARS;
    {
        fae_ktimer kt(ctx, FAE_K_PARTITION);
        if (log >= 6)
            FAE_LAUNCH(ctx, part_classify_kernel<true>, dim3((unsigned)tiles), dim3(PT_THREADS), 0, ctx->stream, a);
        else
            FAE_LAUNCH(ctx, part_classify_kernel<false>, dim3((unsigned)tiles), dim3(PT_THREADS), 0, ctx->stream, a);
        FAE_LAUNCH_CHECK(ctx);
    }
    if (a.scanned) {
        rc = fae_scan_i32(ctx, a.tile_sums, (int64_t)rows * tiles);
        if (rc != FAE_OK)
            return rc;
    }
    {
        fae_ktimer kt(ctx, FAE_K_PARTITION);
        if (log >= 6)
            FAE_LAUNCH(ctx, part_emit_kernel<true>, dim3((unsigned)tiles), dim3(PT_THREADS), 0, ctx->stream, a);
        else
            FAE_LAUNCH(ctx, part_emit_kernel<false>, dim3((unsigned)tiles), dim3(PT_THREADS), 0, ctx->stream, a);
        FAE_LAUNCH_CHECK(ctx);
    }
    rc = fae_readback_status(ctx, nt + 1);
    if (rc == FAE_EHIP)
        return rc;
    *h_n_hot_samples = (int64_t)ctx->h_block[FAE_BLK_SCALARS];
    for (int z = 0; z < nt; ++z)
        h_n_hot_lookups[z] = (int64_t)ctx->h_block[FAE_BLK_SCALARS + 1 + z];
    return rc;
}
