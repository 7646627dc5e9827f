// Input Classifier (Sec. 4.2): a sparse input is hot iff every access in every table
// hits a hot row.  Hot and cold inputs keep their original order; for the hot ones
// the hot slots and a rebuilt CSR are emitted so that consecutive slices are the
// hot mini-batches.  Integer-only work: random 4-byte gathers into the remap, an
// AND-reduction per sample, a stable compaction.
#include <algorithm>

#include "fae_internal.h"

#define PT_THREADS 256
#define PT_MIN_TILE 16
#define PT_MAX_TILE PT_THREADS // samples per tile: one sample per thread
#define PT_SCAN_TILE 1024      // what the size of the workspace goes by
#define PT_SUM_TILES 2048      // tiles up to which every tile adds up the counts of those before it by itself, ...
#define PT_SUM_COUNTS 3072     // ... and with more rows of counts than waves, counts (rows x tiles)
#define PT_LK 8                // lookups per thread and round
#define PT_ROUND (PT_THREADS * PT_LK)
#define PT_OFF_WORDS 1799      // offsets of bags in LDS at a time: (samples per tile + 1) per table
#define PT_HEAVY_MIN 4096      // lookups of bags up to which a tile always walks them itself

enum { PT_LIGHT, PT_HEAVY, PT_MALFORMED };

// The tables with offsets come first (n_csr of them), then those with one lookup per sample (n_one).
struct PartArgs {
    const void *idx[FAE_MAX_TABLES]; // int32 or int64 row ids
    const int32_t *offsets[FAE_MAX_TABLES];
    const int32_t *remap[FAE_MAX_TABLES];
    int32_t *slots[FAE_MAX_TABLES];
    int32_t *hoffsets[FAE_MAX_TABLES];
    int32_t n_rows[FAE_MAX_TABLES];
    int32_t n_lookups[FAE_MAX_TABLES];
    int32_t number[FAE_MAX_TABLES];        // the caller's number of the table
    int32_t blk_start[FAE_MAX_TABLES + 1]; // spread kernel: rounds of lookups per table with offsets
    int32_t wide;                    // the ids are int64
    int32_t n_one, n_csr;
    int32_t n_samples;
    int32_t tile_log;     // samples per tile: 1 << tile_log
    int32_t n_tiles;
    int32_t scanned;      // tile_sums holds running totals over row after row (else the tiles' own counts)
    int32_t heavy_min;    // a tile with more lookups in bags leaves them to the spread kernel
    int32_t leave;        // the emit kernel does nothing if there is a heavy tile
    uint32_t stamp;       // this call's number
    uint32_t *cold;       // [n_samples] 1 = some access is cold
    int32_t *tile_sums;   // [(1 + n_csr) * n_tiles + 1]; row 0 = hot samples, row 1 + c = hot lookups of table c
    int32_t *tile_state;  // [n_tiles] PT_LIGHT, PT_HEAVY or PT_MALFORMED (tables with offsets only)
    uint32_t *any_heavy;  // holds the stamp once some tile is heavy
    int32_t *hot_samples;
    int32_t *cold_samples;
    uint32_t *status;
    uint32_t *host;       // the pinned block: from FAE_BLK_SCALARS on n_hot_samples, then the hot lookups of every table
};
static_assert(sizeof(PartArgs) <= 4096, "kernel arguments are passed by value");

// lookups of sample s, which owns lookups b .. e - 1 of nl; a malformed entry sets *bad and counts none
__device__ __forceinline__ int part_len(int b, int e, int nl, int n_samples, int s, bool *bad)
{
    if (b < 0 || e < b || e > nl || (s == 0 && b != 0) || (s == n_samples - 1 && e != nl)) {
        *bad = true;
        return 0;
    }
    return e - b;
}

// the last of entries 0 .. n - 1 that is <= j (entry 0 is): with offsets, the sample that owns lookup j
__device__ __forceinline__ int part_owner(const int *entries, int n, int j)
{
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (entries[mid] <= j)
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
//   26 one-hot tables, 262 144 samples: 50 us in two kernels, 140 -> 94 us a call (before: 76 us in
//   seven launches: clear, mark, count, scan, lists, offsets, slots; and two waits instead of one)
// Tables with offsets: the offsets of the tile's samples are put into LDS for as many tables at a time
// as fit, and the lookups of all of these are walked as one list, so neither a table nor a sample
// costs a round of its own.  A tile whose lookups are much more than its share (few samples, or a
// sample with a history far longer than the others') would keep one workgroup busy for long after the rest of the
// chip has ended; it is left to part_spread_kernel, which takes lookups 2048 at a time whoever owns them.
//
// The tables with offsets, in LDS: where the lanes of a wave ask for different tables, an entry of the
// kernel's arguments is one more dependent load.  The pointers are said to be global: read back from LDS
// they could otherwise point anywhere.
#define PT_GLOBAL __attribute__((address_space(1)))
struct PartTables {
    const PT_GLOBAL void *idx[FAE_MAX_TABLES];
    const PT_GLOBAL int32_t *offsets[FAE_MAX_TABLES];
    const PT_GLOBAL int32_t *remap[FAE_MAX_TABLES];
    PT_GLOBAL int32_t *slots[FAE_MAX_TABLES];
    PT_GLOBAL int32_t *hoffsets[FAE_MAX_TABLES];
    int32_t rows[FAE_MAX_TABLES], lookups[FAE_MAX_TABLES];
    __device__ __forceinline__ void set(int c, const PartArgs &a)
    {
        idx[c] = (const PT_GLOBAL void *)a.idx[c];
        offsets[c] = (const PT_GLOBAL int32_t *)a.offsets[c];
        remap[c] = (const PT_GLOBAL int32_t *)a.remap[c];
        slots[c] = (PT_GLOBAL int32_t *)a.slots[c];
        hoffsets[c] = (PT_GLOBAL int32_t *)a.hoffsets[c];
        rows[c] = a.n_rows[c];
        lookups[c] = a.n_lookups[c];
    }
    // by the last wave, a lane per table; few tables with loads that every lane shares, which the scalar cache keeps
    __device__ __forceinline__ void fill(const PartArgs &a)
    {
        static_assert(FAE_MAX_TABLES <= FAE_WAVE, "a lane per table");
        const int t = (int)threadIdx.x - (PT_THREADS - FAE_WAVE);
        if (a.n_csr <= 4) {
            for (int c = 0; c < a.n_csr; ++c)
                if (t == 0)
                    set(c, a);
        } else if (t >= 0 && t < a.n_csr) {
            set(t, a);
        }
    }
    __device__ __forceinline__ int row(int c, int j, int wide) const { return fae_load_row((const void *)idx[c], j, wide, rows[c]); }
    __device__ __forceinline__ const PT_GLOBAL int32_t *offset(int c) const { return offsets[c]; }
    __device__ __forceinline__ const PT_GLOBAL int32_t *map(int c) const { return remap[c]; }
    __device__ __forceinline__ PT_GLOBAL int32_t *slot(int c) const { return slots[c]; }
    __device__ __forceinline__ PT_GLOBAL int32_t *hoffset(int c) const { return hoffsets[c]; }
    __device__ __forceinline__ int lookup(int c) const { return lookups[c]; }
    static constexpr int LOADS = PT_LK; // a thread's offsets in flight
    // the table among c0 .. c0 + nb - 1 that lookup i of the tile is in
    __device__ __forceinline__ int owner(const int *pre, int nb, int i) const { return part_owner(pre, nb, i); }
};
// A single table with offsets: every lane asks for the same entry, so the kernel's arguments do, and neither the
// tile's lookups before a table nor a barrier for the entries is needed (microseconds a call, as one of several /
// so: 131 843 samples of bags of 1-39 71.7 / 68.8, 14 000 of 1-3 32.6 / 30.9, beside 25 one-hot tables,
// 4096 samples 57.4 / 54.8).  With two tables the entries in LDS cost nothing any more (34.6 / 34.6).
struct PartOne {
    const PartArgs &a;
    __device__ __forceinline__ int row(int, int j, int wide) const { return fae_load_row(a.idx[0], j, wide, a.n_rows[0]); }
    __device__ __forceinline__ const int32_t *offset(int) const { return a.offsets[0]; }
    __device__ __forceinline__ const int32_t *map(int) const { return a.remap[0]; }
    __device__ __forceinline__ int32_t *slot(int) const { return a.slots[0]; }
    __device__ __forceinline__ int32_t *hoffset(int) const { return a.hoffsets[0]; }
    __device__ __forceinline__ int lookup(int) const { return a.n_lookups[0]; }
    static constexpr int LOADS = 1; // a tile has no more samples than a workgroup has threads
    __device__ __forceinline__ int owner(const int *, int, int) const { return 0; }
};

template <bool ONE> __device__ __forceinline__ const auto &part_tab(const PartTables &all, const PartOne &one)
{
    if constexpr (ONE)
        return one;
    else
        return all;
}

// table of item i (see below); with tiles of whole waves it is the same for every lane, and said so
// its descriptors are scalar loads
template <bool WAVE_TILES> __device__ __forceinline__ int part_table(const PartArgs &a, int i)
{
    const int n = a.n_csr + (i >> a.tile_log);
    return WAVE_TILES ? __builtin_amdgcn_readfirstlane(n) : n;
}

// Offsets of the tile's ns samples (and the closing one) of tables c0 .. c0 + nb - 1, T + 1 words apart.
// Returns whether a sample's are malformed, as far as this thread has seen (CHECK).
template <bool CHECK, typename Tab>
__device__ __forceinline__ bool part_load_offsets(const PartArgs &a, const Tab &tab, int c0, int nb, int s0, int ns, int *s_off)
{
    const int T = 1 << a.tile_log, items = nb << a.tile_log;
    bool bad = false;
    for (int i0 = threadIdx.x; i0 < items; i0 += Tab::LOADS * PT_THREADS) {
        int v[Tab::LOADS], e[Tab::LOADS];
#pragma unroll
        for (int k = 0; k < Tab::LOADS; ++k) { // every load goes out before the first is stored
            const int i = i0 + k * PT_THREADS, s = i & (T - 1);
            v[k] = e[k] = 0;
            if (i < items && s < ns) {
                const auto *off = tab.offset(c0 + (i >> a.tile_log)) + s0 + s;
                v[k] = off[0];
                if (CHECK)
                    e[k] = off[1];
            }
        }
#pragma unroll
        for (int k = 0; k < Tab::LOADS; ++k) {
            const int i = i0 + k * PT_THREADS, s = i & (T - 1), c = i >> a.tile_log;
            if (i < items && s < ns) {
                s_off[c * (T + 1) + s] = v[k];
                if (CHECK)
                    (void)part_len(v[k], e[k], tab.lookup(c0 + c), a.n_samples, s0 + s, &bad);
            }
        }
    }
    if (threadIdx.x < nb)
        s_off[threadIdx.x * (T + 1) + ns] = tab.offset(c0 + threadIdx.x)[s0 + ns];
    return bad;
}

// s_pre[c] = lookups of the tile in the tables before c of c0 .. c0 + nb - 1; returns those of all of them.
// Called by one wave.  A table with more than limit, which is at most 2^24, counts as limit + 1, so that the sum
// stays in range; a malformed one as none.
template <typename Tab>
__device__ __forceinline__ int part_prefix(const Tab &tab, int c0, int nb, int s0, int ns, int limit, int *s_pre)
{
    const int lane = fae_lane();
    int len = 0;
    if (lane < nb) {
        const int lo = tab.offset(c0 + lane)[s0], hi = tab.offset(c0 + lane)[s0 + ns];
        len = lo < 0 || hi < lo ? 0 : hi - lo > limit ? limit + 1 : hi - lo;
    }
    const int incl = fae_wave_incl_scan(len);
    if (lane < nb)
        s_pre[lane] = incl - len;
    if (lane == FAE_WAVE - 1)
        s_pre[nb] = incl;
    return __shfl(incl, FAE_WAVE - 1, FAE_WAVE);
}

// the same of a lone table, whose offsets are in LDS
__device__ __forceinline__ int part_lone_lookups(const int *s_off, int ns, int limit)
{
    const int lo = s_off[0], hi = s_off[ns];
    return lo < 0 || hi < lo ? 0 : hi - lo > limit ? limit + 1 : hi - lo;
}

#define PT_ROWS 4 // rows of counts that a wave takes together: their loads and sums do not depend on one another

// The tile's counts: hot samples, then the hot lookups of each table with offsets.  (In a heavy tile a
// sample counts as hot until the spread kernel finds a cold access of it, and takes it out of the counts.)
// held: offsets of every table in LDS, or null
template <typename Tab>
__device__ __forceinline__ void part_count(const PartArgs &a, const Tab &tab, int tile, const uint32_t *s_cold, const int *held)
{
    const int T = 1 << a.tile_log, s0 = tile << a.tile_log;
    const int ns = a.n_samples - s0 < T ? a.n_samples - s0 : T;
    for (int row0 = __builtin_amdgcn_readfirstlane(threadIdx.x / FAE_WAVE) * PT_ROWS; row0 <= a.n_csr; row0 += PT_THREADS / FAE_WAVE * PT_ROWS) {
        int c[PT_ROWS] = {};
        for (int s = fae_lane(); s < ns; s += FAE_WAVE) {
            int b[PT_ROWS], e[PT_ROWS];
#pragma unroll
            for (int q = 0; q < PT_ROWS; ++q) {
                const int z = row0 + q - 1;
                b[q] = 0;
                e[q] = z < 0 ? 1 : 0; // row 0 counts the samples
                if (z >= 0 && z < a.n_csr) {
                    b[q] = held ? held[z * (T + 1) + s] : a.offsets[z][s0 + s];
                    e[q] = held ? held[z * (T + 1) + s + 1] : a.offsets[z][s0 + s + 1];
                }
            }
            const bool hot = !s_cold[s];
#pragma unroll
            for (int q = 0; q < PT_ROWS; ++q) {
                const int z = row0 + q - 1;
                bool ignored = false;
                if (hot && z < a.n_csr)
                    c[q] += z < 0 ? 1 : part_len(b[q], e[q], a.n_lookups[z], a.n_samples, s0 + s, &ignored);
            }
        }
#pragma unroll
        for (int q = 0; q < PT_ROWS; ++q) {
            c[q] = __shfl(fae_wave_incl_scan(c[q]), FAE_WAVE - 1, FAE_WAVE);
            if (fae_lane() == 0 && row0 + q <= a.n_csr)
                a.tile_sums[(int64_t)(row0 + q) * a.n_tiles + tile] = c[q];
        }
    }
}

// takes the n listed samples of heavy tiles, which counted as hot, out of their tiles' counts
template <typename Tab>
__device__ __forceinline__ void part_uncount(const PartArgs &a, const Tab &tab, const int *samples, int n)
{
    const int rows = 1 + a.n_csr;
    for (int i = threadIdx.x; i < n * rows; i += PT_THREADS) {
        const int s = samples[i / rows], row = i % rows, z = row - 1;
        bool ignored = false;
        int len = 1;
        if (row > 0)
            len = part_len(tab.offset(z)[s], tab.offset(z)[s + 1], tab.lookup(z), a.n_samples, s, &ignored);
        if (len > 0)
            atomicSub(a.tile_sums + (int64_t)row * a.n_tiles + (s >> a.tile_log), len);
    }
}

template <bool WAVE_TILES, bool BAGS, bool ONE = false> __global__ __launch_bounds__(PT_THREADS, 8) void part_classify_kernel(PartArgs a)
{
    __shared__ uint32_t s_cold[PT_MAX_TILE];
    __shared__ int s_off[PT_OFF_WORDS];
    __shared__ int s_pre[FAE_MAX_TABLES + 1];
    __shared__ PartTables s_tab;
    const PartOne one{a};
    const auto &tab = part_tab<ONE>(s_tab, one);
    __shared__ int s_bad, s_heavy;
    const int T = 1 << a.tile_log, s0 = blockIdx.x << a.tile_log;
    const int ns = a.n_samples - s0 < T ? a.n_samples - s0 : T;
    const int t = threadIdx.x;
    bool bad = false;
    s_cold[t] = 0u;
    if (t == 0)
        s_bad = s_heavy = 0;
    if (BAGS && !ONE)
        s_tab.fill(a);
    __syncthreads();
    const int nb_max = PT_OFF_WORDS / (T + 1);
    const bool held = BAGS && a.n_csr <= nb_max; // the offsets of every table fit at once
    // tables with one lookup per sample: item i is sample i % T of table i / T
    const int items = a.n_one << a.tile_log;
    for (int i0 = t; i0 < items; i0 += PT_ROUND) {
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
    if constexpr (BAGS) {
        if (!ONE && t >= PT_THREADS - FAE_WAVE) { // the wave that has offsets to load last
            const int total = part_prefix(tab, 0, a.n_csr, s0, ns, a.heavy_min, s_pre);
            if (t == PT_THREADS - 1)
                s_heavy = total > a.heavy_min;
        }
        for (int c0 = 0; c0 < a.n_csr; c0 += nb_max) {
            const int nb = a.n_csr - c0 < nb_max ? a.n_csr - c0 : nb_max;
            // a sample's offsets are checked whether it is hot or cold
            if (part_load_offsets<true>(a, tab, c0, nb, s0, ns, s_off))
                s_bad = 1;
            __syncthreads();
            const int from = ONE ? 0 : s_pre[c0]; // s_pre: over all tables
            const int total = ONE ? part_lone_lookups(s_off, ns, a.heavy_min) : s_pre[c0 + nb];
            if (ONE && t == 0)
                s_heavy = total > a.heavy_min; // read again behind the next barrier only
            if (s_bad == 0 && (ONE ? total <= a.heavy_min : s_heavy == 0)) { // a malformed tile is not walked: the call reports it
                for (int i0 = from + t; i0 < total; i0 += PT_ROUND) {
                    int r[PT_LK], m[PT_LK], c[PT_LK], j[PT_LK];
#pragma unroll
                    for (int k = 0; k < PT_LK; ++k) {
                        const int i = i0 + k * PT_THREADS;
                        r[k] = -2;
                        c[k] = 0;
                        j[k] = 0;
                        if (i < total) {
                            c[k] = tab.owner(s_pre + c0, nb, i);
                            j[k] = s_off[c[k] * (T + 1)] + (i - (ONE ? 0 : s_pre[c0 + c[k]]));
                            r[k] = tab.row(c0 + c[k], j[k], a.wide);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < PT_LK; ++k)
                        m[k] = r[k] >= 0 ? tab.map(c0 + c[k])[r[k]] : -1;
#pragma unroll
                    for (int k = 0; k < PT_LK; ++k) {
                        if (r[k] == -2)
                            continue;
                        bad = bad || r[k] < 0;
                        if (m[k] < 0)
                            s_cold[part_owner(s_off + c[k] * (T + 1), ns, j[k])] = 1u;
                    }
                }
            }
            if (!held)
                __syncthreads(); // s_off is filled again for the next tables
        }
    }
    __syncthreads();
    if (bad || (t == 0 && s_bad))
        fae_flag(a.status, FAE_STATUS_ERANGE);
    if (t < ns)
        a.cold[s0 + t] = s_cold[t];
    if constexpr (BAGS) {
        if (t == 0) {
            a.tile_state[blockIdx.x] = s_bad ? PT_MALFORMED : s_heavy ? PT_HEAVY : PT_LIGHT;
            if (s_heavy && !s_bad)
                *a.any_heavy = a.stamp; // every writer stores the same value
        }
    }
    part_count(a, tab, blockIdx.x, s_cold, BAGS && held ? s_off : nullptr);
}

// Lookups of the heavy tiles: a workgroup takes a round of PT_ROUND consecutive lookups of a table,
// whichever samples own them.  The first sample is found by a search over the offsets that the workgroup
// makes together, the offsets from there on are put into LDS (PT_SLAB samples at a time; one time is
// enough, but for runs of empty bags).  Two parts, as of the tiles:
//   EMIT = false  marks the samples with a cold access (a.cold) and takes them out of their tile's counts;
//   EMIT = true   writes the slots of the hot samples.  Where they go follows from the counts of the tiles
//                 and the lengths of the samples in front of them, so nothing that the emit kernel's tiles
//                 write is needed, and this part's workgroups are the last ones of that launch.
// Microseconds a call (the tiles alone / one kernel after the other over all lookups, in seven launches):
//   one table, 16 samples of 1 000 000 lookups 224 (98 900 / 257), 1000 of 10 000 172 (1061 / 224),
//   one of 2 M lookups among 30 000 of three 97 (10 090 / 89); 64 tables, 2048 samples of 1-19 155 (577 / 163)
#define PT_SLAB 1024

template <bool EMIT>
__device__ __forceinline__ void part_spread(const PartArgs &a, int g0, int step, int *s_off, int *s_dst, int *s_list, int *s_red, PartTables &s_tab)
{
    const int t = threadIdx.x, S = a.n_samples;
    if (!EMIT)
        s_tab.fill(a); // published by the first barrier below
    bool bad = false;
    for (int g = g0; g < a.blk_start[a.n_csr]; g += step) {
        const int z = fae_find_table(a.blk_start, a.n_csr, g), nl = a.n_lookups[z];
        const int32_t *off = a.offsets[z];
        const uint32_t jb = (uint32_t)(g - a.blk_start[z]) * PT_ROUND; // the end may lie past 2^31
        const uint32_t je = jb + PT_ROUND < (uint32_t)nl ? jb + PT_ROUND : (uint32_t)nl;
        int first = fae_block_sample_of(off, S, (int)jb, s_red);
        int at = 0; // EMIT: where the first hot lookup from `first` on goes
        if (EMIT) {
            const int tile = first >> a.tile_log;
            const int32_t *sums = a.tile_sums + (int64_t)(1 + z) * a.n_tiles;
            first = tile << a.tile_log;
            if (a.scanned) {
                at = sums[tile] - sums[0];
            } else {
                int c = 0;
#pragma unroll 4
                for (int i = t; i < tile; i += PT_THREADS)
                    c += sums[i];
                (void)fae_block_excl_scan<PT_THREADS>(c, s_red, &at);
            }
        }
        for (bool more = true; more;) {
            int n = S - first < PT_THREADS ? S - first : PT_THREADS; // samples at hand, then
            __syncthreads(); // s_off and s_dst may still be read
            if (t <= n)
                s_off[t] = off[first + t];
            if (t == 0)
                s_off[n] = off[first + n];
            __syncthreads();
            if (first + n < S && (uint32_t)s_off[n] < je) { // the same for every thread
                const int all = S - first < PT_SLAB ? S - first : PT_SLAB;
                for (int i = n + 1 + t; i <= all; i += PT_THREADS)
                    s_off[i] = off[first + i];
                n = all;
                __syncthreads();
            }
            // the round's lookups that these samples own
            const uint32_t lo = (uint32_t)s_off[0] > jb ? (uint32_t)s_off[0] : jb;
            const uint32_t end = first + n < S && (uint32_t)s_off[n] < je ? (uint32_t)s_off[n] : je;
            more = end < je;
            bool heavy = false;
            for (int i = (first >> a.tile_log) + t; i <= (first + n - 1) >> a.tile_log; i += PT_THREADS)
                heavy = heavy || a.tile_state[i] == PT_HEAVY;
            heavy = __syncthreads_or(heavy);
            if (EMIT && (heavy || more)) {
                constexpr int PER = PT_SLAB / PT_THREADS;
                int len[PER], own = 0, total;
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    const int i = t * PER + q;
                    bool ignored = false;
                    len[q] = -1; // cold
                    if (i < n && a.cold[first + i] == 0u)
                        len[q] = part_len(s_off[i], s_off[i + 1], nl, S, first + i, &ignored);
                    own += len[q] > 0 ? len[q] : 0;
                }
                int to = at + fae_block_excl_scan<PT_THREADS>(own, s_red, &total);
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    s_dst[t * PER + q] = len[q] < 0 ? -1 : to;
                    to += len[q] > 0 ? len[q] : 0;
                }
                at += total;
            } else if (!EMIT && heavy) {
                for (int i = t; i < n; i += PT_THREADS)
                    s_dst[i] = 0; // 1: a cold access
            }
            __syncthreads();
            if (heavy) {
                const int32_t *remap = a.remap[z];
                int r[PT_LK], s[PT_LK], m[PT_LK];
#pragma unroll
                for (int k = 0; k < PT_LK; ++k) {
                    const uint32_t j = lo + k * PT_THREADS + t; // at most a round in all
                    r[k] = -2;
                    s[k] = 0;
                    if (j < end) {
                        r[k] = fae_load_row(a.idx[z], j, a.wide, a.n_rows[z]);
                        s[k] = part_owner(s_off, n, (int)j);
                    }
                }
#pragma unroll
                for (int k = 0; k < PT_LK; ++k)
                    if (a.tile_state[(first + s[k]) >> a.tile_log] != PT_HEAVY || (EMIT && s_dst[s[k]] < 0))
                        r[k] = -2;
#pragma unroll
                for (int k = 0; k < PT_LK; ++k)
                    m[k] = r[k] >= 0 ? remap[r[k]] : -1;
#pragma unroll
                for (int k = 0; k < PT_LK; ++k) {
                    if (EMIT) {
                        const int d = s_dst[s[k]] + ((int)(lo + k * PT_THREADS + t) - s_off[s[k]]);
                        if (r[k] >= 0 && d >= 0 && d < nl)
                            a.slots[z][d] = m[k];
                    } else if (r[k] != -2) {
                        bad = bad || r[k] < 0;
                        if (m[k] < 0)
                            s_dst[s[k]] = 1;
                    }
                }
                if (!EMIT) {
                    __syncthreads();
                    for (int i0 = 0; i0 < n; i0 += PT_THREADS) { // the same steps for every thread
                        const int i = i0 + t;
                        const bool mine = i < n && s_dst[i] && atomicExch(&a.cold[first + i], 1u) == 0u; // none of its accesses was found cold before
                        int listed;
                        const int p = fae_block_excl_scan<PT_THREADS>(mine ? 1 : 0, s_red, &listed);
                        if (mine)
                            s_list[p] = first + i;
                        __syncthreads();
                        part_uncount(a, s_tab, s_list, listed);
                        __syncthreads();
                    }
                }
            }
            first += n;
        }
    }
    if (bad)
        fae_flag(a.status, FAE_STATUS_ERANGE);
}

__global__ __launch_bounds__(PT_THREADS, 8) void part_spread_kernel(PartArgs a)
{
    __shared__ int s_off[PT_SLAB + 1], s_dst[PT_SLAB], s_list[PT_THREADS], s_red[PT_THREADS / FAE_WAVE + 1];
    __shared__ PartTables s_tab;
    part_spread<false>(a, blockIdx.x, gridDim.x, s_off, s_dst, s_list, s_red, s_tab);
}

template <bool WAVE_TILES, bool BAGS, bool ONE, bool SPREAD> __global__ __launch_bounds__(PT_THREADS, 8) void part_emit_kernel(PartArgs a)
{
    __shared__ int lds[PT_THREADS / FAE_WAVE + 1];
    __shared__ int s_base[FAE_MAX_TABLES + 1]; // per row: what the tiles before this one hold
    __shared__ int s_hot[PT_MAX_TILE];         // position of the sample among the tile's hot ones, -1 if it is cold
    __shared__ int s_off[PT_OFF_WORDS], s_dst[PT_OFF_WORDS]; // of a sample: its first lookup, and its first hot one
    __shared__ int s_pre[FAE_MAX_TABLES + 1];
    __shared__ PartTables s_tab;
    const PartOne one{a};
    const auto &tab = part_tab<ONE>(s_tab, one);
    static_assert(PT_OFF_WORDS > PT_SLAB, "the spread part uses the same room");
    if (SPREAD && blockIdx.x >= (unsigned)a.n_tiles) {
        part_spread<true>(a, blockIdx.x - a.n_tiles, gridDim.x - a.n_tiles, s_off, s_dst, nullptr, lds, s_tab);
        return;
    }
    const int T = 1 << a.tile_log, tile = blockIdx.x, s0 = tile << a.tile_log;
    const int ns = a.n_samples - s0 < T ? a.n_samples - s0 : T;
    const int t = threadIdx.x, lane = fae_lane();
    const bool hot = t < ns && a.cold[s0 + t] == 0u;
    const int state = BAGS ? a.tile_state[tile] : PT_LIGHT;
    const bool leave = BAGS && a.leave && *a.any_heavy == a.stamp;
    // The results go straight to pinned memory (the kernels before this one have reported what they had to), so neither a
    // copy nor a kernel of its own stands between the last tile and the host: 1 table, 3004 samples 26.9 -> 24.3 us a call,
    // 16 tables, 14 059 samples 41.6 -> 39.1, 26 tables, 262 144 samples 88.0 -> 86.9.
    const bool last = tile == a.n_tiles - 1;
    if (last && t == 0) {
        a.host[FAE_BLK_STATUS] = a.status[FAE_BLK_STATUS];
        a.host[FAE_BLK_HEAVY] = *a.any_heavy;
    }
    const int nb_max = PT_OFF_WORDS / (T + 1);
    if (BAGS && !ONE)
        s_tab.fill(a);
    // what the tiles before this one hold
    const int w = __builtin_amdgcn_readfirstlane(t / FAE_WAVE);
    if (a.scanned) {
        if (t <= a.n_csr) {
            const int32_t *sums = a.tile_sums + (int64_t)t * a.n_tiles;
            s_base[t] = sums[tile] - sums[0];
        }
    } else if (a.n_csr < PT_THREADS / FAE_WAVE) { // a row per wave
        if (w <= a.n_csr) {
            const int32_t *sums = a.tile_sums + (int64_t)w * a.n_tiles;
            int c = 0;
#pragma unroll 8
            for (int i = lane; i < tile; i += FAE_WAVE)
                c += sums[i];
            c = __shfl(fae_wave_incl_scan(c), FAE_WAVE - 1, FAE_WAVE);
            if (lane == 0)
                s_base[w] = c;
        }
    } else {
        for (int row0 = w * PT_ROWS; row0 <= a.n_csr; row0 += PT_THREADS / FAE_WAVE * PT_ROWS) {
            int c[PT_ROWS] = {};
#pragma unroll 2
            for (int i = lane; i < tile; i += FAE_WAVE)
#pragma unroll
                for (int q = 0; q < PT_ROWS; ++q)
                    if (row0 + q <= a.n_csr)
                        c[q] += a.tile_sums[(int64_t)(row0 + q) * a.n_tiles + i];
#pragma unroll
            for (int q = 0; q < PT_ROWS; ++q) {
                c[q] = __shfl(fae_wave_incl_scan(c[q]), FAE_WAVE - 1, FAE_WAVE);
                if (lane == 0 && row0 + q <= a.n_csr)
                    s_base[row0 + q] = c[q];
            }
        }
    }
    if constexpr (BAGS) {
        if (!ONE)
            __syncthreads();
        if (!ONE && t >= PT_THREADS - FAE_WAVE)
            (void)part_prefix(tab, 0, a.n_csr, s0, ns, a.heavy_min, s_pre);
        (void)part_load_offsets<false>(a, tab, 0, a.n_csr < nb_max ? a.n_csr : nb_max, s0, ns, s_off);
    }
    int n_here;
    const int pos = fae_block_excl_scan<PT_THREADS>(hot ? 1 : 0, lds, &n_here); // its barriers also publish s_base
    if (leave)
        return;
    const int h0 = s_base[0];
    if (t < ns) {
        s_hot[t] = hot ? pos : -1;
        if (hot)
            a.hot_samples[h0 + pos] = s0 + t;
        else
            a.cold_samples[s0 + t - h0 - pos] = s0 + t;
    }
    __syncthreads();
    uint32_t *const totals = a.host + FAE_BLK_SCALARS; // the last tile also writes the closing offsets and the totals
    if (last && t == 0)
        totals[0] = (uint32_t)(h0 + n_here);
    if (last && t < a.n_one) {
        const int z = a.n_csr + t;
        a.hoffsets[z][h0 + n_here] = h0 + n_here;
        totals[1 + a.number[z]] = (uint32_t)(h0 + n_here);
    }
    const int items = n_here > 0 ? a.n_one << a.tile_log : 0;
    for (int i0 = t; i0 < items; i0 += PT_ROUND) {
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
    if constexpr (BAGS) {
        const int lanes = T < FAE_WAVE ? T : FAE_WAVE, per = T / lanes;
        for (int c0 = 0; c0 < a.n_csr; c0 += nb_max) {
            const int nb = a.n_csr - c0 < nb_max ? a.n_csr - c0 : nb_max;
            if (c0 > 0) {
                (void)part_load_offsets<false>(a, tab, c0, nb, s0, ns, s_off);
                __syncthreads();
            }
            // where a sample's hot lookups go: `lanes` lanes per table, each with `per` consecutive samples
            for (int c = t / lanes; c < nb; c += PT_THREADS / lanes) {
                const int z = c0 + c, nl = tab.lookup(z), l = t & (lanes - 1);
                int len[PT_MAX_TILE / FAE_WAVE], own = 0;
#pragma unroll
                for (int q = 0; q < PT_MAX_TILE / FAE_WAVE; ++q) {
                    const int s = l * per + q;
                    bool ignored = false;
                    len[q] = 0;
                    if (q < per && s < ns && s_hot[s] >= 0)
                        len[q] = part_len(s_off[c * (T + 1) + s], s_off[c * (T + 1) + s + 1], nl, a.n_samples, s0 + s, &ignored);
                    own += len[q];
                }
                int at = own;
                for (int d = 1; d < lanes; d <<= 1) { // the lanes of a table run together
                    const int o = __shfl_up(at, d, FAE_WAVE);
                    at += l >= d ? o : 0;
                }
                at += s_base[1 + z] - own;
#pragma unroll
                for (int q = 0; q < PT_MAX_TILE / FAE_WAVE; ++q) {
                    const int s = l * per + q;
                    if (q < per && s < ns) {
                        s_dst[c * (T + 1) + s] = at;
                        if (s_hot[s] >= 0)
                            tab.hoffset(z)[h0 + s_hot[s]] = at;
                    }
                    at += len[q];
                }
                if (last && l == lanes - 1) {
                    tab.hoffset(z)[h0 + n_here] = at;
                    totals[1 + a.number[z]] = (uint32_t)at;
                }
            }
            __syncthreads();
            const int from = ONE ? 0 : s_pre[c0];
            const int total = state != PT_LIGHT || n_here == 0 ? 0 : ONE ? part_lone_lookups(s_off, ns, a.heavy_min) : s_pre[c0 + nb];
            for (int i0 = from + t; i0 < total; i0 += PT_ROUND) {
                static_assert(FAE_MAX_TABLES <= 256, "a table's number fits a byte");
                uint32_t tables[PT_LK / 4] = {}; // a byte each: as words they cost the eighth wave per SIMD
                int r[PT_LK], dst[PT_LK], m[PT_LK];
#pragma unroll
                for (int k = 0; k < PT_LK; ++k) {
                    const int i = i0 + k * PT_THREADS;
                    r[k] = dst[k] = -1;
                    if (i >= total)
                        continue;
                    const int c = tab.owner(s_pre + c0, nb, i);
                    const int *o = s_off + c * (T + 1);
                    const int j = o[0] + (i - (ONE ? 0 : s_pre[c0 + c]));
                    const int s = part_owner(o, ns, j);
                    if (s_hot[s] >= 0) {
                        tables[k / 4] |= (uint32_t)(c0 + c) << (k % 4 * 8);
                        dst[k] = s_dst[c * (T + 1) + s] + (j - o[s]);
                        r[k] = tab.row(c0 + c, j, a.wide);
                    }
                }
#pragma unroll
                for (int k = 0; k < PT_LK; ++k)
                    m[k] = r[k] >= 0 ? tab.map(tables[k / 4] >> (k % 4 * 8) & 0xff)[r[k]] : -1;
#pragma unroll
                for (int k = 0; k < PT_LK; ++k) {
                    const int z = tables[k / 4] >> (k % 4 * 8) & 0xff;
                    if (r[k] >= 0 && dst[k] >= 0 && dst[k] < tab.lookup(z))
                        tab.slot(z)[dst[k]] = m[k];
                }
            }
            __syncthreads(); // s_off and s_dst are filled again for the next tables
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
    for (int one = 0; one < 2; ++one) // the tables with offsets first
        for (int z = 0; z < nt; ++z) {
            const int32_t *offsets = in->h_offsets ? in->h_offsets[z] : nullptr;
            if ((offsets == nullptr) != (one == 1))
                continue;
            if (!h_remap[z] && tables->h_rows[z] > 0)
                return fae_fail(ctx, FAE_EINVAL, "fae_partition_batch: null remap for table %d", z);
            if (!h_hoffsets[z] || (!h_slots[z] && in->h_n_lookups[z] > 0))
                return fae_fail(ctx, FAE_EINVAL, "fae_partition_batch: null outputs for table %d", z);
            const int i = a.n_csr + a.n_one;
            a.idx[i] = in->h_indices[z];
            a.offsets[i] = offsets;
            a.remap[i] = h_remap[z];
            a.slots[i] = h_slots[z];
            a.hoffsets[i] = h_hoffsets[z];
            a.n_rows[i] = (int32_t)tables->h_rows[z];
            a.n_lookups[i] = (int32_t)in->h_n_lookups[z];
            a.number[i] = z;
            ++(one ? a.n_one : a.n_csr);
        }
    // Samples per tile: enough tiles for eight workgroups on every compute unit, but no more than
    // the workspace has words for (256 samples per tile always fit).
    const int rows = 1 + a.n_csr;
    const bool bags = a.n_csr > 0;
    const size_t words = part_count_words(nt, S);
    const auto tiles_of = [&](int log) { return (S + (1LL << log) - 1) >> log; };
    const auto words_of = [&](int log) { return (size_t)(rows + 1) * (size_t)tiles_of(log) + 1; }; // counts and states
    int log = 4;
    while ((1 << log) < PT_MAX_TILE && (tiles_of(log) > 8LL * ctx->n_cu || words_of(log) > words))
        ++log;
    static_assert(PT_MIN_TILE == 1 << 4, "smallest tile");
    const int64_t tiles = tiles_of(log);
    fae_carver cv(ws, ws_bytes);
    a.cold = cv.take<uint32_t>((size_t)S + 1);
    a.tile_sums = cv.take<int32_t>(words);
    if (!cv.ok || words_of(log) > words)
        return fae_fail(ctx, FAE_ENOSPC, "fae_partition_batch: workspace too small");
    a.tile_state = a.tile_sums + (size_t)rows * (size_t)tiles + 1;
    a.wide = in->index_bits == 64;
    a.n_samples = (int32_t)S;
    a.tile_log = log;
    a.n_tiles = (int32_t)tiles;
    // Every tile adds up the counts in front of it, or one more launch (5 us) turns them into running totals.
    // With a row per wave the first stays the shorter way longest (microseconds a call, added up / running totals):
    //   one table, 2048 tiles 37.7 / 39.5; 26 one-hot tables, 2048 tiles 83 / 85.5, 3907 tiles 452 / 435
    //   5 rows, 375 tiles 42 / 42, 750 tiles 47.5 / 40.5; 9 rows, 750 tiles 53 / 46.6; 27 rows, 375 tiles 83 / 80
    a.scanned = tiles > PT_SUM_TILES || (rows > PT_THREADS / FAE_WAVE && (int64_t)rows * tiles > PT_SUM_COUNTS);
    // A tile is heavy from twice its share of the bags' lookups on if four workgroups per compute unit
    // were to share them (fewer tiles leave much of the chip idle), but not below PT_HEAVY_MIN, two rounds of a
    // workgroup, which cost less than the spread kernel's launch.  Where the average tile is heavy, that launch
    // follows at once.  Else only a few samples can be so far above the others that their tiles are
    // (PT_HEAVY_MIN and twice the average more); such a call finds them when it reads the results back, and
    // only then repeats its second half with that launch in front: the calls without them pay nothing.
    int64_t lookups = 0, rounds = 0;
    for (int c = 0; c < a.n_csr; ++c) {
        lookups += a.n_lookups[c];
        a.blk_start[c] = (int32_t)rounds;
        rounds += (a.n_lookups[c] + (int64_t)PT_ROUND - 1) / PT_ROUND;
    }
    a.blk_start[a.n_csr] = (int32_t)rounds;
    int64_t heavy_min = std::max<int64_t>(lookups / (2LL * ctx->n_cu), PT_HEAVY_MIN);
    bool spread = lookups / tiles > heavy_min;
    if (!spread)
        heavy_min += 2 * (lookups / tiles);
    a.heavy_min = (int32_t)std::min<int64_t>(heavy_min, 1 << 24);
    a.leave = !spread && lookups > a.heavy_min; // else no tile can be heavy
    a.stamp = ++ctx->part_calls;
    a.any_heavy = ctx->d_block + FAE_BLK_HEAVY;
    a.hot_samples = hot_samples;
    a.cold_samples = cold_samples;
    a.status = ctx->d_block;
    a.host = ctx->h_block_dev;
    const dim3 grid((unsigned)tiles), block(PT_THREADS);
    const bool wave_tiles = log >= 6, one_bag = a.n_csr == 1;
    for (bool again = false;; again = true) {
        const dim3 spread_grid((unsigned)std::min<int64_t>(rounds, 8LL * ctx->n_cu)), emit_grid(grid.x + (spread ? spread_grid.x : 0u));
        if (!again || a.scanned) { // the counts are still there, or have become running totals
            fae_ktimer kt(ctx, FAE_K_PARTITION);
            if (one_bag && wave_tiles)
                FAE_LAUNCH(ctx, (part_classify_kernel<true, true, true>), grid, block, 0, ctx->stream, a);
            else if (one_bag)
                FAE_LAUNCH(ctx, (part_classify_kernel<false, true, true>), grid, block, 0, ctx->stream, a);
            else if (bags && wave_tiles)
                FAE_LAUNCH(ctx, (part_classify_kernel<true, true>), grid, block, 0, ctx->stream, a);
            else if (bags)
                FAE_LAUNCH(ctx, (part_classify_kernel<false, true>), grid, block, 0, ctx->stream, a);
            else if (wave_tiles)
                FAE_LAUNCH(ctx, (part_classify_kernel<true, false>), grid, block, 0, ctx->stream, a);
            else
                FAE_LAUNCH(ctx, (part_classify_kernel<false, false>), grid, block, 0, ctx->stream, a);
            FAE_LAUNCH_CHECK(ctx);
        }
        if (spread) {
            fae_ktimer kt(ctx, FAE_K_PARTITION);
            FAE_LAUNCH(ctx, part_spread_kernel, spread_grid, block, 0, ctx->stream, a);
            FAE_LAUNCH_CHECK(ctx);
        }
        if (a.scanned) {
            const int32_t scan = fae_scan_i32(ctx, a.tile_sums, (int64_t)rows * tiles);
            if (scan != FAE_OK)
                return scan;
        }
        {
            fae_ktimer kt(ctx, FAE_K_PARTITION);
            // the spread part costs the tiles registers (five spilled): only where it is launched
            if (spread && wave_tiles)
                FAE_LAUNCH(ctx, (part_emit_kernel<true, true, false, true>), emit_grid, block, 0, ctx->stream, a);
            else if (spread)
                FAE_LAUNCH(ctx, (part_emit_kernel<false, true, false, true>), emit_grid, block, 0, ctx->stream, a);
            else if (one_bag && wave_tiles)
                FAE_LAUNCH(ctx, (part_emit_kernel<true, true, true, false>), grid, block, 0, ctx->stream, a);
            else if (one_bag)
                FAE_LAUNCH(ctx, (part_emit_kernel<false, true, true, false>), grid, block, 0, ctx->stream, a);
            else if (bags && wave_tiles)
                FAE_LAUNCH(ctx, (part_emit_kernel<true, true, false, false>), grid, block, 0, ctx->stream, a);
            else if (bags)
                FAE_LAUNCH(ctx, (part_emit_kernel<false, true, false, false>), grid, block, 0, ctx->stream, a);
            else if (wave_tiles)
                FAE_LAUNCH(ctx, (part_emit_kernel<true, false, false, false>), grid, block, 0, ctx->stream, a);
            else
                FAE_LAUNCH(ctx, (part_emit_kernel<false, false, false, false>), grid, block, 0, ctx->stream, a);
            FAE_LAUNCH_CHECK(ctx);
        }
        const int32_t now = fae_wait_status(ctx);
        if (now == FAE_EHIP)
            return now;
        rc = rc != FAE_OK ? rc : now; // what the first half reported is not reported again
        if (!a.leave || ctx->h_block[FAE_BLK_HEAVY] != a.stamp)
            break;
        a.leave = 0;
        spread = true;
    }
    *h_n_hot_samples = (int64_t)ctx->h_block[FAE_BLK_SCALARS];
    for (int z = 0; z < nt; ++z)
        h_n_hot_lookups[z] = (int64_t)ctx->h_block[FAE_BLK_SCALARS + 1 + z];
    return rc;
}
