// Backward, steps 1 + 2: (hot slot, sample) pairs of a hot mini-batch sorted by slot, per table
// (Sec. 2.2, Sec. 6.2: the embedding update of hot mini-batches runs on the GPU).
//   keys     key = hot slot, value = sample id, per table segment
//   sort     inside LDS for lists of up to 16 K lookups, mostly up to 128 K (split over workgroups by key range),
//            else stable LSD radix passes over only the bits a hot slot can occupy: one kernel per
//            pass for short lists, whose tiles add up their table's digit counts themselves (direct:
//            few tiles, most of them in a few tables) or are chained through published counts;
//            histogram / column scan / scatter for long ones
// Also here: the sort started ahead of the backward (side stream), and the launch that carries
// the forward's row copies and the LDS sort together.
#include "fae_bwd.h"
#include "fae_lsort.h"

// ---------------------------------------------------------------------------------
// 1. keys
// ---------------------------------------------------------------------------------

// Four consecutive lookups of one thread: (slot, sample) pairs, 16-byte loads and stores when
// aligned, plus the digit counts of every radix pass into the workgroup's LDS histograms.
// vs: the samples of the four lookups (tables with offsets; else a lookup is its own sample).
__device__ __forceinline__ void bwd_keys_thread(const BwdArgs &a, int z, int j0, int n, const int32_t *off, const int *vs,
                                                int (*s_hist)[RADIX])
{
    const int32_t *slots = a.slots[z] + j0;
    int32_t *ko = a.keys_in + a.seg_start[z] + j0;
    int32_t *vo = a.vals_in + a.seg_start[z] + j0;
    int k[KEYS_PER_THREAD], v[KEYS_PER_THREAD];
    const bool full = j0 + KEYS_PER_THREAD <= n;
    const bool aligned = full && ((((uintptr_t)slots) | ((uintptr_t)ko) | ((uintptr_t)vo)) & 15) == 0;
    if (aligned) {
        const int4 t = *(const int4 *)slots;
        k[0] = t.x; k[1] = t.y; k[2] = t.z; k[3] = t.w;
    } else {
#pragma unroll
        for (int q = 0; q < KEYS_PER_THREAD; ++q)
            k[q] = j0 + q < n ? slots[q] : 0;
    }
    bool bad = false;
#pragma unroll
    for (int q = 0; q < KEYS_PER_THREAD; ++q) {
        const int j = j0 + q;
        v[q] = j;
        if (j >= n)
            continue;
        if ((unsigned)k[q] >= (unsigned)a.n_hot[z]) {
            bad = true;
            k[q] = a.n_hot[z]; // sorts behind every valid slot of the table; never dereferenced
        }
        if (off) {
            v[q] = vs[q]; // inside [0, n_samples) whatever the offsets hold
            if (off[v[q]] > j || off[v[q] + 1] <= j)
                bad = true; // malformed CSR
        }
    }
    if (bad)
        fae_flag(a.status, FAE_STATUS_ERANGE);
    if (a.n_passes > 0) { // digit counts of this table for every pass (their order does not matter)
#pragma unroll
        for (int q = 0; q < KEYS_PER_THREAD; ++q)
            if (j0 + q < n)
                for (int p = 0; p < a.n_passes; ++p)
                    atomicAdd(&s_hist[p][(k[q] >> (p * a.digit_bits)) & ((1 << a.digit_bits) - 1)], 1);
    }
    if (aligned) {
        *(int4 *)ko = make_int4(k[0], k[1], k[2], k[3]);
        *(int4 *)vo = make_int4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (int q = 0; q < KEYS_PER_THREAD; ++q)
            if (j0 + q < n) {
                ko[q] = k[q];
                vo[q] = v[q];
            }
    }
}

// Each thread handles four consecutive lookups (16-byte loads and stores when aligned).
// Tables with offsets: which sample a lookup belongs to is found by the workgroup together.
//   1. the sample of the workgroup's first lookup;
//   2. every later bag that starts among the workgroup's 1024 lookups marks its first lookup
//      with its sample number (the largest one wins where empty bags share a start);
//   3. a running maximum over the marks gives every lookup its sample.
__global__ __launch_bounds__(256) void bwd_keys_kernel(BwdArgs a)
{
    static_assert(KEYS_PER_BLOCK == SORT_TILE_SMALL, "a block of keys is a tile of the passes that count directly");
    static_assert(KEYS_PER_BLOCK == 256 * KEYS_PER_THREAD, "one workgroup of 256 threads per block of lookups");
    const int z = fae_find_table(a.blk_start, a.n_tables, blockIdx.x);
    const int jb = (blockIdx.x - a.blk_start[z]) * KEYS_PER_BLOCK; // the workgroup's first lookup (inside the table)
    const int j0 = jb + threadIdx.x * KEYS_PER_THREAD;
    const int n = a.seg_start[z + 1] - a.seg_start[z];
    const int32_t *off = a.offsets[z];
    __shared__ int s_hist[SWEEP_MAX_PASSES][RADIX];
    __shared__ int s_mark[KEYS_PER_BLOCK];
    __shared__ int s_red[256 / FAE_WAVE + 1];
    if (a.direct) // the span flags and the later passes' tile counts, which lie behind them
        bwd_clear_flags(a.flags, a.n_clear, a.clear_slice, 256);
    for (int p = 0; p < a.n_passes; ++p)
        s_hist[p][threadIdx.x] = 0;
    int vs[KEYS_PER_THREAD] = {0, 0, 0, 0};
    if (off) {
        const int jend = jb + KEYS_PER_BLOCK < n ? jb + KEYS_PER_BLOCK : n;
#pragma unroll
        for (int q = 0; q < KEYS_PER_THREAD; ++q)
            s_mark[threadIdx.x * KEYS_PER_THREAD + q] = -1;
        // 1.
        const int s_first = fae_block_sample_of(off, a.n_samples, jb, s_red);
        // 2. (also orders the clearing of s_mark above before the marks: fae_block_sample_of has barriers)
        for (int64_t s = (int64_t)s_first + 1 + threadIdx.x; s < a.n_samples; s += 256) {
            const int o = off[s];
            if (o >= jend)
                break;
            if (o >= jb)
                atomicMax(&s_mark[o - jb], (int)s);
        }
        __syncthreads();
        // 3. inclusive running maximum, four positions per thread
        int m[KEYS_PER_THREAD];
        int own = -1;
#pragma unroll
        for (int q = 0; q < KEYS_PER_THREAD; ++q) {
            m[q] = s_mark[threadIdx.x * KEYS_PER_THREAD + q];
            own = own > m[q] ? own : m[q];
        }
        int run = own; // maximum over this and the earlier threads of the wave
#pragma unroll
        for (int d = 1; d < FAE_WAVE; d <<= 1) {
            const int o = __shfl_up(run, d, FAE_WAVE);
            if (fae_lane() >= d)
                run = run > o ? run : o;
        }
        __syncthreads(); // s_red was read by fae_block_sample_of
        if (fae_lane() == FAE_WAVE - 1)
            s_red[threadIdx.x / FAE_WAVE] = run;
        __syncthreads();
        int before = s_first; // everything in front of this thread's positions
        for (int w = 0; w < (int)(threadIdx.x / FAE_WAVE); ++w)
            before = before > s_red[w] ? before : s_red[w];
        const int prev = __shfl_up(run, 1, FAE_WAVE);
        if (fae_lane() > 0)
            before = before > prev ? before : prev;
#pragma unroll
        for (int q = 0; q < KEYS_PER_THREAD; ++q) {
            before = before > m[q] ? before : m[q];
            vs[q] = before;
        }
    }
    __syncthreads();
    if (j0 < n)
        bwd_keys_thread(a, z, j0, n, off, vs, s_hist);
    if (a.direct) { // the block is the first pass's tile: its counts are stored as they are
        __syncthreads();
        a.tcount[(int64_t)blockIdx.x * RADIX + threadIdx.x] = s_hist[0][threadIdx.x];
    } else if (a.n_passes > 0) {
        __syncthreads();
        for (int p = 0; p < a.n_passes; ++p) {
            const int c = s_hist[p][threadIdx.x];
            if (c)
                atomicAdd(&a.ghist[(z * SWEEP_MAX_PASSES + p) * RADIX + threadIdx.x], c);
        }
    }
}


// ---------------------------------------------------------------------------------
// 2. segmented LSD radix sort, one pass = histogram / column scan / scatter
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(SORT_THREADS) void sort_hist_kernel(BwdArgs a)
{
    __shared__ int cnt[RADIX];
    const int z = fae_find_table(a.tile_start, a.n_tables, blockIdx.x);
    const int tl = blockIdx.x - a.tile_start[z];
    const int tiles_z = a.tile_start[z + 1] - a.tile_start[z];
    const int seg1 = a.seg_start[z + 1];
    const int base = a.seg_start[z] + tl * SORT_TILE;
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const int32_t *kp = a.keys_in + base;
    if (base + SORT_TILE <= seg1 && (((uintptr_t)kp) & 15) == 0) {
#pragma unroll
        for (int i = 0; i < SORT_ITEMS / 4; ++i) { // 16-byte loads; the count does not depend on the order
            const int4 t = ((const int4 *)kp)[i * SORT_THREADS + threadIdx.x];
            atomicAdd(&cnt[(t.x >> a.shift) & a.mask], 1);
            atomicAdd(&cnt[(t.y >> a.shift) & a.mask], 1);
            atomicAdd(&cnt[(t.z >> a.shift) & a.mask], 1);
            atomicAdd(&cnt[(t.w >> a.shift) & a.mask], 1);
        }
    } else {
#pragma unroll
        for (int i = 0; i < SORT_ITEMS; ++i) {
            int p = base + i * SORT_THREADS + threadIdx.x;
            if (p < seg1)
                atomicAdd(&cnt[(a.keys_in[p] >> a.shift) & a.mask], 1);
        }
    }
    __syncthreads();
    a.hist[RADIX * a.tile_start[z] + threadIdx.x * tiles_z + tl] = cnt[threadIdx.x];
}

// one wave per (table, digit): exclusive scan of that digit's counts over the table's tiles
__global__ __launch_bounds__(256) void sort_colscan_kernel(BwdArgs a)
{
    const int wid = blockIdx.x * (256 / FAE_WAVE) + threadIdx.x / FAE_WAVE;
    const int lane = fae_lane();
    if (wid >= a.n_tables * RADIX)
        return;
    const int z = wid / RADIX, d = wid % RADIX;
    const int tiles_z = a.tile_start[z + 1] - a.tile_start[z];
    int32_t *col = a.hist + RADIX * a.tile_start[z] + d * tiles_z;
    int carry = 0;
    for (int i0 = 0; i0 < tiles_z; i0 += FAE_WAVE) {
        int i = i0 + lane;
        int v = i < tiles_z ? col[i] : 0;
        int inc = fae_wave_incl_scan(v);
        if (i < tiles_z)
            col[i] = carry + inc - v;
        carry += __shfl(inc, FAE_WAVE - 1, FAE_WAVE);
    }
    if (lane == 0)
        a.tot[wid] = carry;
}

// Stable scatter of one tile.  Ranks come from a wave-level match on the digit plus per-wave
// counters; the tile is then put in digit order inside LDS so that the global writes of a
// digit are runs of consecutive addresses instead of single scattered words.
//
// ITEMS = keys per thread (a tile is 256 * ITEMS keys).
// SCATTER_COUNTED: the tile's output offsets come from the histogram / column-scan kernels.
// SCATTER_DIRECT: every tile adds up the digit counts of all tiles of its table by itself: plain
// loads that do not depend on one another, issued beside the tile's own keys.  The counts of the
// first pass come from the keys kernel (its blocks are the tiles); a pass counts the next digit of
// every key it places at the tile where the next pass will find it, with one atomic per run of
// equal (tile, digit) so that a popular slot does not queue thousands of them on one word.  No
// tile waits for another one, nothing has to be cleared by a launch of its own (the keys kernel
// clears the later passes' counts and the reduce kernel's flags), and the keys kernel counts one
// digit instead of one per pass.  Keys and passes against the chained form:
//   207 K lookups in two tables, 22 bits: 44 -> 39 us; 110 K in five tables, 18 bits: 37 -> 33 us
// The counts read grow with the square of a table's tiles (1 KB each); the rule is in bwd_sort_stage.
// Sixteen of them in flight and four waves per SIMD (99 registers; with the loop unrolled it took 239 and
// ran two): fewer in flight cost more than more waves give (1 x 128 tiles: 43.0 us, eight in flight 44.2, four 47).
// SCATTER_CHAINED: the whole pass is this one kernel.  A tile publishes its digit counts,
// then adds up the published counts of the tiles before it (walking back until it meets a
// tile that already published its running total) and publishes its own running total.  A
// tile only ever waits for tiles with smaller workgroup numbers, which the hardware starts
// first; the wait is bounded all the same and reports an internal error instead of spinning
// forever.  (Handing tiles out through a counter instead makes the order certain but costs
// ~35 ns per workgroup, one device-wide atomic after the other: half the time of a pass over
// a short list.  sort_variant 4 does it that way.)
enum { SCATTER_COUNTED, SCATTER_CHAINED, SCATTER_DIRECT };
template <int MODE, int ITEMS> __global__ __launch_bounds__(SORT_THREADS, MODE == SCATTER_DIRECT ? 4 : 1) void sort_scatter_kernel(BwdArgs a)
{
    constexpr int TILE = SORT_THREADS * ITEMS;
    constexpr bool CHAINED = MODE == SCATTER_CHAINED;
    __shared__ int wcnt[SORT_WAVES][RADIX];  // per wave: running count, then start inside the tile
    __shared__ int gbase[RADIX];             // global position of the tile's first element of a digit
    __shared__ int tbase[RADIX];             // position inside the tile of the first element of a digit
    __shared__ int skey[TILE], sval[TILE];
    __shared__ int scan_lds[SORT_THREADS / FAE_WAVE + 1];
    __shared__ int s_tile;
    __shared__ int s_gave_up; // a chained wait of this tile gave up: nothing of the tile is written
    if (CHAINED && threadIdx.x == 0)
        s_gave_up = 0;
    int tile = blockIdx.x;
    if (CHAINED && a.use_ticket) {
        if (threadIdx.x == 0)
            s_tile = atomicAdd(&a.ticket[a.pass], 1);
        __syncthreads();
        tile = s_tile;
    }
    const int z = fae_find_table(a.tile_start, a.n_tables, tile);
    const int tl = tile - a.tile_start[z];
    const int tiles_z = a.tile_start[z + 1] - a.tile_start[z];
    const int seg1 = a.seg_start[z + 1];
    const int w = threadIdx.x / FAE_WAVE, lane = fae_lane();
    const int tile0 = a.seg_start[z] + tl * TILE;
    const int base = tile0 + w * (FAE_WAVE * ITEMS);
    const int n_tile = seg1 - tile0 < TILE ? seg1 - tile0 : TILE;
    volatile int *my_cnt = wcnt[w];
#pragma unroll
    for (int i = 0; i < RADIX / FAE_WAVE; ++i)
        my_cnt[i * FAE_WAVE + lane] = 0;
    __builtin_amdgcn_wave_barrier();

    int key[ITEMS], val[ITEMS], off[ITEMS];
    const uint64_t lt_mask = (1ull << lane) - 1ull;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int p = base + i * FAE_WAVE + lane;
        const bool valid = p < seg1;
        key[i] = valid ? a.keys_in[p] : 0;
        val[i] = valid ? a.vals_in[p] : 0;
    }
    // direct: keys of every digit in the table's earlier tiles and in all of them.  A wave takes
    // every fourth tile, a lane four digits, sixteen 16-byte loads in flight.
    __shared__ __align__(16) int s_sum[MODE == SCATTER_DIRECT ? 2 : 1][SORT_WAVES][MODE == SCATTER_DIRECT ? RADIX : 4];
    if (MODE == SCATTER_DIRECT) {
        constexpr int UN = 16;
        const int32_t *tc = a.tcount + (int64_t)a.tile_start[z] * RADIX + 4 * lane;
        int4 before = make_int4(0, 0, 0, 0), all = make_int4(0, 0, 0, 0);
        if (4 * lane <= a.mask)
#pragma unroll 1
            for (int r0 = w; r0 < tiles_z; r0 += UN * SORT_WAVES) {
                int4 c[UN];
#pragma unroll
                for (int q = 0; q < UN; ++q) {
                    const int r = r0 + q * SORT_WAVES;
                    c[q] = *(const int4 *)(tc + (int64_t)(r < tiles_z ? r : r0) * RADIX);
                }
#pragma unroll
                for (int q = 0; q < UN; ++q) {
                    const int r = r0 + q * SORT_WAVES;
                    const int in = r < tiles_z ? -1 : 0, lower = r < tl ? -1 : 0;
                    all.x += c[q].x & in;
                    all.y += c[q].y & in;
                    all.z += c[q].z & in;
                    all.w += c[q].w & in;
                    before.x += c[q].x & lower;
                    before.y += c[q].y & lower;
                    before.z += c[q].z & lower;
                    before.w += c[q].w & lower;
                }
            }
        *(int4 *)&s_sum[0][w][4 * lane] = before;
        *(int4 *)&s_sum[1][w][4 * lane] = all;
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool valid = base + i * FAE_WAVE + lane < seg1;
        const int d = (key[i] >> a.shift) & a.mask;
        // lanes of this round that hold the same digit (valid lanes only)
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < RADIX_BITS; ++b) {
            const bool bit = (d >> b) & 1;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const int rank = __popcll(peers & lt_mask);
        const int n_peers = __popcll(peers);
        int old = 0;
        if (valid) {
            old = my_cnt[d];
            if (rank == 0)
                my_cnt[d] = old + n_peers;
        }
        __builtin_amdgcn_wave_barrier();
        off[i] = old + rank;
    }
    __syncthreads();
    {
        // thread t owns digit t: the four waves' counts -> starts inside the tile and in the output
        const int t = threadIdx.x;
        const int c0 = wcnt[0][t], c1 = wcnt[1][t], c2 = wcnt[2][t], c3 = wcnt[3][t];
        int total;
        if (MODE == SCATTER_DIRECT) {
            int d_before = 0, d_all = 0;
#pragma unroll
            for (int i = 0; i < SORT_WAVES; ++i) {
                d_before += s_sum[0][i][t];
                d_all += s_sum[1][i][t];
            }
            gbase[t] = a.seg_start[z] + fae_block_excl_scan<SORT_THREADS>(d_all, scan_lds, &total) + d_before;
        } else if (!CHAINED) {
            const int ex = fae_block_excl_scan<SORT_THREADS>(a.tot[z * RADIX + t], scan_lds, &total);
            gbase[t] = a.seg_start[z] + ex + a.hist[RADIX * a.tile_start[z] + t * tiles_z + tl];
        } else {
            const uint32_t mine = (uint32_t)(c0 + c1 + c2 + c3);
            uint32_t *st = a.state + ((size_t)a.pass * a.total_tiles + tile) * RADIX + t;
            uint32_t before = 0; // lookups with digit t in the earlier tiles of this table
            if (tl == 0) {
                __hip_atomic_store(st, (SWEEP_PREFIX << 30) | mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                __hip_atomic_store(st, (SWEEP_AGGREGATE << 30) | mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                // Walk back over the earlier tiles of the table, eight at a time (their words are
                // loaded together; a tile that has published nothing yet is read again).  The
                // table's first tile publishes a running total, so the walk stops there at the latest.
                int back = 1; // distance of the nearest tile not yet added
                int spins = 0;
                bool done = false;
                while (!done) {
                    uint32_t v[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        const int bq = back + q <= tl ? back + q : tl; // clamped into the table (tile tl back is its first)
                        v[q] = __hip_atomic_load(st - (size_t)bq * RADIX, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        if (done || back > tl)
                            break;
                        const uint32_t flag = v[q] >> 30;
                        if (flag == 0) { // not published yet: start the next round at this tile
                            if (++spins > SWEEP_SPIN_LIMIT) {
                                fae_flag(a.status, FAE_STATUS_EINTERNAL);
                                s_gave_up = 1;
                                done = true;
                            } else {
                                __builtin_amdgcn_s_sleep(1);
                            }
                            break;
                        }
                        before += v[q] & 0x3fffffffu;
                        ++back;
                        if (flag == SWEEP_PREFIX)
                            done = true;
                    }
                    if (back > tl)
                        done = true; // cannot happen before a running total is met; keeps the walk inside the table
                }
                __hip_atomic_store(st, (SWEEP_PREFIX << 30) | (before + mine), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            const int ex = fae_block_excl_scan<SORT_THREADS>(
                a.ghist[(z * SWEEP_MAX_PASSES + a.pass) * RADIX + t], scan_lds, &total);
            gbase[t] = a.seg_start[z] + ex + (int)before;
        }
        const int tb = fae_block_excl_scan<SORT_THREADS>(c0 + c1 + c2 + c3, scan_lds, &total);
        tbase[t] = tb;
        wcnt[0][t] = tb;
        wcnt[1][t] = tb + c0;
        wcnt[2][t] = tb + c0 + c1;
        wcnt[3][t] = tb + c0 + c1 + c2;
    }
    __syncthreads();
    // The running total of a tile whose wait gave up is wrong (it was published all the same, so
    // that later tiles do not wait in turn): its pairs are not written.  The status word is set;
    // the reduce kernel looks at it before it reads any pair and leaves the tables alone.
    if (CHAINED && s_gave_up)
        return;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (base + i * FAE_WAVE + lane < seg1) {
            const int d = (key[i] >> a.shift) & a.mask;
            const int lp = wcnt[w][d] + off[i];
            skey[lp] = key[i];
            sval[lp] = val[i];
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int lp = i * SORT_THREADS + threadIdx.x;
        int at = -1; // direct: where the next pass counts this key
        if (lp < n_tile) {
            const int k = skey[lp];
            const int d = (k >> a.shift) & a.mask;
            const int dst = gbase[d] + (lp - tbase[d]);
            a.keys_out[dst] = k;
            a.vals_out[dst] = sval[lp];
            at = (a.tile_start[z] + (dst - a.seg_start[z]) / TILE) * RADIX + ((k >> (a.shift + a.digit_bits)) & a.mask);
        }
        if (MODE == SCATTER_DIRECT && a.tcount_next) {
            const int prev = __shfl_up(at, 1, FAE_WAVE);
            const bool head = lane == 0 || prev != at;
            const uint64_t later = __ballot(head) & ~((2ull << lane) - 1ull); // lane 63: 2 << 63 is 0, nothing is later
            if (head && at >= 0)
                atomicAdd(&a.tcount_next[at], (later && lane < FAE_WAVE - 1 ? (int)__builtin_ctzll(later) : FAE_WAVE) - lane);
        }
    }
}

// ---------------------------------------------------------------------------------
// 2b. tables of up to LSORT_MAX lookups: sorted inside LDS by a few workgroups per table (fae_lsort.h)
// ---------------------------------------------------------------------------------
template <bool ANY> __global__ __launch_bounds__(LSORT_THREADS, 8) void lds_sort_kernel(LsortArgs a)
{
    bwd_clear_flags(a.flags, a.n_flags, a.flag_slice, LSORT_THREADS);
    const int z = fae_find_table(a.blk_start, a.n_tables, blockIdx.x);
    lds_sort_block<ANY>(a.slots[z], a.offsets[z], a.seg_start[z + 1] - a.seg_start[z], a.n_hot[z], blockIdx.x - a.blk_start[z],
                   a.blk_start[z + 1] - a.blk_start[z], a.part_slots[z], a.n_samples, a.keys_out + a.seg_start[z],
                   a.vals_out + a.seg_start[z], a.status);
}

// ---------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------
// Lists beyond LSORT_SHORT lookups in LDS, instead of a keys kernel and radix passes: up to 100 000 lookups, and up to
// LSORT_MAX where the batch has no more than a million (what every part's way over the whole list costs grows with the square of the
// list), and, by itself, only where some slot needs three passes.  Sort kernels, us, passes / LDS:
//   1 x 17 000 28-34 / 17.6, 1 x 131 000 33.4 / 28.9, 3 x 100 000 43.3 / 33.5, 7 x 65 536 44.6 / 28.9, 13 x 100 000 67.8 / 52.7
//   26 x 17 000 40.9 / 26.7, 26 x 65 536 68.6 / 51.5, 26 x 100 000 81.1 / 76.4, 13 x 131 000 70.5 / 80.1, 26 x 131 000 97.8 / 106.9
//   bags of 20: 1 x 65 536 30.2 / 23.0, 3 x 100 000 45.3 / 45.7, 13 x 65 536 55.7 / 41.3, 13 x 131 000 72.6 / 72.3
//   slots of 13 bits (two passes): 7 x 18 432 26.3 / 17.6, 13 x 60 000 34.6 / 29.9, 2 x 110 000 28.1 / 34.0; 40 rows (one
//   pass): 7 x 18 432 18.1 / 18.0, 13 x 60 000 20.8 / 29.5, 2 x 110 000 13.0 / 35.6.  So two passes or one are left as they are.
#define LSORT_SHORT 16384
#define FUSED_ALONE_LANES 32 // lanes per row from which on a workgroup of the fused launch has a compute unit to itself
// Samples per copying wave of the fused launch: its workgroups fill what the sorting ones leave of the chip, and pieces of 64
// left a nearly empty last round.  26 tables, three batches' inputs in turn, 64 / 32 / 16 samples, us a step: 16 384 samples, dim 64
// 77.6 / 72.8 / 73.4, dim 128 143.6 / 138.9 / 142.6; 50 001 samples, dim 64 218 / 210 / 215; 4096, dim 16 22.9 / 23.0 / 23.0.
// (A loop of no more steps than 32 samples need, against one made for 64: 26 x 8192, dim 256 197 -> 187, 26 x 16 384, dim 64 87.3 -> 82.9,
// 1 x 1024, dim 256 41 -> 34.)  A row of one lane: a slot for each.
#define FUSED_SAMPLES(lanes) ((lanes) == 1 ? FAE_WAVE : 32)
#define LSORT_LONG_ROWS 65536
static bool lsort_takes(int64_t lookups, int64_t all)
{
    return lookups <= 100000 || (lookups <= LSORT_MAX && all <= 1 << 20);
}

// Whether one launch for forward and sort is the shorter way beyond LSORT_SHORT samples.  It is, whatever the slots' bits, since the
// copies hide most of the sort, except where the sort would be a single pass over at most 255 slots and the copies are too few to
// hide what every part's way over the whole list costs.  Steps of 40 slots, three batches' inputs in turn, us, one launch / apart:
//   dim 16: 1 x 30 000 22.1 / 23.5, 50 000 27 / 25, 100 000 37 / 29; 2 x 40 000 26 / 24, 100 000 41 / 33; 4 x 65 536 34 / 31
//   8 x 60 000 40 / 42, 8 x 100 000 67 / 60, 10 x 100 000 80 / 80, 13 x 100 000 84 / 98; dim 64: 1 x 100 000 46 / 40, 8 x 100 000 143 / 148
// 1000 slots (two passes): dim 16 1 x 100 000 35 / 38, 4 x 100 000 44 / 53, 8 x 100 000 70 / 78, dim 128 1 x 100 000 54.5 / 64.
static bool lsort_fuses(int64_t samples, int64_t all, int64_t most_slots, int lanes)
{
    if (samples <= LSORT_SHORT || most_slots >= RADIX)
        return true;
    return !((samples > 40000 && all <= 1 << 18) || (samples > 90000 && all <= 900000 && lanes <= 8));
}

// Workgroups per table for the LDS sort.  Lists that are split into ranges of slots: enough parts to
// occupy the chip, never below ~64 lookups (a part of up to 256 is sorted by counting; a step of 8 x 1024 lookups,
// parts down to 512, 256, 128, 64, 32: 19.3, 17.6, 17.6, 17.5, 17.4 us; of 1 x 512: 15.8, 14.6, 14.8, 14.7, 14.1 us).  The ranges are
// equal, not the slot's top bits, which make half as many parts twice as large just above a power of two (70 000 slots, steps, top bits / equal:
// 40 x 11 000 49.9 / 45.5, 13 x 16 384 31.6 / 29.0, 1 x 1024 13.3 / 12.4; 130 000 slots the same either way).
// Beside more copies than there are compute units of rows of 32 lanes on (there a sorting workgroup has a unit to itself), or than twice as many of
// rows of 16, no more than four a table: steps with up to sixteen / four, 26 x 8192, dim 128 90.8 / 88.2, dim 256 187 / 185; 26 x 10 000, dim 64
// 59.8 / 59.2, dim 128 111 / 106; 13 x 10 200, dim 128 60.0 / 58.9; with fewer copies of 16 lanes 13 x 16 384 49 / 56, 20 x 12 000 55 / 57.
// Those split by rank: one sorting workgroup per compute unit over all tables (no more, where no copies run beside them: two that share one
// end later; sort alone, 3 x 100 000 with 258 / 256 workgroups 37.5 / 28.4, 3 lists of 207 K with 272 / 256 35.7 / 32.8, 5 x 102 400 45 / 35), parts
// of 512 to 5000 lookups (every part goes over its
// table's whole list, so more of them cost more than shorter ones save; 5000 leaves room for the sample's error below
// LSORT_CAP); 5 lists of 111 K in all, parts of 512, 1024: 43.4, 45.3 us.  Beside row copies two for three compute units, and
// one for two where more workgroups copy rows of 16 lanes on than there are compute units, since those need the memory's
// rate from all of them.  Steps, three batches' inputs in turn, two for three / one for two: 26 x 16 384, dim 64 73.9 /
// 72.8 us, 12 000 60.5 / 59.3; 26 x 11 000, dim 16 34.5 / 35.1; 3 x 65 536, dim 8 36.4 / 37.9.  Where a sorting workgroup
// has a compute unit to itself (see fwd_sort_kernel), no less than 3300: 13 x 16 384, dim 128, without / with 79.3 / 76.0.
// part_slots[z]: slots of a part that is a range, 0 where parts are found by rank; blk_start: prefix of workgroups per table (tables not
// sorted in LDS get none).  Returns the number of workgroups.
static int lsort_plan(const fae_ctx *ctx, const fae_tables *hot_tables, const fae_batch *hot_batch, const bool *in_lds,
               int n_lds, int32_t *blk_start, uint32_t *part_slots, int copy_lanes, int64_t copy_blocks)
{
    const int nt = hot_tables->n_tables;
    const bool many = copy_blocks > ctx->n_cu;
    int want = 1;
    while (want < 16 && n_lds * want * 2 <= ctx->n_cu)
        want <<= 1;
    if (want > 4 && (copy_lanes >= FUSED_ALONE_LANES ? many : copy_lanes >= 16 && copy_blocks > 2LL * ctx->n_cu))
        want = 4;
    // Lookups up to which a list is split into ranges of slots: finding the parts by rank takes 2.5 us more, and longer lists gain more from
    // even parts, the more so the more skewed they are.  Steps, a bounded Zipf law of 0.9 / 1.2, us, ranges then by rank: dim 16 1 x 12 000 19.1,
    // 20.3 / 21.6, 21.4; 8 x 12 000 23.2, 25.2 / 26.7, 25.7; 1 x 16 384 19.6, 20.8 / 23.2, 21.4; 8 x 16 384 25.2, 26.9 / 28.8, 27.0; sort alone 4 x 16 384
    // 27.8, 28.9 / 30.6, 28.8, 26 x 16 384 49.5, 50.5 / 49.5, 48.0.  Rows of 16 lanes beside many copies, where the longest part ends last: 26 x 16 384,
    // dim 64 (workload 3) 76.1, 73.1; 26 x 12 000 60.2, 58.9; of 32 lanes 26 x 16 384 139.1, 140.9 / 132.7, 133.6; 13 x 16 384 70.3, 71.1.
    const int64_t ranges = copy_lanes >= FUSED_ALONE_LANES || ctx->opt_sort_order == 1 ? LSORT_SPLIT_MAX : many && copy_lanes >= 16 ? 10240 : 13312;
    int64_t long_lookups = 0;
    int nb = 0;
    for (int z = 0; z < nt; ++z) {
        part_slots[z] = 0; // by rank
        blk_start[z] = 0;
        if (!in_lds[z])
            continue;
        const int64_t n = hot_batch->h_n_lookups[z];
        if (n > ranges) {
            long_lookups += n;
            continue;
        }
        int parts = want;
        while (parts > 1 && n / parts < 64)
            parts >>= 1;
        const int64_t keys = hot_tables->h_rows[z] + 1; // n_hot itself marks an invalid slot
        part_slots[z] = (uint32_t)((keys + parts - 1) / parts);
        blk_start[z] = (int)((keys + part_slots[z] - 1) / part_slots[z]);
        nb += blk_start[z];
    }
    int64_t share = long_lookups * (many && copy_lanes >= 16 ? 4 : copy_blocks > 0 ? 3 : 2) / (2 * ctx->n_cu);
    const int64_t least = many && copy_lanes >= FUSED_ALONE_LANES ? 3300 : 512;
    share = share < least ? least : (share > 5000 ? 5000 : share);
    if (copy_blocks == 0 && long_lookups > 0) { // rounding up may not take them beyond one per compute unit
        const auto parts_of = [&](int64_t per) {
            int64_t p = nb;
            for (int z = 0; z < nt; ++z)
                if (in_lds[z] && hot_batch->h_n_lookups[z] > ranges)
                    p += (hot_batch->h_n_lookups[z] + per - 1) / per;
            return p;
        };
        while (share < 5000 && parts_of(share) > ctx->n_cu)
            share += share / 32 + 1;
        share = share > 5000 ? 5000 : share;
    }
    nb = 0;
    for (int z = 0; z < nt; ++z) {
        const int parts = !in_lds[z] ? 0 : hot_batch->h_n_lookups[z] > ranges ? (int)((hot_batch->h_n_lookups[z] + share - 1) / share) : blk_start[z];
        blk_start[z] = nb;
        nb += parts;
    }
    blk_start[nt] = nb;
    return nb;
}

// Steps 1 + 2 on stream `st`: (slot, sample) pairs sorted by slot per table.  *cur_out names
// the ping-pong buffer that holds the result.
int32_t bwd_sort_stage(fae_ctx *ctx, hipStream_t st, const fae_tables *hot_tables, const fae_batch *hot_batch,
                       BwdSetup &su, int *cur_out)
{
    BwdArgs &a = su.a;
    const BwdWs &w = su.w;
    const int nt = hot_tables->n_tables;
    // Tables that are sorted in LDS take no part in the global passes (zero tiles, zero key blocks).
    bool in_lds[FAE_MAX_TABLES];
    int n_lds = 0;
    int64_t max_hot_global = 0;
    int64_t tiles = 0;
    int64_t max_hot_long = 0; // of the lists beyond LSORT_SHORT
    for (int z = 0; z < nt; ++z)
        if (hot_batch->h_n_lookups[z] > LSORT_SHORT && hot_tables->h_rows[z] > max_hot_long)
            max_hot_long = hot_tables->h_rows[z];
    for (int z = 0; z < nt; ++z) {
        const int64_t nl = hot_batch->h_n_lookups[z];
        in_lds[z] = ctx->opt_sort != 1 && nl > 0 && nl <= LSORT_MAX && (nl <= LSORT_SHORT || !a.offsets[z] || a.n_samples <= LSORT_MAX);
        if (in_lds[z] && nl > LSORT_SHORT && ctx->opt_sort != 2)
            in_lds[z] = ctx->opt_sort == 0 && max_hot_long >= LSORT_LONG_ROWS && lsort_takes(nl, su.plan.N);
        if (!in_lds[z] && nl > 0 && hot_tables->h_rows[z] > max_hot_global)
            max_hot_global = hot_tables->h_rows[z];
    }
    // When some table needs the global passes anyway, a small table whose slots need no more
    // passes than those rides along: its few tiles cost nothing there, and if no small table is
    // left the LDS sort (a launch of its own, ~10 us however small the table) is not needed.
    if (max_hot_global > 0 && ctx->opt_sort != 2) {
        int gbits = 1;
        while ((max_hot_global >> gbits) != 0)
            ++gbits;
        const int gpasses = (gbits + RADIX_BITS - 1) / RADIX_BITS;
        for (int z = 0; z < nt; ++z)
            if (in_lds[z] && hot_tables->h_rows[z] < (1LL << (gpasses * RADIX_BITS)))
                in_lds[z] = false;
    }
    for (int z = 0; z < nt; ++z) {
        const int64_t nl = hot_batch->h_n_lookups[z];
        if (in_lds[z])
            ++n_lds;
        else if (nl > 0 && hot_tables->h_rows[z] > max_hot_global)
            max_hot_global = hot_tables->h_rows[z];
        a.tile_start[z] = (int32_t)tiles;
        if (!in_lds[z])
            tiles += (nl + SORT_TILE - 1) / SORT_TILE;
    }
    a.tile_start[nt] = (int32_t)tiles;
    // only the bits a slot (or the invalid marker n_hot) can occupy are sorted
    int bits = 1;
    while ((max_hot_global >> bits) != 0)
        ++bits;
    const int passes = tiles > 0 ? (bits + RADIX_BITS - 1) / RADIX_BITS : 0;
    const int digit_bits = passes > 0 ? (bits + passes - 1) / passes : RADIX_BITS;
    // Tiles that add up their table's counts themselves (sort_variant 1, 3 and 4 force the other forms).  What
    // that reads grows with the square of a table's tiles, and what it saves is the chain from tile to tile,
    // so it pays where the tiles fit the chip at once (one per compute unit) and a few tables hold most of
    // them.  Backward, microseconds, chained / direct:
    //   1 x 64 tiles 43.2 / 38.9, 1 x 128 49.8 / 43.0, 2 x 64 47.1 / 42.6, 4 x 30 45.2 / 42.1, 4 x 50 50.8 / 48.0
    //   2 x 128 57.4 / 55.7, 4 x 64 54.3 / 55.5, 5 x 22 42.8 / 42.1; 8 x 18 44.6 / 45.2, 8 x 25 48.3 / 49.5, 13 x 18 50.4 / 52.1
    //   3 x 100 59.1 / 63.5, 8 x 64 71 / 78, 26 x 20 70 / 81, 8 x 128 104 / 127
    int64_t small_total = 0, small_most = 0;
    for (int z = 0; z < nt; ++z)
        if (!in_lds[z]) {
            const int64_t t = (hot_batch->h_n_lookups[z] + SORT_TILE_SMALL - 1) / SORT_TILE_SMALL;
            small_total += t;
            small_most = t > small_most ? t : small_most;
        }
    const bool direct = passes > 0 && w.tcount != nullptr && small_total <= ctx->n_cu && small_total <= 6 * small_most &&
                        (ctx->opt_sort == 0 || ctx->opt_sort == 2);
    // Short lists: one kernel per pass (tiles chained through published counts), which saves
    // two launches per pass where launches are what a pass costs.  Long lists keep the
    // three-kernel passes: there the chained kernel's waits cost as much as the launches
    // (measured: 59 us against 63 us per pass at 10.5 M lookups, 16 us against 30 us at 0.2 M).
    // The chained kernel's counters start at zero; the keys kernel fills the per-table digit
    // histograms of all passes.  sort_variant 1 forces the three-kernel passes, 3 the chained ones.
    const bool chained =
        passes > 0 && !direct && ctx->opt_sort != 1 && (ctx->opt_sort == 3 || ctx->opt_sort == 4 || tiles <= 4LL * ctx->n_cu);
    a.use_ticket = ctx->opt_sort == 4;
    // A chained pass over a short list takes small tiles: more workgroups, a shorter chain per tile
    // (the same rule sizes the workspace, so it goes by the lookups of all tables).
    const bool small_tiles = direct || (chained && su.plan.small_tiles <= SORT_SMALL_MAX_TILES);
    if (small_tiles) {
        tiles = 0;
        for (int z = 0; z < nt; ++z) {
            a.tile_start[z] = (int32_t)tiles;
            if (!in_lds[z])
                tiles += (hot_batch->h_n_lookups[z] + SORT_TILE_SMALL - 1) / SORT_TILE_SMALL;
        }
        a.tile_start[nt] = (int32_t)tiles;
    }
    if (chained) {
        a.n_passes = passes;
        a.digit_bits = digit_bits;
        a.total_tiles = (int32_t)tiles;
        a.ticket = (int32_t *)w.sweep;
        a.ghist = (int32_t *)w.sweep + 64;
        a.state = w.sweep + 64 + (size_t)nt * SWEEP_MAX_PASSES * RADIX;
    }
    if (direct) {
        // counts of pass 0 behind those of the later passes: they are stored, not added to
        a.direct = 1;
        a.n_passes = 1;
        a.digit_bits = digit_bits;
        a.tcount = w.tcount + (int64_t)(passes - 1) * tiles * RADIX;
        a.n_clear = (int32_t)((w.tcount - w.flags) + (int64_t)(passes - 1) * tiles * RADIX);
        a.clear_slice = bwd_flag_slice(a.n_clear, tiles);
    }
    if (tiles > 0 && !direct) {
        // The span flags of the reduce kernel start at zero too.  The LDS sort clears them itself;
        // a batch with tables on the global passes gets them cleared here, together with the
        // chained passes' counters that follow them in the workspace.  (Clearing them in the keys
        // kernel instead cost that kernel a third of its time.)
        int64_t words = a.n_flags;
        if (chained)
            words = ((int32_t *)w.sweep - w.flags) +
                    (64 + ((int64_t)nt * SWEEP_MAX_PASSES + (int64_t)passes * tiles) * RADIX);
        int32_t rc = fae_fill_u32_on(ctx, st, w.flags, words, 0u);
        if (rc != FAE_OK)
            return rc;
    }
    // 1. keys
    {
        int64_t blocks = 0;
        for (int z = 0; z < nt; ++z) {
            a.blk_start[z] = (int32_t)blocks;
            if (!in_lds[z])
                blocks += (hot_batch->h_n_lookups[z] + KEYS_PER_BLOCK - 1) / KEYS_PER_BLOCK;
        }
        a.blk_start[nt] = (int32_t)blocks;
        a.keys_in = w.keys[0];
        a.vals_in = w.vals[0];
        if (blocks > 0) {
            fae_ktimer kt(ctx, FAE_K_BWD_KEYS, st);
            FAE_LAUNCH(ctx, bwd_keys_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a);
            FAE_LAUNCH_CHECK(ctx);
        }
    }
    // 2. sort
    int cur = 0;
    for (int pass = 0; pass < passes; ++pass) {
        a.pass = pass;
        a.shift = pass * digit_bits;
        a.mask = (1 << digit_bits) - 1;
        a.keys_in = w.keys[cur];
        a.vals_in = w.vals[cur];
        a.keys_out = w.keys[cur ^ 1];
        a.vals_out = w.vals[cur ^ 1];
        if (direct) {
            a.tcount = w.tcount + (int64_t)(pass > 0 ? pass - 1 : passes - 1) * tiles * RADIX;
            a.tcount_next = pass + 1 < passes ? w.tcount + (int64_t)pass * tiles * RADIX : nullptr;
            fae_ktimer kt(ctx, FAE_K_SORT_SCATTER, st);
            FAE_LAUNCH(ctx, (sort_scatter_kernel<SCATTER_DIRECT, SORT_ITEMS_SMALL>), dim3((unsigned)tiles), dim3(SORT_THREADS), 0, st, a);
            FAE_LAUNCH_CHECK(ctx);
            cur ^= 1;
            continue;
        }
        if (chained) {
            fae_ktimer kt(ctx, FAE_K_SORT_SCATTER, st);
            if (small_tiles)
                FAE_LAUNCH(ctx, (sort_scatter_kernel<SCATTER_CHAINED, SORT_ITEMS_SMALL>), dim3((unsigned)tiles), dim3(SORT_THREADS), 0, st, a);
            else
                FAE_LAUNCH(ctx, (sort_scatter_kernel<SCATTER_CHAINED, SORT_ITEMS>), dim3((unsigned)tiles), dim3(SORT_THREADS), 0, st, a);
            FAE_LAUNCH_CHECK(ctx);
            cur ^= 1;
            continue;
        }
        {
            fae_ktimer kt(ctx, FAE_K_SORT_HIST, st);
            FAE_LAUNCH(ctx, sort_hist_kernel, dim3((unsigned)tiles), dim3(SORT_THREADS), 0, st, a);
            FAE_LAUNCH_CHECK(ctx);
        }
        {
            fae_ktimer kt(ctx, FAE_K_SORT_COLSCAN, st);
            FAE_LAUNCH(ctx, sort_colscan_kernel, dim3((unsigned)((nt * RADIX + 3) / 4)), dim3(256), 0, st, a);
            FAE_LAUNCH_CHECK(ctx);
        }
        {
            fae_ktimer kt(ctx, FAE_K_SORT_SCATTER, st);
            FAE_LAUNCH(ctx, (sort_scatter_kernel<SCATTER_COUNTED, SORT_ITEMS>), dim3((unsigned)tiles), dim3(SORT_THREADS), 0, st, a);
            FAE_LAUNCH_CHECK(ctx);
        }
        cur ^= 1;
    }
    a.keys_in = w.keys[cur];
    a.vals_in = w.vals[cur];
    a.keys_out = nullptr;
    a.vals_out = nullptr;
    if (n_lds > 0) { // small tables: straight from the slots into the final buffer
        LsortArgs la;
        memset(&la, 0, sizeof(la));
        for (int z = 0; z < nt; ++z) {
            la.slots[z] = a.slots[z];
            la.offsets[z] = a.offsets[z];
            la.n_hot[z] = a.n_hot[z];
            la.seg_start[z] = a.seg_start[z];
        }
        const int nb = lsort_plan(ctx, hot_tables, hot_batch, in_lds, n_lds, la.blk_start, la.part_slots, 0, 0);
        la.seg_start[nt] = a.seg_start[nt];
        la.n_tables = nt;
        la.n_samples = a.n_samples;
        la.keys_out = w.keys[cur];
        la.vals_out = w.vals[cur];
        la.status = ctx->d_block;
        la.flags = a.flags;
        la.n_flags = a.n_flags;
        la.flag_slice = bwd_flag_slice(a.n_flags, nb);
        fae_ktimer kt(ctx, FAE_K_LDS_SORT, st);
        if (ctx->opt_sort_order == 1)
            FAE_LAUNCH(ctx, (lds_sort_kernel<true>), dim3(nb), dim3(LSORT_THREADS), 0, st, la);
        else
            FAE_LAUNCH(ctx, (lds_sort_kernel<false>), dim3(nb), dim3(LSORT_THREADS), 0, st, la);
        FAE_LAUNCH_CHECK(ctx);
    }
    *cur_out = cur;
    return FAE_OK;
}

extern "C" int32_t fae_embbag_bwd_presort(fae_ctx *ctx, const fae_tables *hot_tables, const fae_batch *hot_batch,
                                          void *ws, size_t ws_bytes)
{
    BwdSetup su;
    int32_t rc = bwd_setup(ctx, hot_tables, hot_batch, ws, ws_bytes, "fae_embbag_bwd_presort", &su);
    if (rc != FAE_OK)
        return rc;
    FAE_HIP(ctx, hipSetDevice(ctx->device));
    fae_ctx::Presort *ps = ctx->presort_slot(ws);
    if (ps->valid && ps->side) // an unused sort (of this workspace, or the oldest one): nothing else would wait for it
        FAE_HIP(ctx, hipStreamWaitEvent(ctx->stream, ps->ev_join, 0));
    ps->valid = false;
    if (su.empty)
        return FAE_OK;
    // fork: the side stream starts after everything already queued on the main stream
    // (earlier users of this workspace, producers of the slots)
    const int side = ctx->aux_next;
    ctx->aux_next = (side + 1) % fae_ctx::N_AUX;
    FAE_HIP(ctx, hipEventRecord(ctx->ev_fork[side], ctx->stream));
    FAE_HIP(ctx, hipStreamWaitEvent(ctx->aux_stream[side], ctx->ev_fork[side], 0));
    int cur = 0;
    rc = bwd_sort_stage(ctx, ctx->aux_stream[side], hot_tables, hot_batch, su, &cur);
    if (rc != FAE_OK)
        return rc;
    FAE_HIP(ctx, hipEventRecord(ps->ev_join, ctx->aux_stream[side]));
    ps->valid = true;
    ps->side = true;
    ps->ws = ws;
    fae_ctx::presort_bind(ps, hot_tables->n_tables, hot_batch);
    ps->cur = cur;
    ps->age = ++ctx->presort_clock;
    return FAE_OK;
}

// ---------------------------------------------------------------------------------
// Forward and the backward's sort in one launch (one-hot tables whose lists fit the LDS
// sort): the first workgroups sort, the rest copy rows.  The two roles share nothing but
// the slot lists they both read; the sort is latency/ALU bound on a few CUs while the
// row copies stream through the others, so the pair takes about as long as the slower one.
// ---------------------------------------------------------------------------------
struct FusedArgs {
    const float *W[FAE_MAX_TABLES];
    const int32_t *slots[FAE_MAX_TABLES];
    int32_t n_hot[FAE_MAX_TABLES];
    int32_t seg_start[FAE_MAX_TABLES + 1];
    int32_t sort_blk_start[FAE_MAX_TABLES + 1];
    uint32_t part_slots[FAE_MAX_TABLES];
    int32_t n_tables, dim, n_samples;
    int32_t n_sort_blocks, fwd_blocks_per_table;
    int64_t out_stride;
    float *out;
    int32_t *keys_out, *vals_out;
    uint32_t *status;
    int32_t stream_out;
    int32_t *flags; // span flags of the reduce kernel, zeroed here
    int32_t n_flags, flag_slice;
};

// Rows of up to 16 lanes: two workgroups share a compute unit, eight rows per lane group in flight.  Wider ones: with as few
// registers only four rows fit (eight spill: 128 -> 151 us), and 16 rows in one workgroup move more.  Steps of 26 tables, one batch
// over and over, 64 samples per copying wave, before (one workgroup, more LDS) / two with four rows / one with sixteen, us:
// 16 384 samples, dim 128 128.1 / 132.7 / 130.1, 12 000 90.6 / 96.7 / 90.6, 50 001 452 / 420 / 411; dim 100, 16 384 105.9 / 111.4 / 107.1, 50 001 452 / 407 / 415, 4000 39.2 / 36.2 / 38.3.
template <typename V, int LPR, bool ANY> __global__ __launch_bounds__(LSORT_THREADS, (LPR < FUSED_ALONE_LANES ? 8 : 4)) void fwd_sort_kernel(FusedArgs a)
{
    bwd_clear_flags(a.flags, a.n_flags, a.flag_slice, LSORT_THREADS);
    if ((int)blockIdx.x < a.n_sort_blocks) {
        const int z = fae_find_table(a.sort_blk_start, a.n_tables, blockIdx.x);
        lds_sort_block<ANY>(a.slots[z], nullptr, a.seg_start[z + 1] - a.seg_start[z], a.n_hot[z], blockIdx.x - a.sort_blk_start[z],
                       a.sort_blk_start[z + 1] - a.sort_blk_start[z], a.part_slots[z], a.n_samples, a.keys_out + a.seg_start[z],
                       a.vals_out + a.seg_start[z], a.status);
    } else {
        const int b = blockIdx.x - a.n_sort_blocks;
        const int z = b / a.fwd_blocks_per_table, bl = b % a.fwd_blocks_per_table;
        constexpr int SAMPLES = FUSED_SAMPLES(LPR);
        const int64_t s0 = ((int64_t)bl * LSORT_WAVES + threadIdx.x / FAE_WAVE) * SAMPLES;
        const int s1 = s0 + SAMPLES < a.n_samples ? (int)s0 + SAMPLES : a.n_samples;
        fwd_onehot_wave<V, LPR, (LPR < FUSED_ALONE_LANES ? 8 : 16), SAMPLES>((const V *)a.W[z], a.slots[z], a.n_hot[z], s0, s1, a.out + (int64_t)z * a.dim,
                                                                              a.out_stride, a.dim, a.status, a.stream_out != 0);
    }
}

template <int LPR> static void launch_fwd_sort(fae_ctx *ctx, const FusedArgs &a, int blocks)
{
    if (ctx->opt_sort_order == 1)
        FAE_LAUNCH(ctx, (fwd_sort_kernel<float4, LPR, true>), dim3(blocks), dim3(LSORT_THREADS), 0, ctx->stream, a);
    else
        FAE_LAUNCH(ctx, (fwd_sort_kernel<float4, LPR, false>), dim3(blocks), dim3(LSORT_THREADS), 0, ctx->stream, a);
}

extern "C" int32_t fae_embbag_fwd_presort(fae_ctx *ctx, const fae_tables *hot_tables, const float *const *h_hotW,
                                          const fae_batch *hot_batch, float *out, int64_t out_row_stride, void *ws,
                                          size_t ws_bytes)
{
    BwdSetup su;
    int32_t rc = bwd_setup(ctx, hot_tables, hot_batch, ws, ws_bytes, "fae_embbag_fwd_presort", &su);
    if (rc != FAE_OK)
        return rc;
    const int nt = hot_tables->n_tables, dim = hot_tables->dim;
    const int64_t S = hot_batch->n_samples;
    // the fused launch covers the common case of the paper's workloads (every table one-hot,
    // batch within the LDS sort's reach, 16-byte aligned rows); anything else: plain forward
    bool fused = !su.empty && ctx->opt_sort != 1 && ctx->opt_fwd == 0 && h_hotW && out && dim % 4 == 0 &&
                 out_row_stride % 4 == 0 && out_row_stride >= (int64_t)nt * dim && ((uintptr_t)out) % 16 == 0 &&
                 (S <= LSORT_SHORT || ((ctx->opt_sort == 0 || ctx->opt_sort == 2) && lsort_takes(S, su.plan.N)));
    int64_t most_slots = 0;
    for (int z = 0; fused && z < nt; ++z) {
        fused = su.a.offsets[z] == nullptr && h_hotW[z] && ((uintptr_t)h_hotW[z]) % 16 == 0;
        most_slots = hot_tables->h_rows[z] > most_slots ? hot_tables->h_rows[z] : most_slots;
    }
    int lpr = 1;
    while (lpr < dim / 4 && lpr < 64)
        lpr <<= 1;
    if (ctx->opt_sort == 0)
        fused = fused && lsort_fuses(S, su.plan.N, most_slots, lpr);
    if (!fused)
        return fae_embbag_fwd(ctx, hot_tables, h_hotW, hot_batch, out, out_row_stride);
    FAE_HIP(ctx, hipSetDevice(ctx->device));
    fae_ctx::Presort *ps = ctx->presort_slot(ws);
    if (ps->valid && ps->side) // an unused sort (of this workspace, or the oldest one): nothing else would wait for it
        FAE_HIP(ctx, hipStreamWaitEvent(ctx->stream, ps->ev_join, 0));
    ps->valid = false;
    FusedArgs f;
    memset(&f, 0, sizeof(f));
    bool in_lds[FAE_MAX_TABLES];
    for (int z = 0; z < nt; ++z) {
        f.W[z] = h_hotW[z];
        f.slots[z] = su.a.slots[z];
        f.n_hot[z] = su.a.n_hot[z];
        f.seg_start[z] = su.a.seg_start[z];
        in_lds[z] = true;
    }
    f.seg_start[nt] = su.a.seg_start[nt];
    const int64_t piece = LSORT_WAVES * FUSED_SAMPLES(lpr);
    f.fwd_blocks_per_table = (int32_t)((S + piece - 1) / piece);
    f.n_sort_blocks = lsort_plan(ctx, hot_tables, hot_batch, in_lds, nt, f.sort_blk_start, f.part_slots, lpr,
                                 (int64_t)nt * f.fwd_blocks_per_table);
    f.n_tables = nt;
    f.dim = dim;
    f.n_samples = (int32_t)S;
    f.out_stride = out_row_stride;
    f.out = out;
    f.keys_out = su.w.keys[0];
    f.vals_out = su.w.vals[0];
    f.status = ctx->d_block;
    f.stream_out = ctx->opt_fwd_stream != 0;
    f.flags = su.a.flags;
    f.n_flags = su.a.n_flags;
    const int blocks = f.n_sort_blocks + f.fwd_blocks_per_table * nt;
    f.flag_slice = bwd_flag_slice(f.n_flags, blocks);
    {
        fae_ktimer kt(ctx, FAE_K_FWD_SORT);
        switch (lpr) {
        case 1: launch_fwd_sort<1>(ctx, f, blocks); break;
        case 2: launch_fwd_sort<2>(ctx, f, blocks); break;
        case 4: launch_fwd_sort<4>(ctx, f, blocks); break;
        case 8: launch_fwd_sort<8>(ctx, f, blocks); break;
        case 16: launch_fwd_sort<16>(ctx, f, blocks); break;
        case 32: launch_fwd_sort<32>(ctx, f, blocks); break;
        default: launch_fwd_sort<64>(ctx, f, blocks); break;
        }
        FAE_LAUNCH_CHECK(ctx);
    }
    ps->valid = true;
    ps->side = false;
    ps->ws = ws;
    fae_ctx::presort_bind(ps, nt, hot_batch);
    ps->cur = 0;
    ps->age = ++ctx->presort_clock;
    return FAE_OK;
}
