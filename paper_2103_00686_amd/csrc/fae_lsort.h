// Stable sort of one table's lookups by slot inside LDS, by a few workgroups at once (a role of two
// kernels: lds_sort_kernel and fwd_sort_kernel).
#pragma once

#include "fae_device.h"

// A table's keys are split into parts, ranges of slots, a workgroup each.  The parts' outputs are laid end
// to end: a part starts behind all lookups with lower slots.  A workgroup
//   1. goes over all keys of its table and leaves a bit per lookup in registers, in its range or not (a second one for the range's
//      last slot where that is left out of the sort, see below), and adds up the lookups below its range;
//   2. goes over the bits and takes the lookups of its range in batch order into LDS;
//   3. sorts them there (LSD radix passes, or, where they are few, by counting the keys in front of each).
// Lists of up to LSORT_CAP lookups are split into equal ranges of slots, those of up to 10 240 to LSORT_SPLIT_MAX (by lsort_plan) too unless that
// would leave a part with far more than its share (lsort_uneven).  Others are split by the ranks of
// a sample of 1024 lookups, one out of every 1024th of the list (lsort_bounds): to single slots where many lookups
// crowd on few, so that popular slots next to each other (ids in order of popularity) end up in different parts.  A slot that
// owns much of the batch is the last one of its part then: its lookups go straight to their places (their order is
// right as it is) and take no part in the sort, and where it fills several parts the workgroups of
// these share them.  Should a part hold more than LSORT_CAP lookups all the same, it is worked off in pieces whose ends
// are the ranks of other samples (lsort_piece).
//
// Bound by instructions and by the chain of its phases, not by memory (the keys come from the L2): every workgroup
// of a table goes over all its keys, so a key costs five vector instructions there (the sign of a difference,
// shifted into a word).  A pass ranks every key once (the match of a wave's 64 digits is most of it) instead of
// counting digits in one sweep and ranking them in a second one; digits have up to nine bits, so that 18 bits take two
// passes instead of three; loops are left rolled where they can be, since a workgroup runs through the code once
// and unrolled it waits for instructions (26 lists of 4096: 15 us with everything unrolled, 12.9).  With 74 KB of LDS and 64
// registers two workgroups share a compute unit, which is what the row copies of the fused launch need.
// Microseconds a step, one-hot, forward and sort in one launch, before (all keys and a 16-bit permutation in 147 KB
// of LDS, lists of up to 16 384 only, longer ones by the radix passes) and now:
//   three batches' inputs in turn: 26 x 50 001, dim 64 273 -> 210; 26 x 16 384, dim 64 73.0 -> 72.8, dim 32 56.7 -> 47.8;
//   one batch over and over: 26 x 16 384, dim 16 49.3 -> 39.8; 26 x 12 000, dim 16 41.5 -> 37.8;
//   1 x 1024 14.1 -> 12.7; 26 x 4096, dim 16 21.8 -> 22.0; sort alone, ids in order of popularity: 26 x 16 384 36 -> 23
#define LSORT_THREADS 1024
#define LSORT_WAVES (LSORT_THREADS / FAE_WAVE)
#define LSORT_ITEMS 7 // keys per thread in the sort
#define LSORT_CAP (LSORT_THREADS * LSORT_ITEMS)
#define LSORT_POS_BITS 17                 // of a lookup's number, or of a sample's where there are no more of these
#define LSORT_MAX ((1 << LSORT_POS_BITS) - 1) // lookups of a table
#define LSORT_KEYS 16                     // consecutive lookups of a lane in a step: a bit of half a word each
#define LSORT_STEP (FAE_WAVE * LSORT_KEYS)
#define LSORT_STEPS ((LSORT_MAX + LSORT_WAVES * LSORT_STEP) / (LSORT_WAVES * LSORT_STEP)) // of a wave, at most
#define LSORT_SAMPLES 1024
#define LSORT_PARTS 16    // of a list that is split by ranges of slots, at most
#define LSORT_UNEVEN 3072 // lookups beyond an even share that take a part longer than bounds by rank would (1.4 us per 1024 / 2.5 us), and what 64 samples may err by
#define LSORT_PIECE 5000  // lookups of a piece of a part that does not fit
// Lookups of the longest list that is split into ranges of slots (which lists are: lsort_plan)
#define LSORT_SPLIT_MAX 16384
#define LSORT_BITS 9 // of a digit, at most
#define LSORT_DIGITS (1 << LSORT_BITS)
#define LSORT_WORDS (LSORT_WAVES * LSORT_DIGITS / 2) // of the counters, as 32-bit words
#define LSORT_RANK_MAX 256                           // keys of a part up to which places are counted instead of sorted by digits
#define LSORT_RANK_LANES (LSORT_THREADS / LSORT_RANK_MAX)

#define LSORT_COUNTED 16384 // slots of a part up to which lookups may be placed by counting (sort_order 1): a counter of 16 bits each

struct LsortLds {
    union {
        struct {
            int key[LSORT_CAP], pos[LSORT_CAP];
        };
        uint32_t counters[LSORT_COUNTED / 2];
    };
    union {
        unsigned short cnt[LSORT_WAVES][LSORT_DIGITS]; // per wave: running count of a digit, then its start (a part has at most LSORT_CAP keys)
        int word[LSORT_WORDS];
    };
    int in[LSORT_WAVES], last[LSORT_WAVES], below[LSORT_WAVES]; // what each wave has counted
    int scan[LSORT_WAVES + 1];
    int misc[8];
};
static_assert(2 * LSORT_SAMPLES <= LSORT_WORDS, "two histograms of a digit of ten bits");

// The number of sample t out of SAMPLES of n >= SAMPLES lookups: one of every n / SAMPLES, its place among these from a Weyl
// sequence, another part of it for other tries; the same for all workgroups of a table.  (At even distances all samples are the
// same entry of a bag where bags have one length that divides the distance: 2048 bags of 50 on one table, sorted inside or with
// a first entry out of ten, put 100 K lookups into one part, sort alone 30 us without such bags, 1040 to 1120 with them, 29 now.)
template <int SAMPLES> __device__ __forceinline__ int lsort_sample(int t, int n, int tries)
{
    const uint32_t at = (uint32_t)t * (uint32_t)n / SAMPLES, next = (uint32_t)(t + 1) * (uint32_t)n / SAMPLES;
    static_assert((uint64_t)SAMPLES * LSORT_MAX < 1ull << 32, "in 32 bits");
    return (int)(at + __umulhi((uint32_t)(t + tries * SAMPLES) * 0x9E3779B1u, next - at)); // 2^32 times the golden ratio's fraction
}

// For each open b: bound[b] = the lowest slot with at least want[b] (>= 1) of the samples below it, the samples being the threads'
// keys k; found ten bits at a time, from the top, among the samples that agree in the bits above.  A bin with at most `few`
// samples is not looked into (its end is taken), which depends on want[b] and the samples alone, so neighbours agree on the
// bound between them.  crowd[b] = samples of the slot in front of the bound where these are more than `few`, want[b] =
// how many of them are wanted; else crowd[b] = 0.
template <int NB>
__device__ __forceinline__ void lsort_find(LsortLds &s, uint32_t k, uint32_t n_hot, int few, bool (&open)[NB], int (&want)[NB], uint32_t (&bound)[NB],
                                           int (&crowd)[NB])
{
    constexpr int BITS = 10;
    static_assert(LSORT_SAMPLES == LSORT_THREADS && 1 << BITS == LSORT_THREADS, "a sample and a bin per thread");
    const int t = threadIdx.x;
    uint32_t pre[NB];
    bool any = false;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        pre[b] = 0u;
        crowd[b] = 0;
        any = any || open[b];
    }
    for (int sh = 32 - __builtin_clz(n_hot | 1u); any && sh > 0;) {
        const int bits = sh < BITS ? sh : BITS;
        const int up = sh;
        sh -= bits;
#pragma unroll
        for (int b = 0; b < NB; ++b)
            s.word[b * LSORT_SAMPLES + t] = 0;
        __syncthreads();
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (open[b] && k >> up == pre[b])
                atomicAdd(&s.word[b * LSORT_SAMPLES + ((k >> sh) & ((1u << bits) - 1u))], 1);
        __syncthreads();
        int own[NB], sum = 0, all;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            own[b] = s.word[b * LSORT_SAMPLES + t];
            sum += own[b] << 16 * b;
        }
        const int ex = fae_block_excl_scan<LSORT_THREADS, true>(sum, s.scan, &all);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int before = ex >> 16 * b & 0xffff;
            if (open[b] && want[b] > before && want[b] <= before + own[b]) { // one thread
                s.misc[b] = t;
                s.misc[2 + b] = want[b] - before;
                s.misc[4 + b] = own[b];
            }
        }
        __syncthreads();
        any = false;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (open[b]) {
                pre[b] = pre[b] << bits | (uint32_t)__builtin_amdgcn_readfirstlane(s.misc[b]);
                want[b] = __builtin_amdgcn_readfirstlane(s.misc[2 + b]);
                const int here = __builtin_amdgcn_readfirstlane(s.misc[4 + b]);
                if (sh == 0 || here <= few) {
                    bound[b] = (pre[b] + 1u) << sh;
                    open[b] = false;
                    crowd[b] = sh == 0 && here > few ? here : 0;
                }
            }
            any = any || open[b];
        }
    }
}

// Bounds of a part: lsort_find's for part / parts and (part + 1) / parts of the samples.  A slot that owns many lookups may
// fill several parts: the first one ends with it, the others are left empty and take a share of its lookups instead
// (share of shares; slots from hi - 1 on then, without sorting anything).  Returns whether the last slot is to be left out of the sort.
__device__ __forceinline__ bool lsort_bounds(LsortLds &s, const int32_t *slots, int n, uint32_t n_hot, int part, int parts, uint32_t *lo, uint32_t *hi,
                                             int *share, int *shares)
{
    uint32_t k = (uint32_t)slots[lsort_sample<LSORT_SAMPLES>(threadIdx.x, n, 0)];
    k = k < n_hot ? k : n_hot;
    const int upto = (part + 1) * LSORT_SAMPLES / parts;
    int want[2] = {part * LSORT_SAMPLES / parts, upto}, here[2];
    uint32_t bound[2] = {0u, n_hot + 1u};
    bool open[2] = {part > 0, part + 1 < parts};
    lsort_find<2>(s, k, n_hot, LSORT_SAMPLES / (4 * parts), open, want, bound, here);
    *lo = bound[0] < n_hot + 1u ? bound[0] : n_hot + 1u;
    *hi = bound[1] < n_hot + 1u ? bound[1] : n_hot + 1u;
    if (here[1] == 0)
        return false;
    // the parts whose upper bound lies among the samples of this slot: under + 1 .. under + here
    const int under = upto - want[1];
    const int first = ((under + 1) * parts + LSORT_SAMPLES - 1) / LSORT_SAMPLES - 1;
    const int end = ((under + here[1] + 1) * parts + LSORT_SAMPLES - 1) / LSORT_SAMPLES - 1;
    *share = part - first;
    *shares = (end < parts - 1 ? end : parts - 1) - first;
    if (*share > 0)
        *lo = *hi - 1u;
    return true;
}

// Where slots lo .. top - 1 hold `over` lookups, more than fit: the end of a first piece of about LSORT_PIECE, by other samples of the
// list for each try; by halves, which end with a single slot, if these do not help.  *crowd: as lsort_bounds returns.
__device__ __forceinline__ uint32_t lsort_piece(LsortLds &s, const int32_t *slots, int n, uint32_t n_hot, uint32_t lo, uint32_t top, int over, int tries,
                                                bool *crowd)
{
    uint32_t k = (uint32_t)slots[lsort_sample<LSORT_SAMPLES>(threadIdx.x, n, tries)];
    k = k < n_hot ? k : n_hot;
    int both; // samples below lo, and in the range
    (void)fae_block_excl_scan<LSORT_THREADS>((k >= lo && k < top ? 1 << 16 : 0) + (k < lo ? 1 : 0), s.scan, &both);
    const int in = both >> 16, pieces = (over + LSORT_PIECE - 1) / LSORT_PIECE; // at least two
    int want[1] = {(both & 0xffff) + in / pieces}, here[1];
    uint32_t bound[1] = {top - lo > 1u ? lo + (top - lo) / 2u : top};
    bool open[1] = {tries <= 3 && in >= 2 * pieces};
    lsort_find<1>(s, k, n_hot, in / (8 * pieces), open, want, bound, here);
    const uint32_t end = bound[0] < top ? bound[0] : top;
    *crowd = here[0] > 0 || end - lo == 1u;
    return end;
}

// Whether equal ranges of slots make a part of a list of up to LSORT_SPLIT_MAX lookups too large: by 64 samples, the same for
// every wave of every workgroup of a table.
__device__ __forceinline__ bool lsort_uneven(const int32_t *slots, int n, uint32_t n_hot, uint32_t part_slots, int parts)
{
    uint32_t k = (uint32_t)slots[lsort_sample<FAE_WAVE>(fae_lane(), n, 0)];
    k = (k < n_hot ? k : n_hot) / part_slots;
    int most = 0;
#pragma unroll
    for (int p = 0; p < LSORT_PARTS; ++p) {
        const int c = __popcll(__ballot(k == (uint32_t)p));
        most = c > most ? c : most;
    }
    const int limit = n / parts + LSORT_UNEVEN;
    return most * n / FAE_WAVE > (limit < LSORT_CAP - 1024 ? limit : LSORT_CAP - 1024);
}

// The wave's lookups beg .. end - 1, in steps of which a lane has `per` consecutive ones: LSORT_KEYS, or four where
// a wave has no more than 256 in all, so that they are spread over its lanes.  A slot out of range counts as n_hot, behind every valid one.
struct LsortList {
    const int32_t *slots;
    uint32_t n_hot;
    int beg, end, per;
    bool aligned;
};
__device__ __forceinline__ uint32_t lsort_key(const LsortList &l, int e)
{
    const uint32_t k = (uint32_t)l.slots[e];
    return k < l.n_hot ? k : l.n_hot;
}

// (bits << 1) | sign of x
__device__ __forceinline__ uint32_t lsort_shift_in(uint32_t bits, uint32_t x) { return __builtin_amdgcn_alignbit(bits, x, 31); }

// A bit for each of the lane's lookups: step i in half a word (i / 2, the high half first), the step's first lookup's
// bit being the highest.  Four words by name: as an array, with the step known at run time only, they would leave the registers.
struct LsortMask {
    static_assert(LSORT_STEPS <= 8, "four words");
    uint32_t w0, w1, w2, w3;
    __device__ __forceinline__ void clear() { w0 = w1 = w2 = w3 = 0u; }
    __device__ __forceinline__ void put(int step, uint32_t bits)
    {
        const int i = step >> 1;
        bits <<= step & 1 ? 0 : 16;
        w0 |= i == 0 ? bits : 0u;
        w1 |= i == 1 ? bits : 0u;
        w2 |= i == 2 ? bits : 0u;
        w3 |= i == 3 ? bits : 0u;
    }
    __device__ __forceinline__ uint32_t get(int step) const
    {
        const int i = step >> 1;
        const uint32_t m = i == 0 ? w0 : i == 1 ? w1 : i == 2 ? w2 : w3;
        return step & 1 ? m & 0xffffu : m >> 16;
    }
};

// First sweep: the lane's lookups on slots lo .. top - 1 (in) and, if that is left out (CROWD), on the last of these (last); the
// wave's sums, and its lookups below lo.
template <bool CROWD>
__device__ __forceinline__ void lsort_count(const LsortList &l, uint32_t lo, uint32_t top, LsortMask &in, LsortMask &last,
                                            int *n_in, int *n_last, int *n_below)
{
    int below = 0, both = 0, step = 0;
#pragma unroll 1
    for (int j = l.beg; j < l.end; j += FAE_WAVE * l.per, ++step) {
        const int e = j + fae_lane() * l.per;
        // Lookups behind the end are read at its last ones (and masked below): loads under conditions would wait
        // for one another.  Four at once where every four of a lane are all in front of the end or all behind it.
        uint32_t k[LSORT_KEYS];
        if (l.aligned && (j + LSORT_STEP <= l.end || l.end % 4 == 0)) {
#pragma unroll
            for (int i = 0; i < LSORT_KEYS; i += 4) {
                const int4 v = *(const int4 *)(l.slots + (e + i < l.end ? e + i : l.end - 4));
                k[i] = v.x; k[i + 1] = v.y; k[i + 2] = v.z; k[i + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < LSORT_KEYS; ++i)
                k[i] = (uint32_t)l.slots[e + i < l.end ? e + i : l.end - 1];
        }
        uint32_t lt_lo = 0, lt_last = 0, lt_top = 0;
#pragma unroll
        for (int i = 0; i < LSORT_KEYS; ++i) { // slots and bounds are below 2^31, or 2^31 itself as the end
            const uint32_t key = k[i] < l.n_hot ? k[i] : l.n_hot;
            lt_lo = lsort_shift_in(lt_lo, key - lo);
            lt_top = lsort_shift_in(lt_top, key - top);
            if (CROWD)
                lt_last = lsort_shift_in(lt_last, key - (top - 1u));
        }
        const int left = l.end - e < l.per ? l.end - e : l.per;
        const uint32_t valid = left > 0 ? 0xffffu & ~(0xffffu >> left) : 0u;
        lt_lo &= valid;
        lt_top &= valid;
        const uint32_t mine = (CROWD ? lt_last & valid : lt_top) & ~lt_lo, mine_last = CROWD ? lt_top & ~lt_last : 0u;
        below += __popc(lt_lo);
        both += __popc(mine_last) << 16 | __popc(mine); // at most 128 of a lane
        in.put(step, mine);
        if (CROWD)
            last.put(step, mine_last);
    }
    both = __builtin_amdgcn_readlane(fae_wave_incl_scan(both), FAE_WAVE - 1); // at most 8192 of a wave
    *n_in = both & 0xffff;
    *n_last = both >> 16;
    *n_below = __builtin_amdgcn_readlane(fae_wave_incl_scan(below), FAE_WAVE - 1);
}

// Second sweep: the lookups whose bits are set, in their order, as numbers `at`, at + 1, ...; those with the numbers
// from .. to - 1 go to s.pos[number - from].
__device__ __forceinline__ void lsort_take(LsortLds &s, const LsortList &l, const LsortMask &bits, int at, int from, int to)
{
#pragma unroll 1
    for (int j = l.beg, step = 0; j < l.end; j += FAE_WAVE * l.per, ++step) {
        uint32_t m = bits.get(step);
        const int own = __popc(m), incl = fae_wave_incl_scan(own);
        const int e = j + fae_lane() * l.per + LSORT_KEYS - 1;
        for (int number = at + incl - own; m != 0; ++number) {
            const int bit = 31 - __builtin_clz(m);
            if (number >= from && number < to)
                s.pos[number - from] = e - bit;
            m ^= 1u << bit;
        }
        at += __builtin_amdgcn_readlane(incl, FAE_WAVE - 1);
    }
}

// s.key[0 .. n) and s.pos[0 .. n) sorted stably by the low nbits bits of key - lo
__device__ __forceinline__ void lsort_passes(LsortLds &s, int n, uint32_t lo, int nbits)
{
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t / FAE_WAVE), lane = fae_lane();
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    const int passes = (nbits + LSORT_BITS - 1) / LSORT_BITS;
    const int digit_bits = passes > 0 ? (nbits + passes - 1) / passes : 1;
    const uint32_t mask = (1u << digit_bits) - 1u;
    const int rounds = (n + LSORT_THREADS - 1) / LSORT_THREADS; // of 64 keys per wave
    const int at0 = w * rounds * FAE_WAVE + lane;
    volatile unsigned short *my = s.cnt[w];
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = pass * digit_bits;
        for (int i = lane; i <= (int)(mask >> 1); i += FAE_WAVE)
            s.word[w * (LSORT_DIGITS / 2) + i] = 0;
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int i = 0; i < rounds; ++i) {
            const int at = at0 + i * FAE_WAVE;
            const bool valid = at < n;
            const uint32_t d = valid ? ((uint32_t)s.key[at] - lo) >> shift & mask : 0u;
            uint64_t peers = __ballot(valid); // lanes with the same digit
#pragma unroll
            for (int b = 0; b < LSORT_BITS; ++b) {
                if (b >= digit_bits)
                    break;
                const bool bit = d >> b & 1u;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            const int r = __popcll(peers & lt_mask);
            if (valid) {
                const int old = my[d];
                if (r == 0)
                    my[d] = (unsigned short)(old + __popcll(peers));
                s.pos[at] |= (old + r) << LSORT_POS_BITS;
            }
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // digit t: the waves' counts -> their starts, digits in order, waves in order inside a digit
        int c[LSORT_WAVES], own = 0, all;
#pragma unroll
        for (int i = 0; i < LSORT_WAVES; ++i) {
            c[i] = t <= (int)mask ? s.cnt[i][t] : 0; // set in every case: else it would stay in registers from pass to pass
            own += c[i];
        }
        int at = fae_block_excl_scan<LSORT_THREADS, true>(own, s.scan, &all);
        if (t <= (int)mask) {
#pragma unroll
            for (int i = 0; i < LSORT_WAVES; ++i) {
                s.cnt[i][t] = (unsigned short)at;
                at += c[i];
            }
        }
        uint32_t key[LSORT_ITEMS];
        int pos[LSORT_ITEMS];
#pragma unroll
        for (int i = 0; i < LSORT_ITEMS; ++i) {
            const int at = at0 + i * FAE_WAVE;
            key[i] = i < rounds && at < n ? (uint32_t)s.key[at] : 0u;
            pos[i] = i < rounds && at < n ? s.pos[at] : 0;
        }
        __syncthreads(); // every key is in a register by now: the places are free
#pragma unroll
        for (int i = 0; i < LSORT_ITEMS; ++i)
            if (i < rounds && at0 + i * FAE_WAVE < n) {
                const int to = (pos[i] >> LSORT_POS_BITS) + my[(key[i] - lo) >> shift & mask];
                s.key[to] = (int)key[i];
                s.pos[to] = pos[i] & ((1 << LSORT_POS_BITS) - 1);
            }
        __syncthreads();
    }
}

// The sample of a lookup of a table with offsets: a search among every step-th offset in LDS (s.word, m of
// them), then in between.  In range even for a malformed CSR, which is reported.
struct LsortBags {
    const int32_t *off;
    int n_samples, step, m;
    __device__ __forceinline__ LsortBags(const int32_t *offsets, int samples) : off(offsets), n_samples(samples)
    {
        step = n_samples / LSORT_WORDS + 1;
        m = n_samples / step + 1;
    }
    __device__ __forceinline__ void stage(LsortLds &s) const // into the counters' room
    {
        for (int i = threadIdx.x; i < m; i += LSORT_THREADS)
            s.word[i] = off[(int64_t)i * step];
    }
    __device__ __forceinline__ int offset(const LsortLds &s, int i) const { return step == 1 ? s.word[i] : off[i]; }
    __device__ __forceinline__ int check(const LsortLds &s, int at, int e, bool *bad) const
    {
        at = at < n_samples ? at : n_samples - 1;
        if (offset(s, at) > e || offset(s, at + 1) <= e)
            *bad = true;
        return at;
    }
    __device__ __forceinline__ int search(const LsortLds &s, int e) const // the last offset that is <= e, or the first
    {
        int at = 0;
        for (int d = m > 1 ? 1 << (31 - __builtin_clz(m - 1)) : 0; d > 0; d >>= 1)
            at += at + d < m && s.word[at + d < m ? at + d : 0] <= e ? d : 0;
        at *= step;
        for (int d = step > 1 ? 1 << (31 - __builtin_clz(step - 1)) : 0; d > 0; d >>= 1)
            at += d <= n_samples - at && off[d <= n_samples - at ? at + d : 0] <= e ? d : 0;
        return at;
    }
};

// Slots lo .. lo + range - 1 of a list of up to 16 lookups per thread, the lookups of a slot in any order: a counter per slot, a
// scan, and every lookup takes the next free place of its slot.  One sweep each way over keys in registers instead of a
// selection and ranked passes, and no limit on a part's lookups.
// Steps, one-hot, three batches' inputs in turn, us, stable / any order, 30 000 slots: dim 16 1 x 4096 16.7 / 13.8, 4 x 8192 20.5 / 16.2,
// 8 x 16 384 26.1 / 22.9, 26 x 4096 22.7 / 19.0, 26 x 16 384 40.7 / 35.6, dim 64 26 x 8192 45.4 / 47.0.
__device__ __forceinline__ void lsort_place(LsortLds &s, const int32_t *slots, const int32_t *off, int n, uint32_t n_hot, uint32_t lo, uint32_t range,
                                            int n_samples, int32_t *keys_out, int32_t *vals_out, uint32_t *status)
{
    constexpr int PER = LSORT_COUNTED / LSORT_THREADS;
    const int t = threadIdx.x;
    uint32_t k[PER];
    int below = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) { // behind the list: below no slot, in no range
        const int e = i * LSORT_THREADS + t;
        k[i] = e < n ? (uint32_t)slots[e] : 0xffffffffu;
    }
    const int words = (int)(range + 1u) / 2;
    for (int i = t; i < words; i += LSORT_THREADS)
        s.counters[i] = 0u;
    bool bad = false;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (i * LSORT_THREADS + t >= n)
            continue;
        k[i] = k[i] < n_hot ? k[i] : n_hot;
        below += k[i] < lo ? 1 : 0;
        k[i] -= lo;
        if (k[i] < range) {
            bad = bad || k[i] + lo == n_hot;
            atomicAdd(&s.counters[k[i] >> 1], k[i] & 1u ? 1u << 16 : 1u); // up to 16 384 of a slot
        }
    }
    int n_below, n_part, own = 0;
    (void)fae_block_excl_scan<LSORT_THREADS>(below, s.scan, &n_below); // its barriers also end the counting
    const int per = (words + LSORT_THREADS - 1) / LSORT_THREADS; // counters of a thread, in words
#pragma unroll 1
    for (int i = t * per; i < (t + 1) * per && i < words; ++i)
        own += (int)(s.counters[i] & 0xffffu) + (int)(s.counters[i] >> 16);
    uint32_t at = (uint32_t)fae_block_excl_scan<LSORT_THREADS>(own, s.scan, &n_part);
#pragma unroll 1
    for (int i = t * per; i < (t + 1) * per && i < words; ++i) {
        const uint32_t c = s.counters[i], next = at + (c & 0xffffu);
        s.counters[i] = next << 16 | at;
        at = next + (c >> 16);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = i * LSORT_THREADS + t;
        if (e >= n || k[i] >= range)
            continue;
        int sample = e;
        if (off) {
            sample = fae_sample_of(off, n_samples, e);
            bad = bad || off[sample] > e || off[sample + 1] <= e; // malformed CSR
        }
        const uint32_t was = atomicAdd(&s.counters[k[i] >> 1], k[i] & 1u ? 1u << 16 : 1u);
        const int to = n_below + (int)(k[i] & 1u ? was >> 16 : was & 0xffffu);
        keys_out[to] = (int)(lo + k[i]);
        vals_out[to] = sample;
    }
    if (bad)
        fae_flag(status, FAE_STATUS_ERANGE);
}

// Part `part` of `parts` of a table's n lookups; part_slots: slots of a part of a list that is split
// by ranges, 0 where it is split by rank.  keys_out / vals_out: the table's segment of the sorted pairs.  ANY: the lookups of a slot may come in any order.
template <bool ANY>
__device__ __forceinline__ void lds_sort_block(const int32_t *slots, const int32_t *off, int n, int n_hot_z, int part, int parts, uint32_t part_slots,
                                               int n_samples, int32_t *keys_out, int32_t *vals_out, uint32_t *status)
{
    __shared__ __align__(16) LsortLds s;
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t / FAE_WAVE), lane = fae_lane();
    const uint32_t n_hot = (uint32_t)n_hot_z;
    bool by_rank = part_slots == 0u;
    uint32_t lo = (uint32_t)part * part_slots; // the part's slots
    uint32_t hi = n_hot + 1u - lo < part_slots ? n_hot + 1u : lo + part_slots;
    if (ANY && !by_rank && n <= LSORT_COUNTED && part_slots <= LSORT_COUNTED) {
        lsort_place(s, slots, off, n, n_hot, lo, hi - lo, n_samples, keys_out, vals_out, status);
        return;
    }
    bool crowd = false; // the last of them is left out of the sort
    int share = 0, shares = 1;
    if (n > LSORT_CAP && !by_rank)
        by_rank = lsort_uneven(slots, n, n_hot, part_slots, parts);
    if (by_rank) {
        crowd = lsort_bounds(s, slots, n, n_hot, part, parts, &lo, &hi, &share, &shares);
        __syncthreads(); // its counts are read
    }
    LsortList l;
    l.slots = slots;
    l.n_hot = n_hot;
    l.aligned = (((uintptr_t)slots) & 15) == 0;
    const int per_wave = (n + LSORT_WAVES * 256 - 1) / (LSORT_WAVES * 256) * 256; // consecutive lookups
    l.beg = w * per_wave < n ? w * per_wave : n;
    l.end = l.beg + per_wave < n ? l.beg + per_wave : n;
    l.per = per_wave > 256 ? LSORT_KEYS : 4;
    const LsortBags bags(off, n_samples);
    const bool many_samples = n_samples > LSORT_MAX; // the passes have no room for a sample's number beside a key's rank: found behind them
    bool bad = false;
    int left = 0;             // lookups on slots lo .. hi - 1, once they are counted
    int over = 0, tries = 1;  // lookups on slots lo .. top - 1 where these are known not to fit
    for (uint32_t top = hi; lo < hi;) { // slots lo .. top - 1; more than once only if a part does not fit
        if (over > 0) {
            top = lsort_piece(s, slots, n, n_hot, lo, top, over, tries++, &crowd);
            share = 0;
            shares = 1;
            over = 0;
            __syncthreads(); // its counts are read
        }
        if (off && !many_samples)
            bags.stage(s);
        LsortMask in, last;
        in.clear();
        last.clear();
        int n_in, n_last, n_below;
        if (crowd)
            lsort_count<true>(l, lo, top, in, last, &n_in, &n_last, &n_below);
        else
            lsort_count<false>(l, lo, top, in, last, &n_in, &n_last, &n_below);
        if (lane == 0) {
            s.in[w] = n_in;
            s.last[w] = n_last;
            s.below[w] = n_below;
        }
        __syncthreads();
        const int in_upto = fae_row_incl_scan(s.in[lane % LSORT_WAVES]), last_upto = fae_row_incl_scan(s.last[lane % LSORT_WAVES]);
        const int below_upto = fae_row_incl_scan(s.below[lane % LSORT_WAVES]);
        const int n_part = __builtin_amdgcn_readlane(in_upto, LSORT_WAVES - 1);
        const int all_last = __builtin_amdgcn_readlane(last_upto, LSORT_WAVES - 1);
        const int all_below = __builtin_amdgcn_readlane(below_upto, LSORT_WAVES - 1);
        if (top == hi)
            left = n_part + all_last;
        if (n_part > LSORT_CAP) { // then of at least two slots, or of one that is not left out
            over = n_part + all_last;
            continue;
        }
        const bool few = n_part <= LSORT_RANK_MAX, late = many_samples && !few;
        if (off && many_samples && (few || crowd))
            bags.stage(s);
        if (crowd) { // this part's share of the lookups on the last slot, as many at a time as LDS holds
            const int end = (int)((int64_t)all_last * (share + 1) / shares);
            for (int from = (int)((int64_t)all_last * share / shares); from < end; from += LSORT_CAP) {
                const int to = from + LSORT_CAP < end ? from + LSORT_CAP : end;
                lsort_take(s, l, last, __builtin_amdgcn_readlane(last_upto, w) - n_last, from, to);
                __syncthreads();
                for (int i = t; i < to - from; i += LSORT_THREADS) {
                    const int e = s.pos[i];
                    keys_out[all_below + n_part + from + i] = (int)(top - 1u);
                    vals_out[all_below + n_part + from + i] = off ? bags.check(s, bags.search(s, e), e, &bad) : e;
                }
                __syncthreads();
            }
            if (top > n_hot)
                bad = true;
        }
        if (n_part > 0)
            lsort_take(s, l, in, __builtin_amdgcn_readlane(in_upto, w) - n_in, 0, n_part);
        __syncthreads();
        for (int i = t; i < n_part; i += LSORT_THREADS) {
            const int e = s.pos[i];
            s.key[i] = (int)lsort_key(l, e);
            if (off && !late)
                s.pos[i] = bags.check(s, bags.search(s, e), e, &bad);
        }
        __syncthreads();
        int rank = 0; // few: the place of key t / LSORT_RANK_LANES
        if (few) {
            // Every key's place is the number of keys that go before it, counted outright by LSORT_RANK_LANES lanes per
            // key.  The count goes with the square of the length, so it ends at LSORT_RANK_MAX.
            const int i = t / LSORT_RANK_LANES, q = t % LSORT_RANK_LANES;
            const int key = i < n_part ? s.key[i] : 0;
            if (i < n_part) {
#pragma unroll 4
                for (int j = q; j < n_part; j += LSORT_RANK_LANES) {
                    const int o = s.key[j];
                    rank += (o < key || (o == key && j < i)) ? 1 : 0;
                }
            }
#pragma unroll
            for (int m = 1; m < LSORT_RANK_LANES; m <<= 1)
                rank += __shfl_xor(rank, m, FAE_WAVE);
        } else {
            lsort_passes(s, n_part, lo, 32 - __builtin_clz((top - 1u - lo) | 1u));
            if (off && late) {
                bags.stage(s);
                __syncthreads();
                for (int i = t; i < n_part; i += LSORT_THREADS) {
                    const int e = s.pos[i];
                    s.pos[i] = bags.check(s, bags.search(s, e), e, &bad);
                }
            }
        }
        if (few) {
            const int i = t / LSORT_RANK_LANES;
            if (i < n_part && t % LSORT_RANK_LANES == 0) {
                keys_out[all_below + rank] = s.key[i];
                vals_out[all_below + rank] = s.pos[i];
                if (s.key[i] == n_hot_z)
                    bad = true; // a slot out of range
            }
        } else {
            for (int i = t; i < n_part; i += LSORT_THREADS) {
                keys_out[all_below + i] = s.key[i];
                vals_out[all_below + i] = s.pos[i];
            }
            if (n_part > 0 && s.key[n_part - 1] == n_hot_z)
                bad = true;
        }
        left -= n_part + all_last;
        lo = top;
        top = hi;
        crowd = false;
        share = 0;
        shares = 1;
        tries = 1;
        over = left > LSORT_CAP ? left : 0;
        if (lo < hi)
            __syncthreads(); // LDS is filled again
    }
    if (bad)
        fae_flag(status, FAE_STATUS_ERANGE);
}
