// Device code shared by more than one kernel of libfae (gfx950).
#pragma once

#include "fae_internal.h"

#define RADIX_BITS 8
#define RADIX (1 << RADIX_BITS)
#define KEY_NONE 0x7fffffff // no carried run / element past the end of the span

// ---------------------------------------------------------------------------------
// 16-byte (or scalar) column slices
// ---------------------------------------------------------------------------------
template <typename V> struct vec_ops;
// s += v with the rounding error of the addition carried in c (compensated summation): the error
// of a long sum then stays at a few units of the last place whatever its length, also where one
// row is added over and over (a popular row in a long bag), which otherwise drifts one way.
__device__ __forceinline__ void fae_add_comp(float &s, float &c, float v)
{
    const float y = v - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
}

template <> struct vec_ops<float4> {
    static __device__ __forceinline__ float4 zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
    static __device__ __forceinline__ void add(float4 &a, const float4 &b)
    {
        a.x += b.x;
        a.y += b.y;
        a.z += b.z;
        a.w += b.w;
    }
    static __device__ __forceinline__ void scale(float4 &a, float f)
    {
        a.x *= f;
        a.y *= f;
        a.z *= f;
        a.w *= f;
    }
    static __device__ __forceinline__ void add_comp(float4 &s, float4 &c, const float4 &v)
    {
        fae_add_comp(s.x, c.x, v.x);
        fae_add_comp(s.y, c.y, v.y);
        fae_add_comp(s.z, c.z, v.z);
        fae_add_comp(s.w, c.w, v.w);
    }
    static __device__ __forceinline__ float4 shfl_xor(const float4 &a, int m)
    {
        return make_float4(__shfl_xor(a.x, m, FAE_WAVE), __shfl_xor(a.y, m, FAE_WAVE),
                           __shfl_xor(a.z, m, FAE_WAVE), __shfl_xor(a.w, m, FAE_WAVE));
    }
};
template <> struct vec_ops<float> {
    static __device__ __forceinline__ float zero() { return 0.f; }
    static __device__ __forceinline__ void add(float &a, const float &b) { a += b; }
    static __device__ __forceinline__ void scale(float &a, float f) { a *= f; }
    static __device__ __forceinline__ void add_comp(float &s, float &c, const float &v) { fae_add_comp(s, c, v); }
    static __device__ __forceinline__ float shfl_xor(const float &a, int m) { return __shfl_xor(a, m, FAE_WAVE); }
};

typedef float fae_v4f __attribute__((ext_vector_type(4)));
// streaming store: the pooled output is written once and not read again by this kernel
__device__ __forceinline__ void fwd_store(float4 *p, const float4 &v, bool stream)
{
    if (stream)
        __builtin_nontemporal_store(*(const fae_v4f *)&v, (fae_v4f *)p);
    else
        *p = v;
}
__device__ __forceinline__ void fwd_store(float *p, const float &v, bool stream)
{
    if (stream)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// One-hot tables (one lookup per sample): a wave takes SAMPLES consecutive samples from s0 on (those in front of s_end),
// reads their slots with one coalesced load and then copies rows, 64/LPR rows per step, with
// the loads of up to UNMAX steps in flight before the first store.  obase points at the table's
// first output column of sample 0.
template <typename V, int LPR, int UNMAX, int SAMPLES = FAE_WAVE>
__device__ __forceinline__ void fwd_onehot_wave(const V *W, const int32_t *slots, int n_hot, int64_t s0, int s_end,
                                                float *obase, int64_t out_stride, int dim, uint32_t *status,
                                                bool stream_out)
{
    constexpr int G = FAE_WAVE / LPR;
    constexpr int STEPS = SAMPLES / G;
    static_assert(SAMPLES <= FAE_WAVE && SAMPLES % G == 0, "a slot per lane, whole steps");
    constexpr int UN = STEPS < UNMAX ? STEPS : UNMAX;
    const int lane = fae_lane(), g = lane / LPR, l = lane % LPR;
    if (s0 >= s_end)
        return;
    int sreg = -1;
    if ((SAMPLES == FAE_WAVE || lane < SAMPLES) && s0 + lane < s_end) {
        sreg = slots[s0 + lane];
        if ((unsigned)sreg >= (unsigned)n_hot) {
            fae_flag(status, FAE_STATUS_ERANGE);
            sreg = -1; // pooled row of an invalid slot: zeros
        }
    }
    const int ncols = dim / (int)(sizeof(V) / sizeof(float));
    for (int c0 = 0; c0 < ncols; c0 += LPR) {
        const int c = c0 + l;
        const bool active = c < ncols;
#pragma unroll 1
        for (int i0 = 0; i0 < STEPS; i0 += UN) {
            V v[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int sl = __shfl(sreg, (i0 + u) * G + g, FAE_WAVE);
                v[u] = (active && sl >= 0) ? W[(int64_t)sl * ncols + c] : vec_ops<V>::zero();
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int64_t s = s0 + (i0 + u) * G + g;
                if (active && s < s_end)
                    fwd_store((V *)(obase + s * out_stride) + c, v[u], stream_out);
            }
        }
    }
}
