// One output element group at a time, on the allowed pairs alone: what a matrix-core kernel falls back to where its sums
// are not finite.
//
// In a matrix product a pair that is not allowed takes part with an exact zero, and zero times an inf or NaN of the other
// factor is NaN, which would reach rows that may not read it: the rows of another sample in the same tile, an earlier row
// of the same sample, padding.  A sum keeps a NaN, so a kernel only has to look at its finished sums (nothing is spent in
// its loops) and take the groups of four head dims that are not all finite from here.  Whether they then come out finite
// or not depends on the pairs that the mask allows and on nothing else.
//
// One thread per group, no staging, fp32 with expf: orders of magnitude slower than the products, for data that should
// not occur.  A group whose four sums are NaN stays so whatever follows and is left at once.
#pragma once
#include <hip/hip_runtime.h>

#include "psattn_mask.h"

namespace psattn {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// four neighbouring elements; tensors start wherever an element may (one wide access all the same)
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
__device__ inline f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4_any*>(p); }
__device__ inline f32x4 ld4(const uint16_t* p) {
    const u32x2_any u = *reinterpret_cast<const u32x2_any*>(p);
    f32x4 v;
    v[0] = __uint_as_float(u[0] << 16); v[1] = __uint_as_float(u[0] & 0xffff0000u);
    v[2] = __uint_as_float(u[1] << 16); v[3] = __uint_as_float(u[1] & 0xffff0000u);
    return v;
}
__device__ inline uint32_t bf16_bits(float v) {  // round to nearest even
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ inline void st4(float* p, f32x4 v) { *reinterpret_cast<f32x4_any*>(p) = v; }
__device__ inline void st4(uint16_t* p, f32x4 v) {
    const u32x2_any u = {bf16_bits(v[0]) | (bf16_bits(v[1]) << 16), bf16_bits(v[2]) | (bf16_bits(v[3]) << 16)};
    *reinterpret_cast<u32x2_any*>(p) = u;
}

__device__ inline bool allowed(const Tok4& t, int q, int kv) {
    return kv >= t.s && kv <= q && !(kv >= t.hole_lo && kv < t.hole_hi);
}

__device__ inline bool is_finite(const f32x4& x) {
    uint32_t top = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) top = max(top, __float_as_uint(x[c]) & 0x7fffffffu);
    return top < 0x7f800000u;
}
__device__ inline bool all_nan(const f32x4& x) {
    uint32_t low = 0xffffffffu;
#pragma unroll
    for (int c = 0; c < 4; ++c) low = min(low, __float_as_uint(x[c]) & 0x7fffffffu);
    return low > 0x7f800000u;
}

template <int D, typename E>
__device__ inline float exact_dot(const E* x, const E* y) {
    float s = 0.f;
#pragma unroll 4
    for (int i = 0; i < D; i += 4) {
        const f32x4 u = ld4(x + i), v = ld4(y + i);
#pragma unroll
        for (int c = 0; c < 4; ++c) s = fmaf(u[c], v[c], s);
    }
    return s;
}

template <typename E, int D>
__device__ inline const E* exact_row(const void* base, int row, int H, int h) {
    return static_cast<const E*>(base) + (static_cast<size_t>(row) * H + h) * D;
}

// f(key) for the keys that query q reads, ascending, until it returns false
template <typename F>
__device__ inline void exact_keys(const Tok4& t, int q, F f) {
#pragma nounroll
    for (int k = t.s; k <= q; ++k)
        if (allowed(t, q, k) && !f(k)) return;
}

// The scale, loaded on its own.  (Multiplying four values by it, the compiler loads the 16 bytes of the arguments that it starts,
// and for that copies the arguments around them to scratch memory.)
__device__ __forceinline__ float scale_of(const AttnArgs& a) {
    float x = a.scale;
    asm volatile("" : "+s"(x));
    return x;
}

// head dims d .. d + 3 of O
template <typename E, int D>
__device__ inline f32x4 exact_o(const AttnArgs& a, int h, int q, int d) {
    const int kvh = h / (a.Hq / a.Hkv);
    const E* qr = exact_row<E, D>(a.Q, q, a.Hq, h);
    float m = -INFINITY, l = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    exact_keys(token(a.meta, q), q, [&](int k) {
        const float s = exact_dot<D>(qr, exact_row<E, D>(a.K, k, a.Hkv, kvh)) * a.scale;
        const float mn = fmaxf(m, s), alpha = expf(m - mn), p = expf(s - mn);  // m = -inf the first time: alpha = 0
        const f32x4 v = ld4(exact_row<E, D>(a.V, k, a.Hkv, kvh) + d);
        l = l * alpha + p;
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = fmaf(p, v[c], acc[c] * alpha);
        m = mn;
        return !all_nan(acc);
    });
    return acc * (l > 0.f ? 1.f / l : 0.f);
}

// the same of dQ; delta = rowsum(dO o O) of the query
template <typename E, int D>
__device__ inline f32x4 exact_dq(const AttnArgs& a, int h, int q, int d, float delta) {
    const int kvh = h / (a.Hq / a.Hkv);
    const E *qr = exact_row<E, D>(a.Q, q, a.Hq, h), *gr = exact_row<E, D>(a.dO, q, a.Hq, h);
    const float lse = a.LSE[static_cast<size_t>(h) * a.meta.T + q];
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    exact_keys(token(a.meta, q), q, [&](int k) {
        const E* kr = exact_row<E, D>(a.K, k, a.Hkv, kvh);
        const float p = expf(exact_dot<D>(qr, kr) * a.scale - lse);
        const float ds = p * (exact_dot<D>(gr, exact_row<E, D>(a.V, k, a.Hkv, kvh)) - delta);
        const f32x4 x = ld4(kr + d);
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = fmaf(ds, x[c], acc[c]);
        return !all_nan(acc);
    });
    return acc * scale_of(a);
}

// the same of dK (DK) or dV.  DELTA: a.delta holds delta (1) or its negative (-1), or delta is summed from O and dO (0)
template <typename E, int D, bool DK, int DELTA>
__device__ inline f32x4 exact_dkdv(const AttnArgs& a, int kvh, int key, int d) {
    const int G = a.Hq / a.Hkv, q_hi = token(a.meta, key).key_hi;  // queries [key, q_hi) read this key
    const E *kr = exact_row<E, D>(a.K, key, a.Hkv, kvh), *vr = exact_row<E, D>(a.V, key, a.Hkv, kvh);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma nounroll
    for (int h = kvh * G; h < kvh * G + G; ++h)
#pragma nounroll
        for (int q = key; q < q_hi && !all_nan(acc); ++q) {
            const E *qr = exact_row<E, D>(a.Q, q, a.Hq, h), *gr = exact_row<E, D>(a.dO, q, a.Hq, h);
            const size_t stat = static_cast<size_t>(h) * a.meta.T + q;
            float p = expf(exact_dot<D>(qr, kr) * a.scale - a.LSE[stat]);
            if constexpr (DK) {
                const float delta = DELTA == 0 ? exact_dot<D>(exact_row<E, D>(a.O, q, a.Hq, h), gr) : DELTA * a.delta[stat];
                p *= exact_dot<D>(gr, vr) - delta;
            }
            const f32x4 x = ld4((DK ? qr : gr) + d);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = fmaf(p, x[c], acc[c]);
        }
    return DK ? acc * scale_of(a) : acc;
}

}  // namespace psattn
