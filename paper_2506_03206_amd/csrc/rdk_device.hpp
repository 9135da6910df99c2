// Device-side helpers: wavefront reductions and scans, typed row loads, Philox4x32-10.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rdk_common.hpp"

namespace rdk {

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// ---- 64-wide reductions and scans on the data-parallel-primitive (DPP) modifiers of the vector ALU: a lane
// reads another lane of its row of 16 at register speed, where a shuffle goes through the LDS crossbar (an
// order of magnitude more latency, which a lone wavefront cannot hide).  Controls: 0xB1 / 0x4E = quad
// permutations [1,0,3,2] / [2,3,0,1], 0x141 / 0x140 = mirror within 8 / 16 lanes, 0x110 + n = shift right by n
// within the row, 0x142 / 0x143 = lane 15 of each row to the next row / lane 31 to rows 2 and 3.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp_move(float v)   // lanes without a source (or outside ROW_MASK) get 0
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, ROW_MASK == 0xf));
}

template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp_move(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROW_MASK, 0xf, ROW_MASK == 0xf);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROW_MASK, 0xf, ROW_MASK == 0xf);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// value of lane `src` (the same for all lanes) in every lane
__device__ __forceinline__ int lane_value(int v, int src)
{
    return __builtin_amdgcn_readlane(v, __builtin_amdgcn_readfirstlane(src));
}
__device__ __forceinline__ float lane_value(float v, int src)
{
    return __builtin_bit_cast(float, lane_value(__builtin_bit_cast(int, v), src));
}
__device__ __forceinline__ double lane_value(double v, int src)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)lane_value((int)(unsigned)b, src), hi = (unsigned)lane_value((int)(unsigned)(b >> 32), src);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// sum over each row of 16 lanes, the same bits in all 16
template <typename T>
__device__ __forceinline__ T row16_sum(T v)
{
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    v += dpp_move<0x141>(v);
    v += dpp_move<0x140>(v);
    return v;
}

// sum over the 64 lanes, the same bits in every lane
template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
    v = row16_sum(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, dpp_move<0xB1>(v));
    v = fmaxf(v, dpp_move<0x4E>(v));
    v = fmaxf(v, dpp_move<0x141>(v));
    v = fmaxf(v, dpp_move<0x140>(v));
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}

// Inclusive prefix sum over the 64 lanes: Hillis-Steele inside each row, then the row totals are handed on.
__device__ __forceinline__ double wave_inclusive_scan(double v)
{
    v += dpp_move<0x111>(v);
    v += dpp_move<0x112>(v);
    v += dpp_move<0x114>(v);
    v += dpp_move<0x118>(v);
    v += dpp_move<0x142, 0xa>(v);   // rows 1 and 3 take the total of the row before
    v += dpp_move<0x143, 0xc>(v);   // rows 2 and 3 take the total of rows 0 and 1
    return v;
}

// exp(x) for x <= 0 (softmax terms) through the hardware base-2 exponential: one multiply and one v_exp_f32
// instead of the dozen instructions of the library routine, which made the logit paths ALU-bound.  The product
// x * log2(e) is rounded once: relative error of the result about |x| * 6e-8, i.e. below 1e-6 for every term
// larger than e^-15 of the row maximum; exp(-inf) = 0.  Every kernel uses this one function, so normalisers
// and terms carry the same rounding.
__device__ __forceinline__ float soft_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }

// The same with the rounding of the product x * log2(e) carried along (its exact residual and the part of log2(e) that
// a float drops): about one ulp for any x <= 0.  Five more instructions: for factors that a whole chunk of ids shares.
// Differences below -256 (a result of zero either way) are taken as -256, or a product beyond the range of a float would
// make the residual a NaN: the maximum of a masked chunk may be the lowest finite value.
__device__ __forceinline__ float soft_exp_fine(float x)
{
    x = x < -256.f ? -256.f : x;
    const float hi = x * 1.44269504088896341f;
    const float lo = fmaf(x, 1.44269504088896341f, -hi) + x * 1.92596299e-8f;
    return __builtin_amdgcn_exp2f(hi) * fmaf(0.693147180559945309f, lo, 1.0f);
}

// 1 / (mass of a drafter row), and 0 for a row without mass: Eq. 1 is undefined there, and every redistribution
// then returns the zero row (no token can be drafted from it; verification falls back on the target row alone).
__device__ __forceinline__ float inv_mass(float z) { return z > 0.f ? 1.0f / z : 0.f; }

// What the weights of a drafter row of logits are formed against: its maximum, or 0 if all of its ids are masked.  Their weights are
// exp(-inf) = 0 then, where -inf for both would make them NaN, and the row is one without mass like any other.
__device__ __forceinline__ float weight_reference(float row_max) { return row_max > -INFINITY ? row_max : 0.f; }

// ---- softmax statistics (running maximum m and sum of exp(z - m)), merged pairwise
struct SoftStat {
    float m, s;
};

__device__ __forceinline__ SoftStat soft_merge(SoftStat a, SoftStat b)
{
    float m = fmaxf(a.m, b.m);
    SoftStat r;
    r.m = m;
    r.s = (a.s == 0.f ? 0.f : a.s * soft_exp(a.m - m)) + (b.s == 0.f ? 0.f : b.s * soft_exp(b.m - m));
    return r;
}

// The statistics of the 64 lanes in every lane: each lane's sum is brought to the common maximum once (a tree of soft_merge takes two
// exponentials and two trips through the LDS crossbar per level, half a microsecond for a lone wavefront).
__device__ __forceinline__ SoftStat wave_soft_merge(SoftStat v)
{
    SoftStat r;
    r.m = wave_max(v.m);
    r.s = wave_sum(v.s == 0.f ? 0.f : v.s * soft_exp(v.m - r.m));
    return r;
}

// ---- typed loads of 4 consecutive elements of a row; those at or beyond `len` come back as `fill`.
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// Four consecutive elements, which may lie at any multiple of the element's size: the vector memory pipe reads 16 bytes from any
// address (a row of an odd number of ids starts anywhere), and single loads are left for the quad that crosses the row's end.
// Single loads for all of such a row, before, now: ten tree nodes of N = 256987 277 -> 111 us a call, 56 of N = 102359 165 -> 63,
// fused Eq. 3 at N = 55393, 44 positions 22.8 -> 16.8, fused sparse at N = 4797, 336 fp32 logits 32.7 -> 28.3.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u32x2_any __attribute__((ext_vector_type(2), aligned(2)));

// Without any check: the caller knows the four elements are in range.  STREAM marks the load non-temporal: for data that is read
// once and should not displace what the caches hold.
template <int KIND, bool STREAM = false>
__device__ __forceinline__ float4 load4_full(const void *row, int64_t i)
{
    if (KIND == RDK_LOGIT_BF16) {
        const u32x2_any *src = (const u32x2_any *)((const uint16_t *)row + i);
        const u32x2_any raw = STREAM ? __builtin_nontemporal_load(src) : *src;
        return make_float4(__uint_as_float(raw.x << 16), __uint_as_float(raw.x & 0xFFFF0000u), __uint_as_float(raw.y << 16),
                           __uint_as_float(raw.y & 0xFFFF0000u));
    }
    const f32x4_any *src = (const f32x4_any *)((const float *)row + i);
    const f32x4_any v = STREAM ? __builtin_nontemporal_load(src) : *src;
    return make_float4(v.x, v.y, v.z, v.w);
}

template <int KIND>
__device__ __forceinline__ float load1(const void *row, int64_t i)
{
    if (KIND == RDK_LOGIT_BF16) return bf16_to_f32(((const uint16_t *)row)[i]);
    return ((const float *)row)[i];
}

template <int KIND>
__device__ __forceinline__ float4 load4(const void *row, int64_t i, int64_t len, float fill)
{
    if (i + 3 < len) return load4_full<KIND>(row, i);
    return make_float4(i + 0 < len ? load1<KIND>(row, i + 0) : fill, i + 1 < len ? load1<KIND>(row, i + 1) : fill,
                       i + 2 < len ? load1<KIND>(row, i + 2) : fill, i + 3 < len ? load1<KIND>(row, i + 3) : fill);
}

// The 16 elements a lane holds of one chunk of kChunk ids (ids base + i*256 + lane*4 .. +3, i = 0..3).  A chunk that
// lies wholly inside the row is read by four loads behind ONE wavefront-uniform
// branch; per-load range checks cost a dozen scalar and exec-mask instructions each and made the streaming
// kernels issue-bound.  The loads are non-temporal unless STREAM is false: every user reads its rows once per
// launch, and batches are larger than the caches.
template <int KIND, bool STREAM = true>
__device__ __forceinline__ void load_chunk(const void *row, int64_t base, int64_t len, float fill, float4 (&v)[4])
{
    const int64_t first = base + lane_id() * 4;
    if (base + kChunk <= len) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = load4_full<KIND, STREAM>(row, first + i * 256);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = load4<KIND>(row, first + i * 256, len, fill);
    }
}

// Four consecutive raw values as they lie in memory: the conversion of bf16 waits until they are used, or every load would
// be waited for where it is made.
template <int KIND>
struct RawQuad {
    typedef float type __attribute__((ext_vector_type(4), aligned(4)));
    static __device__ __forceinline__ void to(const type r, float (&v)[4])
    {
        v[0] = r.x; v[1] = r.y; v[2] = r.z; v[3] = r.w;
    }
};
template <>
struct RawQuad<RDK_LOGIT_BF16> {
    typedef unsigned type __attribute__((ext_vector_type(2), aligned(2)));
    static __device__ __forceinline__ void to(const type r, float (&v)[4])
    {
        v[0] = __uint_as_float(r.x << 16); v[1] = __uint_as_float(r.x & 0xFFFF0000u);
        v[2] = __uint_as_float(r.y << 16); v[3] = __uint_as_float(r.y & 0xFFFF0000u);
    }
};
template <int KIND>
__device__ __forceinline__ typename RawQuad<KIND>::type raw_quad(const void *row, int i, int len)
{
    typedef typename RawQuad<KIND>::type Raw;
    return *(const Raw *)((const char *)row + (uint32_t)min(i, len - 4) * (KIND == RDK_LOGIT_BF16 ? 2u : 4u));
}
// raw_quad reads the last four values of the row for a quad that crosses its end: `past` places too early.
__device__ __forceinline__ void quad_shift(float (&v)[4], int past)
{
    past = max(past, 0);
    const bool one = past & 1, two = past & 2;
    v[0] = one ? v[1] : v[0]; v[1] = one ? v[2] : v[1]; v[2] = one ? v[3] : v[2];
    v[0] = two ? v[2] : v[0]; v[1] = two ? v[3] : v[1];
}

// The lane's four values of quad i of chunk c; ids beyond N come back as `fill`.
template <int KIND>
__device__ __forceinline__ void row_quad_values(const typename RawQuad<KIND>::type raw, int c, int i, int N, float fill, float (&v)[4])
{
    RawQuad<KIND>::to(raw, v);
    if (N - c * kChunk < kChunk) {                                        // the same for the whole wavefront
        const int left = N - (c * kChunk + 256 * i + 4 * lane_id());      // ids of the row from the lane's quad on
        quad_shift(v, 4 - left);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e >= left) v[e] = fill;
    }
}

template <int KIND>
__device__ __forceinline__ const void *row_ptr(const void *base, int64_t ld, int64_t b)
{
    if (KIND == RDK_LOGIT_BF16) return (const void *)((const uint16_t *)base + b * ld);
    return (const void *)((const float *)base + b * ld);
}

// Four consecutive floats to any address of a float.
__device__ __forceinline__ void store4(float *dst, float a, float b, float c, float d) { *(f32x4_any *)dst = f32x4_any{a, b, c, d}; }

// Turns a raw element into the weight the method works with: probabilities pass through, logits
// become exp(z - m) * inv (inv = 1 / sum exp for a normalised softmax, 1 for an unnormalised one).
template <int KIND>
__device__ __forceinline__ float to_weight(float x, float m, float inv)
{
    if (KIND == RDK_PROB_F32) return x;
    return soft_exp(x - m) * inv;
}

// ---- Philox4x32-10 (Salmon et al., SC'11): counter (c0..c3), key (k0,k1), ten rounds.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                              uint32_t k1, uint32_t out[4])
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

__device__ __forceinline__ void position_words(uint64_t seed, uint64_t index, uint32_t w[4])
{
    philox4x32_10((uint32_t)index, (uint32_t)(index >> 32), 0u, 0u, (uint32_t)seed, (uint32_t)(seed >> 32), w);
}

__device__ __forceinline__ double word_to_unit(uint32_t w) { return (double)(w >> 8) * (1.0 / 16777216.0); }

}  // namespace rdk
