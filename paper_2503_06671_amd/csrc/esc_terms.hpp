// fp32 values as terms for the 16-bit matrix instructions, and the range within which fp16 terms hold them
// (esc_kernels.hpp: large depth-wise kernels; esc_dense.hip; esc_backward.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace esc {
namespace {

// Largest of the 64 values of a wavefront, in lane 63 (the moves are wave_sum's).
__device__ __forceinline__ unsigned wave_max(unsigned v)
{
    constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
    auto dpp = [](unsigned x, auto ctrl, auto row_mask) {
        return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, decltype(row_mask)::value, 0xf, false);
    };
    v = max(v, dpp(v, std::integral_constant<int, kRowShr + 1>{}, std::integral_constant<int, 0xf>{}));
    v = max(v, dpp(v, std::integral_constant<int, kRowShr + 2>{}, std::integral_constant<int, 0xf>{}));
    v = max(v, dpp(v, std::integral_constant<int, kRowShr + 4>{}, std::integral_constant<int, 0xf>{}));
    v = max(v, dpp(v, std::integral_constant<int, kRowShr + 8>{}, std::integral_constant<int, 0xf>{}));
    v = max(v, dpp(v, std::integral_constant<int, kRowBcast15>{}, std::integral_constant<int, 0xa>{}));
    return max(v, dpp(v, std::integral_constant<int, kRowBcast31>{}, std::integral_constant<int, 0xc>{}));
}

__device__ __forceinline__ float power_of_two(int e) { return __uint_as_float((unsigned)(127 + e) << 23); }

// The range of some values: their largest magnitude (NaN if there is one) and the smallest apart from zeros, its sign shifted
// out and one subtracted, so that a zero is beyond all.  Two instructions a value.
struct Range {
    float large = 0.f;
    unsigned small = 0xffffffffu;
    __device__ __forceinline__ void look(float a, float b)
    {
        large = __builtin_elementwise_maximum(__builtin_elementwise_maximum(large, __builtin_fabsf(a)), __builtin_fabsf(b));
        small = min(min(small, (__float_as_uint(a) << 1) - 1u), (__float_as_uint(b) << 1) - 1u);
    }
};
// the same of many values: bits of the largest, and 2^32 - 1 less what Range keeps of the smallest, so that both are maxima
struct BlockRange {
    unsigned large = 0, small = 0;
    __device__ __forceinline__ BlockRange() {}
    __device__ __forceinline__ BlockRange(unsigned l, unsigned s) : large(l), small(s) {}
    __device__ __forceinline__ explicit BlockRange(const Range &r) : large(__float_as_uint(r.large) & 0x7fffffffu), small(~r.small) {}
    __device__ __forceinline__ void merge(unsigned l, unsigned s)
    {
        large = l > large ? l : large;
        small = s > small ? s : small;
    }
    __device__ __forceinline__ bool finite() const { return large < 0x7f800000u; }
    // the exponent of the power of two that brings the largest to 2^14 ... 2^15 (as far as fp32 reaches)
    __device__ __forceinline__ int up() const { return min(14 + 127 - (int)(large >> 23), 126); }
    // There, the smallest is still 2^-13 at least (or all are zeros): three terms hold every value, two to a unit of fp32's last
    // place.  (Values below fp32's smallest normal one have fewer bits than that.)
    __device__ __forceinline__ bool narrow() const { return (int)(large >> 23) - (int)((0u - small) >> 24) <= 27; }
};

// N fp16 terms of two values at a time, of magnitudes up to 2^15: v = t0 + (t1 + t2) / 4096, t0 the nearest fp16 to v, t1 the nearest to
// 4096 times what is left, t2 to what that leaves.  From 2^-13 up (below, fp16 runs out of bits) two terms are within a unit of fp32's last place (and
// miss it in a quarter of the values), three are exact.
constexpr float kLowTerm = 4096.f;
template <int N>
__device__ __forceinline__ void split_f16(float v0, float v1, uint32_t (&t)[N])
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const f16x2 h = __builtin_convertvector(f32x2{v0, v1}, f16x2);
        t[q] = __builtin_bit_cast(uint32_t, h);
        // (all exact)
        const float f = q == 0 ? kLowTerm : 1.f;
        v0 = __builtin_fmaf(-f, (float)h.x, v0 * f), v1 = __builtin_fmaf(-f, (float)h.y, v1 * f);
    }
}

// a value as three bf16 terms by truncation (the top eight mantissa bits, the next eight, the rest): exact, whatever its size (but
// for values within 2^24 of the smallest normal number).  Two values at a time.
__device__ __forceinline__ void split_bf16(float v0, float v1, uint32_t (&t)[3])
{
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const uint32_t a = __float_as_uint(v0) & 0xffff0000u, b = __float_as_uint(v1) & 0xffff0000u;
        t[q] = a >> 16 | b;
        v0 -= __uint_as_float(a), v1 -= __uint_as_float(b);
    }
}

}  // namespace
}  // namespace esc
