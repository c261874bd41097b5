// What the kernels that pool and estimate share: the sums' fixed order, the estimator's arithmetic and
// the pool tiles' geometry (esc_kernels.hpp: the forward's items; esc_dense.hip: the dense call's).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace esc {

constexpr int kPoolTileW = 64, kPoolTileH = 32;  // the GAP is cut into 64 x 32 pixel tiles
constexpr int kPoolBatch = 4;                    // pool tiles a block works on at once

struct bf16_t {
    uint16_t bits;
};

namespace {

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return __uint_as_float((uint32_t)v.bits << 16); }

// four consecutive elements wherever they lie (one access: nothing here needs more than the element's alignment)
template <typename T>
struct __attribute__((packed, aligned(sizeof(T)))) Run4 {
    T e[4];
};

// NR runs of four pixels, run r being (gy[r], gx[r] .. + 3) of plane[r], zeros outside the image; gx a multiple of 4,
// nothing negative.  All loads go out together: no condition around a load, or between two (the compiler waits for what
// is under way at the end of a basic block); the run of a row's end is its last four elements, moved into place.
template <int NR, typename T>
__device__ __forceinline__ void pool_runs(const T *const (&plane)[NR], const int (&gy)[NR], const int (&gx)[NR], int H, int W,
                                          float (&v)[NR][4])
{
    if (W >= 4) {
        Run4<T> raw[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r)
            raw[r] = *reinterpret_cast<const Run4<T> *>(plane[r] + (size_t)(gy[r] < H ? gy[r] : H - 1) * W + (gx[r] + 4 <= W ? gx[r] : W - 4));
        const bool ragged = (W & 3) != 0;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int d = gy[r] < H ? (gx[r] + 4 <= W ? 0 : gx[r] + 4 - W) : 4;   // how many elements the run starts early
            float e[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) e[q] = to_f32(raw[r].e[q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) v[r][q] = d == 0 ? e[q] : 0.f;
            if (ragged) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int k = 1; q + k < 4; ++k) v[r][q] = d == k ? e[q + k] : v[r][q];
            }
        }
    } else {
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool in = gy[r] < H && gx[r] + q < W;
                const float t = to_f32(plane[r][in ? (size_t)gy[r] * W + gx[r] + q : 0]);
                v[r][q] = in ? t : 0.f;
            }
    }
}

// Sum over the 64 lanes of a wavefront, returned in every lane.  Data-parallel-primitive
// moves inside the vector ALU (a handful of cycles each; the LDS-crossbar shuffles they
// replace cost over a hundred): an inclusive scan inside each row of 16 lanes, then the
// row totals are carried over with the two row-broadcast steps; lane 63 ends with the
// total.  The order of the additions is fixed, which is all the callers rely on.
__device__ __forceinline__ float wave_sum(float v)
{
    constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
    auto dpp = [](float x, auto ctrl, auto row_mask) {
        return __builtin_bit_cast(
            float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                               decltype(row_mask)::value, 0xf, false));
    };
    v += dpp(v, std::integral_constant<int, kRowShr + 1>{}, std::integral_constant<int, 0xf>{});
    v += dpp(v, std::integral_constant<int, kRowShr + 2>{}, std::integral_constant<int, 0xf>{});
    v += dpp(v, std::integral_constant<int, kRowShr + 4>{}, std::integral_constant<int, 0xf>{});
    v += dpp(v, std::integral_constant<int, kRowShr + 8>{}, std::integral_constant<int, 0xf>{});
    v += dpp(v, std::integral_constant<int, kRowBcast15>{}, std::integral_constant<int, 0xa>{});
    v += dpp(v, std::integral_constant<int, kRowBcast31>{}, std::integral_constant<int, 0xc>{});
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// Running sum along each row of 16 lanes (lane 15 of a row ends with the row's total).
__device__ __forceinline__ float row_sum(float v)
{
    constexpr int kRowShr = 0x110;
    auto dpp = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x),
                                                                     decltype(ctrl)::value, 0xf, 0xf, false));
    };
    v += dpp(v, std::integral_constant<int, kRowShr + 1>{});
    v += dpp(v, std::integral_constant<int, kRowShr + 2>{});
    v += dpp(v, std::integral_constant<int, kRowShr + 4>{});
    v += dpp(v, std::integral_constant<int, kRowShr + 8>{});
    return v;
}

__device__ __forceinline__ float gelu_erf(float v)
{
    return 0.5f * v * (1.f + erff(v * 0.70710678118654752440f));
}

// bias + sum_k w[k] * in[k], accumulated in ascending k.  Weights are fetched eight at
// a time so their latencies overlap instead of adding up.
__device__ __forceinline__ float dot_row(const float *w, const float *in, int K, float bias)
{
    float s = bias;
    for (int k0 = 0; k0 < K; k0 += 8) {
        float wv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) wv[u] = k0 + u < K ? w[k0 + u] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k0 + u < K) s = fmaf(wv[u], in[k0 + u], s);
    }
    return s;
}

}  // namespace
}  // namespace esc
