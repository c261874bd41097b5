// The A-operand table of the dense large kernel's matrix path (esc_dense.hip), entry by entry:
// built by the launch in front of the dense kernel, beside the pooling where a call has an estimator to run.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "esc_terms.hpp"

namespace esc {

typedef unsigned dw_u32x4 __attribute__((ext_vector_type(4)));

// fp32 -> bf16, round to nearest even, NaN kept quiet
__device__ __forceinline__ uint16_t dw_f32_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// entries of the table: one per (pair of tap columns, kernel row, lane)
__host__ __device__ inline int dense_table_entries(int Kse) { return (Kse + 1) / 2 * Kse * 64; }

// wa[pair of columns jp][kernel row i][2][lane l]: lane l holds output channel l % 16,
// tap (i, 2 jp + l / 32), input channels 8 ((l / 16) % 2) .. + 7 - the A operand of the
// instruction; zero beyond the kernel (the last pair's second column) and beyond C_a.  bf16 storage: two
// operands of terms, hi = bf16(w), lo = bf16(w - hi); fp32 storage: the eight weights as they are, four and four (the
// dense kernel takes them apart).
// Entry idx = (jp * Kse + i) * 64 + l.  Returns the eight weights' range.
__device__ __forceinline__ Range dense_table_entry(const float *lk, int Ca, int Ks, int Kse, bool terms, uint32_t *wa, int idx)
{
    const int q = idx >> 6, l = idx & 63, co = l & 15, kg = l >> 4, off = (Kse - Ks) / 2;
    const int jp = q / Kse, i = q - jp * Kse - off, j = 2 * jp + (kg >> 1) - off;
    // all eight weights are on their way before the first is looked at (a load behind a condition would be waited for
    // by itself)
    float v8[8];
    bool in8[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int ci = 8 * (kg & 1) + e;
        in8[e] = co < Ca && ci < Ca && i >= 0 && i < Ks && j >= 0 && j < Ks;
        v8[e] = lk[in8[e] ? (((size_t)co * Ca + ci) * Ks + i) * Ks + j : 0];
    }
    Range range;
    uint32_t part[2][4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float a = in8[2 * w] ? v8[2 * w] : 0.f, b = in8[2 * w + 1] ? v8[2 * w + 1] : 0.f;
        range.look(a, b);
        if (terms) {
            const uint16_t ha = dw_f32_to_bf16(a), hb = dw_f32_to_bf16(b);
            part[0][w] = (uint32_t)ha | ((uint32_t)hb << 16);
            part[1][w] = (uint32_t)dw_f32_to_bf16(a - __uint_as_float((uint32_t)ha << 16)) |
                         ((uint32_t)dw_f32_to_bf16(b - __uint_as_float((uint32_t)hb << 16)) << 16);
        } else {
            part[w >> 1][2 * (w & 1)] = __float_as_uint(a), part[w >> 1][2 * (w & 1) + 1] = __float_as_uint(b);
        }
    }
    dw_u32x4 *dst = reinterpret_cast<dw_u32x4 *>(wa) + (size_t)q * 128 + l;
#pragma unroll
    for (int t = 0; t < 2; ++t) dst[t * 64] = dw_u32x4{part[t][0], part[t][1], part[t][2], part[t][3]};
    return range;
}

// fp32 storage: behind the table, a block of the preparing launch leaves the ranges of its 256 entries per output channel (BlockRange)
__host__ __device__ inline int dense_table_blocks(int Kse) { return (dense_table_entries(Kse) + 255) / 256; }
__host__ __device__ inline size_t dense_table_words(int Kse) { return (size_t)dense_table_entries(Kse) * 8; }

}  // namespace esc
