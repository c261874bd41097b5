// GELU of ConvFFN for gfx950 (MI355X).
#pragma once
#include <hip/hip_runtime.h>

namespace esc {

// gelu(v) = v Phi(v) = h + |h| (1 - erfc(|v| / sqrt 2)), h = v / 2, the complementary error function as a power
// of two: erfc(t / sqrt 2) = 2^-(t P(t)).  P, of degree seven, is the minimax fit of
// -log2(erfc(t / sqrt 2)) / t on 0 <= t <= 5.9, weighted with what an error of it does to the result (less
// than 1e-8 |v|; linear programming on 2000 Chebyshev nodes), and grows beyond.  Evaluated in fp32 the result
// is within 8.1e-8 |v| and 3.4e-7 of the definition, more than twice as near as by the rational
// approximation 7.1.26 of Abramowitz and Stegun's handbook, which needs a reciprocal besides the exponential:
// eleven plain instructions and one of the slow ones (8 clocks a wavefront, against 4) instead of twelve and two.
// A hidden element costs two of these, which is what the vector units of ConvFFN's kernels spend most of
// their time on.  NaN stays NaN, +inf stays +inf and -inf gives NaN, as 0.5 v (1 + erf(v / sqrt 2)) does (the
// form max(v, 0) - |v| e would save one instruction and give NaN for both).
__device__ __forceinline__ float ffn_gelu(float v)
{
    const float t = fabsf(v);
    float q = fmaf(2.834909764715121e-06f, t, -3.937766086892225e-05f);
    q = fmaf(q, t, 0.0001861801283666864f);
    q = fmaf(q, t, 0.0001369366073049605f);
    q = fmaf(q, t, -0.0070634204894304276f);
    q = fmaf(q, t, 0.052496179938316345f);
    q = fmaf(q, t, 0.4592081904411316f);
    q = fmaf(q, t, 1.1511051654815674f);
    const float e = __builtin_amdgcn_exp2f(-q * t);
    const float h = 0.5f * v;
    return fmaf(fabsf(h), 1.f - e, h);
}

}  // namespace esc
