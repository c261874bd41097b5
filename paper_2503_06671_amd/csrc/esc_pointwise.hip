// Point-wise (1x1) convolutions of the ConvAttn module for gfx950 (MI355X): Conv_fuse on
// Concat(F_res, F_idt) (Eq. 4 line 4 of the ESC paper), the point-wise large-kernel
// factor LK^c of Eq. 5, the residual add of Eq. 3 line 3 in the same pass, and the two
// layers of ConvFFN where they are launches of their own.
//
// A 1x1 convolution in NCHW is the dense contraction  D[M x P] = W[M x K] . B[K x P]
// per image, with P = H*W pixels contiguous in memory for every channel of B and D, so
// it runs on the matrix cores, on v_mfma_f32_32x32x16_bf16 for both storage types:
//
//  fp32 storage: every value and every weight as three bf16 terms (v = t0 + t1 + t2, each the
//    nearest bf16 to what the terms before it left: exact, down to magnitudes of 2^-110, where t2
//    runs out of bits: 64 channels of standard deviation 2^-114 come out to 5.6e-7, of 2^-118 to
//    8.8e-6, ordinary ones to 1.1e-7), and the six of the nine products of
//    terms whose orders add up to at most two, accumulated in fp32.  What is left out lies below
//    2^-24 of a product: fp32 accuracy, at 6 x 32 clocks per 32x32x16 block of products against
//    the 8 x 64 of v_mfma_f32_32x32x2_f32, which moreover holds up the vector units.
//  bf16 storage: the stored values as they are, every fp32 weight as two bf16 terms (w = hi + lo to
//    16 mantissa bits; products exact, fp32 accumulation, the result rounded once at the store).
//
// The input channels come from two tensors (the first K1 from `src1`, the other K2 from
// `src2`): that is the concat, which is never materialised.
//
// Layout.  A wavefront owns 32 NT pixels and 32 MT output channels; a lane of the matrix
// instruction's B operand wants eight consecutive channels of one pixel, which is what eight
// loads of one channel row each bring it (32 lanes on a run of 32 NT pixels: whole cache
// lines), so the inputs go from memory into the operand's registers without passing LDS, asked
// for two stages of 32 channels ahead (runs_body has them under way until they are wanted; in
// pointwise_body the compiler waits for all of them at every stage: see there).  Only the weights pass LDS, split into their terms there by
// the block, a stage at a time in two buffers and one barrier a stage.  The residual's first row
// block is on its way with them, its second takes an input buffer as that falls free; it is added to
// the finished sums: one rounding at its size, where sums started from it are rounded there by every
// matrix instruction (64 -> 64 channels, fp32, a residual ten times the products: error against
// float64 3.2e-8, started from it 1.7e-7; the fused call 339 x 511 83.4 us, started from it 81.2,
// with the whole residual in freed buffers 88).  Nothing here
// asks for alignment: a lane's two pixels are one access wherever they lie (a plane of odd size
// costs 4 %, where the kernel before this one went element by element).
//
// What bounds it: memory.  64 -> 64 channels with a residual, 339 x 511 fp32: 30 us for 133 MB
// (54 us before: element-wise accesses and fp32 matrix instructions), 360 x 640 bf16: 18 us for
// 88 MB (35 us: 16-bit gathers from LDS for every operand); 16 -> 16 channels, 339 x 511: 7.8 us (19).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "esc_gelu.hpp"
#include "esc_pointwise.hpp"

namespace esc {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __amdgpu_buffer_rsrc_t Rsrc;

constexpr int kPwThreads = 256;
constexpr int kPwStage = 32;    // input channels of a stage: two matrix instructions' worth
constexpr int kRawBuffer = 0x00020000;     // raw buffer (no stride, no swizzle), 32-bit data format
constexpr int kNt = 2;                     // non-temporal
constexpr int kSchedNoVmem = 0x38f;        // a scheduling barrier for accesses to memory alone
constexpr unsigned kBeyond = 0x80000000u;  // an offset beyond every resource (an image of a tensor is < 2 GiB)

struct bf16s {
    uint16_t bits;
};

// two fp32 values rounded to nearest even and packed, a in the low half (v_cvt_pk_bf16_f32)
typedef float pw_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 pw_bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pw_pack2_bf16(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(pw_f32x2{a, b}, pw_bf16x2));
}

// N terms of the pair (v0, v1), one packed word per term
template <int N>
__device__ __forceinline__ void split_pair(float v0, float v1, unsigned (&t)[N])
{
#pragma unroll
    for (int q = 0; q < N; ++q) {
        t[q] = pw_pack2_bf16(v0, v1);
        if (q + 1 < N) {
            v0 -= __uint_as_float(t[q] << 16);
            v1 -= __uint_as_float(t[q] & 0xffff0000u);
        }
    }
}

extern __shared__ __align__(16) u32x4 pw_lds[];

// bytes of LDS: the weights of two stages, [2 buffers][2 chunks][MT][terms][64 lanes] operands, and the biases
template <typename T, int MT>
constexpr size_t pw_lds_bytes()
{
    return (size_t)2 * 2 * MT * (sizeof(T) == 4 ? 3 : 2) * 64 * 16 + MT * 32 * sizeof(float);
}

// The finished sums' way to memory: stores, and the elements that came out NaN summed again.
template <typename T, int MT, int NT, bool GELU>
__device__ __forceinline__ void pw_finish(const PointwiseParams &p, const f32x16 (&acc)[MT][NT], unsigned n, int m0, unsigned px, unsigned pxc,
                                          unsigned out_off, bool has_res)
{
    constexpr bool F = sizeof(T) == 4;
    const int lane = (int)threadIdx.x & 63, half = lane >> 5, K1 = p.K1, K = p.K1 + p.K2, M = p.M;
    const unsigned P = (unsigned)p.P, pb = P * (unsigned)sizeof(T);
    auto row_of = [](int mt, int i) { return (unsigned)(32 * mt + 8 * (i >> 2) + (i & 3)); };
    // ConvFFN's hidden layer is read back by the next launch; the other results are not, or lie better in memory
    constexpr int kStoreAux = GELU ? 0 : kNt;   // (step of 192 channels fp32, past the L2 and through it: 169 x 341 259 and 254.6 us, 180 x 320 246.0 and 246.3)
    // (taken afresh: kept from the residual's loads, the offsets would fill registers)
    unsigned st_off = out_off;
    asm volatile("" : "+v"(st_off));
    const Rsrc rdst = __builtin_amdgcn_make_buffer_rsrc((void *)((T *)p.dst + (size_t)n * p.dst_img_stride), 0,
                                                        (int)((unsigned)M * pb), kRawBuffer);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const unsigned row = row_of(mt, i);
            const unsigned off = (px < P && m0 + 4 * half + (int)row < M) ? st_off + row * pb : kBeyond;
            const float v0 = GELU ? ffn_gelu(acc[mt][0][i]) : acc[mt][0][i];
            if constexpr (NT == 1) {
                if constexpr (F)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v0), rdst, (int)off, 0, kStoreAux);
                else
                    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)pw_pack2_bf16(v0, v0), rdst, (int)off, 0, kStoreAux);
            } else {
                const float v1 = GELU ? ffn_gelu(acc[mt][NT - 1][i]) : acc[mt][NT - 1][i];
                if constexpr (F) {
                    typedef decltype(__builtin_amdgcn_raw_buffer_load_b64(rdst, 0, 0, 0)) B64;
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(B64, u32x2{__float_as_uint(v0), __float_as_uint(v1)}), rdst, (int)off, 0, kStoreAux);
                } else {
                    __builtin_amdgcn_raw_buffer_store_b32(pw_pack2_bf16(v0, v1), rdst, (int)off, 0, kStoreAux);
                }
            }
        }

    // An infinite value, or one beyond the largest bf16, has no three terms: its products come out NaN, and so does
    // every output channel of that pixel.  Those elements - none in an ordinary image: one comparison for two
    // accumulators - are summed again in plain fp32, which gives what fp32 arithmetic gives.  Not those that are NaN
    // for good because their row of W or their pixel holds one (found first, each read once): all-NaN
    // inputs must not cost many times an ordinary call (the fused call at 339 x 511: 78 us, with x all NaN 105; 2010
    // with every element of it summed again).
    if constexpr (F) {
        bool bad = false;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i)
#pragma unroll
                for (int t = 0; t < NT; t += 2) bad |= __builtin_isunordered(acc[mt][t][i], acc[mt][NT > 1 ? t + 1 : t][i]);
        bad = bad && px < P;
        if (__builtin_amdgcn_ballot_w64(bad) == 0) return;
        uint64_t todo = 0;   // this lane's elements, bit NT (16 mt + i) + t
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (bad && __builtin_isnan(acc[mt][t][i])) todo |= (uint64_t)1 << (NT * (16 * mt + i) + t);
        bool nan = false;
        const int wm = m0 + (lane & (32 * MT - 1));
        const float *wrow = p.w + (wm < M ? (size_t)wm * p.w_ld : 0);
#pragma unroll 1
        for (int k = 0; k < K; k += 8)
#pragma unroll
            for (int e = 0; e < 8; ++e) nan |= __builtin_isnan(wrow[min(k + e, K - 1)]);
        const uint64_t nan_rows = __builtin_amdgcn_ballot_w64(nan);   // bit r: row m0 + r of W
        const float *b1 = (const float *)p.src1 + (size_t)n * p.src1_img_stride + pxc;
        const float *b2 = (const float *)p.src2 + (size_t)n * p.src2_img_stride + pxc;
        const float *br = (const float *)p.res + (size_t)n * p.res_img_stride + pxc;
        float *bd = (float *)p.dst + (size_t)n * p.dst_img_stride + pxc;
        auto value = [&](int k, int t) { return k < K1 ? b1[(size_t)k * P + t] : b2[(size_t)(k - K1) * P + t]; };
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const uint64_t of_t = NT == 1 ? ~(uint64_t)0 : (uint64_t)0x5555555555555555u << t;
            nan = (todo & of_t) == 0;
#pragma unroll 1
            for (int k = 0; k < K && !nan; k += 8)
#pragma unroll
                for (int e = 0; e < 8; ++e) nan |= __builtin_isnan(value(min(k + e, K - 1), t));
            if (nan) todo &= ~of_t;
        }
#pragma unroll 1
        while (todo != 0) {
            const int bit = __builtin_ctzll(todo), i = bit / NT, t = bit % NT;
            todo &= todo - 1;
            const int row = 32 * (i >> 4) + 8 * ((i & 15) >> 2) + 4 * half + (i & 3), m = m0 + row;
            if (m >= M || (nan_rows >> row & 1) != 0) continue;
            float s = p.bias != nullptr ? p.bias[m] : 0.f;
            const float r = has_res ? br[(size_t)m * P + t] : 0.f;
            if (__builtin_isnan(r)) continue;
#pragma unroll 1
            for (int k = 0; k < K && !__builtin_isnan(s); k += 8) {
                float w[8], v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = p.w[(size_t)m * p.w_ld + min(k + e, K - 1)], v[e] = value(min(k + e, K - 1), t);
#pragma unroll
                for (int e = 0; e < 8; ++e) s = k + e < K ? fmaf(w[e], v[e], s) : s;
            }
            bd[(size_t)m * P + t] = GELU ? ffn_gelu(s) : s + r;
        }
    }
}

template <typename T, int MT, int NT, bool GELU>
__device__ __forceinline__ void pointwise_body(const PointwiseParams &p)
{
    constexpr bool F = sizeof(T) == 4;
    constexpr int TX = F ? 3 : 1, TW = F ? 3 : 2;         // bf16 terms of a value, of a weight
    constexpr int RW = (NT * (int)sizeof(T) + 3) / 4;     // words a load brings
    constexpr int kUnits = (MT * 128 + kPwThreads - 1) / kPwThreads;  // runs of eight weights a thread stages
    typedef typename std::conditional<RW == 2, u32x2, unsigned>::type Raw;
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, half = lane >> 5;
    const int K1 = p.K1, K = p.K1 + p.K2, M = p.M;
    const int stages = (K + kPwStage - 1) / kPwStage;
    const unsigned P = (unsigned)p.P, pb = P * (unsigned)sizeof(T);

    // which pixels, which 32 MT output channels.  Blocks are dealt to the eight dies in turn, each
    // with an L2 of its own: every die gets a contiguous eighth of the image, and the blocks that
    // read the same pixels for other output channels follow one another there
    const unsigned bq = gridDim.x / 8u, br = gridDim.x % 8u, xcd = blockIdx.x % 8u;
    const unsigned piece = xcd * bq + (xcd < br ? xcd : br) + blockIdx.x / 8u;
    const unsigned groups = (unsigned)(M + 32 * MT - 1) / (32u * MT);
    const unsigned tiles = (P + 128u * NT - 1) / (128u * NT);
    const unsigned tile_n = piece / groups, n = tile_n / tiles;
    const int m0 = (int)(piece - tile_n * groups) * 32 * MT;
    const unsigned px = (tile_n - n * tiles) * 128u * NT + 32u * NT * (unsigned)wave + NT * (unsigned)l32;
    // a lane whose pixels reach beyond the plane takes the plane's last NT instead (where it overlaps its
    // neighbour both compute and store the same bits); one that lies wholly beyond stores nothing
    const unsigned pxc = px + NT <= P ? px : P - NT;

    const Rsrc r1 = __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)p.src1 + (size_t)n * p.src1_img_stride), 0,
                                                      (int)((unsigned)K1 * pb), kRawBuffer);
    const Rsrc r2 = __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)p.src2 + (size_t)n * p.src2_img_stride), 0,
                                                      (int)((unsigned)p.K2 * pb), kRawBuffer);
    auto load = [](Rsrc r, unsigned voff, unsigned soff) -> Raw {
        if constexpr (RW == 2)
            return __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0));
        else if constexpr (NT * sizeof(T) == 4)
            return (unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0);
        else
            return (unsigned)__builtin_amdgcn_raw_buffer_load_b16(r, (int)voff, (int)soff, 0);
    };

    // ---- inputs of a stage: channel 32 st + 16 c + 8 half + j of this lane's pixels ----
    const unsigned in_off = 8u * (unsigned)half * pb + pxc * (unsigned)sizeof(T);
    auto fetch = [&](int st, Raw (&r)[16]) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int k0 = st * kPwStage + 16 * c;   // wavefront-uniform, like every condition on it
            if (k0 + 16 <= K1) {
#pragma unroll
                for (int j = 0; j < 8; ++j) r[8 * c + j] = load(r1, in_off, (unsigned)(k0 + j) * pb);
            } else if (k0 >= K1 && k0 + 16 <= K) {
#pragma unroll
                for (int j = 0; j < 8; ++j) r[8 * c + j] = load(r2, in_off, (unsigned)(k0 - K1 + j) * pb);
            } else if (k0 >= K) {
                break;
            } else {
                // the channels where src1 ends, or where src2 does: each lane's channel from the tensor that
                // holds it, nothing (zero) from the other or beyond both
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int k = k0 + 8 * half + j;
                    const unsigned o1 = k < K1 ? (unsigned)k * pb + pxc * (unsigned)sizeof(T) : kBeyond;
                    const unsigned o2 = (k >= K1 && k < K) ? (unsigned)(k - K1) * pb + pxc * (unsigned)sizeof(T) : kBeyond;
                    r[8 * c + j] = load(r1, o1, 0) | load(r2, o2, 0);
                }
            }
        }
    };

    // ---- weights of a stage: unit u = eight weights of one row ----
    const bool k8 = (K & 7) == 0;   // a run of eight is inside or outside as a whole
    struct __attribute__((packed, aligned(4))) W4 {
        float v[4];
    };
    auto wfetch = [&](int st, float (&w)[kUnits][8]) {
#pragma unroll
        for (int i = 0; i < kUnits; ++i) {
            const int u = tid + i * kPwThreads;
            const int m = m0 + (u >> 2), k = st * kPwStage + 8 * (u & 3);
            const bool row_in = m < M;
            if (k8) {
                const float *s = p.w + ((row_in && k < K) ? (size_t)m * p.w_ld + k : 0);
                const W4 a = *reinterpret_cast<const W4 *>(s), b = *reinterpret_cast<const W4 *>(s + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) w[i][e] = a.v[e], w[i][4 + e] = b.v[e];
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) w[i][e] = p.w[(row_in && k + e < K) ? (size_t)m * p.w_ld + k + e : 0];
            }
        }
    };
    auto wput = [&](int st, const float (&w)[kUnits][8]) {
#pragma unroll
        for (int i = 0; i < kUnits; ++i) {
            const int u = tid + i * kPwThreads;
            const int row = u >> 2, kq = u & 3;
            const int in = m0 + row < M ? K - (st * kPwStage + 8 * kq) : 0;   // how many of the eight lie in W
            unsigned t[4][TW];
#pragma unroll
            for (int e = 0; e < 4; ++e) split_pair<TW>(2 * e < in ? w[i][2 * e] : 0.f, 2 * e + 1 < in ? w[i][2 * e + 1] : 0.f, t[e]);
            if (MT * 128 % kPwThreads == 0 || u < MT * 128) {
                u32x4 *d = pw_lds + ((((st & 1) * 2 + (kq >> 1)) * MT + (row >> 5)) * TW) * 64 + 32 * (kq & 1) + (row & 31);
#pragma unroll
                for (int q = 0; q < TW; ++q) d[q * 64] = u32x4{t[0][q], t[1][q], t[2][q], t[3][q]};
            }
        }
    };

    float wr[kUnits][8];
    Raw ra[16], rb[16];
    wfetch(0, wr);
    fetch(0, ra);
    if (stages > 1) fetch(1, rb);
    // the accumulators' layout: lane l of tile t of row block mt holds output channel
    // m0 + 32 mt + 8 (i / 4) + 4 half + i % 4 of pixel px + t in element i
    const unsigned out_off = (unsigned)(m0 + 4 * half) * pb + pxc * (unsigned)sizeof(T);
    auto row_of = [](int mt, int i) { return (unsigned)(32 * mt + 8 * (i >> 2) + (i & 3)); };
    // the residual: row block 0's is on its way from the start, row block 1's takes the first input buffer once nothing
    // will be fetched into it any more
    const bool has_res = !GELU && p.res != nullptr;
    const Rsrc rres = __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)p.res + (size_t)n * p.res_img_stride), 0,
                                                        (int)((unsigned)M * pb), kRawBuffer);
    auto rfetch = [&](int mt, Raw (&r)[16]) {
        int m = m0 + 4 * half;
        asm volatile("" : "+v"(m));  // (not to be computed ahead of the loop and kept through it)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const unsigned row = row_of(mt, i);
            r[i] = load(rres, m + (int)row < M ? out_off : kBeyond, row * pb);
        }
    };
    Raw rv[16];
    if (has_res) rfetch(0, rv);
    float *s_bias = reinterpret_cast<float *>(pw_lds + 2 * 2 * MT * TW * 64);
    if (tid < 32 * MT) s_bias[tid] = (p.bias != nullptr && m0 + tid < M) ? p.bias[m0 + tid] : 0.f;
    wput(0, wr);

    f32x16 acc[MT][NT];
    __syncthreads();  // the first stage's weights are in LDS
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 b = *reinterpret_cast<const f32x4 *>(s_bias + 32 * mt + 8 * g + 4 * half);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[mt][t][4 * g + e] = b[e];
            }
    auto body = [&](int st, Raw (&raw)[16], bool first) {
        if (st + 1 < stages) wfetch(st + 1, wr);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (c == 1 && st * kPwStage + 16 >= K) break;   // wavefront-uniform: nothing left in the second chunk
            // B operands: the terms of this lane's eight channels, per pixel tile
            u32x4 b[NT][TX];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const Raw x0 = raw[8 * c + 2 * e], x1 = raw[8 * c + 2 * e + 1];
                if constexpr (F) {
                    unsigned t[TX];
                    if constexpr (NT == 2) {
                        split_pair<TX>(__uint_as_float(x0.x), __uint_as_float(x1.x), t);
#pragma unroll
                        for (int q = 0; q < TX; ++q) b[0][q][e] = t[q];
                        split_pair<TX>(__uint_as_float(x0.y), __uint_as_float(x1.y), t);
#pragma unroll
                        for (int q = 0; q < TX; ++q) b[NT - 1][q][e] = t[q];
                    } else {
                        split_pair<TX>(__uint_as_float(x0), __uint_as_float(x1), t);
#pragma unroll
                        for (int q = 0; q < TX; ++q) b[0][q][e] = t[q];
                    }
                } else {
                    b[0][0][e] = __builtin_amdgcn_perm(x1, x0, 0x05040100u);                       // the low halves
                    if constexpr (NT == 2) b[NT - 1][0][e] = __builtin_amdgcn_perm(x1, x0, 0x07060302u);  // the high ones
                }
            }
            if (c == 1 || st * kPwStage + 16 >= K) {
                if (st + 2 < stages)
                    fetch(st + 2, raw);
                else if (has_res && MT > 1 && first)
                    rfetch(1, raw);
            }
            const u32x4 *wa = pw_lds + (((st & 1) * 2 + c) * MT * TW) * 64 + lane;
            u32x4 a[MT][TW];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int q = 0; q < TW; ++q) a[mt][q] = wa[(mt * TW + q) * 64];
            // small terms first; neighbouring instructions on different accumulators
#pragma unroll
            for (int qw = TW - 1; qw >= 0; --qw)
#pragma unroll
                for (int qx = TX - 1; qx >= 0; --qx) {
                    if (F && qw + qx > 2) continue;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            acc[mt][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[mt][qw]),
                                                                                 __builtin_bit_cast(bf16x8, b[t][qx]), acc[mt][t], 0, 0, 0);
                }
        }
        if (st + 1 < stages) {
            wput(st + 1, wr);
            __syncthreads();  // the next stage's weights are in LDS; everyone has finished with this one's
        }
    };
    for (int st = 0; st < stages; st += 2) {
        body(st, ra, true);
        if (st + 1 < stages) body(st + 1, rb, false);
    }
    if (has_res) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const Raw r = mt == 0 ? rv[i] : ra[i];
                if constexpr (F && NT == 2) {
                    acc[mt][0][i] += __uint_as_float(r.x);
                    acc[mt][NT - 1][i] += __uint_as_float(r.y);
                } else if constexpr (F) {
                    acc[mt][0][i] += __uint_as_float(r);
                } else {
                    acc[mt][0][i] += __uint_as_float(r << 16);
                    if constexpr (NT == 2) acc[mt][NT - 1][i] += __uint_as_float(r & 0xffff0000u);
                }
            }
    }

    pw_finish<T, MT, NT, GELU>(p, acc, n, m0, px, pxc, out_off, has_res);
}

// ---- the same with everything fetched ahead, where src1's channels, and all of them, are whole runs of sixteen (a chunk
// lies in one tensor, or beyond both): pointwise_body's loads stand behind conditions, which make the compiler wait for
// all that are under way at every stage.  (Its steps are written out a second time: as functions of both bodies they leave
// pointwise_kernel<2, false>, which fills its registers, with 36 to 44 bytes in the private segment.) ----

// what becomes of the sums
enum : int { kPwPlain = 0, kPwGelu = 1, kPwRes = 2 };

// any number of stages; all channels in one (LK^c: 339 x 511 fp32 8.9 us -> 7.8); in two, written out (as a loop: the fused
// call with a residual 64 x 64 x 64 bf16 39.0 us, so 36.7, 360 x 640 bf16 36.7 and 34.6, 180 x 320 fp32 22.2 and 21.4;
// without one at 360 x 640 bf16 31 - 33 either way)
enum : int { kPwRuns = 0, kPwOne = 1, kPwTwo = 2 };

template <typename T, int MT, int NT, int MODE, int LIE>
__device__ __forceinline__ void runs_body(const PointwiseParams &p)
{
    constexpr bool GELU = MODE == kPwGelu, has_res = MODE == kPwRes, ONE = LIE == kPwOne, TWO = LIE == kPwTwo;
    constexpr bool F = sizeof(T) == 4;
    constexpr int TX = F ? 3 : 1, TW = F ? 3 : 2;         // bf16 terms of a value, of a weight
    constexpr int RW = (NT * (int)sizeof(T) + 3) / 4;     // words a load brings
    constexpr int kUnits = (MT * 128 + kPwThreads - 1) / kPwThreads;  // runs of eight weights a thread stages
    typedef typename std::conditional<RW == 2, u32x2, unsigned>::type Raw;
    // what is asked for stays in the order it is written in
    auto order = [] { __builtin_amdgcn_sched_barrier(kSchedNoVmem); };
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, half = lane >> 5;
    const int K1 = p.K1, K = p.K1 + p.K2, M = p.M;
    const int stages = (K + kPwStage - 1) / kPwStage;
    const unsigned P = (unsigned)p.P, pb = P * (unsigned)sizeof(T);

    // which pixels, which 32 MT output channels.  Blocks are dealt to the eight dies in turn, each
    // with an L2 of its own: every die gets a contiguous eighth of the image, and the blocks that
    // read the same pixels for other output channels follow one another there
    const unsigned bq = gridDim.x / 8u, br = gridDim.x % 8u, xcd = blockIdx.x % 8u;
    const unsigned piece = xcd * bq + (xcd < br ? xcd : br) + blockIdx.x / 8u;
    const unsigned groups = (unsigned)(M + 32 * MT - 1) / (32u * MT);
    const unsigned tiles = (P + 128u * NT - 1) / (128u * NT);
    const unsigned tile_n = piece / groups, n = tile_n / tiles;
    const int m0 = (int)(piece - tile_n * groups) * 32 * MT;
    const unsigned px = (tile_n - n * tiles) * 128u * NT + 32u * NT * (unsigned)wave + NT * (unsigned)l32;
    // a lane whose pixels reach beyond the plane takes the plane's last NT instead (where it overlaps its
    // neighbour both compute and store the same bits); one that lies wholly beyond stores nothing
    const unsigned pxc = px + NT <= P ? px : P - NT;

    const Rsrc r1 = __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)p.src1 + (size_t)n * p.src1_img_stride), 0,
                                                      (int)((unsigned)K1 * pb), kRawBuffer);
    const Rsrc r2 = __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)p.src2 + (size_t)n * p.src2_img_stride), 0,
                                                      (int)((unsigned)p.K2 * pb), kRawBuffer);
    auto load = [](Rsrc r, unsigned voff, unsigned soff) -> Raw {
        if constexpr (RW == 2)
            return __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0));
        else if constexpr (NT * sizeof(T) == 4)
            return (unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0);
        else
            return (unsigned)__builtin_amdgcn_raw_buffer_load_b16(r, (int)voff, (int)soff, 0);
    };

    // ---- inputs of a stage: channel 32 st + 16 c + 8 half + j of this lane's pixels ----
    const unsigned in_off = 8u * (unsigned)half * pb + pxc * (unsigned)sizeof(T);
    // Sixteen loads on every way through here and through the loop: at a point that could be reached without them, or
    // behind a wait for some of them, the compiler waits for all that are under way, and nothing is fetched ahead.  A
    // chunk beyond the channels is asked for beyond the tensor: zeros, and no traffic.  (With the fetches behind
    // conditions: residual step of the 192-channel model 64 x 64 fp32 72 us, so 60; 64 channels of 25 images of 63 x 63
    // 119 and 111; Conv_fuse 360 x 640 bf16 21.1 and 19.1.)
    auto fetch = [&](int st, Raw (&r)[16]) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int k0 = st * kPwStage + 16 * c;   // wavefront-uniform, like every condition on it
            {
                const bool one = k0 < K1;
                const unsigned so = (unsigned)(one ? k0 : k0 - K1) * pb, vo = k0 < K ? in_off : kBeyond;
#pragma unroll
                for (int j = 0; j < 8; ++j) r[8 * c + j] = load(one ? r1 : r2, vo, k0 < K ? so + (unsigned)j * pb : 0u);
            }
        }
    };

    // ---- weights of a stage: unit u = eight weights of one row ----
    struct __attribute__((packed, aligned(4))) W4 {
        float v[4];
    };
    auto wfetch = [&](int st, float (&w)[kUnits][8]) {
#pragma unroll
        for (int i = 0; i < kUnits; ++i) {
            const int u = tid + i * kPwThreads;
            const int m = m0 + (u >> 2), k = st * kPwStage + 8 * (u & 3);
            const bool row_in = m < M;
            const float *s = p.w + ((row_in && k < K) ? (size_t)m * p.w_ld + k : 0);   // (a run of eight is inside or outside as a whole)
            const W4 a = *reinterpret_cast<const W4 *>(s), b = *reinterpret_cast<const W4 *>(s + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) w[i][e] = a.v[e], w[i][4 + e] = b.v[e];
        }
    };
    auto wput = [&](int st, const float (&w)[kUnits][8]) {
#pragma unroll
        for (int i = 0; i < kUnits; ++i) {
            const int u = tid + i * kPwThreads;
            const int row = u >> 2, kq = u & 3;
            const int in = m0 + row < M ? K - (st * kPwStage + 8 * kq) : 0;   // how many of the eight lie in W
            unsigned t[4][TW];
#pragma unroll
            for (int e = 0; e < 4; ++e) split_pair<TW>(2 * e < in ? w[i][2 * e] : 0.f, 2 * e + 1 < in ? w[i][2 * e + 1] : 0.f, t[e]);
            if (MT * 128 % kPwThreads == 0 || u < MT * 128) {
                u32x4 *d = pw_lds + ((((st & 1) * 2 + (kq >> 1)) * MT + (row >> 5)) * TW) * 64 + 32 * (kq & 1) + (row & 31);
#pragma unroll
                for (int q = 0; q < TW; ++q) d[q * 64] = u32x4{t[0][q], t[1][q], t[2][q], t[3][q]};
            }
        }
    };

    float wr[kUnits][8];
    Raw ra[16], rb[16];
    // results return in order: the bias and the first weights, wanted first, are asked for first
    float bias = 0.f;
    if (p.bias != nullptr) bias = p.bias[m0 + (tid < 32 * MT && m0 + tid < M ? tid : 0)];
    wfetch(0, wr);
    order();
    fetch(0, ra);
    order();
    if constexpr (!ONE) fetch(1, rb);
    order();
    // the accumulators' layout: lane l of tile t of row block mt holds output channel
    // m0 + 32 mt + 8 (i / 4) + 4 half + i % 4 of pixel px + t in element i
    const unsigned out_off = (unsigned)(m0 + 4 * half) * pb + pxc * (unsigned)sizeof(T);
    auto row_of = [](int mt, int i) { return (unsigned)(32 * mt + 8 * (i >> 2) + (i & 3)); };
    // the residual: row block 0's is on its way from the start, row block 1's takes the first input buffer once nothing
    // will be fetched into it any more
    const Rsrc rres = __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)p.res + (size_t)n * p.res_img_stride), 0,
                                                        (int)((unsigned)M * pb), kRawBuffer);
    auto rfetch = [&](int mt, Raw (&r)[16]) {
        int m = m0 + 4 * half;
        asm volatile("" : "+v"(m));  // (not to be computed ahead of the loop and kept through it)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const unsigned row = row_of(mt, i);
            r[i] = load(rres, m + (int)row < M ? out_off : kBeyond, row * pb);
        }
    };
    Raw rv[16];
    float *s_bias = reinterpret_cast<float *>(pw_lds + 2 * 2 * MT * TW * 64);
    {
        if (tid < 32 * MT) s_bias[tid] = m0 + tid < M ? bias : 0.f;
        wput(0, wr);
        order();
        if constexpr (!ONE) wfetch(1, wr);
        order();
        if (has_res) rfetch(0, rv);
        order();
    }

    f32x16 acc[MT][NT];
    __syncthreads();  // the first stage's weights are in LDS
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 b = *reinterpret_cast<const f32x4 *>(s_bias + 32 * mt + 8 * g + 4 * half);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[mt][t][4 * g + e] = b[e];
            }
    // one stage's products; `next` fetches into the registers it has done with
    auto multiply = [&](int st, Raw (&raw)[16], auto next, bool full = false) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (c == 1 && !full && st * kPwStage + 16 >= K) break;   // wavefront-uniform: nothing left in the second chunk
            // B operands: the terms of this lane's eight channels, per pixel tile
            u32x4 b[NT][TX];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const Raw x0 = raw[8 * c + 2 * e], x1 = raw[8 * c + 2 * e + 1];
                if constexpr (F) {
                    unsigned t[TX];
                    if constexpr (NT == 2) {
                        split_pair<TX>(__uint_as_float(x0.x), __uint_as_float(x1.x), t);
#pragma unroll
                        for (int q = 0; q < TX; ++q) b[0][q][e] = t[q];
                        split_pair<TX>(__uint_as_float(x0.y), __uint_as_float(x1.y), t);
#pragma unroll
                        for (int q = 0; q < TX; ++q) b[NT - 1][q][e] = t[q];
                    } else {
                        split_pair<TX>(__uint_as_float(x0), __uint_as_float(x1), t);
#pragma unroll
                        for (int q = 0; q < TX; ++q) b[0][q][e] = t[q];
                    }
                } else {
                    b[0][0][e] = __builtin_amdgcn_perm(x1, x0, 0x05040100u);                       // the low halves
                    if constexpr (NT == 2) b[NT - 1][0][e] = __builtin_amdgcn_perm(x1, x0, 0x07060302u);  // the high ones
                }
            }
            const u32x4 *wa = pw_lds + (((st & 1) * 2 + c) * MT * TW) * 64 + lane;
            u32x4 a[MT][TW];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int q = 0; q < TW; ++q) a[mt][q] = wa[(mt * TW + q) * 64];
            // small terms first; neighbouring instructions on different accumulators
#pragma unroll
            for (int qw = TW - 1; qw >= 0; --qw)
#pragma unroll
                for (int qx = TX - 1; qx >= 0; --qx) {
                    if (F && qw + qx > 2) continue;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            acc[mt][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[mt][qw]),
                                                                                 __builtin_bit_cast(bf16x8, b[t][qx]), acc[mt][t], 0, 0, 0);
                }
        }
        order();
        next();
        order();
    };
    // row block 1's residual takes the first buffer when it falls free
    if constexpr (ONE || TWO) {
        multiply(0, ra, [&] {
            if (has_res && MT > 1) rfetch(1, ra);
        });
        if constexpr (TWO) {
            wput(1, wr);
            __syncthreads();
            multiply(1, rb, [] {});
        }
    } else {
        // (the last two stages, or the last one, stand behind the loop: with a way out of its middle the compiler takes the
        // values fetched last for the ones wanted first, and waits for everything at every turn)
        int st = 0;
        for (; st + 2 < stages; st += 2) {
            multiply(st, ra, [&] { fetch(st + 2, ra); }, true);
            wput(st + 1, wr);
            order();
            wfetch(st + 2, wr);
            __syncthreads();  // the next stage's weights are in LDS; everyone has finished with this one's
            multiply(st + 1, rb, [&] { fetch(st + 3, rb); }, true);
            wput(st + 2, wr);
            order();
            wfetch(st + 3, wr);
            __syncthreads();
        }
        multiply(st, ra, [&] {
            if (has_res && MT > 1) rfetch(1, ra);
        });
        if (st + 1 < stages) {
            wput(st + 1, wr);
            __syncthreads();
            multiply(st + 1, rb, [] {});
        }
    }
    if (has_res) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const Raw r = mt == 0 ? rv[i] : ra[i];
                if constexpr (F && NT == 2) {
                    acc[mt][0][i] += __uint_as_float(r.x);
                    acc[mt][NT - 1][i] += __uint_as_float(r.y);
                } else if constexpr (F) {
                    acc[mt][0][i] += __uint_as_float(r);
                } else {
                    acc[mt][0][i] += __uint_as_float(r << 16);
                    if constexpr (NT == 2) acc[mt][NT - 1][i] += __uint_as_float(r & 0xffff0000u);
                }
            }
    }

    pw_finish<T, MT, NT, GELU>(p, acc, n, m0, px, pxc, out_off, has_res);
}

// 64 pixels per wavefront.
template <int MT, bool GELU>
__global__ __launch_bounds__(kPwThreads, 2) void pointwise_kernel(const PointwiseParams p)
{
    pointwise_body<float, MT, 2, GELU>(p);
}
template <int MT, bool GELU>
__global__ __launch_bounds__(kPwThreads, 2) void pointwise_bf16_kernel(const PointwiseParams p)
{
    pointwise_body<bf16s, MT, 2, GELU>(p);
}
// Few pixels: 32 pixels per wavefront.
template <typename T, int MT, bool GELU>
__global__ __launch_bounds__(kPwThreads, 2) void pointwise_single_kernel(const PointwiseParams p)
{
    pointwise_body<T, MT, 1, GELU>(p);
}

// Channels in whole runs of sixteen.
template <typename T, int MT, int NT, int MODE, int LIE>
__global__ __launch_bounds__(kPwThreads, 2) void pointwise_runs_kernel(const PointwiseParams p)
{
    runs_body<T, MT, NT, MODE, LIE>(p);
}

template <auto kernel>
hipError_t launch_one(const PointwiseParams &p, unsigned grid, size_t lds, hipStream_t s)
{
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kPwThreads), lds, s, p);
    return hipGetLastError();
}

template <typename T, bool GELU>
hipError_t launch_typed(const PointwiseParams &p, int mt, int nt, unsigned grid, hipStream_t s)
{
    if (nt == 1)
        return mt == 1 ? launch_one<pointwise_single_kernel<T, 1, GELU>>(p, grid, pw_lds_bytes<T, 1>(), s)
                       : launch_one<pointwise_single_kernel<T, 2, GELU>>(p, grid, pw_lds_bytes<T, 2>(), s);
    if constexpr (sizeof(T) == 4)
        return mt == 1 ? launch_one<pointwise_kernel<1, GELU>>(p, grid, pw_lds_bytes<T, 1>(), s)
                       : launch_one<pointwise_kernel<2, GELU>>(p, grid, pw_lds_bytes<T, 2>(), s);
    else
        return mt == 1 ? launch_one<pointwise_bf16_kernel<1, GELU>>(p, grid, pw_lds_bytes<T, 1>(), s)
                       : launch_one<pointwise_bf16_kernel<2, GELU>>(p, grid, pw_lds_bytes<T, 2>(), s);
}

template <typename T, int NT, int MODE, int LIE>
hipError_t launch_runs(const PointwiseParams &p, int mt, unsigned grid, hipStream_t s)
{
    return mt == 1 ? launch_one<pointwise_runs_kernel<T, 1, NT, MODE, LIE>>(p, grid, pw_lds_bytes<T, 1>(), s)
                   : launch_one<pointwise_runs_kernel<T, 2, NT, MODE, LIE>>(p, grid, pw_lds_bytes<T, 2>(), s);
}

// Every way through here ends in a kernel: a variant that is not compiled is not named.
template <typename T, int NT, int MODE>
hipError_t launch_mode(const PointwiseParams &p, int mt, unsigned grid, hipStream_t s)
{
    const int K = p.K1 + p.K2;
    // Fetching ahead pays where latency counts: few pixels (192-channel residual step 64 x 64 fp32 77 us -> 64, 64 channels
    // of 25 images of 63 x 63 120 -> 111), bf16 storage (Conv_fuse 360 x 640 21 -> 19), LK^c's single stage, and more than two
    // stages (192-channel residual step 180 x 320 fp32 240 -> 211, 64 x 64 58 -> 54).  Large calls of fp32 with two are
    // bound by memory: waiting for everything, the residual step of 40 images of 72 x 72 of 64 channels takes 187 us, fetched
    // ahead 206; the fused call 339 x 511 63.0 and 66.2, 360 x 640 49.8 and 52.0.
    if (p.K1 % 16 == 0 && p.K2 % 16 == 0) {
        if constexpr (MODE == kPwPlain)
            if (K <= kPwStage) return launch_runs<T, NT, MODE, kPwOne>(p, mt, grid, s);
        if (K > 2 * kPwStage) return launch_runs<T, NT, MODE, kPwRuns>(p, mt, grid, s);
        if constexpr (sizeof(T) == 2 || NT == 1)
            return K > kPwStage ? launch_runs<T, NT, MODE, kPwTwo>(p, mt, grid, s) : launch_runs<T, NT, MODE, kPwRuns>(p, mt, grid, s);
    }
    return launch_typed<T, MODE == kPwGelu>(p, mt, NT, grid, s);
}

template <typename T, int MODE>
hipError_t launch_pixels(const PointwiseParams &p, int mt, int nt, unsigned grid, hipStream_t s)
{
    return nt == 1 ? launch_mode<T, 1, MODE>(p, mt, grid, s) : launch_mode<T, 2, MODE>(p, mt, grid, s);
}

}  // namespace

// Host side: how many pixels and output channels a wavefront owns.
__attribute__((visibility("hidden"))) hipError_t launch_pointwise(const PointwiseParams &p, bool bf16, hipStream_t s)
{
    if (p.N < 1 || p.P < 1 || p.M < 1 || p.K1 + p.K2 < 1) return hipSuccess;
    const size_t es = bf16 ? 2 : 4;
    // the accesses address an image of a tensor with 32-bit byte offsets below 2 GiB
    const size_t widest = (size_t)(p.M > p.K1 + p.K2 ? p.M : p.K1 + p.K2);
    if (widest * (size_t)p.P * es >= ((size_t)1 << 31)) return hipErrorInvalidValue;
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return hipErrorInvalidDevice;
        cus = n > 0 ? n : 1;
    }
    const int tiles_m = (p.M + 31) / 32;
    auto blocks = [&](int mt, int nt) { return (long)p.N * ((p.P + 128L * nt - 1) / (128L * nt)) * ((tiles_m + mt - 1) / mt); };
    // two pixels per lane (twice the bytes per access and operand read) once that still gives every
    // compute unit two blocks (360 x 640 bf16: 18.2 us, one pixel per lane 26; 180 x 320 fp32, 225
    // blocks: 11.2, one pixel per lane 9.9); more than 64 output channels: groups of 64, each reading the inputs
    const int mt = tiles_m < 2 ? tiles_m : 2;
    const int nt = (p.P >= 2 && blocks(mt, 2) >= 2L * cus) ? 2 : 1;
    const long grid = blocks(mt, nt);
    if (grid >= (1L << 31)) return hipErrorInvalidValue;
    if (p.gelu) return bf16 ? launch_pixels<bf16s, kPwGelu>(p, mt, nt, (unsigned)grid, s) : launch_pixels<float, kPwGelu>(p, mt, nt, (unsigned)grid, s);
    if (p.res != nullptr) return bf16 ? launch_pixels<bf16s, kPwRes>(p, mt, nt, (unsigned)grid, s) : launch_pixels<float, kPwRes>(p, mt, nt, (unsigned)grid, s);
    return bf16 ? launch_pixels<bf16s, kPwPlain>(p, mt, nt, (unsigned)grid, s) : launch_pixels<float, kPwPlain>(p, mt, nt, (unsigned)grid, s);
}

}  // namespace esc
