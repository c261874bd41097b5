// Backward pass of the ConvAttn module (depth-wise form; Eq. 4 lines 1-4 of the ESC paper
// without Conv_fuse) for gfx950 (MI355X).  The paper trains its shared LK end to end
// (Sec. 3) but prints no gradient formulae; these are the derivatives of the definition:
//
//   S[n,c,i,j]  = sum_{y,x} go[n,c,y,x] xz[n,c,y+i-p,x+j-p]      correlation of grad_out with x
//   dLK[c]      = sum_n S[n,c]           dDK[n,c] = centre 3 x 3 of S[n,c]
//   estimator   : dd = dDK;  db_up = sum_n dd;  dw_up = sum_n dd (x) t;  dt = w_up^T dd;
//                 du = dt * gelu'(u);  db_down = sum_n du;  dw_down = sum_n du (x) g;  dg = w_down^T du
//   dx[n,c]     = go[n,c] (*) flip(LK[c] + ZP(DK[n,c])) + dg[n,c] / (H W)     (c < C_a; dx = go elsewhere)
//
// The input gradient's convolution is the forward kernel itself, run on grad_out with the
// flipped kernels (esc_api.hip); this file holds what is new: the correlation S,
// as Toeplitz products on the matrix cores (corr_mfma_kernel), and the small estimator kernels; the GAP term of dx is a constant per plane that the
// input gradient's launch adds at its stores.  Every sum has a fixed order
// (per-tile partial sums in the workspace, then one thread per result), so results do not
// depend on scheduling.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "esc_backward.hpp"
#include "esc_estimator.hpp"
#include "esc_terms.hpp"

namespace esc {
namespace {

constexpr int kBwThreads = 256;

struct bf16b {
    uint16_t bits;
};
__device__ __forceinline__ float bw_load(const float *p) { return *p; }
__device__ __forceinline__ float bw_load(const bf16b *p) { return __uint_as_float((uint32_t)p->bits << 16); }
// running sum along each row of 16 lanes (data-parallel moves inside the vector unit):
// lane 15 of a row ends with the row's total, in a fixed order
__device__ __forceinline__ float row16_sum(float v)
{
    auto dpp = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                                                     0xf, 0xf, false));
    };
    v += dpp(v, std::integral_constant<int, 0x111>{});
    v += dpp(v, std::integral_constant<int, 0x112>{});
    v += dpp(v, std::integral_constant<int, 0x114>{});
    v += dpp(v, std::integral_constant<int, 0x118>{});
    return v;
}

extern __shared__ __align__(16) float bw_lds[];

// ---------------------------------------------------------------------------
// S per tile.  A block takes a 64 x 32 pixel tile of one (image, channel) plane; the window's sums over
// it run on the matrix cores.  For one row y of grad_out's tile the sums over x are a product of two matrices:
//   S[i][j] += sum_c  X_y[i][c] * G_y[c][j],   X_y[i][c] = xz[y + i][c]  (rows of x's halo tile),
//                                              G_y[c][j] = go[y][c - j]  (a Toeplitz matrix of the row)
// with K = the halo tile's columns, 32 per v_mfma_f32_16x16x32: one 16 x 16 block of sums up to 15 x 15, 3
// instructions per tile row; two by two blocks beyond, 12.  With bf16 storage the stored values are the operands
// (products exact, fp32 accumulation).  fp32 values are taken apart into two fp16 terms behind a power of two that brings the
// tile's largest to 2^14 ... 2^15 (within a unit of fp32's last place), kept as two tiles, and three of the four
// products of terms are accumulated (the fourth is below 2^-22 of a product).  A tile whose magnitudes lie further apart than that
// reaches (BlockRange), or with infinities or NaN in it, is summed in fp32 by the vector units (plain_sums).
// A operand: lane (i, kg) reads 16 bytes of halo row y + i - the halo tile is laid out from the
// aligned column x0 - 8 (x0 - 16), so every read is aligned.  B operand: lane (j, kg) wants eight
// consecutive values of the row starting j elements to the left - a start that is odd for
// every other lane.  grad_out's rows are therefore kept twice, zero-extended: as they are and
// moved by one element; a lane reads four whole words from the copy of its parity.  The four
// wavefronts take eight rows each (neighbouring rows share their A operands, see there) and add
// their results through LDS; the sum of x (for the GAP) comes from the halo tile's loads.  The partial sums of a
// tile end with it.  Bound by no unit alone (16 x 64 x 64 fp32 13 x 13: the LDS at work in 47 % of the clocks, vector instructions 37 %, matrix
// cores 15 %): one tile a block, its loads, its range and its sums one behind the other.
// 64 x 64 x 64, the whole backward: 17 x 17 bf16 79 us -> 43, fp32 98 -> 80 (31 x 31 196 -> 71 and 223 -> 101), by a vector kernel
// with the window's rows in registers until then; 13 x 13 fp32 71 -> 61 and 16 x 64 x 64 28.6 -> 26.8, with three bf16 terms and nine
// products until then, error against float64 4.8e-7 -> 1.6e-7 (products with a low term summed apart; together 5.0e-7).
// With a value of 1e10 in every tile 13 x 13 88 us, 17 x 17 142, 31 x 31 266 (by the kernels before 74, 98 and 210).  Widths off the pieces, all loads of a thread
// at once instead of one after the other: 8 x 63 x 63 fp32 29 -> 25 us, 64 x 63 x 63 bf16 47 -> 39.
// ---------------------------------------------------------------------------
constexpr int kCmXP = 104;  // halo tile: elements per row (96 columns are read; 13 x 16 bytes: rows fall on different banks)
// the tiles of a window: one 16 x 16 block of sums up to 15 x 15, two by two beyond
template <int KC, bool F32>
struct CorrGeom {
    static constexpr int NB = KC <= 15 ? 1 : 2;
    static constexpr int BASE = 8 * NB;                // the halo tile starts this many columns left of the tile
    static constexpr int PIECES = 8 + 2 * NB;          // pieces of eight columns of a halo row
    // neighbouring rows of grad_out that share their A operands: a block's sixteen rows serve 16 NB - KC + 1, at most four;
    // two where four rows' sums would leave a block alone on its compute unit
    static constexpr int SH = NB == 1 && 16 - KC + 1 >= 4 ? 4 : 2;
    static constexpr int BLOCKS = F32 ? 4 - NB : NB == 1 ? 6 : 3;   // resident blocks per compute unit the registers are cut for
    static constexpr int XR = NB == 1 ? 48 : 64;       // halo tile rows (those read beyond the window feed discarded results)
    static constexpr int GP = NB == 1 ? 112 : 128;     // elements per zero-extended row of grad_out
    static constexpr size_t G0 = (size_t)XR * kCmXP * 2, G1 = G0 + (size_t)kCorrTileH * GP * 2 + 64;
    static constexpr size_t TERM = G1 + (size_t)kCorrTileH * GP * 2;  // bytes per term
    static constexpr size_t RED = NB == 1 ? (size_t)4 * SH * 256 * 4 + 64 : (size_t)4 * 1024 * 4 + 64;
    // special tiles (below): x's halo from column -P on and grad_out, fp32, rows of whole runs of four
    static constexpr int JG = (KC + 3) / 4, IG = (KC + 1) / 2, XF = kCorrTileW + 4 * JG + 4, XFR = kCorrTileH + 2 * IG;
    static constexpr int SPLIT = 256 / (JG * IG) < 8 ? 256 / (JG * IG) : 8;   // threads that share two rows and four columns of the window, by tile rows
    static constexpr size_t PLAIN = F32 || NB == 2 ? ((size_t)XFR * XF + kCorrTileH * kCorrTileW) * 4 : 0;
    static constexpr size_t tiles(int terms)
    {
        const size_t a = terms * TERM > RED ? terms * TERM : RED;
        return a > PLAIN ? a : PLAIN;
    }
    static constexpr size_t lds() { return tiles(F32 ? 2 : 1) + 4 * sizeof(uint4); }
};

// eight consecutive bf16 values to row[q ...]: whole words where the parity of q allows
template <bool EVEN>
__device__ __forceinline__ void cm_put8(uint16_t *row, int q, const uint16_t (&v)[8])
{
    if (EVEN) {
#pragma unroll
        for (int d = 0; d < 4; ++d) *reinterpret_cast<uint32_t *>(row + q + 2 * d) = (uint32_t)v[2 * d] | ((uint32_t)v[2 * d + 1] << 16);
    } else {
        row[q] = v[0];
#pragma unroll
        for (int d = 0; d < 3; ++d) *reinterpret_cast<uint32_t *>(row + q + 1 + 2 * d) = (uint32_t)v[2 * d + 1] | ((uint32_t)v[2 * d + 2] << 16);
        row[q + 7] = v[7];
    }
}

template <typename T, int KC>
__global__ __launch_bounds__(kBwThreads, (CorrGeom<KC, std::is_same<T, float>::value>::BLOCKS)) void corr_mfma_kernel(const BackwardParams p)
{
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    static_assert(KC % 2 == 1 && KC >= 3 && KC <= 31, "at most two by two blocks of sums");
    constexpr bool kF32 = std::is_same<T, float>::value;
    using CG = CorrGeom<KC, kF32>;
    constexpr int NT = kF32 ? 2 : 1;          // terms per value (fp32 storage: fp16 terms)
    constexpr int NB = CG::NB, P = (KC - 1) / 2, PC = CG::PIECES;
    constexpr int HRU = kCorrTileH + KC - 1;  // halo rows the window reaches
    constexpr int GOFF = P + CG::BASE;        // element of a zero-extended row that holds the tile's column 0
    char *lds = reinterpret_cast<char *>(bw_lds);
    // term t: halo tile [XR][kCmXP] (column c = image column x0 - BASE + c), then grad_out's rows
    // [32][GP] (element q = column q - GOFF) and the same moved by one (element q = column q + 1 - GOFF)
    auto xs = [&](int t) { return reinterpret_cast<uint16_t *>(lds + t * CG::TERM); };
    auto g0 = [&](int t) { return reinterpret_cast<uint16_t *>(lds + t * CG::TERM + CG::G0); };
    auto g1 = [&](int t) { return reinterpret_cast<uint16_t *>(lds + t * CG::TERM + CG::G1); };
    u32x4 *s_range = reinterpret_cast<u32x4 *>(lds + CG::tiles(NT));   // of each wavefront's values of x and of grad_out

    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int H = p.H, W = p.W;
    const int tiles_x = (W + kCorrTileW - 1) / kCorrTileW;
    const int tiles = corr_tiles(H, W);
    const unsigned nc = blockIdx.x / (unsigned)tiles, tile = blockIdx.x - nc * (unsigned)tiles;
    const unsigned n = nc / (unsigned)p.Ca, c = nc - n * (unsigned)p.Ca;
    const int ty0 = (int)(tile / (unsigned)tiles_x) * kCorrTileH, tx0 = (int)(tile % (unsigned)tiles_x) * kCorrTileW;
    const size_t plane = ((size_t)n * p.C + c) * (size_t)H * W;
    const T *xp = (const T *)p.x + plane, *gp = (const T *)p.go + plane;

    // Up to 15 x 15 in bf16 storage a value that is not finite makes what its instructions touch NaN.  Otherwise the ranges of
    // the two tiles are looked for: they give fp32 storage its powers of two, and tiles that reach further than two terms do, or
    // that have infinities or NaN in them, are special.
    constexpr bool kLook = kF32 || NB == 2;
    Range rx, rg;
    BlockRange mx, mg;
    auto agree = [&](bool barrier) {
        if constexpr (kLook) {
            const BlockRange x(rx), g(rg);
            const u32x4 mine{wave_max(x.large), wave_max(x.small), wave_max(g.large), wave_max(g.small)};
            if (lane == 63) s_range[wave] = mine;
        }
        if (kLook || barrier) __syncthreads();
        if constexpr (kLook) {
#pragma unroll
            for (int k = 0; k < kBwThreads / 64; ++k) {
                const u32x4 theirs = s_range[k];
                mx.merge(theirs[0], theirs[1]);
                mg.merge(theirs[2], theirs[3]);
            }
        }
        return kLook && !(mx.finite() && mg.finite() && (!kF32 || (mx.narrow() && mg.narrow())));   // block-uniform
    };
    float *plain_x = bw_lds, *plain_g = bw_lds + CG::XFR * CG::XF;
    auto plain_put = [&](int r, int cc, float v) {   // x, halo row r and column cc (from -BASE)
        const int at = cc - CG::BASE + P;
        if (at >= 0 && at < CG::XF) plain_x[r * CG::XF + at] = v;
    };
    // a value as NT terms: bf16 storage itself; fp32 the nearest fp16 and the nearest to 4096 times what is left
    auto split = [](float v, uint16_t (&t)[NT]) {
        if constexpr (kF32) {
            const _Float16 h = (_Float16)v, l = (_Float16)((v - (float)h) * kLowTerm);
            t[0] = __builtin_bit_cast(uint16_t, h), t[NT - 1] = __builtin_bit_cast(uint16_t, l);
        } else {
            t[0] = (uint16_t)(__float_as_uint(v) >> 16);
        }
    };
    // eight neighbouring values (16 or 32 bytes of memory) at e, or zeros; their sum for the GAP
    auto fetch8 = [](const T *e, bool in, u32x4 (&raw)[kF32 ? 2 : 1]) {
        raw[0] = *reinterpret_cast<const u32x4 *>(e);
        if (kF32) raw[kF32 ? 1 : 0] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(e) + 16);
        if (!in)
            for (int k = 0; k < (kF32 ? 2 : 1); ++k) raw[k] = u32x4{0u, 0u, 0u, 0u};
    };
    auto value8 = [](const u32x4 (&raw)[kF32 ? 2 : 1], int e) {
        if constexpr (kF32)
            return __uint_as_float(raw[e >> 2][e & 3]);
        else
            return __uint_as_float(e & 1 ? raw[0][e >> 1] & 0xffff0000u : raw[0][e >> 1] << 16);
    };
    auto terms8 = [&](const u32x4 (&raw)[kF32 ? 2 : 1], float f, uint16_t (&v)[NT][8], float &sum) {
        sum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float a = value8(raw, e);
            uint16_t t[NT];
            split(kF32 ? a * f : a, t);
#pragma unroll
            for (int q = 0; q < NT; ++q) v[q][e] = t[q];
            sum += a;
        }
    };

    float sx = 0.f;
    bool special = false;
    float *dst = p.partial + ((size_t)nc * tiles + tile) * (KC * KC + 1);
    // A special tile, in fp32: a thread has two rows and four columns of the window, for every SPLIT-th row of the tile.  Per four
    // pixels one read of grad_out and two of x (sixteen bytes each) feed 32 multiply-adds, which bound it.  (grad_out beyond the image is not
    // multiplied: x may be infinite there.)
    auto plain_sums = [&]() {
        if constexpr (kLook) {
            typedef float f4 __attribute__((ext_vector_type(4)));
            constexpr int JG = CG::JG, IG = CG::IG, XF = CG::XF, SPLIT = CG::SPLIT, TASKS = JG * IG;
            const float sxr = row16_sum(sx);
            __syncthreads();
            const int q = tid / TASKS, task = tid - q * TASKS, i0 = 2 * (task / JG), j0 = 4 * (task % JG);
            const int rows = min(kCorrTileH, H - ty0), cols = min(kCorrTileW, W - tx0);
            float s[2][4] = {};
            if (q < SPLIT) {
                for (int y = q; y < rows; y += SPLIT) {
                    const float *gs = plain_g + y * kCorrTileW, *xs0 = plain_x + (y + i0) * XF + j0;
                    f4 xa[2] = {*reinterpret_cast<const f4 *>(xs0), *reinterpret_cast<const f4 *>(xs0 + XF)};
#pragma unroll 1
                    for (int x = 0; x < cols; x += 4) {
                        const f4 g = *reinterpret_cast<const f4 *>(gs + x);
#pragma unroll
                        for (int w = 0; w < 2; ++w) {
                            const f4 xb = *reinterpret_cast<const f4 *>(xs0 + w * XF + x + 4);
                            const float v[8] = {xa[w][0], xa[w][1], xa[w][2], xa[w][3], xb[0], xb[1], xb[2], xb[3]};
                            if (x + 4 <= cols) {
#pragma unroll
                                for (int k = 0; k < 4; ++k)
#pragma unroll
                                    for (int j = 0; j < 4; ++j) s[w][j] = fmaf(g[k], v[k + j], s[w][j]);
                            } else {
#pragma unroll
                                for (int k = 0; k < 3; ++k)
#pragma unroll
                                    for (int j = 0; j < 4; ++j) s[w][j] = x + k < cols ? fmaf(g[k], v[k + j], s[w][j]) : s[w][j];
                            }
                            xa[w] = xb;
                        }
                    }
                }
            }
            __syncthreads();  // the tiles are no longer read
            float *red = bw_lds, *sxs = bw_lds + SPLIT * 4 * IG * 2 * JG;   // [SPLIT][2 IG][4 JG], [16 rows of lanes]
            if (q < SPLIT)
#pragma unroll
                for (int w = 0; w < 2; ++w)
#pragma unroll
                    for (int j = 0; j < 4; ++j) red[(q * 2 * IG + i0 + w) * 4 * JG + j0 + j] = s[w][j];
            if ((lane & 15) == 15) sxs[tid >> 4] = sxr;
            __syncthreads();
            for (int o = tid; o < KC * KC + 1; o += kBwThreads) {
                float sum = 0.f;
                if (o == KC * KC) {
                    for (int k = 0; k < 16; ++k) sum += sxs[k];
                } else {
                    for (int k = 0; k < SPLIT; ++k) sum += red[(k * 2 * IG + o / KC) * 4 * JG + o % KC];
                }
                dst[o] = sum;
            }
        }
    };
    if (p.corr_vec) {
        // whole pieces of eight columns, each entirely inside or outside the image; the loads
        // travel while the LDS is cleared
        constexpr int XT = HRU * PC, XK = (XT + kBwThreads - 1) / kBwThreads;
        u32x4 xv[XK][kF32 ? 2 : 1], gv[kF32 ? 2 : 1];
#pragma unroll
        for (int k = 0; k < XK; ++k) {
            const int t = k * kBwThreads + tid, r = t / PC, pc = t - r * PC;
            const int gy = ty0 - P + r, gx = tx0 - CG::BASE + 8 * pc;
            const bool in = t < XT && gy >= 0 && gy < H && gx >= 0 && gx < W;
            fetch8(xp + (in ? (size_t)gy * W + gx : 0), in, xv[k]);
        }
        {
            const int r = tid >> 3, pc = tid & 7;
            const int gy = ty0 + r, gx = tx0 + 8 * pc;
            const bool in = gy < H && gx < W;
            fetch8(gp + (in ? (size_t)gy * W + gx : 0), in, gv);
        }
        for (int o = tid; o < (int)(NT * CG::TERM / 16); o += kBwThreads) reinterpret_cast<u32x4 *>(lds)[o] = u32x4{0u, 0u, 0u, 0u};
        if constexpr (kLook) {
#pragma unroll
            for (int k = 0; k < XK; ++k)
#pragma unroll
                for (int e = 0; e < 8; e += 2) rx.look(value8(xv[k], e), value8(xv[k], e + 1));
#pragma unroll
            for (int e = 0; e < 8; e += 2) rg.look(value8(gv, e), value8(gv, e + 1));
        }
        special = agree(true);
        if (kLook && special) {
#pragma unroll
            for (int k = 0; k < XK; ++k) {
                const int t = k * kBwThreads + tid, r = t / PC, pc = t - r * PC;
                if (t >= XT) continue;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float v = value8(xv[k], e);
                    plain_put(r, 8 * pc + e, v);
                    if (r >= P && r < P + kCorrTileH && pc >= NB && pc < NB + 8) sx += v;
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) plain_g[(tid >> 3) * kCorrTileW + 8 * (tid & 7) + e] = value8(gv, e);
            return plain_sums();
        }
        const float fx = kF32 ? power_of_two(mx.up()) : 1.f, fg = kF32 ? power_of_two(mg.up()) : 1.f;
#pragma unroll
        for (int k = 0; k < XK; ++k) {
            const int t = k * kBwThreads + tid, r = t / PC, pc = t - r * PC;
            uint16_t v[NT][8];
            float sum;
            terms8(xv[k], fx, v, sum);
            if (t < XT) {
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) cm_put8<true>(xs(tt) + r * kCmXP, 8 * pc, v[tt]);
                // the tile's own pixels, for the GAP
                if (r >= P && r < P + kCorrTileH && pc >= NB && pc < NB + 8) sx += sum;
            }
        }
        {
            const int r = tid >> 3, pc = tid & 7;
            uint16_t v[NT][8];
            float sum;
            terms8(gv, fg, v, sum);
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                cm_put8<GOFF % 2 == 0>(g0(tt) + r * CG::GP, GOFF + 8 * pc, v[tt]);
                cm_put8<GOFF % 2 != 0>(g1(tt) + r * CG::GP, GOFF + 8 * pc - 1, v[tt]);
            }
        }
    } else {
        for (int o = tid; o < (int)(NT * CG::TERM / 16); o += kBwThreads) reinterpret_cast<u32x4 *>(lds)[o] = u32x4{0u, 0u, 0u, 0u};
        // element by element: eight of a thread's on their way at once, or all of them where the largest is looked for first
        constexpr int XT = HRU * 8 * PC, XK = (XT + kBwThreads - 1) / kBwThreads, GK = kCorrTileH * kCorrTileW / kBwThreads;
        constexpr int STEP = kLook ? XK : 8;
        int t0 = tid;
        asm volatile("" : "+v"(t0));  // (nothing of this is to be computed ahead and kept)
        float xv[STEP], gv[GK];
        auto get_x = [&](int k0) {
#pragma unroll
            for (int k = 0; k < STEP; ++k) {
                const int t = (k0 + k) * kBwThreads + t0, r = t / (8 * PC), cc = t - r * (8 * PC);
                const int gy = ty0 - P + r, gx = tx0 - CG::BASE + cc;
                const bool in = t < XT && gy >= 0 && gy < H && gx >= 0 && gx < W;
                const float f = bw_load(xp + (in ? (size_t)gy * W + gx : 0));
                xv[k] = in ? f : 0.f;
            }
        };
        auto put_x = [&](int k0, float f) {
#pragma unroll
            for (int k = 0; k < STEP; ++k) {
                const int t = (k0 + k) * kBwThreads + t0, r = t / (8 * PC), cc = t - r * (8 * PC);
                uint16_t v[NT];
                split(kF32 ? xv[k] * f : xv[k], v);
                if (t < XT) {
#pragma unroll
                    for (int tt = 0; tt < NT; ++tt) xs(tt)[r * kCmXP + cc] = v[tt];
                    if (r >= P && r < P + kCorrTileH && cc >= CG::BASE && cc < CG::BASE + kCorrTileW) sx += xv[k];
                }
            }
        };
        get_x(0);
#pragma unroll
        for (int k = 0; k < GK; ++k) {
            const int t = k * kBwThreads + t0, gy = ty0 + (t >> 6), gx = tx0 + (t & 63);
            const bool in = gy < H && gx < W;
            const float f = bw_load(gp + (in ? (size_t)gy * W + gx : 0));
            gv[k] = in ? f : 0.f;
        }
        if constexpr (kLook) {
#pragma unroll
            for (int k = 0; k < STEP; k += 2) rx.look(xv[k], k + 1 < STEP ? xv[k + 1] : 0.f);
#pragma unroll
            for (int k = 0; k < GK; k += 2) rg.look(gv[k], gv[k + 1]);
        }
        special = agree(true);
        if (kLook && special) {
#pragma unroll
            for (int k = 0; k < XK; ++k) {
                const int t = k * kBwThreads + t0, r = t / (8 * PC), cc = t - r * (8 * PC);
                if (t >= XT) continue;
                const float v = xv[k < STEP ? k : 0];
                plain_put(r, cc, v);
                if (r >= P && r < P + kCorrTileH && cc >= CG::BASE && cc < CG::BASE + kCorrTileW) sx += v;
            }
#pragma unroll
            for (int k = 0; k < GK; ++k) plain_g[k * kBwThreads + t0] = gv[k];
            return plain_sums();
        }
        const float fx = kF32 ? power_of_two(mx.up()) : 1.f, fg = kF32 ? power_of_two(mg.up()) : 1.f;
        put_x(0, fx);
#pragma unroll
        for (int k = 0; k < GK; ++k) {
            const int t = k * kBwThreads + t0, r = t >> 6, cc = t & 63;
            uint16_t v[NT];
            split(kF32 ? gv[k] * fg : gv[k], v);
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                g0(tt)[r * CG::GP + GOFF + cc] = v[tt];
                g1(tt)[r * CG::GP + GOFF + cc - 1] = v[tt];
            }
        }
        for (int k0 = STEP; k0 < XK; k0 += STEP) get_x(k0), put_x(k0, fx);
    }
    __syncthreads();

    // ---- this wavefront's rows of the tile: 8 w .. 8 w + 7, in groups of SH neighbours that
    // share their A operands: the halo rows R .. R + 15 serve tile row R + s as window rows
    // i = i' - s (i' the row of the product), s < SH = 16 - KC + 1 (at most 4); every shift has
    // accumulators of its own, and the shifted results are put together at the end ----
    constexpr int SH = CG::SH;
    const int l16 = lane & 15, kg = lane >> 4;
    // block jb of the window's columns: column 16 jb + l16 (those beyond the window repeat its last one; their sums are
    // dropped), in the copy of its parity, from an even element on
    size_t gsel[NB];
    int o0[NB];
#pragma unroll
    for (int jb = 0; jb < NB; ++jb) {
        const int jc = min(16 * jb + l16, KC - 1);
        gsel[jb] = (jc & 1) ? CG::G1 : CG::G0;
        o0[jb] = 8 * kg - jc + 2 * P - (jc & 1);
    }
    constexpr int NC = NB == 1 ? 3 : 1;   // one 16 x 16 block: the three column blocks' sums apart, so that their chains take turns
    f32x4 acc[SH][NB][NB][NC], low[kF32 ? SH : 1][NB][NB][NC];   // (fp32 storage: products with a low term apart)
#pragma unroll
    for (int sft = 0; sft < SH; ++sft)
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
            for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                for (int b = 0; b < NC; ++b) acc[sft][ib][jb][b] = low[kF32 ? sft : 0][ib][jb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 8 / SH; ++u) {
        const int R = 8 * wave + SH * u;
        u32x4 a[NT][NB][3];
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
            for (int ib = 0; ib < NB; ++ib)
#pragma unroll
                for (int b = 0; b < 3; ++b) a[tt][ib][b] = *reinterpret_cast<const u32x4 *>(xs(tt) + (R + 16 * ib + l16) * kCmXP + 32 * b + 8 * kg);
#pragma unroll
        for (int sft = 0; sft < SH; ++sft) {
            u32x4 bv[NT][NB][3];
#pragma unroll
            for (int tt = 0; tt < NT; ++tt)
#pragma unroll
                for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                    for (int b = 0; b < 3; ++b)
                        __builtin_memcpy(&bv[tt][jb][b],
                                         reinterpret_cast<const uint32_t *>(reinterpret_cast<const uint16_t *>(lds + tt * CG::TERM + gsel[jb]) +
                                                                            (R + sft) * CG::GP + o0[jb] + 32 * b),
                                         16);
            // (small terms first; neighbouring products belong to different sums)
#pragma unroll
            for (int ta = NT - 1; ta >= 0; --ta)
#pragma unroll
                for (int tb = NT - 1; tb >= 0; --tb) {
                    if (ta + tb > 1) continue;   // (below 2^-22 of a product)
#pragma unroll
                    for (int b = 0; b < 3; ++b)
#pragma unroll
                        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
                            for (int jb = 0; jb < NB; ++jb) {
                                f32x4 &d = (ta + tb > 0 ? low[kF32 ? sft : 0] : acc[sft])[ib][jb][NC == 3 ? b : 0];
                                if constexpr (kF32)
                                    d = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a[ta][ib][b]),
                                                                               __builtin_bit_cast(f16x8, bv[tb][jb][b]), d, 0, 0, 0);
                                else
                                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[ta][ib][b]),
                                                                                __builtin_bit_cast(bf16x8, bv[tb][jb][b]), d, 0, 0, 0);
                            }
                }
        }
    }
    if constexpr (kF32) {
#pragma unroll
        for (int sft = 0; sft < SH; ++sft)
#pragma unroll
            for (int ib = 0; ib < NB; ++ib)
#pragma unroll
                for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                    for (int b = 0; b < NC; ++b)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[sft][ib][jb][b][r] = fmaf(low[sft][ib][jb][b][r], 1.f / kLowTerm, acc[sft][ib][jb][b][r]);
    }
    const float sxr = row16_sum(sx);
    __syncthreads();  // the tiles are no longer read: their LDS takes the wavefronts' results
    // one block: [4 wavefronts][SH shifts][16 i'][16 j]; two by two: [4 wavefronts][32 i][32 j], a shift at a time
    float *red = bw_lds, *sxs = bw_lds + (NB == 1 ? 4 * SH * 256 : 4096);    // [16 rows of lanes]
    if constexpr (NB == 1) {
#pragma unroll
        for (int sft = 0; sft < SH; ++sft) {
            const f32x4 tot = (acc[sft][0][0][0] + acc[sft][0][0][1 % NC]) + acc[sft][0][0][2 % NC];
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(wave * SH + sft) * 256 + (4 * kg + r) * 16 + l16] = tot[r];
        }
    } else {
#pragma unroll
        for (int sft = 0; sft < SH; ++sft) {
#pragma unroll
            for (int ib = 0; ib < NB; ++ib)
#pragma unroll
                for (int jb = 0; jb < NB; ++jb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int i = 16 * ib + 4 * kg + r - sft;   // the window row that row i' of the product is for this shift
                        float *d = red + wave * 1024 + i * 32 + 16 * jb + l16;
                        if (sft == 0)
                            *d = acc[sft][ib][jb][0][r];
                        else if (i >= 0)
                            *d += acc[sft][ib][jb][0][r];
                    }
            __syncthreads();  // (the next shift's rows lie in other lanes)
        }
    }
    if (l16 == 15) sxs[tid >> 4] = sxr;
    __syncthreads();
    const int back = kF32 ? -mx.up() - mg.up() : 0;
    for (int o = tid; o < KC * KC + 1; o += kBwThreads) {
        float s2 = 0.f;
        if (o == KC * KC) {
#pragma unroll
            for (int k = 0; k < 16; ++k) s2 += sxs[k];
        } else {
            const int i = o / KC, j = o - i * KC;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                if constexpr (NB == 2) {
                    s2 += red[w * 1024 + i * 32 + j];
                } else {
#pragma unroll
                    for (int sft = 0; sft < SH; ++sft) s2 += red[(w * SH + sft) * 256 + (i + sft) * 16 + j];
                }
            }
            if (kF32) s2 = __builtin_amdgcn_ldexpf(s2, back);
        }
        dst[o] = s2;
    }
}

template <typename T, int KC>
hipError_t launch_corr_mfma(const BackwardParams &p, unsigned grid, hipStream_t s)
{
    constexpr size_t lds = CorrGeom<KC, std::is_same<T, float>::value>::lds();
    static bool granted = false;
    if (lds > 48 * 1024 && !granted) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&corr_mfma_kernel<T, KC>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        granted = true;
    }
    hipLaunchKernelGGL((corr_mfma_kernel<T, KC>), dim3(grid), dim3(kBwThreads), lds, s, p);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_corr_mfma_kc(const BackwardParams &p, int kc, unsigned grid, hipStream_t s)
{
    switch (kc) {
#define ESC_KC(K) case K: return launch_corr_mfma<T, K>(p, grid, s);
        ESC_KC(3) ESC_KC(5) ESC_KC(7) ESC_KC(9) ESC_KC(11) ESC_KC(13) ESC_KC(15) ESC_KC(17)
        ESC_KC(19) ESC_KC(21) ESC_KC(23) ESC_KC(25) ESC_KC(27) ESC_KC(29) ESC_KC(31)
#undef ESC_KC
    }
    return hipErrorInvalidValue;
}

// grad_lk: one row of 16 lanes per element (element idx of the Ks x Ks filters; sums over images
// and tiles, over channels too for a single shared filter).  Lane l adds terms l, l + 16, ...
// in ascending order, then the row's lanes are added in lane order: a fixed order, and
// sixteen loads in flight instead of a chain of dependent ones.
__device__ __forceinline__ void sums_row(const BackwardParams &p, int KC, int tiles, size_t idx, int l)
{
    const int Ks = p.Ks, Ca = p.Ca, off = (KC - Ks) / 2;
    const size_t per = (size_t)KC * KC + 1;
    const int c0 = (int)(idx / ((size_t)Ks * Ks)), r = (int)(idx % ((size_t)Ks * Ks));
    const size_t elem = (size_t)(r / Ks + off) * KC + (size_t)(r % Ks + off);
    // channel c0 of every image, or (one shared filter) every channel of every image
    const size_t nc0 = p.lk_cstride != 0 ? (size_t)c0 : 0;
    const int planes = p.lk_cstride != 0 ? p.N : p.N * Ca, plane_step = p.lk_cstride != 0 ? Ca : 1;
    const int count = planes * tiles;
    float s = 0.f;
    for (int k0 = l; k0 < count; k0 += 64) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + 16 * u;
            const int kk = k < count ? k : count - 1;
            const int pl = kk / tiles, tl = kk - pl * tiles;
            v[u] = p.partial[((nc0 + (size_t)pl * plane_step) * tiles + tl) * per + elem];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) s += k0 + 16 * u < count ? v[u] : 0.f;
    }
    s = row16_sum(s);
    if (l != 15 || p.grad_lk == nullptr) return;
    float *dst = p.grad_lk + (p.lk_cstride != 0 ? (size_t)c0 * p.lk_cstride : 0) + r;
    *dst = p.accumulate ? *dst + s : s;
}

__device__ __forceinline__ float gelu_f(float v) { return 0.5f * v * (1.f + erff(v * 0.70710678118654752440f)); }
__device__ __forceinline__ float gelu_grad_f(float v)
{
    return 0.5f * (1.f + erff(v * 0.70710678118654752440f)) + v * expf(-0.5f * v * v) * 0.39894228040143267794f;
}

// One block per image: its tiles' partial sums are added to dDK[n] and the GAP means g[n]
// (a thread per result); then the estimator forwards from g (DK, stored flipped for the input
// gradient) and backwards from dDK (dL/dt, dL/du, dL/dg) - plain loops, a few thousand
// multiply-adds per image.
__global__ __launch_bounds__(kBwThreads) void estimator_image_kernel(const BackwardParams p, int KC, int tiles)
{
    __shared__ float s_g[256], s_u[256], s_t[256], s_dt[256], s_du[256], s_dd[9 * 256], s_part[kBwThreads];
    const int n = (int)blockIdx.x, tid = (int)threadIdx.x;
    const int Ca = p.Ca, hidden = p.hidden, K = hidden > 0 ? hidden : Ca;
    const float hw = (float)((double)p.H * (double)p.W);
    {
        // this image's sums over its tiles, one thread per result (9 C_a of dDK, C_a of g), the
        // tiles in ascending order, eight loads in flight
        const size_t per = (size_t)KC * KC + 1;
        for (int o = tid; o < 10 * Ca; o += kBwThreads) {
            const bool is_dd = o < 9 * Ca;
            const int c = is_dd ? o / 9 : o - 9 * Ca, r = is_dd ? o - 9 * c : 0;
            const size_t elem = is_dd ? (size_t)(r / 3 + (KC - 3) / 2) * KC + (size_t)(r % 3 + (KC - 3) / 2) : (size_t)KC * KC;
            const float *src = p.partial + ((size_t)n * Ca + c) * tiles * per + elem;
            float sum = 0.f;
            for (int t0 = 0; t0 < tiles; t0 += 8) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = src[(size_t)(t0 + u < tiles ? t0 + u : tiles - 1) * per];
#pragma unroll
                for (int u = 0; u < 8; ++u) sum += t0 + u < tiles ? v[u] : 0.f;
            }
            if (is_dd) {
                s_dd[o] = sum;
                p.ddk[(size_t)n * 9 * Ca + o] = sum;
                if (p.grad_dk != nullptr) p.grad_dk[(size_t)n * 9 * Ca + o] = sum;
            } else {
                const float g = sum / hw;
                s_g[c] = g;
                p.g[(size_t)n * Ca + c] = g;
            }
        }
    }
    if (!p.has_gen) {  // DK as given (or zero): only its flipped copy is needed
        for (int o = tid; o < 9 * Ca; o += kBwThreads) {
            const int c = o / 9, r = o - 9 * c;
            p.dkf[((size_t)n * Ca + c) * 9 + (8 - r)] = p.dk_in != nullptr ? p.dk_in[(size_t)n * 9 * Ca + o] : 0.f;
        }
        for (int k = tid; k < Ca; k += kBwThreads) p.dgc[(size_t)n * Ca + k] = 0.f;
        return;
    }
    __syncthreads();  // s_g and s_dd are written
    if (hidden > 0) {
        for (int m = tid; m < hidden; m += kBwThreads) {
            float s = p.b_down != nullptr ? p.b_down[m] : 0.f;
#pragma unroll 8
            for (int k = 0; k < Ca; ++k) s = fmaf(p.w_down[(size_t)m * Ca + k], s_g[k], s);
            s_u[m] = s;
            s_t[m] = gelu_f(s);
        }
    } else {
        for (int k = tid; k < Ca; k += kBwThreads) s_t[k] = s_g[k];
    }
    __syncthreads();
    for (int k = tid; k < K; k += kBwThreads) p.t[(size_t)n * K + k] = s_t[k];
    for (int o = tid; o < 9 * Ca; o += kBwThreads) {
        float s = p.b_up != nullptr ? p.b_up[o] : 0.f;
#pragma unroll 8
        for (int k = 0; k < K; ++k) s = fmaf(p.w_up[(size_t)o * K + k], s_t[k], s);
        const int c = o / 9, r = o - 9 * c;
        p.dkf[((size_t)n * Ca + c) * 9 + (8 - r)] = s;
    }
    // dL/dt = w_up^T dd: the rows o are dealt to the block's groups of K threads (group g takes
    // rows g, g + groups, ...), whose partial sums are then added in group order - a chain of
    // 9 C_a dependent loads per thread otherwise
    if (K <= kBwThreads / 2) {
        const int groups = kBwThreads / K, g = tid / K, k = tid - g * K;
        float s = 0.f;
        if (g < groups) {
#pragma unroll 4
            for (int o = g; o < 9 * Ca; o += groups) s = fmaf(p.w_up[(size_t)o * K + k], s_dd[o], s);
            s_part[g * K + k] = s;
        }
        __syncthreads();
        if (tid < K) {
            float t = 0.f;
            for (int q = 0; q < groups; ++q) t += s_part[q * K + tid];
            s_dt[tid] = t;
        }
    } else {
        for (int k = tid; k < K; k += kBwThreads) {
            float s = 0.f;
#pragma unroll 8
            for (int o = 0; o < 9 * Ca; ++o) s = fmaf(p.w_up[(size_t)o * K + k], s_dd[o], s);
            s_dt[k] = s;
        }
    }
    __syncthreads();
    if (hidden > 0) {
        for (int m = tid; m < hidden; m += kBwThreads) {
            const float v = s_dt[m] * gelu_grad_f(s_u[m]);
            s_du[m] = v;
            p.du[(size_t)n * hidden + m] = v;
        }
        __syncthreads();
        for (int k = tid; k < Ca; k += kBwThreads) {
            float s = 0.f;
#pragma unroll 8
            for (int m = 0; m < hidden; ++m) s = fmaf(p.w_down[(size_t)m * Ca + k], s_du[m], s);
            p.dgc[(size_t)n * Ca + k] = s / hw;
        }
    } else {
        for (int k = tid; k < Ca; k += kBwThreads) p.dgc[(size_t)n * Ca + k] = s_dt[k] / hw;
    }
}

// One row of 16 lanes per result of the sums over the batch: grad_lk (sums_row) and the
// estimator's parameters (lane l adds images l, l + 16, ... in ascending order, then the
// row's lanes in lane order); the flipped LK takes one lane per element behind them.
__global__ __launch_bounds__(256) void batch_sums_kernel(const BackwardParams p, int KC, int tiles)
{
    const int Ca = p.Ca, hidden = p.hidden, K = hidden > 0 ? hidden : Ca, Ks = p.Ks;
    const size_t n_lk = (size_t)(p.lk_cstride != 0 ? Ca : 1) * Ks * Ks;
    const size_t n_wu = p.has_gen ? (size_t)9 * Ca * K : 0, n_bu = p.has_gen ? (size_t)9 * Ca : 0;
    const size_t n_wd = p.has_gen ? (size_t)hidden * Ca : 0, n_bd = p.has_gen ? (size_t)hidden : 0;
    size_t idx = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;  // uniform per row of 16 lanes
    const int l = (int)(threadIdx.x & 15);
    if (idx < n_lk) {
        sums_row(p, KC, tiles, idx, l);
        return;
    }
    idx -= n_lk;
    if (idx >= n_wu + n_bu + n_wd + n_bd) {  // the flipped large kernel: one element per lane of the rows left over
        const size_t e = (idx - (n_wu + n_bu + n_wd + n_bd)) * 16 + l;
        if (e < n_lk) {
            const size_t c = e / ((size_t)Ks * Ks), r = e % ((size_t)Ks * Ks);
            p.lkf[e] = p.lk[c * (size_t)p.lk_cstride + ((size_t)Ks * Ks - 1 - r)];
        }
        return;
    }
    // result = sum_n a[n * sa + ia] * b[n * sb + ib]   (b == nullptr: the plain sum of a)
    const float *a, *b = nullptr;
    size_t sa, ia, sb = 0, ib = 0;
    float *dst;
    if (idx < n_wu) {
        a = p.ddk, sa = (size_t)9 * Ca, ia = idx / K;
        b = p.t, sb = (size_t)K, ib = idx % K;
        dst = p.grad_w_up ? p.grad_w_up + idx : nullptr;
    } else if ((idx -= n_wu) < n_bu) {
        a = p.ddk, sa = (size_t)9 * Ca, ia = idx;
        dst = p.grad_b_up ? p.grad_b_up + idx : nullptr;
    } else if ((idx -= n_bu) < n_wd) {
        a = p.du, sa = (size_t)hidden, ia = idx / Ca;
        b = p.g, sb = (size_t)Ca, ib = idx % Ca;
        dst = p.grad_w_down ? p.grad_w_down + idx : nullptr;
    } else {
        idx -= n_wd;
        a = p.du, sa = (size_t)hidden, ia = idx;
        dst = p.grad_b_down ? p.grad_b_down + idx : nullptr;
    }
    float s = 0.f;
    for (int n = l; n < p.N; n += 16) s = b != nullptr ? fmaf(a[(size_t)n * sa + ia], b[(size_t)n * sb + ib], s) : s + a[(size_t)n * sa + ia];
    s = row16_sum(s);
    if (l == 15 && dst != nullptr) *dst = p.accumulate ? *dst + s : s;
}


}  // namespace

// the correlation of grad_out with x, tile by tile
__attribute__((visibility("hidden"))) hipError_t launch_backward_sums(const BackwardParams &p, bool bf16, hipStream_t s)
{
    if (p.Ca < 1) return hipSuccess;
    const int kc = corr_window(p.Ks), tiles = corr_tiles(p.H, p.W);
    const size_t grid = (size_t)p.N * p.Ca * tiles;
    if (grid >= ((size_t)1 << 31)) return hipErrorInvalidValue;
    BackwardParams q = p;
    q.corr_vec = (p.W % 8 == 0) && ((uintptr_t)p.x % 16 == 0) && ((uintptr_t)p.go % 16 == 0);
    return bf16 ? launch_corr_mfma_kc<bf16b>(q, kc, (unsigned)grid, s) : launch_corr_mfma_kc<float>(q, kc, (unsigned)grid, s);
}

// per image: dDK and g from the tiles' sums, the estimator forwards and backwards, the
// flipped kernels (all that the input gradient's launch needs); then the sums over the
// batch: grad_lk and the estimator's parameter gradients
__attribute__((visibility("hidden"))) hipError_t launch_backward_estimator(const BackwardParams &p, hipStream_t s)
{
    if (p.Ca < 1) return hipSuccess;
    const int kc = corr_window(p.Ks), tiles = corr_tiles(p.H, p.W);
    hipLaunchKernelGGL(estimator_image_kernel, dim3((unsigned)p.N), dim3(kBwThreads), 0, s, p, kc, tiles);
    return hipGetLastError();
}

__attribute__((visibility("hidden"))) hipError_t launch_backward_batch_sums(const BackwardParams &p, hipStream_t s)
{
    if (p.Ca < 1) return hipSuccess;
    const int kc = corr_window(p.Ks), tiles = corr_tiles(p.H, p.W);
    const size_t K = p.hidden > 0 ? (size_t)p.hidden : (size_t)p.Ca;
    const size_t rows = (size_t)(p.lk_cstride != 0 ? p.Ca : 1) * p.Ks * p.Ks +
                        (p.has_gen ? (size_t)9 * p.Ca * K + 9 * p.Ca + (size_t)p.hidden * p.Ca + p.hidden : 0);
    const size_t n_lkf = (size_t)(p.lk_cstride != 0 ? p.Ca : 1) * p.Ks * p.Ks;  // one lane per element behind the rows
    hipLaunchKernelGGL(batch_sums_kernel, dim3((unsigned)((rows * 16 + n_lkf + 255) / 256)), dim3(256), 0, s, p, kc, tiles);
    return hipGetLastError();
}

}  // namespace esc
