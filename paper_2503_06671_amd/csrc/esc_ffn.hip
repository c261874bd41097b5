// The depth-wise branch of ConvFFN for gfx950 (MI355X): between the two point-wise layers
// of the feed-forward network that precedes every ConvAttn module (Eq. 3 line 3 of the ESC
// paper; Sec. 3 fixes the kernel size at three),
//
//     V = U + gelu(K (*) U + bk),      K depth-wise 3 x 3, zero padding, erf-form GELU.
//
// Nine multiply-adds and one GELU per element on 2 x 4 (or 2 x 2) bytes of traffic: bound by
// memory, so the kernel is laid out for 16-byte accesses, all in flight at once, and little
// else.  A thread owns a column strip one 16-byte piece wide and kFbRows rows high of one plane;
// it asks for the strip's rows and the two around it before it works on the first (left and
// right neighbours' elements come from the neighbouring pieces' cache lines).  Neighbouring
// lanes own neighbouring pieces of a row.  Nothing asks for alignment: the last piece of a row
// is its last 16 bytes, computed and stored twice with the same bits where it overlaps; rows
// shorter than a piece go element by element.  Indices are 32-bit (a thread's three 64-bit
// divisions cost as much as its arithmetic).  384 channels of 180 x 320 fp32: 38 us, 4.6 TB/s.  The
// residual step around it: 192 channels of 169 x 341 fp32 270 -> 254 us, 16 x 64 channels of
// 63 x 63 bf16 65 -> 56 us (element by element before, as every width that pieces do not divide).
// fp32 arithmetic; bf16 storage is widened exactly and rounded once at the store.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "esc_ffn.hpp"
#include "esc_gelu.hpp"

namespace esc {
namespace {

constexpr int kFbThreads = 256;
constexpr int kFbRows = 4;  // rows of a thread's strip

// two fp32 values rounded to nearest even and packed, a in the low half: the hardware's
// packed conversion (v_cvt_pk_bf16_f32)
typedef float fb_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 fb_bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t fb_pack2_bf16(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(fb_f32x2{a, b}, fb_bf16x2));
}

template <typename T>
__device__ __forceinline__ float fb_load1(const T *p)
{
    if constexpr (sizeof(T) == 4)
        return *p;
    else
        return __uint_as_float((uint32_t)*p << 16);
}

// One row of a strip as it lies in memory: the piece, the element left of it, the one right of it.
template <typename T, int PER>
struct __attribute__((packed, aligned(sizeof(T)))) FbPiece {
    T e[PER];
};
template <typename T, int PER>
struct FbRow {
    FbPiece<T, PER> piece;
    T left, right;
};

// The row, widened; zeros outside the image.
template <typename T, int PER>
__device__ __forceinline__ void fb_widen(const FbRow<T, PER> &r, bool row_in, bool left_in, bool right_in, float (&e)[PER + 2])
{
    e[0] = row_in && left_in ? fb_load1(&r.left) : 0.f;
#pragma unroll
    for (int j = 0; j < PER; ++j) e[j + 1] = row_in ? fb_load1(&r.piece.e[j]) : 0.f;
    e[PER + 1] = row_in && right_in ? fb_load1(&r.right) : 0.f;
}

template <typename T, int PER>
__global__ __launch_bounds__(kFbThreads) void ffn_branch_kernel(const FfnBranchParams p)
{
    const unsigned H = (unsigned)p.H, W = (unsigned)p.W;
    const unsigned pieces = (W + PER - 1) / PER;           // per row
    const unsigned strips = (H + kFbRows - 1) / kFbRows;   // per piece column
    const unsigned idx = blockIdx.x * kFbThreads + threadIdx.x;
    const unsigned plane_i = idx / (pieces * strips);
    if (plane_i >= (unsigned)p.planes) return;
    const unsigned rem = idx - plane_i * (pieces * strips);
    const unsigned sy = rem / pieces, px = rem - sy * pieces;
    const unsigned x0 = px + 1 < pieces ? px * PER : W - PER;
    const int y0 = (int)sy * kFbRows;
    const unsigned ch = plane_i % (unsigned)p.Ch;
    const T *up = (const T *)p.u + (size_t)plane_i * H * W;
    T *vp = (T *)p.v + (size_t)plane_i * H * W;
    const bool left_in = x0 > 0, right_in = x0 + PER < W;

    FbRow<T, PER> raw[kFbRows + 2];
#pragma unroll
    for (int r = 0; r < kFbRows + 2; ++r) {
        const int y = y0 - 1 + r;
        const T *row = up + (size_t)(y < 0 ? 0 : (y >= p.H ? p.H - 1 : y)) * W + x0;
        raw[r].piece = *reinterpret_cast<const FbPiece<T, PER> *>(row);
        raw[r].left = row[left_in ? -1 : 0];
        raw[r].right = row[right_in ? PER : PER - 1];
    }
    float k[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) k[t] = p.k[(size_t)ch * 9 + t];
    const float b = p.bk != nullptr ? p.bk[ch] : 0.f;

    float ra[PER + 2], rb[PER + 2], rc[PER + 2];
    fb_widen<T, PER>(raw[0], y0 > 0, left_in, right_in, ra);
    fb_widen<T, PER>(raw[1], true, left_in, right_in, rb);
#pragma unroll
    for (int r = 0; r < kFbRows; ++r) {
        const int y = y0 + r;
        fb_widen<T, PER>(raw[r + 2], y + 1 < p.H, left_in, right_in, rc);
        float o[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            float s = b;
            s = fmaf(k[0], ra[j], s), s = fmaf(k[1], ra[j + 1], s), s = fmaf(k[2], ra[j + 2], s);
            s = fmaf(k[3], rb[j], s), s = fmaf(k[4], rb[j + 1], s), s = fmaf(k[5], rb[j + 2], s);
            s = fmaf(k[6], rc[j], s), s = fmaf(k[7], rc[j + 1], s), s = fmaf(k[8], rc[j + 2], s);
            o[j] = rb[j + 1] + ffn_gelu(s);
        }
        if (y < p.H) {
            FbPiece<T, PER> w;
            if constexpr (sizeof(T) == 4) {
#pragma unroll
                for (int j = 0; j < PER; ++j) w.e[j] = o[j];
            } else {
#pragma unroll
                for (int j = 0; j < PER; ++j) w.e[j] = (T)fb_pack2_bf16(o[j], o[j]);
            }
            *reinterpret_cast<FbPiece<T, PER> *>(vp + (size_t)y * W + x0) = w;
        }
#pragma unroll
        for (int j = 0; j < PER + 2; ++j) ra[j] = rb[j], rb[j] = rc[j];
    }
}


// ---- the whole network in one kernel (C <= 64, Ch <= 128) --------------------------------
//
// A block streams down a strip of the image 32 columns wide (30 output columns and one
// halo column each side) over a band of rows.  Per input row y:
//   1. the row's C x 32 values are in LDS (fetched a row ahead), pixel-major: bf16 storage as
//      stored, fp32 storage as three bf16 terms each (v = t0 + t1 + t2 but for 2^-24 of it);
//   2. wavefront w forms U[32 w .. 32 w + 31][32 columns] = gelu(W1 . x + b1) with
//      v_mfma_f32_32x32x16_bf16, the row as operand A and its 32 x 64 tile of W1 as operand B,
//      held in registers.  The result puts a hidden channel in a lane; the row's columns sit in
//      LDS in the order that gives lane (channel, half) the sixteen neighbouring columns
//      16 half .. 16 half + 15 in its sixteen accumulators;
//   3. so the depth-wise branch for row y - 1 needs nothing but registers: the last three rows
//      of U are 3 x 16 registers of the lane, its channel's nine weights nine more, and the two
//      columns where the halves meet change places once per row (v_permlane32_swap);
//   4. V is rounded (bf16 storage) or taken apart into three terms (fp32 storage) and written to
//      LDS pixel-major; after the step's only barrier - both LDS tiles have two buffers -
//      wavefront w multiplies W2's rows 16 w .. 16 w + 15, in registers too, with all 128 hidden
//      channels of V (v_mfma_f32_16x16x32_bf16) and stores 30 columns of output row y - 1.  Its
//      two products hold the odd and the even columns, so a lane stores pairs of neighbours.
// fp32 storage: three terms per value and weight, the six of nine products of terms that lie
// above 2^-24 of a product; bf16 storage: the value and two terms per weight.  fp32 sums.
//
// With fp32 storage an infinite value, and one of x or a weight beyond the largest bf16, has no three
// terms (inf - inf is left for the second): its products come out NaN.  Elements of U and of out that
// do - none in an ordinary image: twelve comparisons a lane and row - are summed again in fp32, U from x
// in memory and out from V's terms in LDS, which gives what fp32 arithmetic gives - unless a NaN among
// their values or weights (the first terms tell) makes them NaN for good.  V's first term is cut off, not rounded, so that every finite V has three terms and an infinite
// first term means an infinite V.
// What bounds it: the vector instructions.  Two GELUs (ten instructions and an exponential
// each), ten for the branch and, fp32 storage, five and a half to take V apart per hidden
// element; the matrix instructions run beside them (the fp32 ones, four times as long, did not).
// U stays in registers because its way through LDS - sixteen stores and fifty-four loads a lane
// and row - cost as much as the arithmetic.  The band's first two input rows are recomputed by
// the band above (rows_per_band + 2 first-layer rows for rows_per_band output rows), the strips'
// halo columns by their neighbours (32 for 30).

typedef float f32x4s __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x2s __attribute__((ext_vector_type(2)));
typedef unsigned u32x4s __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8s __attribute__((ext_vector_type(8)));

constexpr int kFsThreads = 256;
constexpr int kFsC = 64;        // input (and output) channels the tiles hold
constexpr int kFsCh = 128;      // hidden channels the tiles hold
constexpr int kFsNp = 32;       // columns of a strip, halo included
constexpr int kFsOut = 30;      // output columns of a strip
// pitches, in bf16 elements, of 4 words mod 32: the sixteen-byte reads of eight neighbouring lanes cover all banks
constexpr int kFsXPitch = kFsC + 8;                // between two columns of an input row tile (144 bytes)
constexpr int kFsVPitch = kFsCh + 8;               // ... of V's tile (272 bytes)
constexpr int kFsXTerm = kFsNp * kFsXPitch;        // elements of one term's tile
constexpr int kFsVTerm = kFsNp * kFsVPitch;
constexpr size_t kFsLdsBytes = (size_t)2 * 3 * (kFsXTerm + kFsVTerm) * 2;  // fp32 storage: two buffers of three terms
constexpr size_t kFbLdsBytes = (size_t)2 * (kFsXTerm + kFsVTerm) * 2;
static_assert(2 * kFsLdsBytes <= 160 * 1024, "two blocks per compute unit");
constexpr unsigned kFsNowhere = 0x80000000u;       // a byte offset beyond any image: loads give 0, stores are dropped

extern __shared__ __align__(16) uint16_t fs_lds[];

// eight fp32 values as T bf16 terms each in a matrix operand's layout: every term the nearest bf16 to what
// the terms before it left
template <int T>
__device__ __forceinline__ void fs_split8(const float *v, u32x4s (&t)[T])
{
    unsigned o[T][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float a = v[2 * e], b = v[2 * e + 1];
#pragma unroll
        for (int q = 0; q < T; ++q) {
            o[q][e] = fb_pack2_bf16(a, b);
            a -= __uint_as_float(o[q][e] << 16), b -= __uint_as_float(o[q][e] & 0xffff0000u);
        }
    }
#pragma unroll
    for (int q = 0; q < T; ++q) t[q] = u32x4s{o[q][0], o[q][1], o[q][2], o[q][3]};
}

// whether one of eight first terms is NaN (which it is where the value is)
__device__ __forceinline__ bool fs_any_nan(u32x4s t)
{
    bool n = false;
    asm volatile("" : "+v"(t));  // (not to be known ahead of the rare case that asks)
#pragma unroll
    for (int e = 0; e < 4; ++e) n |= (t[e] & 0x7fffu) > 0x7f80u || (t[e] & 0x7fff0000u) > 0x7f800000u;
    return n;
}

// eight neighbouring weights of a row, zeros outside the rows x cols matrix
__device__ __forceinline__ void fs_weights8(const float *w, int row, int rows, int col, int cols, bool vec, float (&v)[8])
{
    if (vec) {  // cols % 4 == 0 on a 16-byte boundary: four weights are in or out together
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool in = row < rows && col + 4 * h < cols;
            const f32x4s r = *reinterpret_cast<const f32x4s *>(w + (in ? (size_t)row * cols + col + 4 * h : 0));
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * h + e] = in ? r[e] : 0.f;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const bool in = row < rows && col + e < cols;
            const float r = w[in ? (size_t)row * cols + col + e : 0];
            v[e] = in ? r : 0.f;
        }
    }
}

template <bool BF>
__device__ __forceinline__ void ffn_stream(const FfnStreamParams &p)
{
    constexpr int TX = BF ? 1 : 3;         // terms of a value
    constexpr int TW = BF ? 2 : 3;         // terms of a weight
    constexpr int OM = BF ? 1 : 2;         // products of terms whose orders add up to at most this
    constexpr unsigned ES = BF ? 2u : 4u;  // bytes of a stored value
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, half = lane >> 5;
    const int l16 = lane & 15, quad = lane >> 4;
    const int C = p.C, Ch = p.Ch, H = p.H, W = p.W;

    uint16_t *sX = fs_lds;                      // [2][TX][kFsNp][kFsXPitch] bf16
    uint16_t *sV = sX + 2 * TX * kFsXTerm;      // [2][TX][kFsNp][kFsVPitch] bf16

    // which strip, band and image.  Blocks are dealt to the eight dies (XCDs) in turn, each die
    // with an L2 of its own: block b works on piece (b % 8) * (grid / 8) + b / 8 of the image, so
    // that neighbouring strips and bands - which share cache lines (a strip's 128-byte row
    // segments start one column left of a 30-column boundary) and halo rows - meet in one L2
    const unsigned bq = gridDim.x / 8u, br = gridDim.x % 8u, xcd = blockIdx.x % 8u;
    const unsigned piece = xcd * bq + (xcd < br ? xcd : br) + blockIdx.x / 8u;
    const unsigned per_img = (unsigned)p.strips * (unsigned)p.bands;
    const unsigned n = piece / per_img;
    const unsigned rem = piece - n * per_img;
    const int band = (int)(rem / (unsigned)p.strips), strip = (int)(rem - (unsigned)band * (unsigned)p.strips);
    const int x0 = strip * kFsOut - 1;                    // image column of the strip's column 0
    const int y0 = band * p.rows_per_band;                // first output row
    const int steps = min(p.rows_per_band, H - y0) + 2;   // input rows, >= 3
    const unsigned row_bytes = (unsigned)W * ES, plane_bytes = (unsigned)H * row_bytes;
    const unsigned img_bytes = (unsigned)C * plane_bytes;  // < 2^31 (checked by the caller)
    const __amdgpu_buffer_rsrc_t rin =
        __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)p.x + (size_t)n * img_bytes), 0, (int)img_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rout =
        __builtin_amdgcn_make_buffer_rsrc((void *)((char *)p.out + (size_t)n * img_bytes), 0, (int)img_bytes, 0x00020000);

    // ---- this thread's share of an input row: channels 8 (tid / 32) ... + 7 of the column that row
    // tid % 32 of the first layer's product stands for (accumulator i of half h is row 8 (i / 4) + 4 h + i % 4).
    // A column or channel that does not exist has its offset beyond the image and reads as zero; a row that does
    // not exist reads as the nearest one (what comes of it is not used) ----
    const int xslot = tid & 31;
    const int xcol = x0 + 16 * ((xslot >> 2) & 1) + 4 * (xslot >> 3) + (xslot & 3);
    const int xc0 = 8 * (tid >> 5);
    unsigned xoff[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
        xoff[i] = (xcol >= 0 && xcol < W && xc0 + i < C) ? (unsigned)(xc0 + i) * plane_bytes + (unsigned)xcol * ES : kFsNowhere;
    unsigned xr[8];
    // (the loads' results are not touched until they are put into LDS a row later)
    auto fetch_row = [&](int gy) {
        const unsigned so = (unsigned)min(max(gy, 0), H - 1) * row_bytes;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (BF)
                xr[i] = (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rin, (int)xoff[i], (int)so, 0);
            else
                xr[i] = __builtin_amdgcn_raw_buffer_load_b32(rin, (int)xoff[i], (int)so, 0);
        }
    };
    auto put_row = [&](int buf) {
        u32x4s t[TX];
        if constexpr (BF) {
            t[0] = u32x4s{xr[0] | xr[1] << 16, xr[2] | xr[3] << 16, xr[4] | xr[5] << 16, xr[6] | xr[7] << 16};
        } else {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = __uint_as_float(xr[i]);
            fs_split8<TX>(v, t);
        }
        uint16_t *d = sX + buf * (TX * kFsXTerm) + xslot * kFsXPitch + xc0;
#pragma unroll
        for (int q = 0; q < TX; ++q) *reinterpret_cast<u32x4s *>(d + q * kFsXTerm) = t[q];
    };

    fetch_row(y0 - 1);  // the band's first input row travels with the weights

    // ---- weights into registers, in the matrix operands' layouts, sixteen bytes a load where they allow it.
    // first layer: lane holds W1[32 w + l32][16 c + 8 half ... + 7]; second: W2[16 w + l16][32 c + 8 quad ... + 7] ----
    u32x4s a1[4][TW], a2[4][TW];
    {
        const bool vec = C % 4 == 0 && Ch % 4 == 0 && ((uintptr_t)p.w1 | (uintptr_t)p.w2) % 16 == 0;
        float v1[4][8], v2[4][8];
#pragma unroll
        for (int c = 0; c < 4; ++c) fs_weights8(p.w1, 32 * wave + l32, Ch, 16 * c + 8 * half, C, vec, v1[c]);
#pragma unroll
        for (int c = 0; c < 4; ++c) fs_weights8(p.w2, 16 * wave + l16, C, 32 * c + 8 * quad, Ch, vec, v2[c]);
#pragma unroll
        for (int c = 0; c < 4; ++c) fs_split8<TW>(v1[c], a1[c]);
#pragma unroll
        for (int c = 0; c < 4; ++c) fs_split8<TW>(v2[c], a2[c]);
    }
    // the branch's and the first layer's other constants of this lane's hidden channel
    const int chb = 32 * wave + l32;
    float kd[9], bkd, b1d;
    {
        const bool in = chb < Ch;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const float v = p.k[in ? (size_t)chb * 9 + t : 0];
            kd[t] = in ? v : 0.f;
        }
        bkd = (in && p.bk != nullptr) ? p.bk[chb] : 0.f;
        b1d = (in && p.b1 != nullptr) ? p.b1[chb] : 0.f;
    }
    // the output channels 16 w + 4 quad ... + 3 this lane's second product holds, of columns 2 l16 + 1 and 2 l16 + 2
    const int ocol = x0 + 1 + 2 * l16;
    float b2d[4];
    unsigned ooff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int co = 16 * wave + 4 * quad + i;
        b2d[i] = (p.b2 != nullptr && co < C) ? p.b2[co] : 0.f;
        ooff[i] = (l16 < 15 && ocol < W && co < C) ? (unsigned)co * plane_bytes + (unsigned)ocol * ES : kFsNowhere;
    }
    // an even width has no pair with one column outside and, from such a base, none across a boundary of its size
    const bool pairs = W % 2 == 0 && (uintptr_t)p.out % (2 * ES) == 0;
    const bool edge = x0 < 0 || x0 + kFsNp > W;   // some of the strip's columns lie outside the image

    put_row(0);
    fetch_row(y0);
    __syncthreads();

    // first layer on input row r of the band: u[j] is column 16 half + j; u[16], u[17]: the column left of and the
    // column right of the half (used where the other half has it: the strip's outer neighbours are nobody's)
    auto first = [&](int r, float (&u)[18]) {
        const int gy = y0 - 1 + r;
        if (gy < 0 || gy >= H) {  // the branch pads U with zeros
#pragma unroll
            for (int j = 0; j < 18; ++j) u[j] = 0.f;
            return;
        }
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
        const uint16_t *ax = sX + (r & 1) * (TX * kFsXTerm) + l32 * kFsXPitch + 8 * half;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            u32x4s x[TX];
#pragma unroll
            for (int q = 0; q < TX; ++q) x[q] = *reinterpret_cast<const u32x4s *>(ax + q * kFsXTerm + 16 * c);
#pragma unroll
            for (int qw = TW - 1; qw >= 0; --qw)
#pragma unroll
                for (int qx = TX - 1; qx >= 0; --qx)
                    if (qw + qx <= OM)
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8s, x[qx]),
                                                                      __builtin_bit_cast(bf16x8s, a1[c][qw]), acc, 0, 0, 0);
        }
        if constexpr (!BF) {
            bool bad = false;
#pragma unroll
            for (int j = 0; j < 16; j += 2) bad |= __builtin_isunordered(acc[j], acc[j + 1]);
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad) != 0, 0)) {  // (see above)
                bool xn = false, wn = false;
#pragma unroll
                for (int c = 0; c < 4; ++c) xn |= fs_any_nan(*reinterpret_cast<const u32x4s *>(ax + 16 * c)), wn |= fs_any_nan(a1[c][0]);
                const uint64_t xm = __builtin_amdgcn_ballot_w64(xn), wm = __builtin_amdgcn_ballot_w64(wn);
                const unsigned slots = ~(unsigned)(xm | xm >> 32) >> 4 * half;   // columns of x without a NaN
                const bool row = chb < Ch && ((unsigned)(wm | wm >> 32) >> l32 & 1u) == 0;
                unsigned todo = 0;
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    if (chb >= Ch || (__builtin_isnan(acc[j]) && row && (slots >> (8 * (j >> 2) + (j & 3)) & 1u) != 0))
                        acc[j] = 0.f, todo |= 1u << j;
                }
                if (chb >= Ch) todo = 0;
                int gx0 = x0 + 16 * half;
                asm volatile("" : "+v"(gx0));  // (nothing of this is to be computed ahead and kept)
#pragma unroll 1
                for (int c = 0; c < C && todo != 0; ++c) {
                    const float w = p.w1[(size_t)chb * C + c];
                    const unsigned line = (unsigned)c * plane_bytes + (unsigned)gy * row_bytes;
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        if (todo >> j & 1u) {  // (what a column outside the image gives is not used)
                            const unsigned off = line + (unsigned)min(max(gx0 + j, 0), W - 1) * ES;
                            acc[j] = fmaf(__uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rin, (int)off, 0, 0)), w, acc[j]);
                            if (__builtin_isnan(acc[j])) todo &= ~(1u << j);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) u[j] = ffn_gelu(acc[j] + b1d);
        if (edge) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int gx = x0 + 16 * half + j;
                u[j] = gx >= 0 && gx < W ? u[j] : 0.f;
            }
        }
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(u[0]), __float_as_uint(u[15]), false, false);
        u[16] = __uint_as_float(sw[0]), u[17] = __uint_as_float(sw[1]);
    };
    // the branch on the middle one of three rows of U; V into its buffer.  The second layer's lane l wants columns
    // 2 l + 1 and 2 l + 2 (mod 32): column c's slot is c / 2 for odd ones, 16 + (c / 2 - 1) mod 16 for even ones
    uint16_t *const vw = sV + 8 * half * kFsVPitch + chb;
    uint16_t *const vw0 = sV + (half ? 23 : 31) * kFsVPitch + chb;
    auto branch = [&](int r, const float (&ua)[18], const float (&ub)[18], const float (&uc)[18]) {
        const int buf = (r & 1) * (TX * kFsVTerm);
#pragma unroll
        for (int j = 0; j < 16; j += 2) {
            float v[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int m = j + e, l = m == 0 ? 16 : m - 1, g = m == 15 ? 17 : m + 1;
                float s = bkd;
                s = fmaf(kd[0], ua[l], s), s = fmaf(kd[1], ua[m], s), s = fmaf(kd[2], ua[g], s);
                s = fmaf(kd[3], ub[l], s), s = fmaf(kd[4], ub[m], s), s = fmaf(kd[5], ub[g], s);
                s = fmaf(kd[6], uc[l], s), s = fmaf(kd[7], uc[m], s), s = fmaf(kd[8], uc[g], s);
                v[e] = ub[m] + ffn_gelu(s);
            }
            uint16_t *const d0 = (j == 0 ? vw0 : vw + (15 + j / 2) * kFsVPitch) + buf, *const d1 = vw + (j / 2) * kFsVPitch + buf;
#pragma unroll
            for (int q = 0; q < TX; ++q) {
                // (fp32 storage: the first term is the value's upper half, so that every finite value has its three)
                const uint32_t t = BF || q > 0 ? fb_pack2_bf16(v[0], v[1])
                                               : __builtin_amdgcn_perm(__float_as_uint(v[1]), __float_as_uint(v[0]), 0x07060302u);
                d0[q * kFsVTerm] = (uint16_t)t, d1[q * kFsVTerm] = (uint16_t)(t >> 16);
                v[0] -= __uint_as_float(t << 16), v[1] -= __uint_as_float(t & 0xffff0000u);
            }
        }
    };
    // second layer on the V of step r, output row y0 + r - 2
    auto second = [&](int r) {
        // (fp32 storage: the small products in sums of their own, so that they are not rounded at the large ones' size; the
        // bias is added to the finished sums for the same reason)
        f32x4s acc[2], low[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t] = low[t] = f32x4s{0.f, 0.f, 0.f, 0.f};
        const uint16_t *bv = sV + (r & 1) * (TX * kFsVTerm) + l16 * kFsVPitch + 8 * quad;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            u32x4s v[2][TX];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < TX; ++q)
                    v[t][q] = *reinterpret_cast<const u32x4s *>(bv + q * kFsVTerm + 16 * t * kFsVPitch + 32 * c);
#pragma unroll
            for (int qw = TW - 1; qw >= 0; --qw)
#pragma unroll
                for (int qx = TX - 1; qx >= 0; --qx)
                    if (qw + qx <= OM) {
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            f32x4s &sum = !BF && qw + qx > 0 ? low[t] : acc[t];
                            sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8s, a2[c][qw]),
                                                                          __builtin_bit_cast(bf16x8s, v[t][qx]), sum, 0, 0, 0);
                        }
                    }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if constexpr (!BF) acc[t] += low[t];
            acc[t] += f32x4s{b2d[0], b2d[1], b2d[2], b2d[3]};
        }
        if constexpr (!BF) {
            bool bad = false;
#pragma unroll
            for (int i = 0; i < 4; ++i) bad |= __builtin_isunordered(acc[0][i], acc[1][i]);
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad && l16 < 15) != 0, 0)) {  // (see above; V is in LDS, its first term alone where that is infinite)
                bool vn[2] = {false, false}, wn = false;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    wn |= fs_any_nan(a2[c][0]);
#pragma unroll
                    for (int t = 0; t < 2; ++t) vn[t] |= fs_any_nan(*reinterpret_cast<const u32x4s *>(bv + 16 * t * kFsVPitch + 32 * c));
                }
                auto fold = [](bool b) {  // of the four lanes l16, l16 + 16, ... : bit l16
                    const uint64_t m = __builtin_amdgcn_ballot_w64(b);
                    const unsigned h = (unsigned)m | (unsigned)(m >> 32);
                    return h | h >> 16;
                };
                const unsigned cols[2] = {fold(vn[0]) >> l16, fold(vn[1]) >> l16}, rows = fold(wn) >> 4 * quad;
                unsigned todo = 0;
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (__builtin_isnan(acc[t][i]) && l16 < 15 && 16 * wave + 4 * quad + i < C && ((cols[t] | rows >> i) & 1u) == 0)
                            acc[t][i] = b2d[i], todo |= 1u << (4 * t + i);
                int at = (r & 1) * (TX * kFsVTerm) + l16 * kFsVPitch, co = 16 * wave + 4 * quad;
                asm volatile("" : "+v"(at), "+v"(co));
#pragma unroll 1
                for (int ch = 0; ch < Ch && todo != 0; ++ch) {
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const uint16_t *e = sV + at + 16 * t * kFsVPitch + ch;
                        const float t0 = __uint_as_float((uint32_t)e[0] << 16), t1 = __uint_as_float((uint32_t)e[kFsVTerm] << 16);
                        const float v = __builtin_isinf(t0) ? t0 : t0 + t1 + __uint_as_float((uint32_t)e[2 * kFsVTerm] << 16);
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (todo >> (4 * t + i) & 1u) {
                                acc[t][i] = fmaf(p.w2[(size_t)(co + i) * Ch + ch], v, acc[t][i]);
                                if (__builtin_isnan(acc[t][i])) todo &= ~(1u << (4 * t + i));
                            }
                    }
                }
            }
        }
        // (pieces of 60 bytes: half lines, which bf16 storage's L2 puts together - step 360 x 640 90.3 -> 88.9 us - and fp32's
        // streams past it - step 180 x 320 57.0 -> 55.8)
        constexpr int kAux = BF ? 0 : 2 /* non-temporal */;
        // (the same for all lanes, which the compiler must see: otherwise every store is a loop over the lanes' offsets)
        const int so = __builtin_amdgcn_readfirstlane((int)((unsigned)(y0 + r - 2) * row_bytes));
        if (pairs) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (BF)
                    __builtin_amdgcn_raw_buffer_store_b32(fb_pack2_bf16(acc[0][i], acc[1][i]), rout, (int)ooff[i], so, kAux);
                else
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2s{__float_as_uint(acc[0][i]), __float_as_uint(acc[1][i])}, rout,
                                                          (int)ooff[i], so, kAux);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned off1 = ocol + 1 < W ? ooff[i] + ES : kFsNowhere;
                if constexpr (BF) {
                    const uint32_t o = fb_pack2_bf16(acc[0][i], acc[1][i]);
                    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)o, rout, (int)ooff[i], so, kAux);
                    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(o >> 16), rout, (int)off1, so, kAux);
                } else {
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[0][i]), rout, (int)ooff[i], so, kAux);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[1][i]), rout, (int)off1, so, kAux);
                }
            }
        }
    };
    // one input row: the next one into the other buffer (whose readers are behind the last barrier) and the one after
    // it asked for, first layer, and from the third row on branch and second layer for the row above
    auto next_row = [&](int r) {
        if (r + 1 < steps) {
            put_row((r + 1) & 1);
            if (r + 2 < steps) fetch_row(y0 + 1 + r);
        }
    };
    auto step = [&](int r, const float (&ua)[18], const float (&ub)[18], float (&uc)[18]) {
        next_row(r);
        first(r, uc);
        branch(r, ua, ub, uc);
        __syncthreads();  // V of all hidden channels and the next input row are in LDS
        second(r);
    };
    float u0[18], u1[18], u2[18];
    next_row(0);
    first(0, u0);
    __syncthreads();
    next_row(1);
    first(1, u1);
    __syncthreads();
    // three copies of the step, the three rows of U in three sets of registers that take turns
    for (int r = 2;; r += 3) {
        step(r, u0, u1, u2);
        if (r + 1 >= steps) break;
        step(r + 1, u1, u2, u0);
        if (r + 2 >= steps) break;
        step(r + 2, u2, u0, u1);
        if (r + 3 >= steps) break;
    }
}

__global__ __launch_bounds__(kFsThreads, 2) void ffn_stream_kernel(const FfnStreamParams p) { ffn_stream<false>(p); }

__global__ __launch_bounds__(kFsThreads, 2) void ffn_stream_bf16_kernel(const FfnStreamParams p) { ffn_stream<true>(p); }

}  // namespace

__attribute__((visibility("hidden"))) hipError_t launch_ffn_branch(const FfnBranchParams &p, bool bf16, hipStream_t s)
{
    if (p.planes < 1 || p.H < 1 || p.W < 1 || p.Ch < 1) return hipSuccess;
    // 16-byte pieces wherever a row holds one (element by element an odd width costs 8 us of 65, see above)
    const int per = bf16 ? (p.W >= 8 ? 8 : 1) : (p.W >= 4 ? 4 : 1);
    const long per_plane = (long)((p.W + per - 1) / per) * ((p.H + kFbRows - 1) / kFbRows);
    // the kernel's indices are 32-bit: whole images to a launch, as many as fit (an image of U is < 2 GiB, so one does)
    const long images = p.planes / p.Ch;
    long fit = ((1L << 32) - 2 * kFbThreads) / (per_plane * p.Ch);
    if (fit < 1) return hipErrorInvalidValue;
    for (long n = 0; n < images; n += fit) {
        FfnBranchParams q = p;
        const size_t off = (size_t)n * p.Ch * p.H * p.W * (bf16 ? 2 : 4);
        q.u = (const char *)p.u + off;
        q.v = (char *)p.v + off;
        q.planes = (n + fit < images ? fit : images - n) * p.Ch;
        const dim3 grid((unsigned)((per_plane * q.planes + kFbThreads - 1) / kFbThreads)), block(kFbThreads);
        if (bf16) {
            if (per == 8)
                hipLaunchKernelGGL((ffn_branch_kernel<uint16_t, 8>), grid, block, 0, s, q);
            else
                hipLaunchKernelGGL((ffn_branch_kernel<uint16_t, 1>), grid, block, 0, s, q);
        } else {
            if (per == 4)
                hipLaunchKernelGGL((ffn_branch_kernel<float, 4>), grid, block, 0, s, q);
            else
                hipLaunchKernelGGL((ffn_branch_kernel<float, 1>), grid, block, 0, s, q);
        }
    }
    return hipGetLastError();
}

__attribute__((visibility("hidden"))) hipError_t launch_ffn_stream(const FfnStreamParams &p, hipStream_t s)
{
    if (p.N < 1 || p.C < 1 || p.H < 1 || p.W < 1 || p.Ch < 1) return hipSuccess;
    if (p.C > kFsC || p.Ch > kFsCh) return hipErrorNotSupported;
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return hipErrorInvalidDevice;
        cus = n > 0 ? n : 1;
    }
    static bool lds_granted = false;
    if (!lds_granted) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(ffn_stream_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFsLdsBytes);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(ffn_stream_bf16_kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFbLdsBytes);
        if (e != hipSuccess) return e;
        lds_granted = true;
    }
    FfnStreamParams q = p;
    q.strips = (p.W + kFsOut - 1) / kFsOut;
    // Which problems take one launch (C = 64, Ch = 128, the residual step around it; three launches -> one):
    //  * small ones, whose four-row bands fit on the chip in one round, at widths that fill at least half of their
    //    strips and nearly all of the kernel's channels (it always works for 64 and 128: with 32 and 64 the three
    //    launches are as fast).  64 x 64 fp32 38 -> 27 us, bf16 34 -> 24; 135 x 240 50 -> 43, 43 -> 36; 8 x 64 x 64
    //    50 -> 46, 42 -> 37; 2000 x 8, a quarter of a strip: 50 -> 53.
    //  * large ones at widths that fill at least four fifths of their strips: a last strip that is mostly empty costs
    //    as much as a full one (180 x 320 fp32 68 -> 50, 16 x 72 x 72 107 -> 86; 32 x 64 x 64 bf16, whose 64
    //    columns are 30 + 30 + 4: 72 -> 74).
    const long quads = (long)p.N * q.strips * ((p.H + 3) / 4), width = (long)q.strips * kFsOut;
    const bool small = quads <= 2L * cus && 2L * p.W >= width && 4L * p.C * p.Ch >= 3L * kFsC * kFsCh;
    const bool large = 2 * quads >= 3L * cus && 5L * p.W >= 4 * width;
    if (!small && !large) return hipErrorNotSupported;
    // the band height that needs the fewest row steps one after the other: a block takes its rows + 2
    // steps and about a step and a half to get its weights; the blocks run in rounds of two per compute unit.
    // Bands of less than four rows where they leave half of the compute units to a single block (64 x 64 fp32:
    // one row 27 us, two 30, four 35; 135 x 240: 360 blocks of three rows 43, 272 of four 47; 8 x 64 x 64: 528 of three
    // 47, 384 of four 46)
    q.rows_per_band = 4;
    double best = 0.0;
    for (int rb : {4, 1, 2, 3, 8, 16, 32}) {
        const long blocks = (long)p.N * q.strips * ((p.H + rb - 1) / rb);
        if (rb < 4 && (!small || 2 * blocks > 3L * cus)) continue;
        const long rounds = (blocks + 2L * cus - 1) / (2L * cus);
        const double cost = (double)rounds * (rb + 3.5);
        if (rb == 4 || cost < best) {
            best = cost;
            q.rows_per_band = rb;
        }
    }
    q.bands = (p.H + q.rows_per_band - 1) / q.rows_per_band;
    const long grid = (long)p.N * q.strips * q.bands;
    if (grid >= (1L << 31)) return hipErrorNotSupported;
    if (p.bf16)
        hipLaunchKernelGGL(ffn_stream_bf16_kernel, dim3((unsigned)grid), dim3(kFsThreads), kFbLdsBytes, s, q);
    else
        hipLaunchKernelGGL(ffn_stream_kernel, dim3((unsigned)grid), dim3(kFsThreads), kFsLdsBytes, s, q);
    return hipGetLastError();
}

}  // namespace esc
