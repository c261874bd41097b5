// Interface between the host side (esc_api.hip) and the dense large-kernel convolution
// kernels (esc_dense.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace esc {

constexpr int kDenseMaxCa = 64;   // attention channels the dense form handles (four tiles of 16)
constexpr int kDenseMaxKs = 17;   // largest dense kernel (its halo tile and weight rows must fit in LDS)

struct DenseParams {
    const void *x;      // [N,C,H,W] storage type
    void *out;          // [N,C,H,W] storage type
    float *wt;          // weights rearranged by launch_dense_prep (workspace)
    const float *dk;    // [N,Ca,3,3] fp32 or nullptr (DK = 0)
    int N, C, Ca, H, W, Ks;
    int tiles_x, tiles_y;
    // pass-through copy: every block moves `copy_share` bytes (a multiple of 4096, or the whole
    // range by elements when copy_vec is 0) of its image's identity range [idt_off, idt_off + idt_len)
    size_t img_bytes, idt_off, idt_len, copy_share;
    int copy_vec, elem_bytes;
    // set by launch_dense: division by the halo tile's width and by its rows x width as a
    // multiply-high and a shift (the tile fill locates every element with both)
    unsigned hc_mul, hc_shift, hp_mul, hp_shift;
    // bf16 matrix path: whether the tile is fetched in 16-byte pieces
    int fill_vec;
    // bf16 matrix path, DK from the estimator: the first n_gen = N blocks finish the GAP from the pool tiles' sums
    // that launch_dense_prep leaves in pool_box (value in the low word; the high word, where the forward's
    // mailboxes carry a call's tag, says "empty") and publish DK in dk, which launch_dense_prep fills with kDkEmpty.
    // n_gen = 0: dk is there already
    int n_gen, hidden, ptiles_x, ptiles;
    float hw;
    const float *w_down, *b_down, *w_up, *b_up;
    unsigned long long *pool_box;
    unsigned *err;      // raised when the bounded wait for DK expires
};

constexpr unsigned kDkEmpty = 0xffffffffu;  // a NaN no arithmetic gives (a DK of these bits is published as another NaN)

// Does the preparing launch pool (and the main one estimate)?  The one has a block to four pool tiles, the other one more
// to an image, and a launch holds less than 2^32 threads of these kernels' 256 to a block.  Up to 2^25 tiles the first has
// at most 2^31, and its index and stride over DK stay in 32 bits together; the second is counted in its smaller tiles.
// Beyond that (2^21 images of one tile and 16 channels) DK comes from the estimator's own, resident grid, in a launch more;
// 65536 images of 8 x 8 fp32, 2^20 tiles: 2541 us so, 2902 with the estimator in front.
inline bool dense_prep_pools(int N, int Ca, int H, int W, int ptiles)
{
    const size_t tiles = (size_t)N * Ca * ptiles, blocks = (size_t)N * (1 + (size_t)((W + 31) / 32) * ((H + 3) / 4));
    return tiles < ((size_t)1 << 25) && blocks < ((size_t)1 << 24);
}

// the kernel size the device code walks: a 1 x 1 kernel is embedded in a 3 x 3 one
inline int dense_effective_ks(int Ks) { return Ks < 3 ? 3 : Ks; }

// up to 16 channels run on the 16-bit matrix instructions: bf16 storage for every kernel size,
// fp32 storage (a value as three terms, three tiles in LDS) up to 13 x 13
inline bool dense_on_bf16_mfma(int Ca, int Ks, bool bf16) { return Ca <= 16 && (bf16 || dense_effective_ks(Ks) <= 13); }

// floats the rearranged weights take: [CT chunks][Kse rows][Kse taps][CT][16 ci][16 co], or, for
// the 16-bit matrix path, [(Kse + 1) / 2 pairs of tap columns][Kse rows][64 lanes] entries of 32 bytes and, behind them, the
// weights' ranges (room for entries of 48 bytes: callers keep buffers of the size they were told)
inline size_t dense_weight_floats(int Ca, int Ks)
{
    const size_t ct = (size_t)(Ca + 15) / 16, kse = (size_t)dense_effective_ks(Ks);
    return ct == 1 ? kse * (kse + 1) * 384 : ct * kse * kse * ct * 256;
}

hipError_t launch_dense_prep(const DenseParams &p, const float *lk, bool bf16, hipStream_t s);
hipError_t launch_dense(const DenseParams &p, bool bf16, hipStream_t s);

}  // namespace esc
