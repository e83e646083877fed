// Which form of the Dense kernels a shape takes where more than one could (host arithmetic only).
#pragma once
#include <stdint.h>

namespace ivit {

// Layers without a residual that neither hold weights in registers nor are long enough for gemm_tl.hip: streamed tiles of 128 x 128 or 256 x 256
// (gemm_st.hip) or the slab of weights in LDS (gemm_i8.hip, slabs of `slab` channels), which reads activations once per slab and pads rows
// to 128 bytes.  Tiles pad the channels to 128.  us, slab and tiles: 12000 x 1040 x 400 16.9 and 12.3, 4000 x 2000 x 448 13.0 and 9.5,
// 30000 x 656 x 560 26.8 and 24.7, 12000 x 1024 x 896 22.1 and 15.7, 40000 x 2000 x 896 102 and 93, 4000 x 3008 x 1152 27.5 and 18.3.  The slab keeps
//   up to 384 bytes a row (50000 x 2000 x 272 75 and 81, 40000 x 400 x 384 17.3 and 19.2),
//   less than three quarters of a round of 128 x 128 tiles, two a CU (20000 x 208 x 1024 10.4 and 10.9),
//   64 channels and less, half of a tile (tiles / slab at K = 640, 50000 to 400000 rows: 0.97, 1.00, 1.24, 1.17, 1.15, 1.19),
//   more than four rounds, where it has the rows to use a slab many times over: N = 256, K = 400, 50000 rows 0.77, 131072 (four rounds) 0.93,
//   200000 1.22; up to 128 channels two and a half rounds, as one slab reads the rows once (N = 128, K = 400, 131072 rows 0.93, 200000 1.21),
// except that rows of more than 768 bytes have no such end (K = 1152, 200000 rows, N = 128 0.92, 256 0.95, 400 0.99, 640 1.00) if the tiles pad
// little beyond the slabs (200000 x 144 x 1152, 256 channels for 192, 1.21; 272, 384 for 288, 1.20) or those are of 64 channels, for
// longer rows (200000 x 144 x 1664 1.00, 272 0.90).
constexpr bool tiles_before_slab(int64_t M, int64_t N, int64_t K, int slab, int64_t cus) {
    if (K <= 384 || N <= 64) return false;
    const int64_t cols = (N + 127) / 128, tiles = (M + 127) / 128 * cols, slab_cols = (N + slab - 1) / slab * slab;
    if (2 * tiles < 3 * cus) return false;
    const bool any_rows = K > 768 && (4 * 128 * cols <= 5 * slab_cols || slab == 64);
    return any_rows || tiles <= (N > 128 ? 8 : 5) * cus;
}

// Rows of 768 bytes and more, more 128 x 64 tiles than CUs: at most one of 128 x 128 a CU, eight wavefronts of 64 x 32 (gemm_st.hip, launch_linear_st,
// where figures are).  Time with these tiles / with 64 x 64: where two of those a CU take the shape, whose last row of tiles is half
// empty then, K = 1536 and 2048 1.10 to 1.24, with a residual 1.26 to 1.45 (129 x 10736, 257 x 6384, 1341 x 1520; K = 768 0.99 to 1.17); at up
// to two and a half a CU 0.81 to 1.05 (K = 3072 to 768), with a residual 1.02 to 1.19 at K = 768 and 1024, 0.97 to 1.07 at 2048, 0.86 to 1.00 at 3072;
// beyond, 0.71 to 1.03 with or without one.
constexpr bool one_round_of_128(int64_t M, int64_t N, int64_t K, bool residual, int64_t cus) {
    const int64_t small = (M + 63) / 64 * ((N + 63) / 64);
    if ((M + 127) / 128 * ((N + 127) / 128) > cus || small <= 2 * cus) return false;
    return !residual || K >= 2048 || 2 * small > 5 * cus;
}

// Rows of 1024 bytes and more, more 128 x 128 tiles than CUs and at most one of 192 x 128 a CU: eight wavefronts of 96 x 32, one workgroup a
// CU (gemm_st.hip; the last step of the rule in launch_linear_st).  us, what took the shape before and this: 128 x 128 tiles 4000 x 1536 x 1024
// 11.3 and 10.5, 2500 x 2304 x 1024 10.9 and 10.0, 4000 x 1536 x 2048 19.6 and 16.2; 256 x 128 tiles of gemm_tl.hip 6272 x 768 x 3072 26.2 and
// 22.0, 8000 x 768 x 3072 26.5 and 23.6, 5000 x 1024 x 3072 27.0 and 23.2; the K-split kernel 6272 x 768 x 1536 14.3 and 11.4, 16000 x 384 x
// 1536 17.4 and 15.4.  Not for shorter rows (1576 x 3072 x 768 9.6 either way, 1970 x 2304 x 768 8.9 and 9.0), and 256 x 128 tiles for
// the next size up gain nothing (8000 x 1000 x 2048 21.1 and 21.3, 6600 x 900 x 1104 with a residual 17.1 and 18.3).
// Time with these tiles / without: 64 channels and less fill half of one and lose, K = 1024 1.07 to 1.14, 2048 1.00 to 1.07 (with a residual
// to 1.24), until rows of 2560 bytes (0.86 to 0.99, but 16 and 32 channels to 1.06; 4096 0.87 to 1.05), with a residual for more than 48
// channels (64: 0.90 to 1.05; 48: 1.02; 16: 1.09 to 1.17).  At 1024 bytes 128 x 64 tiles, which longer rows do not have then, are faster while
// two a CU take the shape (20000 x 192 1.09, with a residual 1.14; 24500 x 192 0.97 and 0.70), and from two and a half on at up to 128 channels
// without a residual (35000 x 128 0.94, 40000 1.00, 49000 1.03 to 1.06; with one 0.71, 0.75, 0.80).
constexpr bool one_round_of_192(int64_t M, int64_t N, int64_t K, bool residual, int64_t cus) {
    if (K < 1024 || (M + 127) / 128 * ((N + 127) / 128) <= cus || (M + 191) / 192 * ((N + 127) / 128) > cus) return false;
    if (N <= 64) return K >= 2560 && (!residual || N > 48);
    const int64_t tiles = (M + 127) / 128 * ((N + 63) / 64);
    return K > 1024 || (tiles > 2 * cus && (residual || N > 128 || 2 * tiles <= 5 * cus));
}

}  // namespace ivit
