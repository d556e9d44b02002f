// Which tile a product of the encoder goes through.  Host code without HIP types.
#pragma once
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

constexpr int GEMM_BK = 32;  // gemm_kernel's K-slab

// How gemm_stream_kernel's grid covers the 8 XCDs: xr of them side by side over the rows, the rest over the columns.  First
// the arrangement with the fewest rounds of blocks on the fullest XCD, among those the one that reads least (an XCD
// reads its share of the rows of A and of W once).
struct StreamPlan {
    int xr, rounds;
};

inline StreamPlan plan_stream(int cus, int tile_rows, int tile_cols, int rows, int N)
{
    StreamPlan best = {1, INT_MAX};
    double best_bytes = 0;
    const int rt = (rows + tile_rows - 1) / tile_rows, ct = (N + tile_cols - 1) / tile_cols;
    const int per_xcd_cus = std::max(1, cus / 8);
    for (int xr = 1; xr <= 8; xr *= 2) {
        const int xc = 8 / xr;
        const int per_xcd = ((ct + xc - 1) / xc) * ((rt + xr - 1) / xr);
        const int rounds = (per_xcd + per_xcd_cus - 1) / per_xcd_cus;
        const double bytes = (double)rows * xc + (double)N * xr;
        if (rounds < best.rounds || (rounds == best.rounds && bytes < best_bytes)) {
            best = {xr, rounds};
            best_bytes = bytes;
        }
    }
    return best;
}

// Tiles of the stream kernels (width, blocks of rows, wavefronts) and what a launch takes while its blocks fit the chip at once:
// microseconds besides the K loop and per 768 elements of K.
#define LEANN_STREAM_TILES(X)                                                                            \
    X(16, 2, 1, 1.85, 0.85) X(16, 2, 2, 2.25, 0.92) X(16, 2, 3, 2.35, 1.08) X(16, 2, 4, 2.2, 1.3) X(32, 1, 3, 2.5, 1.68) X(32, 1, 4, 2.55, 2.1) \
    X(16, 4, 4, 2.65, 1.75) X(32, 2, 3, 3.2, 2.25) X(32, 2, 4, 3.2, 2.65) X(32, 2, 6, 3.3, 4.15) X(32, 2, 8, 3.4, 5.0) X(32, 4, 6, 4.6, 7.4)   \
    X(32, 4, 8, 4.9, 8.8)

struct GemmChoice {
    int stream;  // number of the stream tile, -1: gemm_kernel
    int xr;      // the stream kernel's grid, see plan_stream
    int large;   // rows of a tile of gemm_kernel (128) or gemm_large_kernel (256)
    int cols;    // its columns
};

// Tile choice of one product.  All tiles add the K-slabs in the same order, so a row's result does not depend on it.
// Measured per launch in a row of dependent launches, W of twelve layers in turn, in microseconds (rows x N x K; "16:" tiles of
// gemm_stream16_kernel, then those of gemm_stream_kernel, behind the bar gemm_kernel's):
//                   16: 32x16   32x32   32x48   32x64   64x64 |   32x96  32x128   64x96  64x128  64x192  64x256 128x192 128x256 | 128x128
//    80 x  768 x  768     2.7     2.8     3.0     3.1     4.0 |     3.6     4.0     4.6     4.9                                 |    8.6
//    80 x  768 x 3072     5.2     5.6     6.2     7.1     9.1 |     8.6    10.6    11.2    12.9                                 |   26.1
//   244 x 2304 x  768                                     4.4 |     4.2     4.6     5.0     5.3     6.3     7.0                 |
//   244 x  768 x 3072             5.8     6.6     7.2     9.2 |     8.8    10.7    11.3    13.0                                 |
//   450 x 2304 x  768                                         |                     5.5     5.9     6.8     7.2                 |    9.8
//   450 x  768 x 3072                     7.1     7.2     9.2 |     8.9    10.7    11.3    12.9                                 |
//  1040 x  768 x  768                                     4.7 |             4.9     5.2     5.4     6.5                         |    9.1
//  1040 x  768 x 3072                                    10.1 |            12.0    11.9    13.4    17.2                         |
//  1040 x 2304 x  768                                         |                                     7.4     7.9    10.7         |   10.7
//  2000 x 3072 x  768                                         |                                    14.6    15.8    13.4    14.1 |   19.0
//  2500 x 1152 x  384                                         |                                     5.7     5.9     7.8     8.2 |    6.6
//  3500 x 1152 x  384                                         |                                     9.4     9.9     8.1     8.6 |    6.9
//  3500 x 3072 x  768                                         |                                                    23.6    25.1 |   28.3
//  8000 x  768 x 3072                                         |                                    42.7    47.1    37.0    37.5 |   51.2
// 10000 x  384 x 1536                                         |                                    21.5    23.9    17.5    18.5 |   18.9
// 12000 x  768 x  768                                         |                                                    22.3    24.3 |   23.7
// The smallest stream tile that needs one round of blocks is the fastest (in a second round nothing hides the first operands' way).
// Tiles of gemm_stream16_kernel with the columns of 32x96 and 32x128 were no faster than those (4.3 and 4.8 where these take 4.2
// and 4.6).  32x128 is for K = 128: the FFN's first product at hidden 128, 1320 to 2000 x 512 x 128, takes 0.1 to 0.3 us longer through 64x64.
// gemm_kernel (128x128) and gemm_large_kernel (256x256, and 256x192 for what those leave of the chip or of the columns) walk over their tiles:
// what decides is how many the busiest CU gets, c = ceil(tiles / CUs), and what one takes.  By 768 elements of K, 256x256 takes 4.8 + 16 k, 256x192
// 4.35 + 12.7 k and 128x128 7 k (3 more for each 768 beyond the first), with 2.45 per launch and, where c > 1, 0.135 per MB of A.  In a row of launches, whose A
// never leaves the caches, 128x128 takes 1 + c (1.2 + 6.4 k); its figures are of launches behind the kernels of a pass, which read what those have just
// written past the caches: least squares of 340 of them, on the scale of the stream tiles' figures, are 2.3 + c (0.6 + 6.6 k) + 0.13 per MB, and near
// these the values were taken whose choices lose least, in the 340 and in whole passes of 384 and 768 columns with one product's tile exchanged.
// Microseconds in a pass (chunks of 76 tokens, five eighths full; "s": the fastest stream tile):
//                        128x128 256x256 256x192     s |                       128x128 256x256 256x192     s
//   6900 x  384 x  128       5.9                   7.0 |  6900 x 1152 x  384      11.3    13.4    12.4  13.8
//  13000 x  512 x  128 G     8.6                  12.3 | 13000 x 1536 x  384 G    25.7    32.4    28.3  31.5
//   6900 x  768 x  256       8.5    10.4    10.2   8.6 | 19000 x  384 x  384      14.5    13.9    12.7  16.1
//   6900 x 1024 x  256 G    10.5    16.0    14.5  12.9 | 38000 x  384 x  384      25.7    25.3    26.2
//   9500 x  384 x 1536      23.0    29.4    28.0  17.8 | 38000 x  384 x 1536      79.7    66.8    62.4
//  25500 x  768 x  256      16.8    19.7    22.5       | 13000 x  768 x  768      30.4    21.8    19.9  26.8
//   3600 x  768 x 3072      40.5    56.0    51.6  22.4 |  3600 x 2304 x  768      21.9    19.8    18.2  20.4
//   6900 x  768 x 3072      67.7    58.4    53.7  36.1 |  6900 x  768 x  768      19.9    18.9    17.0  14.2
//   9500 x  768 x 3072      70.1    59.8    55.6  43.2 |  9500 x  768 x  768      21.1    20.0    18.2  17.2
//  13000 x  768 x 3072     101.8    63.0    57.6  69.5 |  6900 x 3072 x  768 G    49.5    46.1    41.5  49.2
// Over the 340 (K 128 to 4096, 1000 to 100 000 rows) the tile taken is 1.1 % slower than the fastest on average; with 1 + c (0.4 + 9.02 k) for 128x128 1.6 %;
// with 1 + c (2 + 9.2 k), which two products of K = 384 and 1536 suggest, 2.5 %: it leaves 128x128 for stream tiles at K of 128 and 256.  Whole passes
// with the first of these two and now: 384 columns, 6700 tokens 814 and 791 us, 11 600 1229 and 1148, 12 900 1266 and 1191; 256 columns, 20 200 tokens 1208 and 1079.
// Slower than before by 1 to 2 %: 256 columns at 3000 tokens.
// In a row of launches, all three measured (rows x N x K; "G": with GELU):
//                        128x128 256x256 256x192 |                       128x128 256x256 256x192
//   5000 x 2304 x  768      25.1    22.7    22.2 |  8000 x  384 x  384       6.7    12.3    10.4
//  12000 x 2304 x  768      54.6    48.9    52.6 | 20000 x 1152 x  384      26.5    24.6    22.9
//  25500 x  768 x  768      38.0    38.6    34.9 | 37000 x  384 x  384      18.9    23.5    20.4
//  25500 x  768 x 3072     132.6   120.8   101.5 | 37000 x 1152 x  384      45.1    37.2    41.1
//  37000 x  768 x  768      52.9    42.1    48.1 | 48000 x  384 x 1536      68.5    65.3    54.9
//  37000 x  768 x 3072     187.6   135.2   151.4 | 65536 x  384 x  384      28.3    27.8    28.1
//  37000 x 3072 x  768 G   226.8   181.3   204.7 | 65536 x 1536 x  384 G   118.1   112.9   121.9
//
// rows: that the product is expected to have; large_tile, small_rows: see leann_set_gemm_tiles (0 also: no packed weights).
inline GemmChoice choose_gemm(int cus, int large_tile, int small_rows, int rows, int N, int K)
{
    auto busiest = [&](int tile_rows, int tile_cols) {  // tiles of the busiest CU
        const int64_t tiles = (int64_t)((rows + tile_rows - 1) / tile_rows) * ((N + tile_cols - 1) / tile_cols);
        return (double)((tiles + cus - 1) / cus);
    };
    const double k = K / 768.0;
    GemmChoice best = {-1, 1, 128, 128};
    const double c128 = busiest(128, 128);
    double best_us = 2.45 + c128 * (7.03 * k + 3.0 * std::max(0.0, k - 1.0)) + (c128 > 1 ? 0.135e-6 * sizeof(uint16_t) * rows * K : 0.0);
    if (large_tile == 256 && K >= 8 * GEMM_BK) {
        const double us256 = busiest(256, 256) * (4.8 + 16.0 * k), us192 = busiest(256, 192) * (4.35 + 12.7 * k), us = std::min(us256, us192);
        if (us <= best_us) {
            best_us = us;
            best.large = 256;
            best.cols = us192 < us256 ? 192 : 256;
        }
    }
    if (small_rows <= 0) return best;
    int tile = 0;
#define LEANN_TILE(W, R, NM, US, US_K)                                                                                \
    {                                                                                                                 \
        const StreamPlan p = plan_stream(cus, W * R, W * NM, rows, N);                                                \
        const double us = US + US_K * k;                                                                              \
        if (p.rounds == 1 && us < best_us && (W * R * W * NM > 4096 || rows <= small_rows)) {                         \
            best_us = us;                                                                                             \
            best.stream = tile;                                                                                       \
            best.xr = p.xr;                                                                                           \
        }                                                                                                             \
        ++tile;                                                                                                       \
    }
    LEANN_STREAM_TILES(LEANN_TILE)
#undef LEANN_TILE
    return best;
}

// Padded rows above which a pass whose caller does not know its tokens asks the device for their number before it chooses
// tiles (four layers of 768: 48 x 256 tokens, all valid, 1237 us with tiles for five eighths of them, 1159 us asked; 24 x 256, a
// quarter valid, 456 and 345; five eighths valid, 4 us are lost to the wait).  Below, the wrong tile costs no more than the
// wait: 17 x 128, all valid, 436 us guessed, 448 asked.
constexpr int ASK_ROWS = 4096;

// Rows that a smaller one of those is taken to hold: chunks are five eighths full.
inline int guessed_rows(int max_rows) { return (int)(((int64_t)max_rows * 5 + 7) / 8); }
