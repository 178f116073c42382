// Internal: host-side launch interface of the GEMM + LeakyReLU kernels (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>

struct GemmLaunch {
    const void* a;
    const void* b;
    void* c;
    int batch, M, N, K;
    float slope;
    int dtype;     // 0 binary16, 1 bfloat16
    void* stream;
};

// Pieces of t that cover x, for any x >= 0 (as int, x + t - 1 would overflow where x is near 2^31).
constexpr int gemm_pieces(int x, int t) { return (int)(((unsigned)x + (unsigned)(t - 1)) / (unsigned)t); }

// 128 x 128 with fewer than 192 of them, too?  Where tiles of 64 x 128 (below) would begin a second round, 64 x 64 tiles are more than two
// to a compute unit (512), and K is long enough (us with 128 and 64, 140 to 191 of them: 1536 x 1536, K = 4096 32 50; 1599 x 1696, K = 1408 14.7
// 20.4; 2 x 3476 x 288, K = 560 9.5 11.1; 2370 x 1216, K = 384 7.3 7.9; 4 x 576 x 904, K = 512 8.2 10.9; 4 x 846 x 576, K = 384, 140 of
// them, 6.7 5.5; 4 x 324 x 1408, K = 448, 132, 7.2 6.9; 2761 x 704, K = 608, 132, 8.6 7.3).  Up to 512 of 64 x 64 only for a long K, sooner where rows of b do not
// begin at cache lines (6395 x 264, K = 2048, 500 of 64 x 64, 18.5 19.7; 4224 x 440, K = 1344, 462, 14.3 15.1; 2 x 2784 x 288, K = 1440, 440, 15.8 14.6; 5952 x
// 264, K = 704, 465, 10.4 9.8; but 2 x 2176 x 448, K = 1024 12.7 11.4; 5952 x 320, K = 1024 12.7 11.3; 2 x 1728 x 576, K = 2048 19.3 18.1; 4 x 704 x
// 704, K = 3368 28.6 31.8, but 2 x 2171 x 448, K = 3616 30.9 27.5).  Not where a quarter more of them lies outside c (8 x 556 x 448, K = 1536 14.9 13.7; 8 x 398 x 544, K = 1560 16.5 15.7.)
inline bool gemm_middle_round(int batch, int M, int N, int K) {
    auto tiles = [&](int bm, int bn) { return (long long)batch * gemm_pieces(M, bm) * gemm_pieces(N, bn); };
    const long long t64 = tiles(64, 64), t128 = tiles(128, 128);
    if (K < 384 || tiles(64, 128) <= 256 || 16 * t128 > 5 * t64) return false;
    return t64 > 512 ? K >= 640 || t128 >= 152 : K >= (t64 > 448 && N % 64 != 0 ? 1200 : 3000);
}

// Tiles of c for a problem whose rows are 16-byte aligned: 1: 256 x 256, 2: 128 x 128, 3: 64 x 64, 5: 32 x 32 with K
// split over the wavefronts of a workgroup.  The largest tile that still gives three quarters of the 256 compute units
// a workgroup, and that is not more than half empty: a tile costs the same however little of it lies inside c (us with 256,
// 128, 64: 1024 x 8 x 64, K = 40, 30 8.8 5.1; 4096 x 16 x 16, K = 64, 95 28 12; 262144 x 64, K = 64, 30 20 15; 262144 x 128, K = 64, 37
// 27 35; K = 2048 the same way).  Except few rows with a long K, where what counts is how often a is read, once per column of
// tiles (us with 128 and 64: 4 x 64 x 8192, K = 512 9.5 9.1, 1024 14.6 15.0, 4096 54 69; 232 x 33 x 232, K = 1024 29 33).  A problem that fits the chip in one round of 32 x 32 tiles and has a K worth splitting
// takes those.
// And 256 x 256 already where 128 x 128 tiles would begin a second round of the chip (two to a compute unit, 512) and K is
// long enough to matter (us with 128 and 256: 2816 x 3072, K = 1024, 528 of them, 29.0 26.1; 3072 x 3072, K = 2048, 50 43, K = 4096, 93 75; 2 x 2048 x 2304, K =
// 3000, 86 66; but 4096 x 2048, K = 1024, 512 of them, 22.9 25.5; 3072 x 3584, K = 256, 14.0 14.4).
#ifndef GEMM_SK_TILES
#define GEMM_SK_TILES 256
#endif
inline int gemm_tile_of(int batch, int M, int N, int K) {
    auto tiles = [&](int t) { return (long long)batch * gemm_pieces(M, t) * gemm_pieces(N, t); };
    if (tiles(32) <= GEMM_SK_TILES && K >= 256) return 5;
    const int largest = N <= 64 || (M <= 64 && K < 768) ? 64 : N <= 128 || M <= 128 ? 128 : 256;
    return largest == 256 && (tiles(256) >= 192 || (tiles(128) > 512 && K >= 512)) ? 1 : largest >= 128 && (tiles(128) >= 192 || gemm_middle_round(batch, M, N, K)) ? 2 : 3;
}

// The loads of a tile, not its matrix instructions, are what most problems of one or two rounds of the chip wait for: a compute unit
// takes 16 bytes per lane into LDS at 35 to 60 bytes per cycle, half of that where the rows are short and not aligned to cache lines (measured
// with the loads alone).  So: as few bytes as possible for a round, and rows of a in pieces of 128 bytes (blocks of 64 in K) where
// they start at multiples of that.

// Instead of 128 x 128: 128 x 256 with eight wavefronts, where the first begin a second round and the second do not?  (us with 128 x 128 and 128 x
// 256: 3072 x 1536, K = 3072 50 40; 2 x 2048 x 2048, K = 1000 26 23; 2703 x 2432, K = 448 12.3 11.6; 4 x 522 x 2784, K = 416 11.7 11.1; 3770 x
// 864 x 2, K = 480 13.1 12.2.  Short sums are start and end: 2 x 1292 x 3680, K = 96 10.8 12.3.  A
// single column of them, where nobody shares rows of a, pays for a larger part of the second round only: 8 x 2297 x 256, K = 3200, 288 of 128 x 128, 53 61; 4 x 4271 x
// 256, K = 2400, 272, 42 45; 8 x 2531 x 256, K = 2816, 320, 0.84 of the time.)
inline bool gemm_tiles_128x256(int batch, int M, int N, int K) {
    const long long columns = (long long)batch * gemm_pieces(M, 128);
    return N > 128 && K >= 384 && columns * gemm_pieces(N, 128) > (N > 256 ? 256 : 300) && columns * gemm_pieces(N, 256) <= 256;
}

// 128 x 128 in one round: eight wavefronts in two parts, each with half of every block of 64 in K, instead of four with blocks of 32?  The
// parts' sums are added at the end, worth it for a long K (us with four and eight: 2 x 3374 x 384, K = 3328 30.5 25.4; 3978 x 216 x 4, K =
// 2896 48.6 42.0; 3000 x 1024, K = 2040 23.3 20.6; 2644 x 1440, K = 1472 17.0 16.2; 2285 x 1280, K = 1248 14.1 15.1).  Not for odd multiples of 32,
// whose last block is half empty (4 x 224 x 3168, K = 1312 14.6 15.5; 4 x 1912 x 512, K = 3872 34.2 35.9).
inline bool gemm_two_parts(int batch, int M, int N, int K) {
    return (long long)batch * gemm_pieces(M, 128) * gemm_pieces(N, 128) <= 256 && K >= 1280 && K % 64 != 32;
}

// Instead of 64 x 64: 64 x 128, blocks of 64 in K, where the first begin a second round and the second do not (gemm_tile_of takes 128 x
// 128 where they would, from K = 640 on)?  (us with 64 x 64 and 64 x 128: 2 x 777 x 1000, K = 1000 13.2 10.4; 1304 x 1304, K = 1304 16.5 12.5; 2107 x 720, K =
// 2968 31.7 21.2; 2 x 338 x 2688, K = 640 7.8 7.1; 456 x 2304, K = 576 5.9 6.2; 4 x 594 x 416, K = 512 5.5 5.9;
// 802 x 1536, K = 608, whose last block is half empty, 6.7 7.1.)  Where it takes three columns for five and the like, only for a long K (N = 320: 4071, K = 704 6.3
// 6.8; 8 x 431, K = 2016 11.5 13.7; 4 x 1272 x 312, K = 3968 0.73 of the time; N = 152, K = 1848 0.77).
inline bool gemm_tiles_64x128(int batch, int M, int N, int K) {
    const long long columns = (long long)batch * gemm_pieces(M, 64);
    if (N > 192 && 12 * gemm_pieces(N, 128) > 7 * gemm_pieces(N, 64) && K < 2560) return false;
    return N > 64 && (M > 64 || K >= 768) && K >= (K % 64 == 32 ? 800 : 600) && columns * gemm_pieces(N, 64) > 256 && columns * gemm_pieces(N, 128) <= 256;
}

// 64 x 64 with at most one tile per compute unit: five stages of 64 in K instead of six of 32?  (us with 32 and 64: 512 x 1024, K =
// 4096 18.1 14.9; 4 x 512 x 512, K = 2048 11.6 9.7; 4 x 242 x 832, K = 3328 14.2 12.6; 1024 x 1024, K = 1024 7.4 6.8; 248 x 2688, K = 640 4.8
// 4.7.  K not a multiple of 64 gains nothing: 896 x 424, K = 1712, and 1724 x 160, K = 3600, 1.00; 1100 x 640, K = 928 6.1 6.6.)
inline bool gemm_long_blocks(int batch, int M, int N, int K) {
    return K >= 640 && K % 64 == 0 && (long long)batch * gemm_pieces(M, 64) * gemm_pieces(N, 64) <= 256;
}

// 64 x 64 tiles: six LDS stages instead of four?  A block is two matrix instructions per wavefront, so the loads' latency
// shows where K is long (us with four and six: 1000 x 1000 x 2048 15.7 12.5, 4 x 512 x 512 x 2048 14.5 11.2, 300 x 1400 x 640 5.8
// 5.4); with a short K the loads that run ahead are waste and the larger LDS leaves fewer workgroups on a compute unit (1024 x 64
// x 64, K = 64, 6.7 7.8; 32768 x 64 x 384 7.6 8.1; 1000 x 1000 x 128 3.67 3.75).  Between, operands that an XCD's L2 does not
// hold, with at most one workgroup per compute unit, want the depth too (64 x 9000 x 320 4.8 4.4).
inline bool gemm_deep(int batch, int M, int N, int K) {
    if (K >= 640) return true;
    const long long tiles = (long long)batch * gemm_pieces(M, 64) * gemm_pieces(N, 64), bytes = 2LL * batch * ((long long)M * K + (long long)K * N);
    return K >= 288 && tiles <= 256 && bytes > (4 << 20);
}

// 256 x 256 tiles: eight wavefronts of 64 x 128 instead of four of 128 x 128?  Two wavefronts per SIMD start, read and write a
// tile faster than one, which shows where there are few blocks of K and either fewer tiles than compute units, all whole, or a
// single whole column of them (us with eight and four, K = 64: 3584 x 3584 10.6 11.5, 3 x 2048 x 2048 10.5 11.1, 524288 x 256 79
// 87; K = 32: 9.9 10.6, 9.8 10.3, 69 67; 90000 x 256, K = 32 16.2 17.2).  4096 x 4096, K = 64: 12.0 11.6; 27134 x 480, K = 40 12.6 11.9.
// Up to four blocks of K where at least a sixth of the compute units has no tile (K = 96: 3584 x 3584 11.4 12.2, 256 x 49152 11.3 12.4;
// K = 128: 12.1 12.7, 11.9 12.8, 1536 x 8192 12.3 12.1; with 240 tiles, 3840 x 4096, 13.2 12.8), eight in a single row of them
// (256 x 52224, K = 224: 14.1 14.9).
// And in a single column of tiles with a long K, whole in M, where the launch waits for rows of a from memory and not for the matrix
// instructions (65536 x 256, K = 1536 62.5 63.8, 2048 90 96, 8192 305 344; 131072 x 256, K = 8192 561 609; 65536 x 136, K = 3072
// 107 110; but K = 1280: 51.0 51.1, 57000 x 136, K = 4096 130 122, 200 x 256 x 256, K = 4096 174 172, 262144 x 200, K = 2048 295 279).
inline bool gemm_eight_waves(int batch, int M, int N, int K) {
    const long long tiles = (long long)batch * gemm_pieces(M, 256) * gemm_pieces(N, 256);
    if (N <= 256 && M >= 1024 && M % 256 == 0 && K >= 1536 && K % 32 == 0) return tiles <= 512;
    if (N % 256 != 0) return false;
    if (K > 64) return tiles <= 208 && M % 256 == 0 && K <= (M == 256 ? 256 : 128);
    return N == 256 ? K == 64 || (K == 32 && tiles <= 448) : tiles < 256 && M % 256 == 0;
}

// Do the rows of a and b start at 16-byte aligned addresses (and stay within 32-bit offsets inside a tile)?  Then
// blocks of K go straight from global memory into LDS.
inline bool gemm_rows_aligned(int N, int K) { return K > 0 && K % 8 == 0 && N % 8 == 0 && K <= (1 << 22) && N <= (1 << 22); }

// Rows that are not aligned: 64 x 64 tiles by way of registers instead of 32 x 32 with K split over the wavefronts?  Where the second are more
// than two to a compute unit, a little later for a long K, which they split (us with 32 and 64: 1049 x 565, K = 76 6.5 4.6; 4 x 142 x 2905, K =
// 201 13.5 7.5; 660 x 3283, K = 112 12.3 5.8; 2 x 320 x 2426, K = 1288 27.7 17.7; 4 x 395 x 475, K = 2659, 780 of 32 x 32, 37.4 32.7; 540 of them 0.71 of the time
// at K = 128, 0.89 at 1200, 1.08 above; 648 of them, K = 3087,
// 33.3 34.8; 468 of them, K = 400, 1.19).  The kernel wants N >= 8 and 32-bit offsets in a tile.
inline bool gemm_unaligned_64(int batch, int M, int N, int K) {
    const long long tiles = (long long)batch * gemm_pieces(M, 32) * gemm_pieces(N, 32);
    return tiles > (K > 2400 ? 768 : K > 1200 ? 640 : 512) && N >= 8 && N <= (1 << 22) && K >= 1 && K <= (1 << 22);
}
// Its blocks: 64 in K instead of 32?  With a long K, where the loads' latency shows, unless many more workgroups than fit at once hide it (us with 32 and
// 64: 2 x 320 x 2426, K = 1288 22.4 17.7; 560 x 1415, K = 296 6.3 6.1; 1888 x 1381, K = 184 6.9 7.1; with 836 tiles, K = 400, 64 takes 1.25 of the time).
inline bool gemm_unaligned_blocks_64(int batch, int M, int N, int K) {
    return K > 700 || (K > 256 && (long long)batch * gemm_pieces(M, 64) * gemm_pieces(N, 64) <= 600);
}

// A size that fits no tile (K % 32 != 0, or rows that are not aligned): one thread per element of c instead?  The tile
// kernels compute whole tiles and whole blocks of 32 in K and begin with a chain of LDS stages; with few products per element that
// is mostly waste.  Both times are estimated, in us, from constants fitted to 495 measured sizes of this kind (1 to 70000 in
// M and N, 1 to 104 in K, 1 to 20000 matrices); the choice is the faster kernel, or within 15 %, for 97 % of them.  Measured, us per
// element / in tiles: 4000 x 1 x 9, K = 3, 2.4 28; 4000 x 1 x 35, K = 17, 5.1 48; 65537 in N, K = 7, 2.8 15; 33 x 33, K = 1, 2.3 4.7; 1500 x
// 1500, K = 8, 9.8 12; 1003 x 1003, K = 129, 41 8.2; 65536 x 64, K = 40, 48 9.
//   one thread per element: a launch and a chain of K loads; or all the elements, with K terms each, and, past the first
//   line or so of a row of a, one line per thread and term where a row of c is shorter than a wavefront's 64 elements;
//   tiles: a launch and a workgroup's chain, or all the workgroups.
inline bool gemm_per_element(int batch, int M, int N, int K) {
    if (K > 100) return false;
    const double k = K, elements = 1e-6 * batch * M * N;
    const double chain = 2.25 + (N < 32 ? 0.06 : 0.08) * k, work = 1.6 + elements * (1.3 + 0.4 * k + (K > 12 ? 3.0 / N * (k - 12) : 0.0));
    const double each = chain > work ? chain : work;
    double tiled;
    if (gemm_rows_aligned(N, K)) {
        static constexpr double FLOOR[] = {0, 7.0, 4.5, 3.3}, PER_TILE[] = {0, 25e-3, 6.6e-3, 2.7e-3};
        static constexpr int SIDE[] = {0, 256, 128, 64};
        const int t = gemm_tile_of(batch, M, N, K);   // not 5: K < 256
        tiled = 1.5 + PER_TILE[t] * batch * gemm_pieces(M, SIDE[t]) * gemm_pieces(N, SIDE[t]);
        tiled = tiled > FLOOR[t] ? tiled : FLOOR[t];
    } else {
        const double tiles = 1e-3 * batch * gemm_pieces(M, 32) * gemm_pieces(N, 32);
        tiled = 4.3 + 3.6 * tiles > 5.2 * tiles ? 4.3 + 3.6 * tiles : 5.2 * tiles;
        // (64 x 64, from 60 sizes with K = 64 to 120: 660 x 3283, K = 112 5.8; 2 x 2318 x 2350, K = 86 14.0, one thread per element 47)
        if (K > 32 && gemm_unaligned_64(batch, M, N, K)) tiled = 4.0 + 3.7e-3 * batch * gemm_pieces(M, 64) * gemm_pieces(N, 64);
    }
    return each < (K > 24 ? 0.9 : 1.0) * tiled;   // the estimate for one thread per element is the less certain one the longer K is
}

// What gemm_path reports: the tile, or 4 where K is cut in its last block or rows are not aligned.
inline int gemm_path_of(int batch, int M, int N, int K) {
    return gemm_rows_aligned(N, K) && K % 32 == 0 ? gemm_tile_of(batch, M, N, K) : 4;
}

// The grid over the tiles of bm x bn of a problem: one workgroup per tile, in two dimensions above GEMM_GRID_X of them (a
// dimension of a grid holds fewer than 2^32 threads).  The last row of workgroups may be surplus.
constexpr long long GEMM_GRID_X = 1 << 22;
struct GemmGrid {
    int tiles_m, tiles_n;
    long long total;    // tiles
    unsigned x, y;      // workgroups, x y >= total; y > 65535: more than a grid holds
};
constexpr GemmGrid gemm_grid_of(int batch, int M, int N, int bm, int bn) {
    const int tm = gemm_pieces(M, bm), tn = gemm_pieces(N, bn);
    const long long total = (long long)tm * tn * batch;
    if (total <= GEMM_GRID_X) return {tm, tn, total, (unsigned)total, 1u};
    return {tm, tn, total, (unsigned)GEMM_GRID_X, (unsigned)((total + GEMM_GRID_X - 1) / GEMM_GRID_X)};
}

// Workgroup b of `total` -> position in the list of tiles.  Workgroup b runs on XCD b % 8, each with an L2 of its own, so
// every XCD takes a contiguous run of the list.  The list goes through c in groups of `group` tiles, column by column: where the
// runs are whole groups or whole parts of one, the XCDs would be in the same column all the time, in rows of c a multiple of 16 KiB
// apart, and write to the same memory channels.  XCD x then begins x eighths into its run (8192 x 8192, bfloat16, K = 64: 47 us in
// step, 36 us like this; K = 2048: 231 and 212; 8028 x 24200, K = 64: 134 and 113), if the launch takes more than two rounds of the 256
// compute units (else within 3 % either way).  Other runs are out of step already (7203 x 16848, K = 1280: 297 as it is, 311 like
// this).
constexpr bool gemm_runs_in_step(long long total, long long group) {
    const long long q = total >> 3;
    return total > 512 && (q % group == 0 || group % q == 0);
}

// apart: as above.  I: int where it holds every count, else long long.
template <class I>
constexpr I gemm_list_position(I b, I total, bool apart) {
    const I q = total >> 3, r = total & 7, x = b & 7;
    I j = b >> 3;
    if (apart) {
        const I len = q + (x < r);
        j += (x * len) >> 3;
        j = j < len ? j : j - len;
    }
    return x * q + (x < r ? x : r) + j;
}

// Or one after the other?  With a single column of tiles no two of them share rows of a, and what the XCDs run together is best
// one stretch of memory, as long as that streaming is what a launch waits for and not the matrix instructions (us in runs /
// in order: 200 x 256 x 256, K = 32 10.7 10.1, K = 64 12.1 11.5, K = 2048 94.4 96.1; 50000 x 256, K = 128 12.8 12.5).  Past one round of the
// chip only for whole columns and K = 64 (524288 x 256 81.6 79.1; K = 256 135 147; 56 x 13824 x 184, K = 64 106 114; 30 x 4096 x 256, K = 96
// 24.4 25.8; 24 x 96512 x 256, K = 16 274 288; 126976 x 256, K = 32 17.9 18.6).
constexpr bool gemm_in_order(int N, int K, int total) { return N <= 256 && (total <= 256 ? K <= 128 : N == 256 && K == 64); }

// Position t in matrix bi's list of tiles -> tile.  The list goes through GEMM_GROUP_M tile rows at a time, column by column:
// the workgroups that an XCD runs together then cover a compact block of c (4 x 8 tiles when it holds 32) and share both
// their rows of a and their columns of b.  join: the last group takes the remainder too, GEMM_GROUP_M to 2 GEMM_GROUP_M - 1 rows;
// a last group of one row gives an XCD 32 columns of b to read (288 x 4096 x 2240, five rows of 64 x 64 tiles: 19.7 us with
// groups of 4 and 1, 16.7 us with one of 5).  Not in 256 x 256 tiles: 69 products of 5 to 27 rows of them were 1.2 % slower on average
// with it (8 x 1792 x 4096, K = 256 57.6 63.2; 1 x 2304 x 25600, K = 256 54.7 60.1, K = 1536 166 174; 8 x 2304 x 4096, K = 1536 226 219).
#ifndef GEMM_GROUP_M
#define GEMM_GROUP_M 4
#endif
struct GemmTile {
    int bi, tm, tn;
};
constexpr int gemm_group(int tiles_m, int tiles_n) { return (tiles_m > GEMM_GROUP_M ? GEMM_GROUP_M : tiles_m) * tiles_n; }
// The order of a launch of 256 x 256 tiles (smaller ones always go in runs: nothing else gained there).  Decided once, on the host: a
// workgroup that does not share its compute unit would pay for every division, about 0.05 us each.
enum GemmOrder { GEMM_RUNS, GEMM_RUNS_APART, GEMM_IN_ORDER };
constexpr GemmOrder gemm_order_of(const GemmGrid& g, int N, int K) {
    return g.y == 1 && gemm_in_order(N, K, (int)g.total) ? GEMM_IN_ORDER : gemm_runs_in_step(g.total, gemm_group(g.tiles_m, g.tiles_n)) ? GEMM_RUNS_APART : GEMM_RUNS;
}
constexpr GemmTile gemm_tile_in_list(int bi, int t, int tiles_m, int tiles_n, bool join) {
    const int last = tiles_m <= GEMM_GROUP_M ? 0 : join ? tiles_m / GEMM_GROUP_M - 1 : (tiles_m - 1) / GEMM_GROUP_M;   // number of the last group
    int g = last == 0 ? 0 : t / (GEMM_GROUP_M * tiles_n);
    g = g < last ? g : last;
    const int u = t - g * GEMM_GROUP_M * tiles_n, rows = g < last ? GEMM_GROUP_M : tiles_m - last * GEMM_GROUP_M;
    const int tn = u / rows;
    return {bi, g * GEMM_GROUP_M + (u - tn * rows), tn};
}

hipError_t gemm_launch(const GemmLaunch& a);
