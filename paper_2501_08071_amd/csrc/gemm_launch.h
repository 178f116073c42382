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

// Pieces of t that cover x, for any x >= 0 (x + t - 1 would overflow where x is near 2^31).
constexpr int gemm_pieces(int x, int t) { return x / t + (x % t != 0); }

// Tiles of c for a problem whose rows are 16-byte aligned: 1: 256 x 256, 2: 128 x 128, 3: 64 x 64, 5: 32 x 32 with K
// split over the wavefronts of a workgroup.  The largest tile that still gives three quarters of the 256 compute units
// a workgroup; a problem that fits the chip in one round of 32 x 32 tiles and has a K worth splitting takes those.
#ifndef GEMM_SK_TILES
#define GEMM_SK_TILES 256
#endif
inline int gemm_tile_of(int batch, int M, int N, int K) {
    auto tiles = [&](int t) { return (long long)batch * gemm_pieces(M, t) * gemm_pieces(N, t); };
    if (tiles(32) <= GEMM_SK_TILES && K >= 256) return 5;
    return tiles(256) >= 192 ? 1 : tiles(128) >= 192 ? 2 : 3;
}

// Do the rows of a and b start at 16-byte aligned addresses (and stay within 32-bit offsets inside a tile)?  Then
// blocks of K go straight from global memory into LDS.
inline bool gemm_rows_aligned(int N, int K) { return K > 0 && K % 8 == 0 && N % 8 == 0 && K <= (1 << 22) && N <= (1 << 22); }

// What gemm_path reports: the tile, or 4 where K is cut in its last block or rows are not aligned.
inline int gemm_path_of(int batch, int M, int N, int K) {
    return gemm_rows_aligned(N, K) && K % 32 == 0 ? gemm_tile_of(batch, M, N, K) : 4;
}

hipError_t gemm_launch(const GemmLaunch& a);
