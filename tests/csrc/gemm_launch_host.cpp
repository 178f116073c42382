// The host-side rules of the GEMM launch (gemm_launch.h) behind plain C functions, for tests without a GPU.
#include "../../paper_2501_08071_amd/csrc/gemm_launch.h"

extern "C" {
int pieces(int x, int t) { return gemm_pieces(x, t); }
int tile_of(int batch, int M, int N, int K) { return gemm_tile_of(batch, M, N, K); }
// tiles_m, tiles_n, total, x, y
void grid_of(int batch, int M, int N, int bm, int bn, long long* out) {
    const GemmGrid g = gemm_grid_of(batch, M, N, bm, bn);
    out[0] = g.tiles_m; out[1] = g.tiles_n; out[2] = g.total; out[3] = g.x; out[4] = g.y;
}
int position32(int b, int total, int group) { return gemm_list_position(b, total, group > 0 && gemm_runs_in_step(total, group)); }
long long position64(long long b, long long total, long long group) { return gemm_list_position(b, total, group > 0 && gemm_runs_in_step(total, group)); }
int tile_in_list(int t, int tiles_m, int tiles_n, int join) {
    const GemmTile g = gemm_tile_in_list(0, t, tiles_m, tiles_n, join != 0);
    return g.tm * tiles_n + g.tn;
}
int in_order(int N, int K, int total) { return gemm_in_order(N, K, total); }
int order_of(int batch, int M, int N, int K) { return gemm_order_of(gemm_grid_of(batch, M, N, 256, 256), N, K); }
int eight_waves(int batch, int M, int N, int K) { return gemm_eight_waves(batch, M, N, K); }
int tiles_128x256(int batch, int M, int N, int K) { return gemm_tiles_128x256(batch, M, N, K); }
int two_parts(int batch, int M, int N, int K) { return gemm_two_parts(batch, M, N, K); }
int tiles_64x128(int batch, int M, int N, int K) { return gemm_tiles_64x128(batch, M, N, K); }
int long_blocks(int batch, int M, int N, int K) { return gemm_long_blocks(batch, M, N, K); }
int unaligned_64(int batch, int M, int N, int K) { return gemm_unaligned_64(batch, M, N, K); }
int unaligned_blocks_64(int batch, int M, int N, int K) { return gemm_unaligned_blocks_64(batch, M, N, K); }
int deep(int batch, int M, int N, int K) { return gemm_deep(batch, M, N, K); }
int per_element(int batch, int M, int N, int K) { return gemm_per_element(batch, M, N, K); }
}
