// The host-side rules of the GEMM launch (gemm_launch.h) behind plain C functions, for tests without a GPU.
#include "../../paper_2501_08071_amd/csrc/gemm_launch.h"

extern "C" {
int pieces(int x, int t) { return gemm_pieces(x, t); }
int tile_of(int batch, int M, int N, int K) { return gemm_tile_of(batch, M, N, K); }
}
