// Fused GEMM + LeakyReLU for gfx950 (the paper's mmLeakyReLu, Table 2): c = f(a b), a [M,K], b [K,N]
// row-major, 16-bit in and out, fp32 accumulation.
//
// Matrix-core kernel (K % 8 == 0, N % 8 == 0):
//   * a workgroup of four wavefronts (2 x 2) owns a 64 TM x 64 TN tile of c, a wavefront 32 TM x 32 TN of
//     it as TM x TN accumulator blocks of v_mfma_f32_32x32x16: 128 x 128, 64 x 128 or 64 x 64; eight wavefronts own 128 x 256 or
//     256 x 256, or 128 x 128 in two parts, each with half of every block of K; larger problems: 256 x 256 tiles,
//     gemm_lrelu_wide_kernel; gemm_tile_of chooses, and the rules behind it;
//   * computed transposed, c^T = b^T a^T: the first operand is a 32 x 16 piece of b^T, fetched from the
//     row-major b tile in LDS with transposing reads (ds_read_b64_tr_b16), the second 16 contiguous bytes
//     of a row of a; a lane then holds four consecutive n of one row m of c, and the tile of c goes out
//     through LDS so that the stores write whole rows of it;
//   * K runs in blocks of 32 or 64 through four to six LDS stages; tiles come straight from
//     global memory into LDS (global_load_lds_dwordx4, 16 bytes per lane, 1 KiB of consecutive LDS per
//     instruction), all stages but one ahead, with the bank-conflict swizzle applied to the global address of each lane;
//   * rows past M repeat the last row and column chunks past N the last chunk (results masked at the
//     store), so the loop has no edge cases.
// Small problems (at most 256 tiles of 32 x 32, K >= 256): 32 x 32 tiles with K split over the four wavefronts of
// the workgroup, see gemm_lrelu_splitk_kernel.
// K % 32 != 0: the same kernels with the last block cut (K % 8 == 0), or, where rows of a or b do not start at 16-byte
// aligned addresses, 64 x 64 tiles or the 32 x 32 kernel with their loads through registers; either way one thread per element where there are
// too few products to pay for tiles, see gemm_lrelu_element_kernel.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include <utility>

#include "gemm_launch.h"
#include "gfx950_common.h"

// LDS stages of 32 in K; all but one of them in flight ahead of the one in use.  128 x 128 tiles: 2048 cubed 21.7 us with four
// and six, 22.4 with eight.  64 x 64 tiles take four or six (gemm_deep), or five of 64 (gemm_long_blocks: 1024 x 1024, K = 1024 7.0 with
// four and 6.8 with five, 512 x 1024, K = 4096 16.7 and 14.9); 64 x 128 tiles four of 64 (1000 x 1000 x 1000 9.9, with six 10.8).
#ifndef GEMM_NST128
#define GEMM_NST128 4
#endif
#ifndef GEMM_NST
#define GEMM_NST 4   // the same for 256 x 256 tiles (all that LDS holds)
#endif

namespace {

using namespace gfx950;

template <int N>
__device__ __forceinline__ void wait_tile_loads() { wait_lds_dma<N>(); }

// XOR swizzle of the 16-byte chunk index within a row, by row length (chunks per row 4, 8, 16): rows
// that a wavefront reads together land in different banks both for the 16-byte row reads and for
// the transposing 8-byte reads.
__device__ __forceinline__ constexpr int swz_a(int row) { return (row >> 2) & 3; }
// The same for rows of a of eight chunks (blocks of 64 in K).
__device__ __forceinline__ constexpr int swz_a8(int row) { return (row >> 1) & 7; }
// The same for 16-byte reads of 16 rows and 4 chunks (lane = chunk * 16 + row).  LDS serves such a read in four parts, lanes 0-3,
// 12-15, 20-27 the first and 4-11, 16-19, 28-31 the second, the other half alike: with this swizzle the sixteen lanes of each
// lie in different banks.
__device__ __forceinline__ constexpr int swz_a16(int row) { return (row >> 2) & 2; }
template <int CHUNKS>
__device__ __forceinline__ constexpr int swz_b(int row) {
    return CHUNKS >= 16 ? (((row & 3) << 2) | ((row >> 2) & 3))   // the low four chunk bits = 256 bytes = all banks
                        : ((((row >> 1) & 1) << 2) | (((row >> 2) & 1) << 1) | ((row >> 3) & 1));
}

// Workgroup -> tile: its place in the list (gemm_order_of), then gemm_tile_in_list.  LARGE: 256 x 256 tiles; the others always go in runs.
template <bool LARGE>
__device__ __forceinline__ GemmTile tile_of_workgroup(int tiles_m, int tiles_n, long long total, int order) {
    const int per = tiles_m * tiles_n;
    const bool apart = LARGE && order == GEMM_RUNS_APART;
    if (gridDim.y == 1) {
        const int total1 = (int)gridDim.x, b = (int)blockIdx.x;
        const int c = LARGE && order == GEMM_IN_ORDER ? b : gemm_list_position(b, total1, apart);
        const int bi = total1 == per ? 0 : c / per;   // (a division is 0.05 us)
        return gemm_tile_in_list(bi, c - bi * per, tiles_m, tiles_n, !LARGE);
    }
    long long b = (long long)blockIdx.y * gridDim.x + blockIdx.x;
    b = b < total ? b : total - 1;   // surplus workgroups repeat the last one's tile
    const long long c = gemm_list_position(b, total, apart);
    const int bi = (int)(c / per);
    return gemm_tile_in_list(bi, (int)(c - (long long)bi * per), tiles_m, tiles_n, !LARGE);
}

__device__ __forceinline__ float leaky(float t, float slope) { return t >= 0.f ? t : slope * t; }

extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];

// dynamic LDS of a kernel instance: the stages of the loop, or (if larger) the padded blocks of c on their way out and, behind
// them, the other parts' sums
template <int WM, int WN, int TM, int TN, int BK, int NST, int KS>
struct GemmLds {
    static constexpr int STAGES = NST * 2 * BK * (32 * TM * WM + 32 * TN * WN);
    static constexpr int OUT = WM * WN * (32 * TM) * (64 * TN + 16);
    static constexpr int SUMS = WM * WN * TM * TN * 4096;
    static constexpr int BYTES = STAGES > OUT + (KS - 1) * SUMS ? STAGES : OUT + (KS - 1) * SUMS;
    static_assert(BYTES <= 160 * 1024, "LDS");
};

// ANY: rows of a and b that start at any even address (N >= 8; offsets in a tile below 2^32).  Loads into LDS need aligned addresses, so the
// blocks go through registers, 16 bytes per lane as they come, NST blocks ahead, and from there to the same places in LDS.  Bound by
// those loads: a piece of a row that begins inside a cache line costs two lines (2 x 320 x 2426, K = 1288: 17.7 us; 32 x 32 tiles with K
// split 27.7).  Four stages of LDS and registers: 12 % slower, fewer workgroups fit; 64 x 128 tiles 25 %, 128 x 128 60 %.
// What follows a row's end is the next row's and counts for columns of c that are not stored; in the last block, the only one with k
// past the end, it is zeroed in the registers, and nothing past a matrix's end is read.
template <int DT, int WM, int WN, int TM, int TN, int BK, int NST, int KS, bool KTAIL, bool ANY>
__global__ __launch_bounds__(KS * WM * WN * 64) void gemm_lrelu_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                                        uint16_t* __restrict__ C, int M, int N, int K, int tiles_m,
                                                        int tiles_n, long long total, int order, float slope) {
    using E = Elem<DT>;
    constexpr int NW = WM * WN;               // wavefronts of a part, WM x WN over the tile
    constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN;
    constexpr int A_ROWB = 2 * BK, A_TILE = BM * A_ROWB;   // BM rows of BK elements
    constexpr int B_ROWB = 2 * BN;           // bytes per row of the b tile
    constexpr int B_TILE = BK * B_ROWB;      // BK rows (k) of BN elements
    constexpr int STAGE = A_TILE + B_TILE;
    constexpr int NKS = BK / 16 / KS;        // k steps of 16 of a block per part
    constexpr int A_LPR = BK / 8, A_RPI = 64 / A_LPR;   // as below, for the a tile
    constexpr int B_LPR = B_ROWB / 16;       // lanes (16-byte chunks) per row of the b tile
    constexpr int B_RPI = 64 / B_LPR;        // rows per load instruction
    constexpr int LA = A_TILE / 1024 / (KS * NW), LB = B_TILE / 1024 / (KS * NW);   // load instructions per stage and wavefront
    constexpr int IPS = LA + LB;
    static_assert(LA * KS * NW * 1024 == A_TILE && LB * KS * NW * 1024 == B_TILE && LA >= 1 && LB >= 1, "the wavefronts share the loads evenly");
    static_assert(NST * STAGE <= 160 * 1024, "LDS");
    constexpr bool CLEAR = KTAIL && BK != 32;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int loader = __builtin_amdgcn_readfirstlane(tid >> 6);   // its share of the loads
    const int part = KS == 1 ? 0 : loader / NW;                    // its k steps of every block
    const int wave = loader - part * NW;                           // its piece of the tile
    const int l32 = lane & 31, h = lane >> 5;
    const int wm = wave % WM, wn = wave / WM;

    const auto [bi, tm_i, tn_i] = tile_of_workgroup<BM == 256>(tiles_m, tiles_n, total, order);
    const int m0 = tm_i * BM, n0 = tn_i * BN;
    const uint16_t* Ab = A + ((size_t)bi * M + m0) * K;
    const uint16_t* Bb = B + (size_t)bi * K * N + n0;
    uint16_t* Cb = C + (size_t)bi * M * N;
    const int nk = gemm_pieces(K, BK);
    auto swz = [](int row) { return BK == 64 ? swz_a8(row) : swz_a(row); };

    const uint32_t lds0 = (uint32_t)(uintptr_t)(LDS_AS uint8_t*)smem;

    // ---- loads: byte offset of this lane's source chunk inside the tile's rows ----
    const int kr = K - BK * (nk - 1);   // valid k of the last block (KTAIL: a multiple of 8, else BK)
    uint32_t goff_a[LA], goff_b[LB], tail_a[LA], tail_b[LB];   // tail: the same for the last block, chunks past K replaced
#pragma unroll
    for (int j = 0; j < LA; ++j) {
        const int r = A_RPI * (loader * LA + j) + lane / A_LPR, pos = lane % A_LPR;
        const int rr = r < M - 1 - m0 ? r : M - 1 - m0;
        goff_a[j] = (uint32_t)(rr * K + ((pos ^ swz(r)) << 3)) * 2u;
        if constexpr (KTAIL) tail_a[j] = 8 * (pos ^ swz(r)) < kr ? goff_a[j] : (uint32_t)(rr * K) * 2u;
    }
    {
        const int inside = ANY ? (N - n0 + 7) / 8 : (N - n0) / 8;
        const int nvalid = inside < BN / 8 ? inside : BN / 8;   // chunks of this tile inside the matrix
#pragma unroll
        for (int j = 0; j < LB; ++j) {
            const int r = B_RPI * (loader * LB + j) + lane / B_LPR, pos = lane % B_LPR;
            int ch = pos ^ swz_b<B_LPR>(r);
            ch = ch < nvalid - 1 ? ch : nvalid - 1;
            goff_b[j] = (uint32_t)(r * N + (ch << 3)) * 2u;
            if constexpr (KTAIL) tail_b[j] = (uint32_t)((r < kr ? r : 0) * N + (ch << 3)) * 2u;
        }
    }
    // k block kb into stage st; a block past the end repeats the last one (nobody reads it): every step
    // issues the same number of loads and the wait count is a constant
    auto issue = [&](int kb, int st) {
        const int kc = kb < nk - 1 ? kb : nk - 1;
        const uint16_t* sa = Ab + (size_t)kc * BK;
        const uint16_t* sb = Bb + (size_t)kc * BK * N;
        const bool tail = KTAIL && kc == nk - 1;
#pragma unroll
        for (int j = 0; j < LA; ++j) lds_dma16(lds0 + st * STAGE + (loader * LA + j) * 1024, sa, tail ? tail_a[j] : goff_a[j]);
#pragma unroll
        for (int j = 0; j < LB; ++j) lds_dma16(lds0 + st * STAGE + A_TILE + (loader * LB + j) * 1024, sb, tail ? tail_b[j] : goff_b[j]);
    };

    // ANY: the same by way of registers
    struct Blk {
        u32x4 a[LA], b[LB];
    };
    auto load_block = [&](Blk& x, int kb) {
        if (kb >= nk) return;
        const char* sa = (const char*)(Ab + (size_t)kb * BK);
        const char* sb = (const char*)(Bb + (size_t)kb * BK * N);
        if (kb < nk - 1) {
#pragma unroll
            for (int j = 0; j < LA; ++j) __builtin_memcpy(&x.a[j], sa + goff_a[j], 16);
#pragma unroll
            for (int j = 0; j < LB; ++j) __builtin_memcpy(&x.b[j], sb + goff_b[j], 16);
            return;
        }
        // 16 bytes at p, of which the first n elements (any number) count
        auto cut_load = [](const char* p, long long n) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (n >= 8) {
                __builtin_memcpy(&v, p, 16);
            } else {
#pragma unroll
                for (int e = 0; e < 7; ++e)
                    if (e < n) v[e / 2] |= (uint32_t)((const uint16_t*)p)[e] << (16 * (e % 2));
            }
            return v;
        };
#pragma unroll
        for (int j = 0; j < LA; ++j) {
            const int row = A_RPI * (loader * LA + j) + lane / A_LPR;
            x.a[j] = cut_load(sa + goff_a[j], kr - 8 * ((lane % A_LPR) ^ swz(row)));
        }
#pragma unroll
        for (int j = 0; j < LB; ++j) {
            const int row = B_RPI * (loader * LB + j) + lane / B_LPR;
            x.b[j] = cut_load(sb + goff_b[j], row < kr ? (long long)kr * N - n0 - (long long)(goff_b[j] / 2) : 0);   // up to the matrix's end
        }
    };
    auto store_block = [&](const Blk& x, int st) {
#pragma unroll
        for (int j = 0; j < LA; ++j) lds_write_b128(lds0 + st * STAGE + (loader * LA + j) * 1024 + 16 * lane, x.a[j]);
#pragma unroll
        for (int j = 0; j < LB; ++j) lds_write_b128(lds0 + st * STAGE + A_TILE + (loader * LB + j) * 1024 + 16 * lane, x.b[j]);
    };
    Blk x[ANY ? NST : 1];

    // ---- operand addresses (stage 0, k step 0 of the b tile) ----
    uint32_t a_addr[TM][NKS];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            a_addr[tm][ks] = lds0 + ((wm * TM + tm) * 32 + l32) * A_ROWB + (((2 * (part * NKS + ks) + h) ^ swz(l32)) << 4);
    // b^T operand: lane addresses 8 bytes of row (k) 8 h + 4 hi + x, elements (n) 16 g1 + 4 y .. +3 of the
    // 32-wide block; the transposing read hands lane l the four k of element n = l % 32
    uint32_t b_addr[2][TN];
    {
        const int x = (lane & 15) >> 2, y = lane & 3, g1 = (lane >> 4) & 1;
#pragma unroll
        for (int hi = 0; hi < 2; ++hi)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                const int row = 8 * h + 4 * hi + x;
                const int chunk = 4 * (wn * TN + tn) + 2 * g1 + (y >> 1);
                b_addr[hi][tn] = lds0 + A_TILE + (part * NKS * 16 + row) * B_ROWB + ((chunk ^ swz_b<B_LPR>(row)) << 4) + ((y & 1) << 3);
            }
    }

    f32x16 acc[TN][TM];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[tn][tm][r] = 0.f;

    if constexpr (ANY) {
#pragma unroll
        for (int s = 0; s < NST; ++s) load_block(x[s], s);
    } else {
#pragma unroll
        for (int s = 0; s < NST - 1; ++s) issue(s, s);
    }

    // The operands of one k step (16 k of a block) of stage st
    struct Ops {
        u32x4 a[TM], b[TN];
    };
    auto read_ops = [&](Ops& o, int st_bytes, int ks) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) o.a[tm] = lds_read_b128(a_addr[tm][ks] + st_bytes);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const u32x2 lo = lds_read_tr16(b_addr[0][tn] + st_bytes + ks * 16 * B_ROWB);
            const u32x2 hi = lds_read_tr16(b_addr[1][tn] + st_bytes + ks * 16 * B_ROWB);
            o.b[tn] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
    };
    // The last block of a K that is not a multiple of BK: both operands' k past the end become zero (whatever was loaded in their
    // place may be infinite).  Blocks of 64: every wavefront clears what its own loads brought, once they have landed and before the
    // barrier behind which the block may be read: nothing of it is left in the loop, whose four k steps would each have to ask.  Blocks of
    // 32: in the operands' registers, which takes a product of 128 x 128 tiles with K = 48 6.3 us where clearing takes 6.7 (4664 x 776), one
    // of 64 x 64 tiles with K = 424 7.1 and 7.7 (4 x 123 x 3968).
    auto clear_tail = [&](int st) {
#pragma unroll
        for (int j = 0; j < LA; ++j) {
            const int r = A_RPI * (loader * LA + j) + lane / A_LPR, pos = lane % A_LPR;
            if (8 * (pos ^ swz(r)) >= kr) lds_write_b128(lds0 + st * STAGE + (loader * LA + j) * 1024 + 16 * lane, u32x4{0u, 0u, 0u, 0u});
        }
#pragma unroll
        for (int j = 0; j < LB; ++j)
            if (B_RPI * (loader * LB + j) + lane / B_LPR >= kr) lds_write_b128(lds0 + st * STAGE + A_TILE + (loader * LB + j) * 1024 + 16 * lane, u32x4{0u, 0u, 0u, 0u});
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    auto cut_tail = [&](Ops& o, int ks) {
        const bool past = 16 * ks + 8 * h >= kr;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) o.a[tm] = past ? u32x4{0u, 0u, 0u, 0u} : o.a[tm];
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) o.b[tn] = past ? u32x4{0u, 0u, 0u, 0u} : o.b[tn];
    };
    auto multiply = [&](const Ops& o) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) acc[tn][tm] = E::mfma(o.b[tn], o.a[tm], acc[tn][tm]);
    };

    // Block kb: its first k step runs on operands read during block kb-1 (`ahead`), every other on operands
    // read under the one before, and under the last the first operands of block kb+1 are read: the matrix
    // pipe never waits for an LDS round trip behind a barrier.  For that, block kb+1 must be complete one
    // barrier early: every wavefront checks its share of it before the barrier of block kb.
    Ops ahead;
    if constexpr (ANY) {
        store_block(x[0], 0);
        load_block(x[0], NST);
    } else {
        wait_tile_loads<(NST - 2) * IPS>();
        if (CLEAR && nk == 1) clear_tail(0);
    }
    __syncthreads();
    read_ops(ahead, 0, 0);
    auto step = [&](int kb, auto phase) {
        constexpr int PH = decltype(phase)::value;
        if constexpr (ANY) {
            // block kb+1 to its stage, last read (block kb+1-NST) two barriers ago or more, and the registers to block kb+1+NST
            if (kb + 1 < nk) store_block(x[(PH + 1) % NST], (PH + 1) % NST);
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            load_block(x[(PH + 1) % NST], kb + 1 + NST);
        } else {
            // blocks up to kb+1 have landed when at most the loads of the NST-3 later blocks are still out
            wait_tile_loads<(NST - 3) * IPS>();
            if (CLEAR && kb == nk - 2) clear_tail((PH + 1) % NST);
            asm volatile("s_barrier" ::: "memory");
            // ... for everybody, and everybody is done with block kb-1: its stage takes block kb+NST-1
            issue(kb + NST - 1, (PH + NST - 1) % NST);
        }
        [&]<int... S>(std::integer_sequence<int, S...>) {
            ([&] {
                Ops now = ahead;
                read_ops(ahead, (S + 1 < NKS ? PH : (PH + 1) % NST) * STAGE, (S + 1) % NKS);
                if (KTAIL && !CLEAR && S == 0 && kb == nk - 1) {
                    cut_tail(now, 0);
                    cut_tail(ahead, 1);
                }
                __builtin_amdgcn_sched_barrier(0);
                multiply(now);
                __builtin_amdgcn_sched_barrier(0);
            }(), ...);
        }(std::make_integer_sequence<int, NKS>{});
    };
    static_assert(NST >= 3, "one block in use, one read ahead, at least one in flight");
    for (int k0 = 0; k0 < nk; k0 += NST) {
        [&]<int... PH>(std::integer_sequence<int, PH...>) {
            ((k0 + PH < nk ? step(k0 + PH, std::integral_constant<int, PH>{}) : (void)0), ...);
        }(std::make_integer_sequence<int, NST>{});
    }
    wait_tile_loads<0>();   // the repeated loads of the last steps must not outlive the workgroup's LDS

    // ---- epilogue: activation in fp32, round; the tile leaves through LDS ----
    // A lane holds four consecutive n of one row m: stored from there, an instruction would touch 32 rows with
    // 16 bytes each.  Every wavefront writes its 32 TM x 32 TN block into a region of its own (the stages are
    // free once every wavefront is past the loop and its loads have landed), rows padded by 16 bytes against
    // bank conflicts, and reads it back with 4 TN lanes side by side on a row: a store instruction then writes
    // whole rows of the block, 64 TN bytes each.
    __syncthreads();
    if constexpr (KS > 1) {
        // the sums of the other parts go through LDS, 16 bytes per lane and access, and are added in the order of the parts
        using Lds = GemmLds<WM, WN, TM, TN, BK, NST, KS>;
        auto at = [&](int p, int i) { return (f32x4*)(smem + Lds::OUT + (p - 1) * Lds::SUMS + ((wave * TM * TN * 4 + i) * 64 + lane) * 16); };
        if (part > 0) {
#pragma unroll
            for (int i = 0; i < TM * TN * 4; ++i) {
                const f32x16& t = acc[i / 4 / TM][i / 4 % TM];
                const int r = 4 * (i % 4);
                *at(part, i) = f32x4{t[r], t[r + 1], t[r + 2], t[r + 3]};
            }
        }
        __syncthreads();
        if (part > 0) return;
#pragma unroll
        for (int p = 1; p < KS; ++p)
#pragma unroll
            for (int i = 0; i < TM * TN * 4; ++i) {
                const f32x4 u = *at(p, i);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i / 4 / TM][i / 4 % TM][4 * (i % 4) + e] += u[e];
            }
    }
    {
        constexpr int RW = 32 * TM, RB = 64 * TN, RS = RB + 16;
        static_assert(NW * RW * RS <= GemmLds<WM, WN, TM, TN, BK, NST, KS>::BYTES, "LDS for the way out");
        uint8_t* reg = smem + wave * (RW * RS);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int gg = 0; gg < 4; ++gg) {
                    const f32x16& t = acc[tn][tm];
                    const u32x2 v = {E::pack2(leaky(t[4 * gg], slope), leaky(t[4 * gg + 1], slope)),
                                     E::pack2(leaky(t[4 * gg + 2], slope), leaky(t[4 * gg + 3], slope))};
                    *(u32x2*)(reg + (32 * tm + l32) * RS + 64 * tn + 16 * gg + 8 * h) = v;
                }
        constexpr int LPR = RB / 16, RPP = 64 / LPR;   // lanes per row, rows per store instruction
#pragma unroll
        for (int p = 0; p < RW / RPP; ++p) {
            const int row = p * RPP + lane / LPR, ch = lane % LPR;
            const u32x4 v = *(const u32x4*)(reg + row * RS + ch * 16);
            const int m = m0 + wm * RW + row, n = n0 + wn * (32 * TN) + ch * 8;
            if (m >= M || n >= N) continue;
            uint16_t* cp = Cb + (size_t)m * N + n;
            if constexpr (!ANY) {
                *(u32x4*)cp = v;
            } else if (n <= N - 8) {
                __builtin_memcpy(cp, &v, 16);
            } else {
#pragma unroll
                for (int e = 0; e < 7; ++e)
                    if (n + e < N) cp[e] = (uint16_t)(v[e / 2] >> (16 * (e % 2)));
            }
        }
    }
}


// Large problems: 256 x 256 tiles, four wavefronts (2 x 2), one per SIMD with the whole register file, 128 x 128 of c
// per wavefront.
// What bounds it: the clock, which the chip lowers with the switching activity of the matrix pipes and of what feeds
// them, and LDS.  So the kernel is laid out for energy per operation:
//   * v_mfma_f32_16x16x32 with 8 x 8 accumulators: an operand read from LDS feeds eight instructions, 64 KiB of LDS reads
//     per 32 of K and workgroup instead of 96 KiB with eight wavefronts of 64 x 128;
//   * the accumulators are visited in a snake, so that only one of an instruction's two operands changes.
// Nothing but the order of issue keeps the matrix pipe fed: under the 64 matrix instructions of block kb the operands of block
// kb + 1 are read, one LDS read per two of them, and the eight loads of block kb + NST - 1 issued, one per eight of them, evenly over
// the block.  (All within the first sixteen instructions, where the reads are too, they come in bursts from all compute units at
// once: 4096 cubed 104.5 us in bursts, 99.2 evenly; 8192 cubed 817 and 749; 2 x 3000 cubed 154 and 138; 5000 x 4104, K = 1000, 65.5 and 59.4,
// bfloat16.  A fifth stage: 0.5 to 3 % slower.  v_mfma_f32_32x32x16 with 4 x 4 accumulators instead: 109 and 826, 147, 62.)
// N(0,1), over the boxes seen: 4096 cubed 92 to 104 us = 1320 to 1490 TFLOP/s, 8192 cubed 749 to 763 = 1440 to 1470 (in bursts 96 to
// 107 and 785 to 817; with eight wavefronts of 64 x 128 113 to 121 and 844).
template <int DT, bool KTAIL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void gemm_lrelu_wide_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, uint16_t* __restrict__ C, int M,
                            int N, int K, int tiles_m, int tiles_n, long long total, int order, float slope) {
    using E = Elem<DT>;
    constexpr int NST = GEMM_NST;
    // LDS: the a tiles of all stages, then the b tiles: every read is one base register plus a 16-bit immediate
    constexpr int A_TILE = 256 * 64, B_ROWB = 512, B_TILE = 32 * B_ROWB, B_BASE = NST * A_TILE;
    constexpr int LA = 4, LB = 4, IPS = LA + LB;   // load instructions (1 KiB) per stage and wavefront
    static_assert(NST >= 3 && NST % 2 == 0 && IPS == 8 && NST * (A_TILE + B_TILE) <= 160 * 1024, "stages");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int wm = wave & 1, wn = wave >> 1;

    const auto [bi, tm_i, tn_i] = tile_of_workgroup<true>(tiles_m, tiles_n, total, order);
    const int m0 = tm_i * 256, n0 = tn_i * 256;
    const uint16_t* Ab = A + ((size_t)bi * M + m0) * K;
    const uint16_t* Bb = B + (size_t)bi * K * N + n0;
    uint16_t* Cb = C + (size_t)bi * M * N;
    const int nk = gemm_pieces(K, 32);

    const uint32_t lds0 = (uint32_t)(uintptr_t)(LDS_AS uint8_t*)smem;

    // ---- loads: byte offset of this lane's source chunk inside the tile's rows ----
    const int kr = K - 32 * (nk - 1);   // valid k of the last block (KTAIL: 8, 16 or 24, else 32)
    uint32_t goff_a[LA], goff_b[LB], tail_a[LA], tail_b[LB];   // tail: the same for the last block, chunks past K replaced
    {
        const int nvalid = (N - n0) / 8 < 32 ? (N - n0) / 8 : 32;   // chunks of this tile inside the matrix
#pragma unroll
        for (int j = 0; j < LA; ++j) {
            const int r = 16 * (wave * LA + j) + lane / 4, pos = lane % 4;
            const int rr = r < M - 1 - m0 ? r : M - 1 - m0;
            goff_a[j] = (uint32_t)(rr * K + ((pos ^ swz_a16(r)) << 3)) * 2u;
            if constexpr (KTAIL) tail_a[j] = 8 * (pos ^ swz_a16(r)) < kr ? goff_a[j] : (uint32_t)(rr * K) * 2u;
        }
#pragma unroll
        for (int j = 0; j < LB; ++j) {
            const int r = 2 * (wave * LB + j) + lane / 32, pos = lane % 32;
            int ch = pos ^ swz_b<32>(r);
            ch = ch < nvalid - 1 ? ch : nvalid - 1;
            goff_b[j] = (uint32_t)(r * N + (ch << 3)) * 2u;
            if constexpr (KTAIL) tail_b[j] = (uint32_t)((r < kr ? r : 0) * N + (ch << 3)) * 2u;
        }
    }
    // load instruction j of block kc's tile of a / of b
    auto issue_a = [&](int kc, int j, int st) {
        lds_dma16(lds0 + st * A_TILE + (wave * LA + j) * 1024, Ab + (size_t)kc * 32, KTAIL && kc == nk - 1 ? tail_a[j] : goff_a[j]);
    };
    auto issue_b = [&](int kc, int j, int st) {
        lds_dma16(lds0 + B_BASE + st * B_TILE + (wave * LB + j) * 1024, Bb + (size_t)kc * 32 * N, KTAIL && kc == nk - 1 ? tail_b[j] : goff_b[j]);
    };

    // A block past the end repeats the last one (nobody uses it): every step issues the same number of loads and the wait
    // count is a constant
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) {
        const int kc = s < nk - 1 ? s : nk - 1;
#pragma unroll
        for (int j = 0; j < LA; ++j) issue_a(kc, j, s);
#pragma unroll
        for (int j = 0; j < LB; ++j) issue_b(kc, j, s);
    }
    __builtin_amdgcn_sched_barrier(0);   // the loads are on their way before anything else is set up

    // ---- operand addresses (stage 0) ----
    // a: row l16 of a block of 16, chunk g.  b^T: lane addresses 8 bytes of row (k) 8 g + 4 hi + x, elements (n) 4 y .. +3
    // of a block of 16 columns; the transposing read hands lane l the four k of column l % 16.  Two neighbouring blocks
    // of columns differ in one bit of the swizzled chunk index, further ones by a constant.
    const uint32_t a_addr = lds0 + (wm * 128 + l16) * 64 + ((g ^ swz_a16(l16)) << 4);
    uint32_t b_addr[2][8];
    {
        const int x = l16 >> 2, y = l16 & 3;
#pragma unroll
        for (int hi = 0; hi < 2; ++hi)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int row = 8 * g + 4 * hi + x, chunk = 2 * (wn * 8 + i) + (y >> 1);
                b_addr[hi][i] = lds0 + B_BASE + row * B_ROWB + ((chunk ^ swz_b<32>(row)) << 4) + ((y & 1) << 3);
            }
    }
    struct Ops {
        u32x4 a[8], b[8];
    };
    // the i-th of the 24 LDS reads of a block, in the order of use: b 0, all of a, the other b
    auto read_one = [&](Ops& o, auto idx, int st) {
        constexpr int I = decltype(idx)::value;
        if constexpr (I >= 2 && I < 10) {
            o.a[I - 2] = lds_read_b128(a_addr + (I - 2) * 1024 + st * A_TILE);
        } else {
            constexpr int J = I < 2 ? I : I - 8, i = J / 2, hi = J % 2;
            const u32x2 t = lds_read_tr16(b_addr[hi][i] + st * B_TILE);
            o.b[i][2 * hi] = t[0];
            o.b[i][2 * hi + 1] = t[1];
        }
    };

    f32x4 acc[8][8];   // [n block][m block]
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    Ops ops[2];
    wait_tile_loads<(NST - 2) * IPS>();
    __syncthreads();
    [&]<int... I>(std::integer_sequence<int, I...>) {
        (read_one(ops[0], std::integral_constant<int, I>{}, 0), ...);
    }(std::make_integer_sequence<int, 24>{});
    auto step = [&](int kb, auto phase) {
        constexpr int PH = decltype(phase)::value;
        // block kb+1 has landed when at most the loads of the NST-3 later blocks are still out
        wait_tile_loads<(NST - 3) * IPS>();
        asm volatile("s_barrier" ::: "memory");
        // ... for everybody, and everybody has the operands of block kb-1 in registers: its stage takes block kb+NST-1
        const int kn = kb + NST - 1;
        const int kc = kn < nk - 1 ? kn : nk - 1;
        if (KTAIL && kb == nk - 1) {   // both operands' k past the end become zero (what was loaded there may be infinite)
            const bool past = 8 * g >= kr;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                ops[PH % 2].a[i] = past ? u32x4{0u, 0u, 0u, 0u} : ops[PH % 2].a[i];
                ops[PH % 2].b[i] = past ? u32x4{0u, 0u, 0u, 0u} : ops[PH % 2].b[i];
            }
        }
        auto unit = [&](auto un) {
            constexpr int U = decltype(un)::value;
            constexpr int i = U / 8, j = i % 2 == 0 ? U % 8 : 7 - U % 8;
            acc[i][j] = E::mfma16(ops[PH % 2].b[i], ops[PH % 2].a[j], acc[i][j]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (U % 2 == 1 && U < 48) read_one(ops[(PH + 1) % 2], std::integral_constant<int, U / 2>{}, (PH + 1) % NST);
            if constexpr (U % 8 == 4) {
                constexpr int P = U / 8;
                if constexpr (P < LA) issue_a(kc, P, (PH + NST - 1) % NST);
                else issue_b(kc, P - LA, (PH + NST - 1) % NST);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        [&]<int... U>(std::integer_sequence<int, U...>) {
            (unit(std::integral_constant<int, U>{}), ...);
        }(std::make_integer_sequence<int, 64>{});
    };
    for (int k0 = 0; k0 < nk; k0 += NST) {
        [&]<int... PH>(std::integer_sequence<int, PH...>) {
            ((k0 + PH < nk ? step(k0 + PH, std::integral_constant<int, PH>{}) : (void)0), ...);
        }(std::make_integer_sequence<int, NST>{});
    }
    wait_tile_loads<0>();   // the repeated loads of the last steps must not outlive the workgroup's LDS

    // ---- epilogue: activation in fp32, round, store from registers ----
    // A lane holds four consecutive n of row l16 of every 16 x 16 block.  Exchanging the odd quarters of the wavefront's
    // results of one block with the even quarters of the next makes that eight: an instruction stores 64 bytes of
    // 16 rows.  (By way of LDS, in whole rows, the way out took this one wavefront per SIMD 11.7 k cycles, half of
    // them waits for LDS; like this 8.6 k.)
    {
        // the lane's number anew: nothing that only the way out needs occupies a register during the loop
        const int el = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        const int m = m0 + wm * 128 + (el & 15), n = n0 + wn * 128 + 16 * ((el >> 4) & 1) + 8 * (el >> 5);
        uint16_t* cp = Cb + (size_t)m * N + n;
        auto way_out = [&](auto act, auto inside) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    f32x4 t = acc[2 * p][j], u = acc[2 * p + 1][j];
                    // taken out of the accumulation registers here, not on a common path in front of all the variants
                    asm volatile("" : "+v"(t), "+v"(u));
                    const auto lo = __builtin_amdgcn_permlane16_swap(E::pack2(act(t[0]), act(t[1])), E::pack2(act(u[0]), act(u[1])), false, false);
                    const auto hi = __builtin_amdgcn_permlane16_swap(E::pack2(act(t[2]), act(t[3])), E::pack2(act(u[2]), act(u[3])), false, false);
                    const u32x4 v = {lo[0], hi[0], lo[1], hi[1]};
                    if (decltype(inside)::value || (m + 16 * j < M && n + 32 * p < N)) *(u32x4*)(cp + (size_t)(16 * j) * N + 32 * p) = v;
                }
                __builtin_amdgcn_sched_barrier(0);   // the results of one group of rows at a time in vector registers
            }
        };
        auto way_out_act = [&](auto inside) {
            // 0 < slope <= 1: the larger of t and slope t, one instruction less per element
            if (slope > 0.f && slope <= 1.f) way_out([&](float t) { return vmax(t, slope * t); }, inside);
            else way_out([&](float t) { return leaky(t, slope); }, inside);
        };
        if (m0 + 256 <= M && n0 + 256 <= N) way_out_act(std::true_type{});
        else way_out_act(std::false_type{});
    }
}

// Small problems: 32 x 32 tiles of c, K split over the four wavefronts of the workgroup.
// A problem of few 64 x 64 tiles leaves most compute units without work, and every workgroup pulls its whole
// strip of a and b through one compute unit's memory pipeline: that, not arithmetic, is what such a launch waits
// for.  Here a workgroup owns a 32 x 32 tile (four times the workgroups, half the bytes per compute unit) and
// wavefront w the k blocks w, w + 4, w + 8, ...: it streams them through LDS stages of its own (no barrier in
// the loop: what a wavefront loads only that wavefront reads), accumulates a 32 x 32 partial result in two
// independent accumulators, and at the end the four partial results meet in LDS: wavefront q adds up, activates
// and stores columns 8q .. 8q+7 of the tile.
//
// LOAD 0: K % 32 == 0 and N % 8 == 0; 1: K % 8 == 0 and N % 8 == 0, the last block is cut; both load straight into LDS.
// LOAD 2: any K and N.  Rows of a and b then start at any even address, and loads into LDS need 4-byte aligned ones:
// the blocks go through registers, 16 unaligned bytes per lane, two blocks ahead, and from there into two LDS stages.
// Elements past the end of a row are the next row's and fall under the masks of k and n; only what would pass the end
// of the whole matrix is read element by element.  (777 x 1001 x 1003: 16.2 us; one thread per element of c: 350 us.)
#ifndef GEMM_SK_NST
#define GEMM_SK_NST 4   // LDS stages per wavefront (4 KiB each); more gained nothing and a larger LDS request starts later
#endif
template <int DT, int LOAD>
__global__ __launch_bounds__(256) void gemm_lrelu_splitk_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                                               uint16_t* __restrict__ C, int M, int N, int K, int tiles_m,
                                                               int tiles_n, long long total, int order, float slope) {
    using E = Elem<DT>;
    constexpr int NST = GEMM_SK_NST, STAGE = 4096, IPS = 4;
    constexpr bool KTAIL = LOAD != 0;
    static_assert(NST >= 3 && 4 * NST * STAGE <= 160 * 1024 && (NST - 2) * IPS <= 63, "stages");
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const auto [bi, tm_i, tn_i] = tile_of_workgroup<false>(tiles_m, tiles_n, total, order);
    const int m0 = tm_i * 32, n0 = tn_i * 32;
    const uint16_t* Ab = A + ((size_t)bi * M + m0) * K;
    const uint16_t* Bb = B + (size_t)bi * K * N + n0;
    uint16_t* Cb = C + (size_t)bi * M * N;
    const int nk = gemm_pieces(K, 32);
    const int kr = K - 32 * (nk - 1);   // valid k of the last block
    const int mine = nk > wave ? (nk - wave + 3) / 4 : 0;   // k blocks of this wavefront: wave, wave + 4, ...

    const uint32_t lds0 = (uint32_t)(uintptr_t)(LDS_AS uint8_t*)smem;
    const uint32_t ldsw = lds0 + wave * (NST * STAGE);
    // operands (stage 0): a: row l32, chunk 2 ks + h; b^T: 8 bytes of row (k) 8 h + 4 hi + x, elements 16 g1 + 4 y .. +3
    uint32_t a_addr[2], b_addr[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) a_addr[ks] = ldsw + l32 * 64 + (((2 * ks + h) ^ swz_a(l32)) << 4);
    {
        const int x = (lane & 15) >> 2, y = lane & 3, g1 = (lane >> 4) & 1;
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            const int row = 8 * h + 4 * hi + x, chunk = 2 * g1 + (y >> 1);
            b_addr[hi] = ldsw + 2048 + row * 64 + ((chunk ^ swz_a(row)) << 4) + ((y & 1) << 3);
        }
    }
    f32x16 acc[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[ks][r] = 0.f;

    // the operands of the block in the stage at st_bytes, and their matrix instructions; kb: which block it is
    auto use_stage = [&](int st_bytes, int kb) {
        u32x4 a[2], b[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            a[ks] = lds_read_b128(a_addr[ks] + st_bytes);
            const u32x2 lo = lds_read_tr16(b_addr[0] + st_bytes + ks * 16 * 64);
            const u32x2 hi = lds_read_tr16(b_addr[1] + st_bytes + ks * 16 * 64);
            b[ks] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
        // the last block: both operands' k past the end become zero (whatever was loaded in their place may be infinite)
        if (KTAIL && kb == nk - 1) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int valid = kr - 16 * ks - 8 * h;   // of the eight k in this lane's operand
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const uint32_t keep = 2 * d + 2 <= valid ? 0xffffffffu : 2 * d + 1 <= valid ? 0xffffu : 0u;
                    a[ks][d] &= keep;
                    b[ks][d] &= keep;
                }
            }
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) acc[ks] = E::mfma(b[ks], a[ks], acc[ks]);
    };

    if constexpr (LOAD != 2) {
        // loads: instruction j covers rows 16 j .. 16 j + 15 of a tile (64 bytes each); lane = row * 4 + chunk position
        uint32_t goff_a[2], goff_b[2], tail_a[2], tail_b[2];   // tail: the same for the last block, chunks past K replaced
        {
            const int nvalid = (N - n0) / 8 < 4 ? (N - n0) / 8 : 4;   // 16-byte chunks of this tile inside the matrix
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int r = 16 * j + lane / 4, pos = lane % 4;
                const int rr = r < M - 1 - m0 ? r : M - 1 - m0;
                goff_a[j] = (uint32_t)(rr * K + ((pos ^ swz_a(r)) << 3)) * 2u;
                int ch = pos ^ swz_a(r);
                if constexpr (KTAIL) tail_a[j] = 8 * ch < kr ? goff_a[j] : (uint32_t)(rr * K) * 2u;
                ch = ch < nvalid - 1 ? ch : nvalid - 1;
                goff_b[j] = (uint32_t)(r * N + (ch << 3)) * 2u;
                if constexpr (KTAIL) tail_b[j] = (uint32_t)((r < kr ? r : 0) * N + (ch << 3)) * 2u;
            }
        }
        // the i-th block of this wavefront into stage st; past its last block the last one again (nobody reads it):
        // every step issues the same number of loads.  A wavefront without blocks issues nothing.
        auto issue = [&](int i, int st) {
            if (mine == 0) return;
            const int kb = wave + 4 * (i < mine - 1 ? i : mine - 1);
            const bool tail = KTAIL && kb == nk - 1;
            const uint16_t* sa = Ab + (size_t)kb * 32;
            const uint16_t* sb = Bb + (size_t)kb * 32 * N;
#pragma unroll
            for (int j = 0; j < 2; ++j) lds_dma16(ldsw + st * STAGE + j * 1024, sa, tail ? tail_a[j] : goff_a[j]);
#pragma unroll
            for (int j = 0; j < 2; ++j) lds_dma16(ldsw + st * STAGE + 2048 + j * 1024, sb, tail ? tail_b[j] : goff_b[j]);
        };
#pragma unroll
        for (int s = 0; s < NST - 1; ++s) issue(s, s);
        auto step = [&](int i, auto phase) {
            constexpr int PH = decltype(phase)::value;
            // block i has landed when at most the loads of the NST-2 later blocks are still out
            wait_tile_loads<(NST - 2) * IPS>();
            use_stage(PH * STAGE, wave + 4 * i);
            // the operands are in registers: the stage takes this wavefront's block i + NST - 1
            issue(i + NST - 1, (PH + NST - 1) % NST);
        };
        for (int i0 = 0; i0 < mine; i0 += NST) {
            [&]<int... PH>(std::integer_sequence<int, PH...>) {
                ((i0 + PH < mine ? step(i0 + PH, std::integral_constant<int, PH>{}) : (void)0), ...);
            }(std::make_integer_sequence<int, NST>{});
        }
        wait_tile_loads<0>();   // the repeated loads of the last steps must have landed before LDS is used again
    } else {
        // lane = row * 4 + chunk as above, the swizzle applied to the LDS address
        const int r0 = lane / 4, ch = lane % 4;
        const uint32_t w_addr[2] = {ldsw + r0 * 64 + ((ch ^ swz_a(r0)) << 4), ldsw + (16 + r0) * 64 + ((ch ^ swz_a(16 + r0)) << 4)};
        // 16 bytes from element `off` of a matrix of `size` elements; what lies past its end reads as zero
        auto load8 = [](const uint16_t* base, size_t off, size_t size) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (off + 8 <= size) {
                __builtin_memcpy(&v, base + off, 16);   // an unaligned 16-byte load
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (off + e < size) v[e / 2] |= (uint32_t)base[off + e] << (16 * (e % 2));
            }
            return v;
        };
        const uint16_t* Ai = A + (size_t)bi * M * K;
        const uint16_t* Bi = B + (size_t)bi * K * N;
        const size_t size_a = (size_t)M * K, size_b = (size_t)K * N;
        size_t row_a[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int r = m0 + 16 * j + r0;
            row_a[j] = (size_t)(r < M ? r : M - 1) * K + 8 * ch;
        }
        struct Blk {
            u32x4 a[2], b[2];
        };
        auto load = [&](Blk& x, int i) {
            const int kb = wave + 4 * i;
            if (i >= mine) return;
#pragma unroll
            for (int j = 0; j < 2; ++j) x.a[j] = load8(Ai, row_a[j] + 32 * (size_t)kb, size_a);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int k = 32 * kb + 16 * j + r0;
                x.b[j] = load8(Bi, (size_t)(k < K ? k : K - 1) * N + n0 + 8 * ch, size_b);
            }
        };
        Blk x[2];
        load(x[0], 0);
        load(x[1], 1);
        auto step = [&](int i, auto phase) {
            constexpr int PH = decltype(phase)::value;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                *(LDS_AS u32x4*)(uintptr_t)(w_addr[j] + PH * STAGE) = x[PH].a[j];
                *(LDS_AS u32x4*)(uintptr_t)(w_addr[j] + PH * STAGE + 2048) = x[PH].b[j];
            }
            load(x[PH], i + 2);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // only this wavefront reads what it wrote
            use_stage(PH * STAGE, wave + 4 * i);
        };
        for (int i0 = 0; i0 < mine; i0 += 2) {
            step(i0, std::integral_constant<int, 0>{});
            if (i0 + 1 < mine) step(i0 + 1, std::integral_constant<int, 1>{});
        }
    }
    __syncthreads();
    // the partial results meet: [wavefront][group of four registers][lane] as 16 bytes each
    {
        float* part = (float*)smem;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            f32x4 t;
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = acc[0][4 * g + e] + acc[1][4 * g + e];
            *(f32x4*)(part + ((wave * 4 + g) * 64 + lane) * 4) = t;
        }
        __syncthreads();
        f32x4 t = *(const f32x4*)(part + ((0 * 4 + wave) * 64 + lane) * 4);
#pragma unroll
        for (int w = 1; w < 4; ++w) {
            const f32x4 u = *(const f32x4*)(part + ((w * 4 + wave) * 64 + lane) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] += u[e];
        }
        // registers 4 q .. 4 q + 3 of lane (l32, h) are c[m0 + l32][n0 + 8 q + 4 h .. + 3]
        const int m = m0 + l32, n = n0 + 8 * wave + 4 * h;
        const u32x2 v = {E::pack2(leaky(t[0], slope), leaky(t[1], slope)), E::pack2(leaky(t[2], slope), leaky(t[3], slope))};
        uint16_t* cp = Cb + (size_t)m * N + n;
        if constexpr (LOAD != 2) {
            if (m < M && n < N) *(u32x2*)cp = v;
        } else if (m < M) {
            if (n <= N - 4) {   // (n + 4 overflows where N is near 2^31)
                __builtin_memcpy(cp, &v, 8);   // an unaligned 8-byte store
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (n + e < N) cp[e] = (uint16_t)(v[e / 2] >> (16 * (e % 2)));
            }
        }
    }
}

// Any shape, one thread per element of c: the sizes that fit no tile and have too few products to pay for one
// (gemm_per_element).  Bound by the launch and by the loads of a and b, one element each; fp32 fused multiply-adds in the
// order of k.
template <int DT>
__global__ __launch_bounds__(256) void gemm_lrelu_element_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                                                uint16_t* __restrict__ C, long long total, int M, int N, int K,
                                                                float slope) {
    using E = Elem<DT>;
    for (long long idx = (long long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long long)gridDim.x * 256) {
        const int n = (int)(idx % N);
        const long long bm = idx / N;          // batch * M + m
        const long long bi = bm / M;
        const uint16_t* a = A + (size_t)bm * K;
        const uint16_t* b = B + (size_t)bi * K * N + n;
        float t = 0.f;
        for (int k = 0; k < K; ++k) t = __builtin_fmaf(E::widen(a[k]), E::widen(b[(size_t)k * N]), t);
        const uint32_t p = E::pack2(leaky(t, slope), 0.f);
        C[idx] = (uint16_t)(p & 0xFFFFu);
    }
}

template <int DT>
hipError_t launch_element(const GemmLaunch& g) {
    const uint16_t* a = (const uint16_t*)g.a;
    const uint16_t* b = (const uint16_t*)g.b;
    uint16_t* c = (uint16_t*)g.c;
    long long total = (long long)g.batch * g.M * g.N;
    int M = g.M, N = g.N, K = g.K;
    float slope = g.slope;
    const long long groups = (total + 255) / 256;
    const unsigned grid = (unsigned)(groups < 65536 ? groups : 65536);
    void* args[] = {&a, &b, &c, &total, &M, &N, &K, &slope};
    return hipLaunchKernel(reinterpret_cast<const void*>(&gemm_lrelu_element_kernel<DT>), dim3(grid), dim3(256), args, 0, (hipStream_t)g.stream);
}

// one workgroup of `threads` per tile of bm x bn; `told` as announce_lds has it
hipError_t launch_grid(const GemmLaunch& g, const void* fn, int bm, int bn, int threads, unsigned lds_bytes, std::atomic<uint64_t>& told) {
    GemmGrid grid = gemm_grid_of(g.batch, g.M, g.N, bm, bn);
    if (grid.y > 65535u) return hipErrorInvalidConfiguration;
    int order = bm == 256 ? gemm_order_of(grid, g.N, g.K) : GEMM_RUNS;
    const uint16_t* a = (const uint16_t*)g.a;
    const uint16_t* b = (const uint16_t*)g.b;
    uint16_t* c = (uint16_t*)g.c;
    int M = g.M, N = g.N, K = g.K;
    float slope = g.slope;
    void* args[] = {&a, &b, &c, &M, &N, &K, &grid.tiles_m, &grid.tiles_n, &grid.total, &order, &slope};
    if (const hipError_t e = announce_lds(fn, lds_bytes, told); e != hipSuccess) return e;
    return hipLaunchKernel(fn, dim3(grid.x, grid.y), dim3(threads), args, lds_bytes, (hipStream_t)g.stream);
}

template <int DT, int WM, int WN, int TM, int TN, int BK, int NST, int KS, bool KTAIL, bool ANY = false>
hipError_t launch_tiles(const GemmLaunch& g) {
    static std::atomic<uint64_t> told{0};   // per kernel instance: the devices whose runtime knows its LDS size
    return launch_grid(g, reinterpret_cast<const void*>(&gemm_lrelu_kernel<DT, WM, WN, TM, TN, BK, NST, KS, KTAIL, ANY>), 32 * TM * WM, 32 * TN * WN,
                       KS * WM * WN * 64, (unsigned)GemmLds<WM, WN, TM, TN, BK, NST, KS>::BYTES, told);
}

// 256 x 256 tiles
template <int DT, bool KTAIL>
hipError_t launch_wide(const GemmLaunch& g) {
    static std::atomic<uint64_t> told{0};
    return launch_grid(g, reinterpret_cast<const void*>(&gemm_lrelu_wide_kernel<DT, KTAIL>), 256, 256, 256, GEMM_NST * (256 * 64 + 32 * 512), told);
}

template <int DT, int LOAD>
hipError_t launch_splitk(const GemmLaunch& g) {
    static std::atomic<uint64_t> told{0};
    return launch_grid(g, reinterpret_cast<const void*>(&gemm_lrelu_splitk_kernel<DT, LOAD>), 32, 32, 256, 4u * GEMM_SK_NST * 4096u, told);
}

template <int DT, bool KTAIL>
hipError_t launch_tile_size(const GemmLaunch& g) {
    switch (gemm_tile_of(g.batch, g.M, g.N, g.K)) {
        case 1:                                                                // 256 x 256, eight wavefronts of 64 x 128 or four of 128 x 128
            return gemm_eight_waves(g.batch, g.M, g.N, g.K) ? launch_tiles<DT, 4, 2, 2, 4, 32, 4, 1, KTAIL>(g) : launch_wide<DT, KTAIL>(g);
        case 2:
            if (gemm_tiles_128x256(g.batch, g.M, g.N, g.K)) return launch_tiles<DT, 2, 4, 2, 2, 32, 4, 1, KTAIL>(g);   // eight wavefronts of 64 x 64
            if (gemm_two_parts(g.batch, g.M, g.N, g.K)) return launch_tiles<DT, 2, 2, 2, 2, 64, 4, 2, KTAIL>(g);       // twice four of 64 x 64
            return launch_tiles<DT, 2, 2, 2, 2, 32, GEMM_NST128, 1, KTAIL>(g);                                         // four of 64 x 64
        case 3:
            if (gemm_tiles_64x128(g.batch, g.M, g.N, g.K))                                                            // four of 32 x 64
                return g.K % 64 != 0 ? launch_tiles<DT, 2, 2, 1, 2, 64, 4, 1, true>(g) : launch_tiles<DT, 2, 2, 1, 2, 64, 4, 1, false>(g);
            if (gemm_long_blocks(g.batch, g.M, g.N, g.K)) return launch_tiles<DT, 2, 2, 1, 1, 64, 5, 1, false>(g);    // four of 32 x 32
            return gemm_deep(g.batch, g.M, g.N, g.K) ? launch_tiles<DT, 2, 2, 1, 1, 32, 6, 1, KTAIL>(g) : launch_tiles<DT, 2, 2, 1, 1, 32, 4, 1, KTAIL>(g);
        default: return launch_splitk<DT, KTAIL ? 1 : 0>(g);                  // 32 x 32, K split over the four wavefronts
    }
}
template <int DT>
hipError_t dispatch(const GemmLaunch& g) {
    const bool aligned = gemm_rows_aligned(g.N, g.K);
    if (aligned && g.K % 32 == 0) return launch_tile_size<DT, false>(g);
    if (gemm_per_element(g.batch, g.M, g.N, g.K)) return launch_element<DT>(g);
    if (aligned) return launch_tile_size<DT, true>(g);
    if (!gemm_unaligned_64(g.batch, g.M, g.N, g.K)) return launch_splitk<DT, 2>(g);
    return gemm_unaligned_blocks_64(g.batch, g.M, g.N, g.K) ? launch_tiles<DT, 2, 2, 1, 1, 64, 3, 1, false, true>(g) : launch_tiles<DT, 2, 2, 1, 1, 32, 3, 1, false, true>(g);
}

}  // namespace

hipError_t gemm_launch(const GemmLaunch& g) { return g.dtype == 0 ? dispatch<0>(g) : dispatch<1>(g); }
