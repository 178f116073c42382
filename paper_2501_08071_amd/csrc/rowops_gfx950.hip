// Row softmax and RMS normalisation for gfx950: the paper's two memory-bound kernels (Table 2).
//
// Both are bound by HBM: every element is read once and written once, 4 bytes of traffic per element
// and a handful of fp32 operations.  So the whole design is about the memory side:
//   * a row of 8 to 65536 elements stays in registers between its read and its write: one pass over
//     HBM, not two or three;
//   * every lane moves 16 bytes per instruction and neighbouring lanes neighbouring addresses, so a
//     wavefront's load or store is 1 KiB of consecutive bytes (whole 128-byte lines where the row length
//     is a multiple of 8);
//   * short rows (rmsnorm over a head dimension of 64 is 128 bytes) share a wavefront, TPR lanes per
//     row, so that the instruction stays 1 KiB wide; long rows take a whole workgroup;
//   * reductions run across the TPR lanes with cross-lane moves, across the wavefronts of a
//     workgroup through LDS.
// Rows shorter than 8 or longer than 65536 elements go through a general path that reads the row two
// (rmsnorm) or three (softmax) times with 2-byte accesses.
#include <hip/hip_runtime.h>
#include <cstdint>

#include "gfx950_common.h"
#include "rowops_launch.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 __attribute__((aligned(2))) u32x4_any;   // at any even address

constexpr float LOG2E = 1.4426950408889634f;

template <int DT>
__device__ __forceinline__ float widen(uint16_t b) {
    if (DT == 0) return (float)__builtin_bit_cast(_Float16, b);
    return __builtin_bit_cast(float, (uint32_t)b << 16);
}
// round to nearest even into the 16-bit type (finite values; binary16 overflows to infinity)
template <int DT>
__device__ __forceinline__ uint16_t narrow(float f) {
    return (uint16_t)gfx950::Elem<DT>::pack2(f, 0.f);
}
// 16 bytes of a row
__device__ __forceinline__ u32x4 load16(const uint16_t* p) { return *(const u32x4_any*)p; }
// Ordinary stores.  Non-temporal ones make this kernel faster where x comes from beyond the L2 and y fits it (16 MiB each: 6.6 us
// instead of 8.4), but whoever reads y next finds it in no cache: a copy of y right after takes 0.3 us (4 MiB) to 11 us (64
// MiB: 54 us for both instead of 44) longer, and on new buffers of 256 MiB this kernel itself 105 us instead of 94.
__device__ __forceinline__ void store16(uint16_t* p, u32x4 v) { *(u32x4_any*)p = v; }
template <int DT>
__device__ __forceinline__ void widen8(const u32x4& p, float (&f)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = widen<DT>((uint16_t)(p[i] & 0xFFFFu));
        f[2 * i + 1] = widen<DT>((uint16_t)(p[i] >> 16));
    }
}
template <int DT>
__device__ __forceinline__ u32x4 narrow8(const float (&f)[8]) {
    u32x4 p;
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = gfx950::Elem<DT>::pack2(f[2 * i], f[2 * i + 1]);
    return p;
}

struct Max {
    static __device__ __forceinline__ float op(float a, float b) { return gfx950::vmax(a, b); }
};
struct Sum {
    static __device__ __forceinline__ float op(float a, float b) { return a + b; }
};

// Reduction over the TPR threads that share a row (TPR <= 64: lanes of one wavefront; TPR > 64: the
// whole workgroup, `red` holds one float per wavefront and row), of U independent rows at once.  Every
// thread gets the results.
template <class R, int TPR, int U>
__device__ __forceinline__ void reduce_rows(float (&v)[U], float (*red)[TPR > 64 ? TPR / 64 : 1]) {
    constexpr int W = TPR < 64 ? TPR : 64;
#pragma unroll
    for (int off = W / 2; off >= 1; off >>= 1)
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = R::op(v[u], __shfl_xor(v[u], off, 64));
    if constexpr (TPR > 64) {
        constexpr int NW = TPR / 64;
        if ((threadIdx.x & 63) == 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) red[u][threadIdx.x >> 6] = v[u];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float t[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) t[w] = red[u][w];
#pragma unroll
            for (int h = NW / 2; h >= 1; h >>= 1)
#pragma unroll
                for (int w = 0; w < h; ++w) t[w] = R::op(t[2 * w], t[2 * w + 1]);
            v[u] = t[0];
        }
    }
}

// Registers path.  OP 0: softmax, 1: rmsnorm.  TPR threads share a row, each holds CH chunks of 8
// elements: chunk c of thread t covers elements 8 (c TPR + t) .. +7, so the TPR threads of a row read
// 16 TPR consecutive bytes per instruction.  BLOCK / TPR rows per workgroup at a time, and U such groups
// per step, all their loads issued before the first is used: the bytes in flight are what hides the
// latency of HBM.
// TAIL: the row length is at least 8 but no multiple of it.  Rows then start at any even address (the
// accesses are unaligned, which costs a 128-byte line more per KiB), and the last chunk of a row moves back
// to the row's last eight elements: its first `dup` ones are also the previous chunk's, are left out of
// the sums, and are stored twice with the same value.
// Measured (us a launch, three sets of buffers in turn; general path, or aligned rows of the kernel before, in brackets): softmax 4097 x
// 4095 13.6 (32), 2048 x 32768 58 (166), rmsnorm 33588 x 999 27.6 (93), 1048576 x 64 49.1 = 5470 GB/s (50.3), 16777 x 1000 12.0 (13.9).
template <int DT, int OP, int TPR, int CH, int U, bool TAIL>
__global__ __launch_bounds__(TPR > 64 ? TPR : 256) void rowop_reg_kernel(const uint16_t* x, const uint16_t* __restrict__ w,
                                                                         uint16_t* y, long long n_rows, int n, float eps) {
    constexpr int BLOCK = TPR > 64 ? TPR : 256, RPW = BLOCK / TPR;
    __shared__ float red[2][U][TPR > 64 ? TPR / 64 : 1];
    const int t = threadIdx.x % TPR, rin = threadIdx.x / TPR;
    const int c8 = TAIL ? (n + 7) >> 3 : n >> 3;
    // element offset of a chunk, and how many of its leading elements belong to the chunk before it
    auto offset = [&](int chunk) { return TAIL && chunk == c8 - 1 ? n - 8 : 8 * chunk; };
    auto dup = [&](int chunk) { return TAIL && chunk == c8 - 1 ? 8 * c8 - n : 0; };
    auto sum8 = [&](int chunk, float s, auto term) {
        if (TAIL && chunk == c8 - 1) {
#pragma unroll
            for (int i = 0; i < 8; ++i) s = i >= dup(chunk) ? term(i, s) : s;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) s = term(i, s);
        }
        return s;
    };

    // rmsnorm's weights: held for all the rows of this thread, or, where they would not fit the registers next to a row (1024
    // threads have 128 each), read again for every row
    constexpr bool HOLD = OP == 1 && CH < 8;
    auto weights = [&](int c) {
        const int chunk = c * TPR + t;
        int off = offset(chunk);
        if constexpr (!HOLD) asm volatile("" : "+v"(off));   // computed here, not kept as an address per chunk over the loop
        u32x4 g = {0u, 0u, 0u, 0u};
        if (chunk < c8) g = load16(w + off);
        return g;
    };
    u32x4 wr[HOLD ? CH : 1];
    if constexpr (HOLD) {
#pragma unroll
        for (int c = 0; c < CH; ++c) wr[c] = weights(c);
    }

    int turn = 0;   // which of the two LDS slots the next workgroup-wide reduction uses
    for (long long row0 = (long long)blockIdx.x * (RPW * U); row0 < n_rows; row0 += (long long)gridDim.x * (RPW * U)) {
        u32x4 raw[U][CH];
        bool ok[U][CH];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long row = row0 + u * RPW + rin;
            const uint16_t* xr = x + (size_t)row * n;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int chunk = c * TPR + t;
                ok[u][c] = row < n_rows && chunk < c8;
                // outside the row: zeros do not count in rmsnorm's sum, minus infinity neither in softmax's
                constexpr uint32_t NONE = OP == 1 ? 0u : DT == 0 ? 0xfc00fc00u : 0xff80ff80u;
                raw[u][c] = u32x4{NONE, NONE, NONE, NONE};
                if (ok[u][c]) raw[u][c] = load16(xr + offset(chunk));
            }
        }
        auto store_row = [&](int u, int c, const float (&f)[8]) {
            if (ok[u][c]) store16(y + (size_t)(row0 + u * RPW + rin) * n + offset(c * TPR + t), narrow8<DT>(f));
        };
        if constexpr (OP == 0) {
            float v[U][CH][8];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int c = 0; c < CH; ++c) widen8<DT>(raw[u][c], v[u][c]);
            float m[U], s[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                m[u] = v[u][0][0];
#pragma unroll
                for (int c = 0; c < CH; ++c)
#pragma unroll
                    for (int i = 0; i < 8; ++i) m[u] = gfx950::vmax(m[u], v[u][c][i]);
            }
            reduce_rows<Max, TPR, U>(m, red[turn]);
            turn ^= 1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                s[u] = 0.f;
#pragma unroll
                for (int c = 0; c < CH; ++c) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[u][c][i] = __builtin_amdgcn_exp2f((v[u][c][i] - m[u]) * LOG2E);
                    s[u] = sum8(c * TPR + t, s[u], [&](int i, float s) { return s + v[u][c][i]; });
                }
            }
            reduce_rows<Sum, TPR, U>(s, red[turn]);
            turn ^= 1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float inv = 1.0f / s[u];
#pragma unroll
                for (int c = 0; c < CH; ++c) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[u][c][i] *= inv;
                    store_row(u, c, v[u][c]);
                }
            }
        } else {
            float ss[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                ss[u] = 0.f;
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    float f[8];
                    widen8<DT>(raw[u][c], f);
                    ss[u] = sum8(c * TPR + t, ss[u], [&](int i, float s) { return __builtin_fmaf(f[i], f[i], s); });
                }
            }
            reduce_rows<Sum, TPR, U>(ss, red[turn]);
            turn ^= 1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float r = 1.0f / __builtin_sqrtf(ss[u] / (float)n + eps);
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    // widened again: held as they came, a row and its weights take half the registers
                    float f[8], g[8];
                    widen8<DT>(raw[u][c], f);
                    if constexpr (HOLD) widen8<DT>(wr[c], g);
                    else widen8<DT>(weights(c), g);
#pragma unroll
                    for (int i = 0; i < 8; ++i) f[i] = f[i] * r * g[i];
                    store_row(u, c, f);
                }
            }
        }
    }
}

// General path: one workgroup per row, 2-byte accesses, the row is read again for every pass.
template <int DT, int OP>
__global__ __launch_bounds__(256) void rowop_gen_kernel(const uint16_t* x, const uint16_t* __restrict__ w,
                                                       uint16_t* y, long long n_rows, int n, float eps) {
    __shared__ float red[2][1][4];
    int turn = 0;
    auto reduce_row = [&]<class R>(R, float v) {
        float a[1] = {v};
        reduce_rows<R, 256, 1>(a, red[turn]);
        turn ^= 1;
        return a[0];
    };
    for (long long row = blockIdx.x; row < n_rows; row += gridDim.x) {
        const uint16_t* xr = x + (size_t)row * n;
        uint16_t* yr = y + (size_t)row * n;
        if constexpr (OP == 0) {
            float m = -3.0e38f;
            for (int j = threadIdx.x; j < n; j += 256) {
                const float f = widen<DT>(xr[j]);
                m = f > m ? f : m;
            }
            m = reduce_row(Max{}, m);
            float s = 0.f;
            for (int j = threadIdx.x; j < n; j += 256) s += __builtin_amdgcn_exp2f((widen<DT>(xr[j]) - m) * LOG2E);
            s = reduce_row(Sum{}, s);
            const float inv = 1.0f / s;
            // y may be x: every thread rewrites only the elements it alone reads in this pass, and all
            // reads of the earlier passes lie before the barrier of the second reduction
            for (int j = threadIdx.x; j < n; j += 256)
                yr[j] = narrow<DT>(__builtin_amdgcn_exp2f((widen<DT>(xr[j]) - m) * LOG2E) * inv);
        } else {
            float ss = 0.f;
            for (int j = threadIdx.x; j < n; j += 256) {
                const float f = widen<DT>(xr[j]);
                ss = __builtin_fmaf(f, f, ss);
            }
            ss = reduce_row(Sum{}, ss);
            const float r = 1.0f / __builtin_sqrtf(ss / (float)n + eps);
            for (int j = threadIdx.x; j < n; j += 256) yr[j] = narrow<DT>(widen<DT>(xr[j]) * r * widen<DT>(w[j]));
        }
    }
}

template <int DT, int OP, int TPR, int CH, int U, bool TAIL>
hipError_t launch_reg(const RowopLaunch& a) {
    constexpr int BLOCK = TPR > 64 ? TPR : 256, RPW = (BLOCK / TPR) * U;
    constexpr long long FIT = 2048LL * 256 / BLOCK;   // 2048 threads per compute unit: all that fit, then a stride
    long long groups = (a.n_rows + RPW - 1) / RPW;
    const unsigned grid = (unsigned)(groups < FIT ? groups : FIT);
    const uint16_t* x = (const uint16_t*)a.x;
    const uint16_t* w = (const uint16_t*)a.w;
    uint16_t* y = (uint16_t*)a.y;
    long long n_rows = a.n_rows;
    int n = a.n;
    float eps = a.eps;
    void* args[] = {&x, &w, &y, &n_rows, &n, &eps};
    return hipLaunchKernel(reinterpret_cast<const void*>(&rowop_reg_kernel<DT, OP, TPR, CH, U, TAIL>), dim3(grid), dim3(BLOCK), args,
                           0, (hipStream_t)a.stream);
}

template <int DT, int OP>
hipError_t launch_gen(const RowopLaunch& a) {
    const unsigned grid = (unsigned)(a.n_rows < 2048 ? a.n_rows : 2048);
    const uint16_t* x = (const uint16_t*)a.x;
    const uint16_t* w = (const uint16_t*)a.w;
    uint16_t* y = (uint16_t*)a.y;
    long long n_rows = a.n_rows;
    int n = a.n;
    float eps = a.eps;
    void* args[] = {&x, &w, &y, &n_rows, &n, &eps};
    return hipLaunchKernel(reinterpret_cast<const void*>(&rowop_gen_kernel<DT, OP>), dim3(grid), dim3(256), args, 0,
                           (hipStream_t)a.stream);
}

// Threads per row, chunks per thread and rows per step by row length and number of rows: many rows want bytes in flight
// per thread and few barriers, few rows want as many wavefronts as there can be.  All times in microseconds.
// Rows within a wavefront: four groups per step where that still makes 1024 workgroups, else one (softmax 8192 x 256:
// 2.8 with one, 3.5 with four).
template <int DT, int OP, int TPR, int CH, bool TAIL>
hipError_t launch_short(const RowopLaunch& a) {
    return a.n_rows >= 1024LL * 4 * (256 / TPR) ? launch_reg<DT, OP, TPR, CH, 4, TAIL>(a) : launch_reg<DT, OP, TPR, CH, 1, TAIL>(a);
}

template <int DT, int OP, bool TAIL>
hipError_t dispatch_reg(const RowopLaunch& a) {
    const int c8 = (a.n + 7) / 8;   // 16-byte chunks per row
    const long long rows = a.n_rows;
    if (c8 <= 8) return launch_short<DT, OP, 8, 1, TAIL>(a);
    if (c8 <= 16) return launch_short<DT, OP, 16, 1, TAIL>(a);
    if (c8 <= 32) return launch_short<DT, OP, 32, 1, TAIL>(a);
    if (c8 <= 64) return launch_short<DT, OP, 64, 1, TAIL>(a);
    // two chunks for a wavefront, not one for four: 65536 x 515 takes 26, not 57
    if (c8 <= 128) return launch_short<DT, OP, 64, 2, TAIL>(a);
    // rmsnorm 30000 x 1601: 34 with 64 threads a row, 37 with 256; softmax 512 x 2048 would have half the workgroups
    if (c8 <= 256) return rows >= 4096 ? launch_reg<DT, OP, 64, 4, 1, TAIL>(a) : launch_reg<DT, OP, 256, 1, 1, TAIL>(a);
    // softmax 512 x 4096: 3.6 with two rows per step, 3.1 with one; rmsnorm 16384 x 4095: 51 and 56
    if (c8 <= 512) return rows >= 8192 ? launch_reg<DT, OP, 256, 2, 2, TAIL>(a) : launch_reg<DT, OP, 256, 2, 1, TAIL>(a);
    if (c8 <= 1024) {
        // rmsnorm 512 x 8192: 4.6 with 512 threads, 4.9 with 1024; 2796 x 6000: 11.5 and 13.1; 8192 x 8192: 48.4 and 48.2; unaligned 8193 x
        // 8191: 58 and 52.  15978 x 4200 leaves half of 1024 threads without work: 56, 51 with 256 and two rows.  softmax 512 x
        // 8192: 5.1 with 512, 5.7 with 256 and two rows; 3994 x 4200: 15.9 and 14.6; 8193 x 8191: 59 and 52
        if (rows < (OP == 1 && !TAIL ? 8192 : 2048)) return launch_reg<DT, OP, 512, 2, 1, TAIL>(a);
        if (OP == 0 || c8 <= 640) return launch_reg<DT, OP, 256, 4, 2, TAIL>(a);
        if constexpr (OP == 1) return launch_reg<DT, OP, 1024, 1, 1, TAIL>(a);
    }
    if (c8 <= 2048) {
        // softmax 1398 x 12000: 11.5 with 512 threads, 15.9 with 1024, 12.8 with 256; 1198 x 14000: 11.8, 13.7, 12.0; unaligned 1397 x
        // 9001: 11.2, 15.0, 12.6.  rmsnorm 5592 x 12000: 52.9 with 512, 50.0 with 1024; unaligned 1397 x 9001: 12.0 and 15.0, 209 x 10003: 4.6
        // and 4.2
        if constexpr (OP == 0 || TAIL) {
            if (OP == 0 || rows >= 400) return c8 <= 1536 ? launch_reg<DT, OP, 512, 3, 1, TAIL>(a) : launch_reg<DT, OP, 512, 4, 1, TAIL>(a);
        }
        if constexpr (OP == 1) return launch_reg<DT, OP, 1024, 2, 1, TAIL>(a);
    }
    if (c8 <= 4096) return launch_reg<DT, OP, 1024, 4, 1, TAIL>(a);
    return launch_reg<DT, OP, 1024, 8, 1, TAIL>(a);   // c8 <= 8192 = ROWOPS_MAX_REG_ROW / 8
}
template <int DT, int OP>
hipError_t dispatch(const RowopLaunch& a) {
    if (a.n < 8 || a.n > ROWOPS_MAX_REG_ROW) return launch_gen<DT, OP>(a);
    return a.n % 8 == 0 ? dispatch_reg<DT, OP, false>(a) : dispatch_reg<DT, OP, true>(a);
}

}  // namespace

hipError_t rowop_launch(const RowopLaunch& a) {
    if (a.dtype == 0) return a.op == 0 ? dispatch<0, 0>(a) : dispatch<0, 1>(a);
    return a.op == 0 ? dispatch<1, 0>(a) : dispatch<1, 1>(a);
}
