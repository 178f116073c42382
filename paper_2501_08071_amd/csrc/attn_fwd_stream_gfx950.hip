// Attention forward for problems that do not fill the chip evenly with tiles of 128 or 256 query rows (attn_stream_groups): every
// wavefront streams keys of its own, and the parts of a row are put together at the end.
//
// What bounds such a problem is latency: the launch, a chain over the keys, the loads it waits for (1.4 us from the request of a
// block to its arrival).  So a workgroup owns only RG groups of 32 consecutive query rows of one (b,h), and all its wavefronts
// (two halves of NH) work on all of them, wavefront w on the key blocks (32 keys) w, w + 2 NH, ...: the chain of a row is 2 NH
// times shorter than the number of its blocks, all compute units have work, and the loop has no barrier.
//   * K and V blocks go straight from global memory into LDS (global_load_lds_dwordx4), into buffers of the wavefront's own: one
//     per tensor at D = 128, as many as row groups at 64, two at 32.  A block's buffer is loaded again as soon as its operands are
//     in registers.  (K straight into the operand registers, 32 rows of 32 bytes per instruction, was twice as slow: 8 heads x
//     1024, D = 128 18.9 us, 10.8 by way of LDS.)
//   * At D = 32, and at 64 with one row group, that is 64 KiB and at most 128 registers, so that two workgroups share a compute
//     unit: four wavefronts to a SIMD fill each other's waits, one workgroup's start and end overlap with the other's loop, and the
//     kernel also serves problems of several rounds (us, with twice the buffers and two wavefronts to a SIMD -> so: D = 32, 6 x 6422
//     74 -> 61, with the mask 41 -> 34, 18 x 7992 276 -> 227; D = 64, 8 x 1024 7.2 -> 6.4, 20 x 1041 with the mask 15.1 -> 10.9).
//   * q is read once per workgroup and kept in registers (D = 128 with two groups: in LDS).
//   * An operand read from LDS feeds the matrix instructions of all RG row groups.
// Registers and the transposed formulation are those of attn_fwd_gfx950.hip: a lane holds values of one query row only, the
// weights of a block go from the accumulators straight into the second product.
//
// The end: every wavefront leaves accumulators, row sum and reference maximum in LDS, one barrier, and every wavefront adds up
// its share of the columns against the largest reference.  That and the start are 3.5 (D = 32) to 4.8 us (D = 128), with two
// groups 4.2 to 7 us.
//
// Measured in turn, two wavefronts for every 32 rows that share blocks -> this kernel (us, heads x S): D = 128, 8 x 333 with the mask 10.9 ->
// 6.3; D = 64, 8 x 1024 11.8 -> 6.6; D = 32, 4 x 4096 29.2 -> 19.5 (18.0 where nothing else runs in between).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include <utility>

#include "attn_launch.h"
#include "gfx950_common.h"
#include "attn_device.h"

namespace {

using namespace gfx950;
using namespace attn_device;

extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];

template <int D, int RG, int NW>
struct StreamLds {
    static constexpr int BLK = 32 * 2 * D;                            // one block of K or V
    // buffers per wavefront and tensor: 64 KiB in all where the registers let two workgroups share a compute unit, else 128 KiB
    static constexpr int BUFS = D == 128 ? 1 : D == 64 ? RG : 2;
    static constexpr int WAVE = 2 * BUFS * BLK;                       // a wavefront's K buffers, then its V buffers
    static constexpr int Q = NW * WAVE, STREAM = Q + RG * BLK;
    static constexpr int PASS = 4 * 32 / D < RG ? 4 * 32 / D : RG;    // the end: row groups added up at a time,
    static constexpr int PART = PASS * 32 * D * 4;                    // the accumulators of a wavefront in such a pass,
    static constexpr int STATS = NW * PART;                           // then {reference, row sum} by part, group and row
    static constexpr int MERGE = STATS + NW * RG * 32 * 8;
    static constexpr int BYTES = STREAM > MERGE ? STREAM : MERGE;
    static_assert(BYTES <= 160 * 1024 && RG % PASS == 0, "LDS");
};

template <int DT, int D, bool CAUSAL, int RG, int NH>
__global__ __launch_bounds__(NH * 128) __attribute__((amdgpu_waves_per_eu(RG * D <= 64 ? 4 : 2)))
void attn_fwd_halves_stream_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                            void* __restrict__ o, float* __restrict__ lse, int S, int BH, int nqt, float c, uint32_t qsign, int o16) {
    using E = Elem<DT>;
    using L = StreamLds<D, RG, 2 * NH>;
    constexpr int NW = 2 * NH, BUFS = L::BUFS, BLK = L::BLK;
    constexpr int KSTEPS = D / 16, DB = D / 32, ROWB = 2 * D, CPR = D / 8;
    constexpr int RPI = 1024 / ROWB, IPT = 32 / RPI;   // rows per direct-to-LDS load instruction, instructions per block
    constexpr bool QLDS = RG * D >= 256;               // q stays in LDS where the registers are short of room for it
    // binary16 at D = 64: row sums from the rounded weights (as in attn_fwd_gfx950.hip)
    constexpr bool SUM_DOT = ATTN_F16_SUM_DOT != 0 && DT == 0 && D == 64;

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Workgroup -> rows.  (b,h) fastest: workgroups that read the same K and V are BH apart, and with BH a multiple of 8 on one
    // XCD; under the causal mask the longest rows first.  With two groups and no mask an XCD (workgroup b runs on XCD b % 8) gets a
    // run of whole heads instead, so that its L2 holds what its workgroups read (us before -> after: D = 128, 13 x 1188 22.3 -> 19.0,
    // D = 64, 9 x 1518 13.3 -> 12.1; D = 32, 18 x 7992 238 -> 227, 4 x 4096 the same).  Under the mask that takes the long rows
    // from the front: 1.1 to 1.4 times the time.
    int bh, qt;
    if (CAUSAL || RG == 1) {
        bh = (int)blockIdx.x % BH;
        qt = (int)blockIdx.x / BH;
        if (CAUSAL) qt = nqt - 1 - qt;
    } else {
        const int x = (int)blockIdx.x & 7, each = (int)gridDim.x >> 3, more = (int)gridDim.x & 7;   // (the first `more` XCDs have one more)
        const int item = x * each + (x < more ? x : more) + ((int)blockIdx.x >> 3);
        bh = item / nqt;
        qt = item - bh * nqt;
    }
    const int q0 = qt * (32 * RG);
    const size_t head = (size_t)bh * S * D;
    const uint16_t* kh = k + head;
    const uint16_t* vh = v + head;
    const int kv_end = CAUSAL && q0 + 32 * RG < S ? q0 + 32 * RG : S;
    const int nblk = (kv_end + 31) / 32;

    const uint32_t lds0 = (uint32_t)(uintptr_t)(LDS_AS uint8_t*)smem;
    const uint32_t ldsw = lds0 + wave * L::WAVE;

    // Load instruction i of the 32 rows from row0 on (row0 < S, a multiple of 32), with the bank-conflict swizzle on the global
    // side.  The instructions' offsets differ in the swizzle bits that come from i and in whole rows.  Rows past the end of the
    // sequence are copies of the last one (masked, or never stored); a block that has none skips the arithmetic for them (D = 32, 4 x 4096 18.5 ->
    // 18.0 us, 8 heads x 1024 at D = 64 6.5 -> 6.4).
    constexpr int XM = D == 128 ? 3 : D == 64 ? 1 : 0;
    const uint32_t off0 = (uint32_t)((lane / CPR) * ROWB + (((lane % CPR) ^ swz<D>(lane / CPR)) << 4));
    auto load_piece = [&](const uint16_t* src, int i, int past, uint32_t dst) {
        if constexpr (ATTN_DEBUG_POISON != 0) {
            // Debug build: NaN patterns where this load will land, so that an operand read before its block has landed (a wait that
            // counts too few loads), or after its buffer was given away, shows in the output.
            lds_write_b128(dst + 16 * lane, u32x4{0x7fff7fffu, 0x7fff7fffu, 0x7fff7fffu, 0x7fff7fffu});
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        lds_dma16(dst, src, (off0 ^ ((i & XM) << 4)) + (uint32_t)((i * RPI - past) * ROWB));
    };
    auto load_rows = [&](const uint16_t* base, int row0, int i, uint32_t dst) {
        const int over = row0 + i * RPI + lane / CPR - (S - 1);
        load_piece(base + (size_t)row0 * D, i, over > 0 ? over : 0, dst);
    };
    auto load_block = [&](const uint16_t* base, int j, uint32_t dst) {
        if (32 * j + 32 <= S) {
            // (debug build: keeps the compiler from sharing the first write with the other path, so that each path's loads have their own)
            if constexpr (ATTN_DEBUG_POISON != 0) asm volatile("; a whole block" ::: "memory");
#pragma unroll
            for (int i = 0; i < IPT; ++i) load_piece(base + (size_t)j * (32 * D), i, 0, dst + i * 1024);
        } else {
#pragma unroll
            for (int i = 0; i < IPT; ++i) load_rows(base, 32 * j, i, dst + i * 1024);
        }
    };
    // The loads land in the order of issue: Q, K(0), V(0), K(1), V(1), ... (blocks of this wavefront); to wait for one is to
    // count what was issued after it.
    auto wait_blocks = [&](int later) {
        [&]<int... N>(std::integer_sequence<int, N...>) {
            ((later == N ? wait_lds_dma<N * IPT>() : (void)0), ...);
        }(std::make_integer_sequence<int, 2 * BUFS + 1>{});
    };
    constexpr int QI = RG * IPT;   // load instructions of Q, dealt out to the wavefronts
#pragma unroll
    for (int i = 0; i < (QI + NW - 1) / NW; ++i)
        if (i * NW + wave < QI) load_rows(q + head, q0, i * NW + wave, lds0 + L::Q + (i * NW + wave) * 1024);
    const int mine = wave < nblk ? (nblk - wave + NW - 1) / NW : 0;   // blocks of this wavefront
#pragma unroll
    for (int b = 0; b < BUFS; ++b)
        if (b < mine) {
            load_block(kh, wave + b * NW, ldsw + b * BLK);
            load_block(vh, wave + b * NW, ldsw + (BUFS + b) * BLK);
        }

    f32x16 acc[RG][DB];
    float m_ref[RG], l_run[RG];
#pragma unroll
    for (int g = 0; g < RG; ++g) {
        m_ref[g] = -3.402823466e38f;
        l_run[g] = 0.f;
#pragma unroll
        for (int i = 0; i < DB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[g][i][r] = 0.f;
    }
    // operand addresses in the first buffers, as in attn_fwd_gfx950.hip
    uint32_t kaddr[KSTEPS], vaddr[2][DB];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) kaddr[ks] = ldsw + l32 * ROWB + (((2 * ks + h) ^ swz<D>(l32)) << 4);
    {
        const int x = (lane & 15) >> 2, y = lane & 3, g1 = (lane >> 4) & 1;
#pragma unroll
        for (int hi = 0; hi < 2; ++hi)
#pragma unroll
            for (int i = 0; i < DB; ++i) {
                const int row = 8 * hi + 4 * h + x, chunk = 4 * i + 2 * g1 + (y >> 1);
                vaddr[hi][i] = ldsw + BUFS * BLK + row * ROWB + ((chunk ^ swz<D>(row)) << 4) + ((y & 1) << 3);
            }
    }

    wait_blocks(2 * (mine < BUFS ? mine : BUFS));
    __syncthreads();   // all of Q
    const uint32_t qbase = lds0 + L::Q - ldsw;
    // a negative scale is folded into the sign of q (exact)
    auto read_q = [&](int g, int ks) { return lds_read_b128(kaddr[ks] + qbase + g * BLK) ^ qsign; };
    u32x4 qf[QLDS ? 1 : RG][KSTEPS];
    if constexpr (!QLDS) {
#pragma unroll
        for (int g = 0; g < RG; ++g)
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) qf[g][ks] = read_q(g, ks);
    }

    constexpr int WARY = D == 128 ? 0 : ATTN_WARY;   // (at D = 128 the code for it costs 2 to 4 % of the shortest calls)
    int wary = 0;  // blocks still to go whose row maxima are taken before the weights
    bool watched = false;   // is this block one of them?  (from a move on also for the row group that comes after)
    // The largest sum of a lane's weights that leaves the reference where it is.  Besides range a move gains that the largest weight of
    // every row is one and loses nothing to rounding.  Rows that move in groups of 32 (and not, as at D = 64 with two groups, of 64) are
    // moved less often, and in a chain of few blocks no later move makes up for it: there they have less slack.  Error of O against 64 bits
    // over that of rows moving in groups of 64, 2500 problems with logits peaked 1.5- to 8-fold: with ATTN_MAX_SLACK throughout 0.88 on average, 379
    // problems above 1.001, up to 1.92 (lse 1.61), 44 % of those with two blocks to a wavefront and none with six or more; so 0.73, five
    // above 1.001, 1.04 at most (lse 1.008).  Flat logits (standard normal) do not reach the limit; 2^5 they do now and then, which costs a launch of one
    // round 5 to 8 %, and with 2^7 the error is 0.75, eleven above 1.001.
    const float limit = RG * D <= 64 && mine <= 6 ? __builtin_exp2f(6.0f) : __builtin_exp2f(ATTN_MAX_SLACK);
    int buf = 0;   // byte offset of the block's buffers
#pragma unroll 1
    for (int it = 0; it < mine; ++it) {
        const int j = wave + it * NW, left = mine - 1 - it;   // blocks still to come
        // ---- S = K Q^T ----
        // (the usual count without the search through all of them: D = 32, 4 x 4096 18.9 -> 18.0 us)
        if (left >= BUFS - 1) wait_lds_dma<(2 * BUFS - 1) * IPT>();
        else wait_blocks(1 + 2 * left);
        f32x16 s[RG];
        {
            u32x4 kf[KSTEPS];
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) kf[ks] = lds_read_b128(kaddr[ks] + buf);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before the buffer is loaded again
            if (left >= BUFS) load_block(kh, j + BUFS * NW, ldsw + buf);
#pragma unroll
            for (int g = 0; g < RG; ++g) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[g][r] = 0.f;
#pragma unroll
                for (int ks = 0; ks < KSTEPS; ++ks) {
                    if constexpr (QLDS) s[g] = E::mfma(kf[ks], read_q(g, ks), s[g]);
                    else s[g] = E::mfma(kf[ks], qf[g][ks], s[g]);
                }
            }
        }
        // ---- weights ----
        // Masked logits become -3e38; a row that sees nothing of the block (under the mask, in all but the last group) takes its
        // reference from a floor just above them, so that its weights are zeros.
        const bool cut = (CAUSAL && j * 32 + 31 > q0) || j * 32 + 32 > S;
        if (cut) {
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                const int row = q0 + 32 * g + l32;
                const int lim = (CAUSAL && row < S ? row : S - 1) - j * 32 - 4 * h;
#pragma unroll
                for (int r = 0; r < 16; ++r) s[g][r] = 8 * (r / 4) + r % 4 > lim ? -3.0e38f : s[g][r];
            }
        }
        // the reference policy of attn_fwd_gfx950.hip: the true maxima of the first block, moved only when the weights outgrow it;
        // after that, for ATTN_WARY blocks, moved to every new maximum before the weights are taken (the code for it costs flat logits 3 %, D = 32, 4 x 4096 17.4
        // -> 18.0 us; 144 problems with peaked logits: 0.98 of the time of doing without, and the error of O against 64 bits, where a row's largest weight is exactly one, 0.81 of
        // what it was instead of 0.94)
        auto look = [&](int g) {
            // vmax and vmax3 are asm, for which the compiler does not wait out a matrix instruction's latency
            asm volatile("s_nop 15\n\ts_nop 7" : "+v"(s[g]));
            float mx = vmax3(s[g][0], s[g][1], s[g][2]);
#pragma unroll
            for (int t = 1; t < 7; ++t) mx = vmax3(mx, s[g][2 * t + 1], s[g][2 * t + 2]);
            mx = vmax(mx, s[g][15]);
            float m = vmax(mx, other_half(mx)) * c;    // c >= 0
            if (CAUSAL && RG > 1 && cut) m = vmax(m, -2.99999e38f * c);
            return m > m_ref[g] ? m : m_ref[g];
        };
        u32x4 pf[RG][2];
        float psum[RG];
        auto weights = [&](int g) {
            psum[g] = 0.f;
            f32x16 p;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                p[r] = __builtin_amdgcn_exp2f(fmaf(s[g][r], c, -m_ref[g]));
                if (r % 2 == 1) pf[g][r / 8][(r % 8) / 2] = E::pack2(p[r - 1], p[r]);
                if (!SUM_DOT) psum[g] += p[r];
            }
            if constexpr (SUM_DOT) {
#pragma unroll
                for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) psum[g] = E::dot2_ones(pf[g][tt][e], psum[g]);
            }
        };
        auto move = [&](int g, float m_new) {
            const float alpha = __builtin_amdgcn_exp2f(m_ref[g] - m_new);
            m_ref[g] = m_new;
            l_run[g] *= alpha;
#pragma unroll
            for (int i = 0; i < DB; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[g][i][r] *= alpha;
            wary = WARY;
            watched = WARY > 0;
        };
        if (it == 0) {
#pragma unroll
            for (int g = 0; g < RG; ++g) m_ref[g] = look(g);
        }
        watched = WARY > 0 && wary > 0;
        wary -= watched;
        // One group after the other at D = 32, where four wavefronts share a SIMD: the scores of the first need no registers any more in
        // the second's turn (4 x 4096 19.5 -> 18.0 us).  Both together where two do (one by one 5 % slower at D = 64).
        constexpr int TOGETHER = D == 32 ? 1 : RG;
#pragma unroll
        for (int g0 = 0; g0 < RG; g0 += TOGETHER) {
            bool outgrown = false;
#pragma unroll
            for (int g = g0; g < g0 + TOGETHER; ++g) {
                if (watched) {
                    const float m_new = look(g);
                    if (__builtin_amdgcn_ballot_w64(m_new != m_ref[g]) != 0) move(g, m_new);
                }
            }
#pragma unroll
            for (int g = g0; g < g0 + TOGETHER; ++g) {
                weights(g);
                outgrown |= !(psum[g] <= limit);
            }
            if (__builtin_amdgcn_ballot_w64(outgrown) != 0) {
#pragma unroll
                for (int g = g0; g < g0 + TOGETHER; ++g) {
                    move(g, look(g));
                    weights(g);
                }
            }
        }
#pragma unroll
        for (int g = 0; g < RG; ++g) l_run[g] += psum[g];
        // ---- O += V^T P ----
        if (left >= BUFS) wait_lds_dma<(2 * BUFS - 1) * IPT>();
        else wait_blocks(2 * left);
        u32x4 va[2][DB];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int i = 0; i < DB; ++i) {
                const u32x2 lo = lds_read_tr16(vaddr[0][i] + buf + 16 * tt * ROWB), hi = lds_read_tr16(vaddr[1][i] + buf + 16 * tt * ROWB);
                va[tt][i] = u32x4{lo[0], lo[1], hi[0], hi[1]};
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before the buffer is loaded again
        if (left >= BUFS) load_block(vh, j + BUFS * NW, ldsw + BUFS * BLK + buf);
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int i = 0; i < DB; ++i) acc[g][i] = E::mfma(va[tt][i], pf[g][tt], acc[g][i]);
        if (BUFS > 1) buf = buf == (BUFS - 1) * BLK ? 0 : buf + BLK;
    }

    // ---- the parts of a row are put together (a wavefront without a block adds zeros) ----
    // a unit: eight columns of a row group, four of them in each half
    constexpr int UNITS = L::PASS * DB * 4, PER = UNITS < NW ? 1 : UNITS / NW;
    static_assert(UNITS < NW || PER * NW == UNITS, "the wavefronts share the columns evenly");
#pragma unroll
    for (int g0 = 0; g0 < RG; g0 += L::PASS) {
        wait_lds_dma<0>();
        __syncthreads();   // nobody reads or loads what is overwritten now
#pragma unroll
        for (int g = g0; g < g0 + L::PASS; ++g) {
#pragma unroll
            for (int i = 0; i < DB; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    *(f32x4*)(smem + wave * L::PART + ((((g - g0) * DB + i) * 4 + e) * 64 + lane) * 16) =
                        f32x4{acc[g][i][4 * e], acc[g][i][4 * e + 1], acc[g][i][4 * e + 2], acc[g][i][4 * e + 3]};
            const float l_tot = l_run[g] + other_half(l_run[g]);
            if (h == 0) *(f32x2*)(smem + L::STATS + ((wave * RG + g) * 32 + l32) * 8) = f32x2{m_ref[g], l_tot};
        }
        __syncthreads();
        if (wave * PER >= UNITS) continue;
        const int g = g0 + wave * PER / (DB * 4);
        const int row = q0 + 32 * g + l32;
        f32x2 st[NW];
#pragma unroll
        for (int p = 0; p < NW; ++p) st[p] = *(const f32x2*)(smem + L::STATS + ((p * RG + g) * 32 + l32) * 8);
        float m_all = st[0][0], l_all = 0.f;
#pragma unroll
        for (int p = 1; p < NW; ++p) m_all = fmaxf(m_all, st[p][0]);
#pragma unroll
        for (int p = 0; p < NW; ++p) {
            st[p][0] = __builtin_amdgcn_exp2f(st[p][0] - m_all);
            l_all = fmaf(st[p][0], st[p][1], l_all);
        }
        const float inv = 1.0f / l_all;
#pragma unroll
        for (int t = 0; t < PER; ++t) {
            const int u = wave * PER + t;
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < NW; ++p) {
                const f32x4 y = *(const f32x4*)(smem + p * L::PART + (u * 64 + lane) * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = fmaf(st[p][0], y[e], x[e]);
            }
            const size_t at = head + (size_t)row * D + 8 * (u % (DB * 4)) + 4 * h;
            if (row < S) {
                if (o16 == 0) *(f32x4*)((float*)o + at) = f32x4{x[0] * inv, x[1] * inv, x[2] * inv, x[3] * inv};
                else *(u32x2*)((uint16_t*)o + at) = u32x2{E::pack2(x[0] * inv, x[1] * inv), E::pack2(x[2] * inv, x[3] * inv)};
            }
        }
        if (lse != nullptr && h == 0 && wave * PER % (DB * 4) == 0 && row < S)
            lse[(size_t)bh * S + row] = (m_all + __builtin_amdgcn_logf(l_all)) * 0.6931471805599453f;
    }
}

template <int DT, int D, bool CAUSAL, int RG>
hipError_t launch(const AttnLaunch& a) {
    constexpr int NH = ATTN_NW / 2, BR = 32 * RG;
    int nqt = (a.S + BR - 1) / BR;
    const long long blocks = (long long)nqt * a.BH;
    if (!attn_grid_fits(blocks, NH * 128)) return hipErrorInvalidConfiguration;
    const uint16_t *q = (const uint16_t*)a.q, *k = (const uint16_t*)a.k, *v = (const uint16_t*)a.v;
    void* o = a.o;
    float* lse = a.lse;
    int S = a.S, BH = a.BH, o16 = a.o16;
    float c = a.c;
    uint32_t qsign = a.qsign;
    void* args[] = {&q, &k, &v, &o, &lse, &S, &BH, &nqt, &c, &qsign, &o16};
    const void* fn = reinterpret_cast<const void*>(&attn_fwd_halves_stream_kernel<DT, D, CAUSAL, RG, NH>);
    constexpr unsigned lds_bytes = StreamLds<D, RG, 2 * NH>::BYTES;
    static std::atomic<uint64_t> told{0};   // per kernel instance: the devices whose runtime knows its LDS size
    if (const hipError_t e = announce_lds(fn, lds_bytes, told); e != hipSuccess) return e;
    return hipLaunchKernel(fn, dim3((unsigned)blocks), dim3(NH * 128), args, lds_bytes, (hipStream_t)a.stream);
}

}  // namespace

hipError_t attn_launch_stream(const AttnLaunch& a, int groups) {
#define STREAM_CASE(DT, DD, RG) \
    if (a.dtype == DT && a.D == DD && groups == RG) return a.causal ? launch<DT, DD, true, RG>(a) : launch<DT, DD, false, RG>(a);
#define STREAM_CASES(DD, RG) STREAM_CASE(0, DD, RG) STREAM_CASE(1, DD, RG)
    STREAM_CASES(32, 1)
    STREAM_CASES(32, 2)
    STREAM_CASES(64, 1)
    STREAM_CASES(64, 2)
    STREAM_CASES(128, 1)
    STREAM_CASES(128, 2)
#undef STREAM_CASE
    return hipErrorInvalidValue;
}
