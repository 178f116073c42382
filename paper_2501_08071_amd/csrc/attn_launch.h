// Internal: validated launch request handed from the C-ABI layer to the kernel dispatcher.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#ifndef ATTN_NW
#define ATTN_NW 8   // wavefronts per workgroup, each owning 32 query rows
#endif
#ifndef ATTN_PP_KEYS
#define ATTN_PP_KEYS 64   // keys per inner-loop block in the alternating-phase loop at D = 128 (32 or 64)
#endif
#ifndef ATTN_PP_KEYS_D64
#define ATTN_PP_KEYS_D64 (2 * ATTN_PP_KEYS)   // the same at D = 64 (32, 64 or 128), where a key costs half the matrix work and half the LDS: twice the keys per phase
#endif
#define ATTN_BC 32  // keys per inner-loop block in the interleaved loop
#ifndef ATTN_MAX_SLACK
#define ATTN_MAX_SLACK 15.0f  // log2 of the largest sum of a lane's softmax weights of one block tolerated before the reference maximum is moved
#endif
#ifndef ATTN_WARY
#define ATTN_WARY 16  // alternating-phase loop: after a reference maximum moved, blocks whose row maxima are taken before the weights
#endif
#ifndef ATTN_NBUF
#define ATTN_NBUF 8   // LDS buffers per tensor for blocks of up to 8 KiB (a power of two); larger blocks get half as many: 4 x 2 x 16 KiB = 128 KiB with the shipped blocks at D = 128 and 64, one workgroup per CU
#endif
#ifndef ATTN_BARRIER_EVERY
#define ATTN_BARRIER_EVERY 2  // key blocks per workgroup barrier (1 or 2)
#endif
#ifndef ATTN_PINGPONG
#define ATTN_PINGPONG 1  // D = 128 and 64: alternate matrix and vector phases between two groups of wavefronts
#endif
#ifndef ATTN_HEAD_GROUP
#define ATTN_HEAD_GROUP 4  // (b,h) pairs whose query tiles an XCD works on at the same time (0: no grouping)
#endif
#ifndef ATTN_FETCH
#define ATTN_FETCH 4  // units between the LDS read of an operand and the matrix instruction that uses it
#endif
#ifndef ATTN_PP_FETCH
#define ATTN_PP_FETCH 4  // alternating-phase loop: K operands of the next matrix phase read ahead, in the vector phase
#endif
#ifndef ATTN_F16_SUM_DOT
#define ATTN_F16_SUM_DOT 1  // binary16 at D = 64: row sums from the rounded weights, two per v_dot2c_f32_f16, at the end of the vector phase (0: from the fp32 weights, one addition each, as everywhere else)
#endif
#ifndef ATTN_PP_PRIO_M
#define ATTN_PP_PRIO_M 1  // alternating-phase loop: issue priority of a wavefront in its matrix phase ...
#endif
#ifndef ATTN_PP_PRIO_V
#define ATTN_PP_PRIO_V 0  // ... and in its vector phase (0 .. 3; equal: the priority is never touched)
#endif
#ifndef ATTN_DEBUG_POISON
#define ATTN_DEBUG_POISON 0  // debug build: an LDS buffer is filled with NaN patterns right before the load that overwrites it
#endif
#ifndef ATTN_WPE
#define ATTN_WPE 2  // wavefronts per SIMD the register budget is sized for
#endif

#ifndef ATTN_ROWS64
#define ATTN_ROWS64 0  // D = 128, problems that fill the chip: the kernel with 64 query rows per wavefront, one wavefront per SIMD
#endif
#ifndef ATTN64_NBUF
#define ATTN64_NBUF 8  // that kernel's LDS buffers of 32 keys per tensor
#endif

// Which loop a head dimension runs, the keys per inner-loop block and the LDS buffers per tensor that go with it.
constexpr bool attn_alternating(int D) { return ATTN_PINGPONG != 0 && (D == 128 || D == 64); }
// (the interleaved loop works on 32 keys at a time: each part of a workgroup brings 32 of its own)
constexpr int attn_block_keys(int D, int parts = 1) { return attn_alternating(D) ? (D == 64 ? ATTN_PP_KEYS_D64 : ATTN_PP_KEYS) : ATTN_BC * parts; }
constexpr int attn_buffers(int D, int parts = 1) { return attn_block_keys(D, parts) * D > 32 * 128 ? ATTN_NBUF / 2 : ATTN_NBUF; }   // blocks of more than 8 KiB: half as many (128 KiB in all with the shipped blocks, D = 128 and 64)
// Can the keys of a block be split between two halves of the wavefronts (32 keys for each at least)?
constexpr bool attn_can_split(int D) { return attn_alternating(D) ? attn_block_keys(D) >= 64 : D == 32; }

static_assert(ATTN_PP_KEYS == 32 || ATTN_PP_KEYS == 64, "block size of the alternating-phase loop");
static_assert(ATTN_PP_KEYS_D64 == 32 || ATTN_PP_KEYS_D64 == 64 || ATTN_PP_KEYS_D64 == 128, "block size of the alternating-phase loop at D = 64");

// Wavefronts per workgroup for a problem of BH (b,h) pairs and S rows: ATTN_NW (256 query rows per workgroup),
// or half of that when the larger tiles would leave at least half of the 256 compute units without a
// workgroup (the smaller workgroups also fit two to a compute unit at D = 32).
#ifndef ATTN_SMALL_TILES
#define ATTN_SMALL_TILES 128
#endif
inline int attn_pick_nw(long long BH, int S) {
    const long long tiles = BH * ((S + 32 * ATTN_NW - 1) / (32 * ATTN_NW));
    return tiles <= ATTN_SMALL_TILES ? ATTN_NW / 2 : ATTN_NW;
}

// Workgroups of half the rows: are the keys split too?  What it costs is the final addition (and, in it, the wait for loads
// nobody reads): worth it from a few blocks on.  Measured, us without -> with: D = 32, 8 heads: S = 64 3.5 -> 4.0, 200
// 5.2 -> 5.2, 333 6.5 -> 6.0, 512 7.8 -> 6.5; D = 64: S = 128 (one block) 5.9 -> 5.8, 200 7.9 -> 7.0, 512 9.2 -> 8.3;
// D = 128: S = 128 7.2 -> 8.3, 333 causal 10.9 -> 10.9, 512 12.7 -> 11.9, 2048 35.2 -> 27.9.  Over 488 problems it is done for (1
// to 128 heads, S up to 16384, with and without the causal mask) the time is 0.63 to 1.01 of the unsplit kernel's, the error
// of O against 64 bits (97 problems) 0.67 to 1.001 of it.
inline bool attn_splits_keys(long long BH, int S, int D) {
    return attn_can_split(D) && attn_pick_nw(BH, S) != ATTN_NW && S > (D == 128 ? 384 : D == 64 ? 128 : 256);
}

// Problems that do not fill the chip with large tiles: row groups (of 32 rows) per workgroup of the kernel whose wavefronts each
// stream keys of their own (attn_fwd_stream_gfx950.hip), or 0: not that kernel.  One group while that is one round of the 256
// compute units, two while that is; beyond it the larger workgroups above read less of K and V per row.  Under the mask, where
// the workgroups of a second round are the short ones, a little further.  Measured, us as before / one group / two (heads x S, 8
// wavefronts of the other kernels before): D = 128, 8 x 333 11.6 6.6 9.7, 8 x 1024 17.6 10.8 15.7, 1 x 4096 44.6 23.8 39.0,
// 16 x 1024 19.4 19.9 17.6, 32 x 1024 25.3 39.5 34.2; D = 64, 8 x 1024 12.3 8.0 9.9, 16 x 1024 12.6 13.9
// 10.4, 32 x 1024 14.8 26.0 19.5; D = 32, 8 x 1024 10.1 6.4 8.0, 4 x 4096 29.0 27.2 19.6, 8 x 4096 30.4 50.7 35.9.  With the mask:
// D = 128, 4 x 4096 46.6 32.0 40.3, 8 x 2887 37.6 37.1 33.5, 16 x 2048 31.5 38.2 33.8; D = 64, 4 x 4096 32.4
// 23.0 25.1, 6 x 1670 17.8 10.2 13.4, 32 x 512 9.8 9.0 7.9, 10 x 1701 18.9 16.7 14.6, 32 x 1024 14.1 19.7 15.3; D = 32, 8 x 4096 29.4 31.1
// 23.9, 32 x 1024 11.2 15.4 11.6.
// A single tile of up to 128 rows keeps four wavefronts, not for its time but because attn_kernel_name's answer for it is pinned
// (us with four wavefronts / streaming, one head, S = 1, 64, 128: D = 32 3.0 3.0, 3.2 3.1, 3.9 3.2; D = 64 6.3 3.4, 6.2 3.6, 5.7
// 3.7, the only problems at D = 64 that still take four wavefronts; D = 128 5.6 4.2, 5.4 4.5, 7.0 4.9).
inline bool attn_stream_wide_heads(long long BH, int S, bool causal, int groups);
inline int attn_stream_groups(long long BH, int S, int D, bool causal) {
    if (attn_pick_nw(BH, S) == ATTN_NW || (BH == 1 && S <= 128)) return 0;
    const long long n32 = BH * ((S + 31) / 32), n64 = BH * ((S + 63) / 64);
    if (n32 <= 256) return 1;
    if (D == 128) return attn_stream_wide_heads(BH, S, causal, 1) ? 1 : attn_stream_wide_heads(BH, S, causal, 2) ? 2 : 0;
    if (causal && n32 <= 512 && (S >= 2048 || (n32 <= 400 && S >= 640))) return 1;
    if (n64 <= 256 || (causal && (S >= 2048 ? n64 <= 512 : S >= 1000 && n64 <= 384))) return 2;
    return 0;
}

// The same at D = 128 past one round of single groups.  A key costs the most bytes there, so it counts how many XCDs read a head's K and
// V: workgroup b runs on XCD b % 8 and works on head b % BH, so one XCD does where BH is a multiple of 8, two where it is one of 4, all
// eight where it is odd.  Even numbers of heads are better off streaming from 320 keys on, shorter sequences only where few XCDs
// share a head, odd numbers only while the workgroups are few or the sequence is long.  Measured, us as before / one group / two, on
// either side: 60 x 256 11.7 12.6 11.6, 62 x 256 11.8 16.0 13.3; 24 x 512 13.9 14.0 12.4, 27 x 512 14.6 20.7 16.2; 17 x 600 15.2 16.7 14.0, 25 x
// 576 15.6 22.3 16.5; 15 x 1000 20.2 25.4 19.3; 110 x 100 9.1 11.2 10.2.  With the mask: 64 x 256 11.9 11.4 11.0, 55 x 256 11.6 13.0 11.8; 36 x 333 12.6
// 11.5 11.6, 33 x 333 12.6 13.1 12.5; 24 x 640 15.6 13.2 13.3, 25 x 640 15.9 17.2 15.3; 64 x 200 10.8 10.6 10.0, 62 x 200 11.0 12.3 11.6; 18 x 1000
// 19.5 20.3 18.6, 20 x 1000 19.7 20.8 20.4, 23 x 1000 20.8 29.9 24.1; 11 x 2000 29.7 33.0 28.0.
inline bool attn_stream_wide_heads(long long BH, int S, bool causal, int groups) {
    const long long tiles = BH * ((S + 32 * groups - 1) / (32 * groups));
    const bool even = BH % 2 == 0;
    if (groups == 1) return causal && S >= 256 && tiles <= (S >= 900 || (even && S > 320) ? 512 : S >= 480 ? 440 : even ? 340 : S > 320 ? 352 : 300);
    if (!causal)
        return tiles <= 256 && (S >= 780 || (S > 320 && tiles <= (even ? 256 : S > 512 ? 210 : 165)) || (S > 256 && even && tiles <= 170) || (S > 128 && BH % 4 == 0));
    if (tiles <= 256) return S >= 480 || (S >= 90 && S <= 160 && BH % 8 == 0) || (S > 192 && (BH % 4 == 0 || (even && tiles <= 140)));
    return S >= 1000 && tiles <= (S >= 2000 ? 384 : S >= 1400 ? 340 : S >= 1200 ? 320 : S >= 1100 ? 310 : 300);
}

struct AttnLaunch {
    const void* q;
    const void* k;
    const void* v;
    void* o;          // fp32, or the input type when o16 is set
    float* lse;       // may be null
    int BH, S, D;
    int causal;
    int dtype;        // 0 binary16, 1 bfloat16
    float c;          // |scale| * log2(e)
    uint32_t qsign;   // 0x80008000 when scale < 0 (sign folded into q), else 0
    int o16;          // write O rounded to the input type instead of fp32
    void* stream;
};

hipError_t attn_launch(const AttnLaunch& a);
hipError_t attn_launch_stream(const AttnLaunch& a, int groups);   // with that many row groups per workgroup
hipError_t attn_launch_rows64(const AttnLaunch& a);   // D = 128 only: 64 query rows per wavefront

// Does this problem take the kernel with 64 query rows per wavefront?  (Workgroups of 256 rows either way.)
inline bool attn_takes_rows64(long long BH, int S, int D) {
    return ATTN_ROWS64 != 0 && D == 128 && attn_pick_nw(BH, S) == ATTN_NW;
}
