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
#define ATTN_WARY 16  // alternating-phase loop, streaming kernel at D = 32 and 64: after a reference maximum moved, blocks whose row maxima are taken before the weights
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

// Can a grid of so many workgroups be launched?  The runtime takes fewer than 2^32 work-items.
constexpr bool attn_grid_fits(long long blocks, int threads) { return blocks <= 0xffffffffLL / threads; }

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
//
// Past ATTN_SMALL_TILES, D = 64 and 128.  With the mask the workgroup of a head's last rows takes as long as the whole launch while
// there is one for every compute unit at most: half the rows with twice the wavefronts each are 0.6 of that.  Without it, where a second
// round of 256-row tiles would hold a few only.  Measured, us with 256 rows / split: D = 64 with the mask, 6 x 5392 66 43, 22 x 1325 21.7 15.9,
// 12 x 4071 52 37, 19 x 3162 48.2 38.4, 14 x 5193 74 70, but 58 x 937 21.0 21.6, 43 x 1375 26.4 26.7, 33 x 2528 43 48; D = 128, 14 x 2797 53 40,
// 30 x 1500 34.4 32.4, 20 x 2949 60 56, but 40 x 1421 33.4 35.2, 26 x 2491 57 62.  Without the mask, D = 64, 55 x 1056 42.5 35.5, 10 x 7496 208 187,
// 141 x 363 21.7 19.3, but 297 x 233 19.0 23.7, 95 x 671 38.2 42.0, 33 x 2715 88 99; D = 128, 10 x 6495 276 205, 16 x 4380 194 186, 88 x 633 38.8 33.1, but 265 x 224 28 36.
inline bool attn_splits_wide(long long BH, int S, int D, bool causal) {
    const long long tiles = BH * ((S + 255) / 256), n128 = BH * ((S + 127) / 128);
    if (causal) return D == 64 ? (tiles <= 256 && S >= 1150) || (tiles <= 320 && S >= 5000)
                               : D == 128 && ((tiles <= 190 && S >= 1450) || (tiles <= 250 && S >= 2000));
    if (tiles <= 256) return false;
    return D == 64 ? (n128 <= 512 && S >= 360) || (tiles <= 300 && S >= 3500) : D == 128 && ((n128 <= 512 && S >= 500) || (tiles <= 310 && S >= 4000));
}
inline bool attn_splits_keys(long long BH, int S, int D, bool causal) {
    if (!attn_can_split(D)) return false;
    if (attn_pick_nw(BH, S) == ATTN_NW) return ATTN_NW == 8 && attn_splits_wide(BH, S, D, causal);
    return S > (D == 128 ? 384 : D == 64 ? 128 : 256);
}

// Problems that do not fill the chip with large tiles: row groups (of 32 rows) per workgroup of the kernel whose wavefronts each
// stream keys of their own (attn_fwd_stream_gfx950.hip), or 0: not that kernel.  One group while that is one round of the 256
// compute units, two while that is; beyond it the larger workgroups above read less of K and V per row.  Under the mask, where
// the workgroups of a second round are the short ones, a little further.  Measured, us with 128 rows (keys split or not) / one group / two (heads x
// S): D = 128, 8 x 333 11.1 6.3 9.5, 8 x 1024 17.3 10.0 15.1, 1 x 4096 44.1 23.0 36.3, 16 x 1024 18.3 18.7 16.7, 32 x 1024 23.5 35.0 31.3; D = 64, 8 x 1024 11.7 6.5 9.5,
// 16 x 1024 12.2 10.1 9.9, 32 x 1024 14.2 17.7 19.2; D = 32, 8 x 1024 9.6 5.5 7.4, 4 x 4096 28.4 18.9 18.6, 8 x 4096 29.5 34.5 30.2.  With the mask: D = 128, 4 x 4096
// 44.9 29.4 37.6, 8 x 2887 35.6 33.6 30.4, 16 x 2048 30.0 35.5 31.5; D = 64, 4 x 4096 31.7 18.1 24.0, 6 x 1670 16.7 9.0 13.2, 32 x 512 9.8 6.5 8.1, 10 x 1701 17.8 11.3
// 14.4, 32 x 1024 14.3 13.7 15.3; D = 32, 8 x 4096 29.1 20.5 21.8, 32 x 1024 11.0 10.0 9.5.
// A single tile of up to 128 rows keeps four wavefronts, not for its time but because attn_kernel_name's answer for it is pinned
// (us with four wavefronts / streaming, one head, S = 1, 64, 128: D = 32 3.0 3.0, 3.2 3.1, 3.9 3.2; D = 64 6.3 3.4, 6.2 3.6, 5.7
// 3.7, the only problems at D = 64 that still take four wavefronts; D = 128 5.6 4.2, 5.4 4.5, 7.0 4.9).
//
// At D = 32, and at 64 with one group, two workgroups share a compute unit, so a round is 512 of them; the lines of those two for few
// tiles stand in attn_stream_few_tiles, past ATTN_SMALL_TILES in attn_stream_many_tiles.
inline bool attn_stream_wide_heads(long long BH, int S, bool causal, int groups);
inline int attn_stream_few_tiles(long long BH, int S, int D, bool causal);
inline int attn_stream_many_tiles(long long BH, int S, int D, bool causal);
inline int attn_stream_groups(long long BH, int S, int D, bool causal) {
    if (attn_pick_nw(BH, S) == ATTN_NW) return ATTN_NW == 8 ? attn_stream_many_tiles(BH, S, D, causal) : 0;
    if (BH == 1 && S <= 128) return 0;
    if (BH * ((S + 31) / 32) <= 256) return 1;
    if (D == 128) return attn_stream_wide_heads(BH, S, causal, 1) ? 1 : attn_stream_wide_heads(BH, S, causal, 2) ? 2 : 0;
    return attn_stream_few_tiles(BH, S, D, causal);
}

// D = 32 and 64, more than 256 single groups.  One group halves a workgroup's chain and its registers (two workgroups to a compute unit: 512
// are a round), two read K and V half as often.  Which XCDs read a head counts for that: workgroup b runs on XCD b % 8; with one group or the mask
// it works on head b % BH, so that with an odd number of heads every XCD reads every head, with an even one that is no multiple of
// four every other, while without the mask two groups have whole heads to an XCD.  Times of one over the other, geometric mean (least .. most), three
// sets of buffers in turn:
//   D = 64, no mask, one group / two, n64 <= 256: up to 96 keys 0.90 (0.86 .. 0.93); 97 to 128 and multiples of four heads 0.90 (0.87 .. 0.92), others up to 320 groups 0.90
//   (0.86 .. 0.98), with more 1.10 (0.91 .. 1.18); 129 to 256 and multiples of four heads 0.95 (0.84 .. 0.99), other even numbers up to 320 groups 0.95
//   (0.93 .. 0.99), with more 1.09 (0.90 .. 1.22), odd ones 1.15 (0.87 .. 1.36).  Longer ones, where a wavefront has more than
//   one block: 0.95 (0.89 .. 1.02), 1.00, 1.13, but peaked logits lose up to 9 % of that, and with two blocks an exact largest weight now and
//   then (bfloat16, error of O up to 1.03 times that of two groups, whose rows move together): two groups.
//   D = 64 with the mask, one group / two, n32 <= 512: 0.77 (0.61 .. 1.04), but odd numbers of heads with 225 to 320 keys and more than 300 groups 1.02 (1.00 .. 1.07).  One group /
//   keys split, up to 690 groups: even numbers of heads from 289 keys on 0.76 (0.55 .. 1.01), odd ones from 513 on 0.75 (0.56 .. 1.00), between 1.00 (0.93 .. 1.10).
//     Beyond that two groups / keys split, up to 512 pairs from 1985 keys on 0.82 (0.70 .. 1.00), up to 384 from 1000 on 0.93 (0.82 .. 1.07).
//   D = 32, no mask: two groups while they are one to a compute unit (one group / two 0.99, 0.88 .. 1.21); then, up to 512 groups, one group / keys split 0.82 (0.69
//   .. 1.00), with more 1.00 (0.87 .. 1.27).
//   D = 32 with the mask, one group / two, n64 <= 256: 0.80 (0.67 .. 0.97); up to 512 with more than 1100 keys 0.92 (0.70 .. 1.10), and 0.67 (0.44 .. 0.92) of
//   split keys.  Two groups / keys split, up to 512 pairs of 321 to 1100 keys: even numbers of heads 0.86 (0.73 .. 0.99), odd ones with up to 384 0.94
//   (0.92 .. 0.97), with 385 to 512 1.01 (0.94 .. 1.07), with more 0.90 (0.76 .. 1.01); up to 320 keys 0.98 (0.94 .. 1.00).
inline int attn_stream_few_tiles(long long BH, int S, int D, bool causal) {
    const long long n32 = BH * ((S + 31) / 32), n64 = BH * ((S + 63) / 64);
    const bool even = BH % 2 == 0;
    if (!causal) {
        if (D == 64 && n64 <= 256 && S <= 256 && (S <= 96 || BH % 4 == 0 || (n32 <= 320 && (even || S <= 128)))) return 1;
        return n64 <= 256 ? 2 : D == 32 && n32 <= 512 && S > 256 ? 1 : 0;
    }
    if (D == 64) {
        if (n32 <= 512) return even || S <= 224 || S > 320 || n32 <= 300 || n64 > 256 ? 1 : 2;
        if (n32 <= 690 && S > (even ? 288 : 512)) return 1;
        return (S > 1984 && n64 <= 512) || (S >= 1000 && n64 <= 384) ? 2 : 0;
    }
    if (n64 <= 256 || (n64 <= 512 && S > 1100)) return 1;
    return n64 <= 512 && S > 320 && (even || S <= 384 || S > 512) ? 2 : 0;
}

// More than ATTN_SMALL_TILES tiles of 256 rows.  A tile takes the whole launch's time where there is about one for every compute
// unit, more so under the mask, and its rows past the end of the sequence take as long as the others; workgroups of 32 or 64 rows, two to a
// compute unit, even that out, but read K and V four or eight times as often.  So they pay while the tiles are one round, unevenly filled, while many of their
// rows do not exist, or while the last round is mostly empty.  At the lines: time streamed over 256 rows, geometric mean (least .. most), 4500
// problems, three sets of buffers in turn.
inline int attn_stream_many_tiles(long long BH, int S, int D, bool causal) {
    const long long t = (S + 255) / 256, tiles = BH * t, n64 = BH * ((S + 63) / 64), n32 = BH * ((S + 31) / 32);
    // (past the launch limit for its workgroups a problem keeps the larger tiles)
    if (D == 64) {
        if (!attn_grid_fits(n32, 64 * ATTN_NW)) return 0;
        if (S <= 96) return 1;                       // up to 32 keys 0.32 (0.26 .. 0.38), to 64 0.60 (0.50 .. 0.69), to 96 0.77 (0.60 .. 1.01)
        // 0.97 (0.94 .. 1.10) up to 550 groups, 1.07 (0.92 .. 1.27) above; past a round of tiles 0.77 (0.73 .. 0.82) up to 1200, 0.92 (0.73 .. 1.09) above
        if (S <= 128) return n32 <= 550 || (tiles > 256 && n32 <= 1200) ? 1 : 0;
        return S <= 160 && n32 <= 800 ? 1 : 0;       // 0.89 (0.82 .. 0.94), with more 0.95 (0.73 .. 1.22)
    }
    if (D != 32 || !attn_grid_fits(n64, 64 * ATTN_NW)) return 0;
    const long long last = (tiles - 1) % 256;                                        // tiles of the last round, less one
    auto waste = [&](int percent) { return t * 25600 >= (100LL + percent) * S; };    // so many percent of rows past the end, at least
    if (causal) {
        // 0.63 (0.39 .. 0.98); an odd number of heads, which every XCD reads, up to 1500 pairs 0.57 (0.37 .. 1.03), between 0.90 (0.76 .. 1.13), beyond 1.03 (0.81 ..
        // 1.27), even ones beyond 0.92 (0.76 .. 1.25)
        if (S >= 1200 && n64 <= (BH % 2 == 0 ? 2000 : 1500)) return 2;
        // up to three quarters of a round of tiles 0.54 (0.37 .. 0.94), above 0.61 (0.44 .. 1.06); shorter sequences 1.01 (0.60 .. 1.36)
        if (tiles <= 256) return S >= (n64 <= 768 ? 480 : 512) ? 2 : 0;
        // from 480 keys on 0.85 (0.73 .. 1.01), 257 to 384 0.80 (0.63 .. 0.96), 100 to 128 0.89 (0.80 .. 0.97), 129 to
        // 256 up to a round and a half 0.89 (0.79 .. 1.05), with more tiles 1.09 (0.94 .. 1.20), 385 to 479 where the last round is at most half full 0.88 (0.78 .. 1.01),
        // else 1.01 (0.95 .. 1.10); with less waste 0.99 (0.76 .. 1.34)
        return waste(15) && (S >= 480 || (S > 256 ? S <= 384 || last < 128 : S >= 100 && (S <= 128 || tiles <= 384))) ? 2 : 0;
    }
    // one round of pairs 0.75 (0.56 .. 0.89), three quarters of a round of tiles 0.78 (0.56 .. 0.90), else 1.02 (0.84 .. 1.39)
    if (tiles <= 256) return S >= 256 && n64 <= (S >= 1200 ? 768 : 512) ? 2 : 0;
    // 0.82 (0.51 .. 1.05).  Whole rounds of whole tiles are as fast with 256 rows, which read K and V a quarter as often: 0.99 (0.92 .. 1.07) with up to 5 % of waste, with more
    // 0.95 (0.91 .. 1.00).  (us, binary16, 256 rows / streamed: 64 x 2048 63.5 61.0, 128 x 1024 32.7 34.8, 32 x 4096 106.4 107.5, 8 x 16384 405 396, 256 x 512 21.0 24.2.)
    if (S >= 1000) return last >= 248 && !waste(5) ? 0 : 2;
    if (S >= 500) return waste(last < 192 ? 5 : 20) ? 2 : 0;    // 0.84 (0.61 .. 1.02), others of that length 0.96 (0.83 .. 1.14)
    return S > 256 && waste(5) && tiles <= 340 ? 2 : 0;         // 0.74 (0.65 .. 0.89); more tiles 0.93 (0.76 .. 1.20), shorter 1.03 (0.83 .. 1.38)
}

// The same at D = 128 past one round of single groups.  A key costs the most bytes there, so it counts how many XCDs read a head's K and
// V.  Without the mask two groups have a run of whole heads to an XCD (workgroup b runs on XCD b % 8), whatever the number of heads: while the pairs are one round they are
// 0.87 of the time of 128 rows (0.82 .. 1.00; 1000 problems of more than 128 keys, odd numbers of heads 0.86, multiples of four 0.88), with up to 128 keys 1.00 (0.95 .. 1.07), in a
// second round 1.52 (1.39 .. 1.69).  us, 128 rows / two groups: 17 x 600 14.5 12.0, 25 x 576 14.7 12.6, 23 x 700 16.3 14.8, 27 x 512 13.6 11.9, 41 x 333 12.8 10.8, 62 x 256 11.2 10.2.
// With the mask a workgroup works on head b % BH, so one XCD reads a head where BH is a multiple of 8, two where it is one of 4, all
// eight where it is odd.  Even numbers of heads are better off streaming from 320 keys on, shorter sequences only where few XCDs
// share a head, odd numbers only while the workgroups are few or the sequence is long.  Measured, us as before / one group / two, on
// either side: 64 x 256 11.9 11.4 11.0, 55 x 256 11.6 13.0 11.8; 36 x 333 12.6
// 11.5 11.6, 33 x 333 12.6 13.1 12.5; 24 x 640 15.6 13.2 13.3, 25 x 640 15.9 17.2 15.3; 64 x 200 10.8 10.6 10.0, 62 x 200 11.0 12.3 11.6; 18 x 1000
// 19.5 20.3 18.6, 20 x 1000 19.7 20.8 20.4, 23 x 1000 20.8 29.9 24.1; 11 x 2000 29.7 33.0 28.0.
inline bool attn_stream_wide_heads(long long BH, int S, bool causal, int groups) {
    const long long tiles = BH * ((S + 32 * groups - 1) / (32 * groups));
    const bool even = BH % 2 == 0;
    if (groups == 1) return causal && S >= 256 && tiles <= (S >= 900 || (even && S > 320) ? 512 : S >= 480 ? 440 : even ? 340 : S > 320 ? 352 : 300);
    if (!causal) return tiles <= 256 && S > 128;
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
