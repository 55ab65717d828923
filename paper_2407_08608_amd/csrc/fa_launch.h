// Host-side launch entry points, one per kernel family.  H_kv is the number of key/value heads
// (H for ordinary multi-head attention; a divisor of H for multi-query / grouped-query attention).  Each validates nothing (the C ABI
// layer has done that), enqueues on `stream`, and returns an fa_status.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

#include "../../include/fa_mi355.h"

namespace fa {

// Whether an fp32 forward is short enough for fa_fwd_f32_short_kernel.
inline bool f32_short(int N) { return N <= 32; }

// Whether N rows make an odd number of 128-row tiles.
inline bool odd_row_tiles(int N) { return ((N + 127) / 128) & 1; }

// Whether a causal forward launch pairs its query tiles (query_tiles in fa_device.h).  Pairs all take the same time, so
// they are the better choice when they fill whole rounds of the chip; what decides is the share of the rounds that is
// work (a pair without a partner, the middle tile of an odd number, counts half).  A round is one workgroup on each of
// the 256 CUs while 256 per_cu pairs take them all, `per_cu` on each beyond.  (A fitted number with the rest of a rule: the
// workgroups that a CU holds, but one less for the four-wave tiles, 16-bit and FP8 d = 64, whose rules were drawn when
// they took more registers.)  Against
// single tiles dealt longest first pairs win from `share` on, with up to `most_tiles` tiles: where two or three workgroups
// share a CU, single tiles even out by themselves.  With `many_heads` heads or more pairs win from `many_share` on: single
// tiles read the K and V of all heads at once, which costs most where few rows share a read.  On at most one workgroup per
// CU single tiles lose to pairs only over long sequences (most of all a few very long ones, which pairs finish as soon on
// two thirds of the chip), unless a CU holds but one.
// Causal, bf16 unless said, us, pairs / single tiles (share, heads x N):
//   ping-pong     1.00 151 / 159 (128 x 2048), 0.88 67.8 / 71.6 (56 x 2048), 0.84 53.9 / 56.1 (72 x 1408), 0.75 197 / 209
//                 (12 x 8192);  0.75 176 / 154 (64 x 3001), 0.25 99.5 / 90.1 (8 x 4096)
//   d = 128, 4w   1.00 78.8 / 79.5 (512 x 512), 0.83 87.5 / 102 (640 x 512), 0.85 223 / 225 (390 x 1183);  0.94 59.5 / 53.4
//                 (96 x 1200: lost), 0.75 29.0 / 24.8 (256 x 384: lost);  0.86 120 / 102 (160 x 1300), 0.69 134 / 120 (192 x 1300)
//   d = 256       1.00 79.7 / 94.1 (256 x 512), 1.00 107 / 115 (128 x 1024), 0.81 441 / 536 (224 x 1664), 0.83 227 / 301
//                 (512 x 640);  0.88 243 / 223 (32 x 3500: lost), 0.88 648 / 593 (80 x 3500: lost)
//   FP8 d = 128   1.00 96.6 / 101 (128 x 2048);  0.83 163 / 148 (128 x 2500), 0.75 126 / 106 (64 x 3001)
//   FP8 d = 256   1.00 118 / 125 (256 x 1024);  0.75 588 / 486 (48 x 6000)
//   d = 64, 8w    0.75 308 / 323 (6 x 16384), 1.00 on half the slots 167 / 180 (16 x 8192);  1.00 158 / 155 (64 x 4096: never
//                 beyond one per CU)
//   d = 64, 4w    1.00 28.7 / 29.4 (768 x 256), 1.00 32.2 / 33.0 (384 x 512);  1.00 52.2 / 48.7 (64 x 2048: up to 4 tiles, FP8 2)
// Over 4500 causal shapes of the four-wave 16-bit tiles as they are the rule is 0.1 % (d = 64) and 0.5 % (d = 128) off the better
// of the two on average; at d = 128 one shape in 23 is more than 2 % off, 21 % at worst.  The other kernels' rules were
// drawn on 4400 shapes, up to 0.5 % off on average, by kernel, before the key splits took the shapes of few heads.
struct PairRule {
    int per_cu;
    float share;
    int many_heads;
    float many_share;
    int most_tiles;
};
constexpr int kAny = 0x7fffffff;
inline bool pair_causal_tiles(long heads, int n_qtiles, const PairRule& rule) {
    constexpr long kCus = 256;
    if (n_qtiles < 2) return true;  // nothing to deal out: items, in runs of heads per XCD (FP8 1024 x 100 17.1 / 17.8)
    const long pairs = heads * ((n_qtiles + 1) / 2);
    const long slots = pairs <= kCus * rule.per_cu ? kCus : kCus * rule.per_cu, rounds = (pairs + slots - 1) / slots;
    const float work = (float)(heads * n_qtiles) / (float)(2 * slots * rounds);
    if (pairs <= kCus && (n_qtiles >= 32 || rule.per_cu > 1))
        return rule.per_cu < 3 && n_qtiles >= 16 && work >= (n_qtiles >= 32 ? 2.f / 3 : 7.f / 8);
    return n_qtiles <= rule.most_tiles && work >= (heads >= rule.many_heads ? rule.many_share : rule.share);
}

// How a forward launch is divided goes to its kernel in two arguments, `paired` and `total_wg`:
//   0  single query tiles: the number of work items (the 128-row 16-bit tiles: of heads, query_tiles)
//   1  causal pairs of tiles: the number of work items
//   2, 3  key splits, by FewForward (fa_fwd.hip) or FewFp8Forward (fa_fwd_fp8.hip): few_split(), log2 of the groups into which a
//      head's tiles go so that the XCDs get the same number of groups each, or -1: no groups, where they would come out too
//      uneven (few tiles; all are on the chip at once)
constexpr int kFewForward = 2, kFewForward8 = 3;  // (by as many waves as the kernel's tiles have; by eight where those have four)
inline int few_split(long heads, int N) {
    if (heads % 8 == 0) return 0;
    return N <= 32 * 32 ? -1 : heads % 4 == 0 ? 1 : heads % 2 == 0 ? 2 : 3;
}

// How often workgroups of 32 queries fill the CUs, by what the rules below go, and the tiles of 32 rows of a head.
struct KeySplitFill {
    long tiles;
    float fillings;
    KeySplitFill(long heads, int N) : tiles((N + 31) / 32) {
        const int split = few_split(heads, N);
        const long round_up = (1L << (split > 0 ? split : 0)) - 1;
        fillings = (float)(heads * ((tiles + round_up) & ~round_up)) / 256.f;
        if (split < 0 && fillings > 1.f) fillings *= 1.15f;  // an XCD's share of the tiles cuts through heads
    }
    bool at(float base, float step, float most) const {  // at most that many: more with a longer chain
        const float x = base + (float)tiles / step;
        return fillings <= (x < most ? x : most);
    }
};

// Whether a 16-bit forward is divided so: workgroups of 32 queries whose waves split the keys, against 128 or 256 queries that
// walk all of them.  What counts is how often those workgroups fill the CUs (`fillings`) and how long the chain of 32-key
// tiles is that they shorten; under a causal mask, where the large workgroups wait for their longest, they win further.
// The kernel stays the same (fa_fwd_kernel_name): this is only its work.  bf16, us, large / these, heads x N:
//   d = 64   no mask: 72 x 96 5.8 / 4.9, 32 x 512 10.1 / 8.1, 16 x 1400 21.0 / 16.6, 1 x 4096 50 / 19.5;
//            lost: 72 x 256 7.4 / 8.1, 24 x 1400 25.9 / 27.4;  N <= 64: equal to 2 %
//            causal:  32 x 512 10.9 / 7.1, 16 x 2000 29.6 / 18.4, 8 x 4096 54 / 32;  lost: 24 x 3000 46.0 / 48.5
//   d = 128  no mask: 80 x 96 7.1 / 6.0, 16 x 512 13.5 / 8.6, 32 x 512 14.2 / 12.2, 8 x 2000 41 / 28;
//            lost: 96 x 100 6.9 / 7.4, 16 x 1400 30.5 / 31.0, 8 x 3000 61.9 / 63.7
//            causal:  32 x 512 15.7 / 10.5, 16 x 1000 25.1 / 13.9, 16 x 2000 45.9 / 31.2, 8 x 4096 90 / 54
//   d = 256  no mask: 16 x 333 17.5 / 12.0, 4 x 2048 57 / 32;  lost: 28 x 333 17.9 / 21.5, 8 x 2048 62 / 62
//            causal:  16 x 1000 34 / 27, 2 x 8192 204 / 117;  lost: 32 x 333 18.5 / 19.5, 12 x 2048 61 / 61
// Drawn on 2900 shapes (heads 1 to 384, N from 24 to 16384): up to 4.6 times as fast.  Against the tiles as they are now,
// over 1710 others in the last third before the rule's edge: 0.79 of the time on average, 8 of them above 1.02, at worst 1.06
// (d = 64 causal, 24 x 2929 51.9 / 48.9).
inline bool few_forward(long heads, int N, int d, int causal) {
    const KeySplitFill fill(heads, N);
    if (fill.tiles < 3) return false;
    if (fill.fillings <= 1.f) return true;
    switch (d) {
        case 64: return causal ? (fill.tiles > 6 ? fill.at(1.5f, 9, fill.tiles < 90 ? 7.25f : 9.5f) : fill.fillings <= 1.75f)
                               : (fill.tiles > 6 ? fill.at(1.75f, 16, 4.9f) : fill.fillings <= 1.25f);
        case 128: return fill.tiles > 6 && (causal ? fill.at(1.5f, 18, 4.75f) : fill.fillings <= (fill.tiles < 40 ? 2.f : 3.f));
        default: return causal && fill.at(0.7f, 28, 2.9f);
    }
}

// How many waves such a workgroup has in the four-wave tile kernels: eight halve the chain of a long sequence, four let
// twice as many workgroups share a CU.  bf16, us, eight / four, heads x N:
//   d = 64   no mask: 8 x 700 7.4 / 7.4, 16 x 700 10.2 / 9.2, 32 x 700 14.4 / 11.7;  causal: 8 x 2049 13.1 / 14.5, 6 x 3000 16.3 / 18.3,
//            8 x 2560 18.2 / 17.2, 5 x 3669 19.6 / 22.4, 16 x 2049 22.7 / 19.0, 6 x 4096 26.1 / 25.5, 6 x 6144 48.6 / 51.8, 8 x 6144 62 / 58
//   d = 128  no mask: 16 x 700 17.9 / 13.6;  causal: 6 x 1600 14.7 / 16.1, 12 x 1600 24.6 / 18.7, 16 x 1700 35 / 27
inline int few_forward_waves(long heads, int N, int d, int causal) {
    if (N <= (causal ? (d == 64 ? 2048 : 1408) : 640)) return 4;
    const KeySplitFill fill(heads, N);
    const float most = !causal ? 1.f : d == 128 ? 1.5f : fill.tiles > 150 ? (float)fill.tiles / 42 : 2.4f;
    return fill.fillings <= most ? 8 : 4;
}

// The same for the FP8 forward (FewFp8Forward).  us, large / these, heads x N:
//   d = 64   no mask: 16 x 333 7.9 / 5.6, 4 x 4096 71 / 27, 1 x 16384 270 / 87;  lost: 128 x 256 8.4 / 8.8, 48 x 1000 21 / 22
//            causal:  16 x 1000 14 / 8.1, 8 x 4096 68 / 33;  lost: 96 x 512 10.8 / 11.0
//   d = 128  no mask: 16 x 512 11.2 / 7.2, 2 x 8192 168 / 71;  N <= 128: level;  lost: 48 x 333 9.5 / 11.1, 16 x 2048 46 / 54 (causal 45 / 34)
//            causal:  16 x 1000 18 / 9.7, 8 x 4096 84 / 48;  lost: 48 x 512 11.8 / 12.3
//   d = 256  no mask: 16 x 333 14.0 / 7.1, 4 x 2048 64 / 19;  lost: 48 x 333 15.0 / 16.3, 20 x 2048 69 / 79
//            causal:  16 x 1000 33 / 17, 4 x 8192 206 / 107;  lost: 32 x 1500 53 / 57
// Drawn on 2900 shapes.  Over 790 others in the last third before the edge 0.81 of the time on average, 12 of them above 1.02,
// at worst 1.12 (d = 256 causal, 40 x 438 20.2 / 18.1).  The error against 64 bits is smaller so (each part of the keys gets its own
// reference), with outliers, 4 heads x 1600: d = 64 1.01e-2 / 0.66e-2, d = 128 1.01e-2 / 0.85e-2, d = 256 causal 1.48e-2 / 1.36e-2.
inline bool few_forward_fp8(long heads, int N, int d, int causal) {
    const KeySplitFill fill(heads, N);
    if (fill.tiles < (d == 128 ? 5 : 3)) return false;
    if (fill.fillings <= 1.f) return true;
    if (fill.tiles <= (d == 64 ? 4 : 6)) return false;
    switch (d) {
        case 64: return causal ? fill.at(1.25f, 5.5f, 11.5f) : fill.at(1.4f, 12, 6);
        case 128: return causal ? fill.at(1.4f, 20, 7) : fill.fillings <= (fill.tiles < 32 ? 2.f : fill.tiles < 56 ? 3.f : 4.f);
        default: return causal ? fill.at(1.5f, 20, 7) : fill.fillings <= (fill.tiles < 20 ? 2.f : fill.tiles < 32 ? 2.5f : fill.tiles < 64 ? 3.f : 4.f);
    }
}

// The grid of a forward launch of `total` work items (query_tiles): heads x tiles for single causal tiles (of 128 rows
// or more, so at most 65504 of them at the largest N of any head dimension, which a grid's y takes) and for FewForward.
inline dim3 forward_grid(long heads, int N, int n_qtiles, long total, int causal, int paired) {
    if (paired == kFewForward) {
        const int split = few_split(heads, N), tiles = (N + 31) / 32;
        return split < 0 ? dim3((unsigned)(heads * tiles)) : dim3((unsigned)heads << split, (unsigned)((tiles + (1 << split) - 1) >> split));
    }
    return causal && !paired ? dim3((unsigned)heads, (unsigned)n_qtiles) : dim3((unsigned)total);
}

// ---- The backward at d = 64 and 128: which forms its passes take
//
// Large: a launch for dQ (128 or 256 queries to a workgroup, D beside it), one for dK and dV (128 keys).  The others are
// fa_bwd_few_kernel's: 32 keys to a workgroup, by itself behind the large dQ pass, or together with the dQ work in one launch,
// which then comes in workgroups of 32 queries or of 128.
enum BwdForm { kBwdLarge, kBwdKeys32, kBwdOne32, kBwdOneRows, kBwdForms };

// Up to which length the large dQ pass takes 128-query workgroups of four waves with 32-key blocks, two or three to a CU,
// instead of 256-query ones of eight with 64-key blocks: finer tiles waste less on the diagonal and on ragged ends, and
// the start and end of one workgroup run under the loop of another; over long sequences staging every block twice as
// often costs more.  Whole backward, bf16, H = 16, us, 256 / 128 queries:
//   d = 64   no mask: N = 512 160 / 151, 1300 368 / 347, 2048 485 / 487;  causal: 512 128 / 121, 1300 223 / 200,
//            2048 282 / 274, 3001 437 / 423, 4096 503 / 501
//   d = 128  no mask: 512 356 / 340, 1300 710 / 690, 2048 931 / 950;  causal: 512 289 / 267, 1300 455 / 427,
//            2048 575 / 570, 3001 845 / 863
// Without a mask the line is drawn lower than it would be for these 16 heads: N = 1536, H = 20 68.5 / 65.9 (d = 64) and
// 112 / 106 (d = 128), but H = 24 82.6 / 86.9 and 153 / 161.
constexpr int bwd_short_rows(int d, int causal) { return causal ? (d == 64 ? 3072 : 1536) : 1280; }

// What the forms cost, us.  A workgroup takes `start` and `tile` for each 32-row tile that its longest wave walks, next to as
// many others as its CU holds.  (Fitted, like everything here, to the choice between the forms and not to the times: they are
// within 10 to 15 % where the forms are close to one another.)
struct BwdWork {
    float start, tile;
    float edge;   // causal: the share of the longest workgroup that is left when the others have ended
    float crowd;  // how much longer the work takes where it fills the chip four times and more
};
struct BwdCost {
    float large, keys, one, row_sums;            // of a form, whatever its work; a launch for D before the one launch
    BwdWork dq128, dq256, keys128, keys32;
    float q32_start, q32_tile, rows_start, rows_tile;  // the dQ work of the one launch
    float last_q32, last_rows;                   // of a workgroup dealt last in the one launch, the share that runs past the mean
    float whole;                                 // no mask: how much whole rounds of the one launch count against its mean
    float alone;                                 // time of a workgroup alone on a CU that holds two
    float crowd, spread;                         // the one launch: how much longer at ten fillings; with heads that do not divide over the XCDs
};

// Whether the one launch that runs both passes computes D for itself: cheaper than a launch for it (2 us and the gap
// behind it) while a wave of a key block has few tiles, each of which then reads its rows of O once more, and nearly all
// workgroups are on the chip at once, so that few wait for them.  Whole backward, bf16, over 6450 drawn shapes, time without a
// launch for D of the time with one, by the tiles of a key block (four waves share them):
//   d = 64   1: 0.73, 4: 0.79, 8: 0.87, 12: 0.93, 16: 0.97, 18: 1.01, 24: 1.04;  d = 128  1: 0.83, 4: 0.92, 6: 0.99, 8: 1.02, 16: 1.11
// while the workgroups fill the chip half; between one filling and one and a half d = 64 4: 0.89, 16: 0.95, d = 128 4: 0.98, 6: 0.97, and
// beyond 0.96, 1.00 to 1.05, 1.00 to 1.04 and 1.00 to 1.03.
inline bool bwd_own_row_sums(long heads, long kv_heads, int N, int d) {
    const long tiles = (N + 31) / 32;
    return tiles * (heads / kv_heads) <= (d == 64 ? 16 : 6) && (heads + kv_heads) * tiles <= (d == 64 ? 768 : 384);
}

// Why an estimate: the forms differ in how many workgroups they make, how long the longest of them is and how many rounds they
// come to, and each of these decides somewhere.  Lines drawn through fillings of the chip kept large forms of 1.02 to 1.25 rounds.
// Timed as graphs of calls, every form of 15730 drawn shapes (1 to 512 heads, groups of 1 to 32, N from 16 to 16384), the choice against
// the best form, by such lines / by these estimates: time on average, shapes more than 10 % behind, the worst
//   d = 64   no mask  1.030 / 1.010, 12.3 / 3.0 %, 1.52 / 1.33;  causal 1.021 / 1.007, 8.1 / 1.6 %, 1.50 / 1.20
//   d = 128  no mask  1.035 / 1.006, 13.0 / 1.3 %, 1.71 / 1.24;  causal 1.022 / 1.007, 7.7 / 1.3 %, 1.90 / 1.32
// The constants were fitted to these and 11900 other shapes, weighted against choices slower than the lines': 1.1, 0.9, 0.3 and 0.2 % of
// the shapes take more than 5 % longer than by the lines.  Over 2150 more of 15 to 500 fillings and up to 70000 keys the time is
// 0.97 of the lines' on average.
// bf16, whole backward, us; large, 32 keys alone, one launch with 32 queries, with 128 (* the choice):
//   d = 64   no mask  9 x 7680 -, -, -, 488* (lines: large, 671);  472 on 59 x 640 245, 310, 449, 307* (lines: large);  44 x 1555 162*, 151, 135, 122;  79 x 256 17.2*, 22.6, 23.9, 18.8
//            causal   62 x 128 13.0, 11.2, 7.0, 7.8* (lines: 32);  36 on 18 x 165 19.2, 12.5, 8.4*, 7.2;  399 on 133 x 195 40.7*, 36.5, 46.4, 34.0
//   d = 128  no mask  28 x 1203 138*, 134, 132, 114;  165 on 33 x 512 122, 164, 201, 152* (lines: large);  192 on 64 x 128 27.1, 19.9, 29.2, 21.6*
//            causal   23 x 181 23.1, 18.0, 13.4*, 10.2;  25 x 1621 108, 136, 160, 119* (lines: large);  16 x 512 40, 29.9, 17.1, 18.0* (lines: 32);  480 on 15 x 137 217, 64, 66, 49*
// (With a number of heads that 8 divides, each on one XCD, few-workgroup forms gain up to 15 %, which `spread` follows for large ones
// only: 80 x 256, d = 64 16.6*, 19.3, 17.3, 15.6.  Fitted for all, it was right hardly more often.)  A call takes 0.05 to 0.2 us of the host.
constexpr BwdCost kBwdCost[2][2] = {  // d = 64, 128; no mask, causal
    {
        {7.89f, 3.4f, 0, 0.129f, {0.724f, 0.196f, 0, 11.2f}, {0.001f, 0.386f, 0, 2.48f}, {0.516f, 1.08f, 0, 0}, {5.41f, 0.582f, 0, 5.29f},
         5.72f, 0.268f, 5.31f, 0.397f, 0.129f, 0.479f, 0, 0.748f, 1.81f, 0.346f},
        {8.55f, 0.116f, 0.199f, 0.101f, {0.001f, 0.296f, 0.279f, 2.16f}, {1.38f, 0.633f, 0, 0.256f}, {0, 1.23f, 0.155f, 0}, {5.17f, 0.614f, 1.12f, 1.25f},
         5.06f, 0.748f, 5.0f, 0.62f, 0.179f, 0, 0, 0.744f, 0.713f, 0.347f},
    },
    {
        {6.84f, 2.58f, 0.279f, 0.627f, {3.43f, 0.808f, 0, 1.43f}, {5.23f, 0.995f, 0, 1.41f}, {0.817f, 0.881f, 0, 0.394f}, {4.79f, 0.746f, 0, 1.2f},
         5.01f, 0.508f, 4.08f, 0.605f, 0.106f, 0.134f, 1.0f, 1.0f, 0.944f, 0.153f},
        {10.8f, 3.7f, 0, 0, {1.39f, 1.03f, 0.071f, 0.964f}, {0, 1.28f, 0, 0}, {0.216f, 0.764f, 0.128f, 0.294f}, {6.45f, 0.829f, 0.093f, 0.36f},
         6.63f, 0.649f, 6.72f, 0.656f, 0.219f, 0.001f, 0, 1.0f, 0.307f, 0.013f},
    },
};

// The larger, and a little of the others: two bounds that are close are both felt
inline float bwd_bound(float a, float b, float c = 0) {
    const float m = a > b ? (a > c ? a : c) : (b > c ? b : c);
    return m + 0.08f * (a + b + c - m);
}
inline float bwd_share(float x) { return x < 0 ? 0 : x < 1 ? x : 1; }
inline float bwd_up(float x) { return x > 0 ? (float)(long)(x + 0.999f) : 0; }  // whole rounds

// A launch of `count` workgroups, `slots` of them on the chip at once: without a mask whole rounds, under one, where they are
// dealt longest first, the mean and an edge.
inline float bwd_pass(const BwdWork& w, float count, float longest, float mean, int slots, float alone, int causal) {
    const float all = w.start + mean * w.tile, most = w.start + longest * w.tile, fill = count / slots;
    float one = most, rounds = bwd_up(fill);
    if (slots == 512) {
        const long deep = (long)bwd_up(count / 256);
        one *= alone + (1 - alone) * bwd_share(count / 256 - 1);
        rounds = (float)(deep / 2) + alone * (float)(deep % 2);
    }
    return bwd_bound(one, (causal ? fill * all + w.edge * most : rounds * all) * (1 + w.crowd * bwd_share(fill / 4)));
}

// When the last of `n2` workgroups of `t2` each ends that are dealt behind `n1` of `t1`
inline float bwd_second_end(float slots, float n1, float t1, float n2, float t2) {
    const float mean = (n1 * t1 + n2 * t2) / slots, rounds = (float)(long)(n1 / slots), late = n1 - rounds * slots;
    float end = mean + 2 * t2;
    for (int i = 0; i < 4; ++i) {  // ends of a workgroup on a slot of either kind, from the mean on
        const float from = (rounds + (float)(i / 2)) * t1, t = from + (bwd_up((mean - from) / t2) + (float)(i % 2)) * t2;
        const float early_ones = t > rounds * t1 ? (float)(long)((t - rounds * t1) / t2 + 1e-3f) : 0;
        const float late_ones = t > (rounds + 1) * t1 ? (float)(long)((t - (rounds + 1) * t1) / t2 + 1e-3f) : 0;
        const float at = late > 0 && t < (rounds + 1) * t1 ? (rounds + 1) * t1 : t;
        if ((slots - late) * early_ones + late * late_ones >= n2 && at < end) end = at;
    }
    return end;
}

// Whether 128-query workgroups go ahead of the key blocks in the one launch: where they have the longer chains.  Key blocks of a
// group of g have g / 4 of them; without a mask, where all blocks of a kind are alike, they go first up to two.
inline bool bwd_rows_first(long group, int causal) { return group <= (causal ? 4 : 2); }

inline void bwd_form_times(long heads, long kv_heads, int N, int d, int causal, float (&us)[kBwdForms]) {
    const BwdCost& c = kBwdCost[d == 128][causal != 0];
    const int slots = d == 64 ? 512 : 256;
    const float h = (float)heads, kv = (float)kv_heads, group = h / kv, tiles = (float)((N + 31) / 32);
    auto mean = [&](float rows) { return causal ? (tiles + rows) / 2 : tiles; };  // of tiles that blocks of so many rows walk
    const float n128 = (float)((N + 127) / 128), n256 = (float)((N + 255) / 256);
    const float dq = N <= bwd_short_rows(d, causal) ? bwd_pass(c.dq128, h * n128, tiles, mean(4), d == 64 ? 768 : 512, c.alone, causal)
                                                    : bwd_pass(c.dq256, h * n256, tiles, mean(8), 256, c.alone, causal);
    us[kBwdLarge] = c.large + dq + bwd_pass(c.keys128, kv * n128, group * tiles, group * mean(4), slots, c.alone, causal);
    // 32-key workgroups: their four waves share the tiles
    const float longest_k = (float)(((long)(group * tiles) + 3) / 4);
    const float mean_k = causal ? group * mean(1) / 4 + 0.375f : 0.6f * longest_k + 0.1f * group * tiles;
    us[kBwdKeys32] = c.keys + dq + bwd_pass(c.keys32, kv * tiles, longest_k, mean_k, slots, c.alone, causal);

    // One launch: as long as either kind's longest workgroup, from when it is dealt, and as the work of both
    const float sums = bwd_own_row_sums(heads, kv_heads, N, d) ? 0 : c.row_sums;
    auto one = [&](float n_q, float longest_q, float mean_q, float start, float tile, bool q_first, float last) {
        const float n_k = kv * tiles, fill = (n_q + n_k) / slots;
        const float near = d == 64 ? c.alone + (1 - c.alone) * bwd_share(2 * fill - 1) : 1;
        const float chain_q = (start + longest_q * tile) * near, chain_k = (c.keys32.start + longest_k * c.keys32.tile) * near;
        const float load = 1 + c.crowd * bwd_share(fill / 10) + (kv_heads % 8 ? c.spread * bwd_share(h * (float)N * (float)d * 1e-7f) : 0);
        const float t_q = (start + mean_q * tile) * load, t_k = c.keys32.start + mean_k * c.keys32.tile, t_k_load = t_k * load;
        const float n_1 = q_first ? n_q : n_k, t_1 = q_first ? t_q : t_k_load, n_2 = q_first ? n_k : n_q, t_2 = q_first ? t_k_load : t_q;
        float work = (n_q * t_q + n_k * t_k_load) / (float)slots + last * t_2;
        if (c.whole > 0) work += c.whole * (bwd_second_end((float)slots, n_1, t_1, n_2, t_2) - work);
        const float part = (float)slots / n_1, dealt = q_first ? t_1 : t_k;  // when the first kind has been dealt
        const float second = n_1 <= (float)slots ? 0 : causal ? n_1 * dealt / (float)slots * (1 - part * part) : (float)(long)((n_1 - 1) / (float)slots) * dealt;
        return c.one + sums + (q_first ? bwd_bound(chain_q, second + chain_k, work) : bwd_bound(chain_k, second + chain_q, work));
    };
    const float quarter = (float)((long)(tiles + 3) / 4);
    us[kBwdOne32] = one(h * tiles, quarter, causal ? tiles / 8 + 0.5f : 0.6f * quarter + 0.1f * tiles, c.q32_start, c.q32_tile, false, c.last_q32);
    us[kBwdOneRows] = one(h * n128, tiles, mean(4), c.rows_start, c.rows_tile, bwd_rows_first(heads / kv_heads, causal), c.last_rows);
}

// d = 64 or 128.  Up to 64 rows 128 queries are the head and 32 half of it.  Where the one launch fills the chip 16 times and more it
// was best with 32 queries on none of 2150 shapes, and the estimate is too low (no mask, 48 on 6 x 11705, d = 64: large 7.24 ms,
// 32 queries 10.07); with 128 the shapes drawn end at 24, and with the 32-key form alone at 500, far from the most workgroups a launch takes.
inline BwdForm choose_bwd_form(long heads, long kv_heads, int N, int d, int causal) {
    float us[kBwdForms];
    bwd_form_times(heads, kv_heads, N, d, causal, us);
    const long both = (heads + kv_heads) * ((N + 31) / 32), chip = d == 64 ? 512 : 256;
    BwdForm best = both <= 500 * chip && us[kBwdKeys32] < us[kBwdLarge] ? kBwdKeys32 : kBwdLarge;
    if (both <= 16 * chip && us[kBwdOne32] < us[best]) best = kBwdOne32;
    if (both <= 24 * chip && N > 64 && us[kBwdOneRows] < us[best]) best = kBwdOneRows;
    return best;
}

int launch_fwd_bf16(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int H_kv, int N, int d,
                    float scale, int causal, int schedule, hipStream_t stream);
int launch_fwd_f16(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int H_kv, int N, int d,
                   float scale, int causal, int schedule, hipStream_t stream);
int launch_fwd_f32(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int H_kv, int N, int d,
                   float scale, int causal, hipStream_t stream);
int launch_fwd_fp8(const void* q8, const void* k8, const void* v8, const float* q_scale, const float* k_scale,
                   const float* v_scale, void* o, float* lse, int B, int H, int H_kv, int N, int d, float scale, int causal,
                   hipStream_t stream);
const char* fwd_16bit_kernel_name(bool f16, int N, int d, int causal);
const char* fwd_fp8_kernel_name(int N, int d, int causal);
int launch_quant_hadamard(const void* x, int in_dtype, void* x8, float* scales, int B, int H, int N, int d,
                          const signed char* signs, int per_tensor, hipStream_t stream);
size_t bwd_workspace_bytes(int B, int H, int N, int d);
int launch_bwd(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dout,
               void* dq, void* dk, void* dv, void* workspace, int B, int H, int H_kv, int N, int d, float scale,
               int causal, int dtype, hipStream_t stream);
int launch_probe_mfma(const void* operands, size_t operand_bytes, float* sink, int iters, bool fp8, hipStream_t stream);
double probe_mfma_flops(int iters, bool fp8);

}  // namespace fa
