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
