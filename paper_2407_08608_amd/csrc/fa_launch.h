// Host-side launch entry points, one per kernel family.  H_kv is the number of key/value heads
// (H for ordinary multi-head attention; a divisor of H for multi-query / grouped-query attention).  Each validates nothing (the C ABI
// layer has done that), enqueues on `stream`, and returns an fa_status.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

#include "../../include/fa_mi355.h"

namespace fa {

// Whether N rows make an odd number of 128-row tiles.
inline bool odd_row_tiles(int N) { return ((N + 127) / 128) & 1; }

// Whether a causal forward launch pairs its query tiles (query_tiles in fa_device.h): when the pairs fill whole rounds
// of the chip, or nearly.  `slots`: workgroups of that kernel that the chip holds at once, 0 for kernels that never
// pair; `slack` / 8: how much of the last round may be empty once there is more than one.  Measured causal, bf16 unless
// said, us, pairs / single tiles dealt longest first:
//   ping-pong     3 rounds 269 / 270 (B = 4, H = 16, N = 4096), 2 158 / 162 (N = 2048); 1.5 183 / 164 (H = 64, N = 3001),
//                 2.25 517 / 439 (H = 48, N = 6000), 0.25 101 / 89 (H = 8, N = 4096)
//   d = 128, 4w   1 round 61 / 69 (H = 512, N = 512); 1.5 50.6 / 53.5 (H = 384, N = 512: hence its wider slack while
//                 tiles are short), 2.25 136 / 126 (H = 192, N = 1300), 0.75 28.4 / 27.1 (H = 192, N = 512)
//   d = 256       2 rounds 357 / 374 (H = 128, N = 2048); 4.5 1007 / 985 (H = 48, N = 6000)
//   FP8 d = 128   2 rounds 101 / 104 (N = 2048); 2.25 347 / 295 (N = 6000), 2.5 166 / 156 (H = 128, N = 2500)
//   never paired  d = 64: 164 / 157 (B = 4, H = 16, N = 4096), 329 / 259 (H = 48, N = 6000); FP8 d = 64 136 / 125,
//                 230 / 196; FP8 d = 256 324 / 319, 617 / 514
inline bool pair_causal_tiles(long heads, int n_qtiles, int slots, int slack = 9) {
    if (slots == 0) return false;
    const long items = heads * ((n_qtiles + 1) / 2), rounds = (items + slots - 1) / slots;
    return rounds * slots * 8 <= items * (rounds == 1 ? 9 : slack);
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
