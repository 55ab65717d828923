// FP8 pre-pass (paper section 3.3): optional incoherent processing  y = (x * s) H_d / sqrt(d)
// followed by block quantisation to e4m3 with one fp32 scale per 128 rows of a head.
//
// Every element is read once (2 or 4 bytes) and written once (1 byte); bound by HBM where the 128-row blocks, one workgroup
// each, fill the chip several times, and by the vector instructions of the transform otherwise: with one round of
// workgroups loads, arithmetic and stores hardly overlap.  So instructions per element are what was counted (Hadamard, d = 128:
// 21 before, 17 now; without it 9 and 6):
//   - four or eight lanes share a row, each with 8-element chunks interleaved across them (16-byte loads that cover 64 or
//     128 contiguous bytes of a row).  The Hadamard butterflies run in the order of the element index bits (strides 1, 2,
//     ..., d/2): 1 to 4 inside a chunk, 8 and 16 (32 with eight lanes) between lanes by DPP, the rest between the lane's
//     own chunks.  Eight lanes at d = 128 would need ds_swizzle or one DPP stage more: 23.2 / 24.7 us (32 x 8192).
//   - rows go through one resource per block: past its end reads give zeros and stores are dropped, so there is no branch
//     and all loads are in flight at once;
//   - signs are put on 16-bit words before they are unpacked, two elements an instruction (should any not be 1 or -1, a second
//     way multiplies by the magnitudes too: 0.1 us of a launch for the look at them);
//   - 1 / sqrt(d) is a power of two at d = 64 and 256 and goes into the code's factor there, exactly;
//   - the clamp, which changes nothing in a block of ordinary values, is left to a second way for those that are not;
//   - lanes trade codes in pairs and store 16 bytes each.
// us, before / now, heads x N, bf16, with the transform: d = 64 128 x 2500 18.7 / 15.4; d = 128 32 x 8192 27.3 / 23.2 (4.35 TB/s),
// 32 x 3664 15.8 / 13.1, 16 x 1000 5.7 / 4.7; d = 256 16 x 8192 32.0 / 23.8, 6 x 5056 9.5 / 8.4; without it d = 128
// 32 x 8192 23.4 / 21.1, d = 64 128 x 2500 18.1 / 14.0.
// All arithmetic that decides a code is fp32: add/sub butterflies, one multiply by float(1/sqrt(d)), one multiply by 448/amax,
// clamp, round-to-nearest-even conversion.
#include "fa_device.h"
#include "fa_launch.h"

namespace fa {

constexpr int kBlockRows = 128;
constexpr float kE4m3Max = 448.0f;

template <int CTRL>
static __device__ __forceinline__ int quad_perm(int x) {
    return __builtin_amdgcn_mov_dpp(x, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
static __device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(float, quad_perm<CTRL>(__builtin_bit_cast(int, x)));
}

// A lane's chunk of 8 elements as it lies in memory, and as floats.  Rows past the resource's end read as zero.
template <int IN_DTYPE> struct Chunk {
    static constexpr int ELEM = IN_DTYPE == FA_F32 ? 4 : 2;
    i32x4 w[ELEM / 2];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rsrc, int byte_off) {
#pragma unroll
        for (int i = 0; i < ELEM / 2; ++i) w[i] = buffer_load_16B(rsrc, byte_off + 16 * i);
    }
    __device__ __forceinline__ float at(int t) const {
        if constexpr (IN_DTYPE == FA_F32) return __builtin_bit_cast(float, (int)w[t >> 2][t & 3]);
        const uint32_t u = (uint32_t)w[0][t >> 1];
        if constexpr (IN_DTYPE == FA_BF16) return __builtin_bit_cast(float, t & 1 ? u & 0xFFFF0000u : u << 16);
        return Elem<f16_tag>::to_float((uint16_t)(t & 1 ? u >> 16 : u));
    }
};

// The larger of two magnitudes: a NaN stays one (KEEP_NAN) or gives way to the other
template <bool KEEP_NAN>
static __device__ __forceinline__ float larger(float a, float b) {
    return KEEP_NAN ? __builtin_elementwise_maximum(a, b) : fmaxf(a, b);
}

// Not fused with a sum that takes it
static __device__ __forceinline__ float rounded_product(float a, float b) {
#pragma clang fp contract(off)
    return a * b;
}

// 32 values of the block to a lane: 64 took longer at d = 128 (25.3 / 22.8 us, 32 x 8192) and d = 256 (24.9 / 23.8, 16 x 8192)
constexpr int quant_threads(int d) { return 4 * d; }

// MODE 0: per-block scales.  MODE 1: only fold the block's amax into *amax_bits (atomic max on
// the bit pattern of a non-negative float).  MODE 2: quantise with the scale taken from
// *amax_bits, leave `scales` alone.
template <int D, int IN_DTYPE, int MODE, bool HADAMARD>
__global__ void __launch_bounds__(quant_threads(D))
fa_quant_kernel(const void* __restrict__ x, uint8_t* __restrict__ x8, float* __restrict__ scales,
                const signed char* __restrict__ signs, unsigned* amax_bits, int N, int n_blocks) {
    using C = Chunk<IN_DTYPE>;
    constexpr int NT = quant_threads(D), NW = NT / 64;
    constexpr int LPR = D == 256 ? 8 : 4;       // lanes per row
    constexpr int CH = D / (8 * LPR);          // 8-element chunks per lane and row
    constexpr int RPP = NT / LPR;              // rows per pass of the workgroup
    constexpr int PASSES = kBlockRows / RPP;
    constexpr bool POW2 = HADAMARD && D != 128;  // 1 / sqrt(d) is a power of two
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the lane's place in its row; the upper four of eight stand in reverse, so that DPP's half mirror joins p and p ^ 4
    const int p = LPR == 8 ? (tid & 7) ^ (tid & 4 ? 3 : 0) : tid & 3;
    const int row = tid / LPR;
    const int bh = blockIdx.x / n_blocks, blk = blockIdx.x % n_blocks;
    const size_t off = ((size_t)bh * N + (size_t)blk * kBlockRows) * D;  // of the block
    const int n_el = min(N - blk * kBlockRows, kBlockRows) * D;
    const float inv_sqrt_d = (float)(1.0 / __builtin_sqrt((double)D));

    // Four signs to a lane, to see whether all are 1 or -1; requested ahead of the rows, so that the branch on it waits for no row
    int four_signs = 0x01010101;
    if constexpr (HADAMARD && IN_DTYPE != FA_F32) __builtin_memcpy(&four_signs, signs + 4 * (lane % (D / 4)), 4);
    const __amdgpu_buffer_rsrc_t rsrc = make_buffer(static_cast<const char*>(x) + off * C::ELEM, (uint32_t)(n_el * C::ELEM));
    C raw[PASSES][CH];
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps)
#pragma unroll
        for (int c = 0; c < CH; ++c) raw[ps][c].load(rsrc, ((ps * RPP + row) * D + 8 * (p + LPR * c)) * C::ELEM);

    if constexpr (HADAMARD && IN_DTYPE != FA_F32) {  // the signs go on in the words as they lie in memory
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            i32x2 s8;
            __builtin_memcpy(&s8, signs + 8 * (p + LPR * c), 8);
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int m = s8[g] & (int)0x80808080;
#pragma unroll
                for (int ps = 0; ps < PASSES; ++ps) {
                    raw[ps][c].w[0][2 * g] ^= __builtin_amdgcn_perm(0, m, 0x010c000c);
                    raw[ps][c].w[0][2 * g + 1] ^= __builtin_amdgcn_perm(0, m, 0x030c020c);
                }
            }
        }
    }

    float y[PASSES][CH][8];
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps)
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int t = 0; t < 8; ++t) y[ps][c][t] = raw[ps][c].at(t);
    if constexpr (HADAMARD) {
        // what the words do not have yet: the signs of fp32 rows, and magnitudes other than 1
        auto multiply = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                int at = 8 * (p + LPR * c);
                if constexpr (IN_DTYPE != FA_F32) asm volatile("" : "+v"(at));  // read again: kept, they would cost the ordinary way registers
                i32x2 s8;
                __builtin_memcpy(&s8, signs + at, 8);
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const float s = (float)(signed char)(s8[t >> 2] >> (8 * (t & 3)));
#pragma unroll
                    for (int ps = 0; ps < PASSES; ++ps) y[ps][c][t] = rounded_product(y[ps][c][t], IN_DTYPE == FA_F32 ? s : fabsf(s));
                }
            }
        };
        if constexpr (IN_DTYPE == FA_F32) {
            multiply();
        } else {
            const int negative = (four_signs >> 7) & 0x01010101, unit = ((negative << 8) - negative) | 0x01010101;
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(four_signs != unit) != 0, 0)) multiply();
        }
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            // element index e = t + 8 p + 8 LPR c
#pragma unroll
            for (int c = 0; c < CH; ++c) {
#pragma unroll
                for (int h = 1; h < 8; h <<= 1)  // strides 1, 2, 4
#pragma unroll
                    for (int t = 0; t < 8; ++t)
                        if ((t & h) == 0) {
                            const float a = y[ps][c][t], b = y[ps][c][t + h];
                            y[ps][c][t] = a + b;
                            y[ps][c][t + h] = a - b;
                        }
            }
            // strides 8 and 16: partner lane p^1, then p^2; low lane gets a+b, high lane a-b
            const float s1 = (p & 1) ? -1.f : 1.f, s2 = (p & 2) ? -1.f : 1.f;
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    float v = y[ps][c][t];
                    v = __builtin_fmaf(v, s1, dpp<0xB1>(v));  // lanes (1,0,3,2)
                    v = __builtin_fmaf(v, s2, dpp<0x4E>(v));  // lanes (2,3,0,1)
                    if constexpr (LPR == 8) v = __builtin_fmaf(v, p & 4 ? -1.f : 1.f, dpp<0x141>(v));  // lanes 7 .. 0: p^4
                    y[ps][c][t] = v;
                }
#pragma unroll
            for (int h = 1; h < CH; h <<= 1)  // strides 8 LPR and up
#pragma unroll
                for (int c = 0; c < CH; ++c)
                    if ((c & h) == 0)
#pragma unroll
                        for (int t = 0; t < 8; ++t) {
                            const float a = y[ps][c][t], b = y[ps][c + h][t];
                            y[ps][c][t] = a + b;
                            y[ps][c + h][t] = a - b;
                        }
            if constexpr (!POW2)
#pragma unroll
                for (int c = 0; c < CH; ++c)
#pragma unroll
                    for (int t = 0; t < 8; ++t) y[ps][c][t] *= inv_sqrt_d;
        }
    }

    __shared__ float red[NW];  // one slot per wave
    auto block_amax = [&](auto keep_nan) __attribute__((always_inline)) {
        constexpr bool KEEP = decltype(keep_nan)::value;
        float m = 0.f;
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps)
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int t = 0; t < 8; t += 2) m = larger<KEEP>(larger<KEEP>(fabsf(y[ps][c][t]), fabsf(y[ps][c][t + 1])), m);
        m = larger<KEEP>(m, dpp<0xB1>(m));
        m = larger<KEEP>(m, dpp<0x4E>(m));
        m = larger<KEEP>(m, dpp<0x141>(m));  // row_half_mirror
        m = larger<KEEP>(m, dpp<0x140>(m));  // row_mirror
        m = larger<KEEP>(m, __shfl_xor(m, 16));
        m = larger<KEEP>(m, __shfl_xor(m, 32));
        if (lane == 0) red[wave] = m;
        __syncthreads();
        m = red[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) m = larger<KEEP>(m, red[w]);
        return m;
    };
    // codes of y * factor, 16 bytes a lane: the even lane of a pair takes both lanes' codes of a chunk, the odd lane those of the next
    const __amdgpu_buffer_rsrc_t out = make_buffer(x8 + off, (uint32_t)n_el);
    auto store_codes = [&](float factor, auto limit) __attribute__((always_inline)) {
        const bool odd = p & 1;
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps)
#pragma unroll
            for (int c = 0; c < CH; c += 2) {
                int w[2][2];
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int g = 0; g < 2; ++g) {
                        float z[4];
#pragma unroll
                        for (int t = 0; t < 4; ++t) z[t] = limit(y[ps][c + i][4 * g + t] * factor);
                        w[i][g] = __builtin_amdgcn_cvt_pk_fp8_f32(z[0], z[1], 0, false);
                        w[i][g] = __builtin_amdgcn_cvt_pk_fp8_f32(z[2], z[3], w[i][g], true);
                    }
                const int r0 = quad_perm<0xB1>(odd ? w[0][0] : w[1][0]), r1 = quad_perm<0xB1>(odd ? w[0][1] : w[1][1]);
                const i32x4 v = {odd ? r0 : w[0][0], odd ? r1 : w[0][1], odd ? w[1][0] : r0, odd ? w[1][1] : r1};
                const int at = (ps * RPP + row) * D + 8 * LPR * (c + (odd ? 1 : 0)) + 8 * (p & ~1);
                __builtin_amdgcn_raw_buffer_store_b128(v, out, at, 0, 0);
            }
    };

    if constexpr (MODE == 0) {
        const float m = block_amax(std::true_type{}), amax = POW2 ? m * inv_sqrt_d : m;
        // Ordinary values: no NaN (it fails the comparison) or infinity, and 448 / amax is finite.  Then |y| * inv <= 448 (1 + 2^-22),
        // which rounds to 448 without a clamp, and (u / 2^k) inv = u (inv / 2^k) but for products of less than 1e-5, code 0.
        if (amax > 1e-30f && amax < 1e38f) {
            if (tid == 0) scales[(size_t)bh * n_blocks + blk] = amax / kE4m3Max;
            const float inv = kE4m3Max / amax;
            store_codes(POW2 ? inv * inv_sqrt_d : inv, [](float z) { return z; });
            return;
        }
        __syncthreads();  // red is written again
    }
    if constexpr (POW2)
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps)
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int t = 0; t < 8; ++t) y[ps][c][t] *= inv_sqrt_d;
    float amax = MODE == 2 ? __builtin_bit_cast(float, *amax_bits) : block_amax(std::false_type{});
    if constexpr (MODE == 1) {
        if (tid == 0) atomicMax(amax_bits, __builtin_bit_cast(unsigned, amax));
        return;
    }
    if (MODE == 0 && tid == 0) scales[(size_t)bh * n_blocks + blk] = amax != 0.f ? amax / kE4m3Max : 1.0f;
    store_codes(amax != 0.f ? kE4m3Max / amax : 1.0f, [](float z) { return fminf(fmaxf(z, -kE4m3Max), kE4m3Max); });
}

__global__ void fa_zero_word_kernel(unsigned* p) { *p = 0u; }

// one workgroup: read the tensor-wide amax (stored as bits in slot 0), then fill every slot
__global__ void __launch_bounds__(256) fa_fill_scales_kernel(float* scales, long n) {
    float amax = __builtin_bit_cast(float, *reinterpret_cast<unsigned*>(scales));
    __syncthreads();  // every thread has read slot 0 before anyone overwrites it
    float scale = amax != 0.f ? amax / kE4m3Max : 1.0f;
    for (long i = threadIdx.x; i < n; i += 256) scales[i] = scale;
}

template <int D, int IN_DTYPE, bool HADAMARD>
static int launch_quant(const void* x, void* x8, float* scales, int B, int H, int N, const signed char* signs,
                        int per_tensor, hipStream_t stream) {
    int n_blocks = (N + kBlockRows - 1) / kBlockRows;
    long total = (long)B * H * n_blocks;
    if (total > 0x7fffffffL) return FA_ERR_SHAPE;
    dim3 grid((unsigned)total), block(quant_threads(D));
    auto out = static_cast<uint8_t*>(x8);
    unsigned* slot0 = reinterpret_cast<unsigned*>(scales);
    if (!per_tensor) {
        hipLaunchKernelGGL((fa_quant_kernel<D, IN_DTYPE, 0, HADAMARD>), grid, block, 0, stream, x, out, scales, signs,
                           slot0, N, n_blocks);
    } else {
        hipLaunchKernelGGL(fa_zero_word_kernel, dim3(1), dim3(1), 0, stream, slot0);
        if (hipGetLastError() != hipSuccess) return FA_ERR_LAUNCH;
        hipLaunchKernelGGL((fa_quant_kernel<D, IN_DTYPE, 1, HADAMARD>), grid, block, 0, stream, x, out, scales, signs,
                           slot0, N, n_blocks);
        if (hipGetLastError() != hipSuccess) return FA_ERR_LAUNCH;
        hipLaunchKernelGGL((fa_quant_kernel<D, IN_DTYPE, 2, HADAMARD>), grid, block, 0, stream, x, out, scales, signs,
                           slot0, N, n_blocks);
        if (hipGetLastError() != hipSuccess) return FA_ERR_LAUNCH;
        hipLaunchKernelGGL(fa_fill_scales_kernel, dim3(1), dim3(256), 0, stream, scales, total);
    }
    return hipGetLastError() == hipSuccess ? FA_OK : FA_ERR_LAUNCH;
}

template <int D, int IN_DTYPE>
static int launch_quant_h(const void* x, void* x8, float* scales, int B, int H, int N, const signed char* signs,
                          int per_tensor, hipStream_t stream) {
    return signs ? launch_quant<D, IN_DTYPE, true>(x, x8, scales, B, H, N, signs, per_tensor, stream)
                 : launch_quant<D, IN_DTYPE, false>(x, x8, scales, B, H, N, signs, per_tensor, stream);
}

template <int IN_DTYPE>
static int launch_quant_d(const void* x, void* x8, float* scales, int B, int H, int N, int d,
                          const signed char* signs, int per_tensor, hipStream_t stream) {
    switch (d) {
        case 64: return launch_quant_h<64, IN_DTYPE>(x, x8, scales, B, H, N, signs, per_tensor, stream);
        case 128: return launch_quant_h<128, IN_DTYPE>(x, x8, scales, B, H, N, signs, per_tensor, stream);
        case 256: return launch_quant_h<256, IN_DTYPE>(x, x8, scales, B, H, N, signs, per_tensor, stream);
        default: return FA_ERR_UNSUPPORTED;
    }
}

int launch_quant_hadamard(const void* x, int in_dtype, void* x8, float* scales, int B, int H, int N, int d,
                          const signed char* signs, int per_tensor, hipStream_t stream) {
    switch (in_dtype) {
        case FA_F32: return launch_quant_d<FA_F32>(x, x8, scales, B, H, N, d, signs, per_tensor, stream);
        case FA_BF16: return launch_quant_d<FA_BF16>(x, x8, scales, B, H, N, d, signs, per_tensor, stream);
        case FA_F16: return launch_quant_d<FA_F16>(x, x8, scales, B, H, N, d, signs, per_tensor, stream);
        default: return FA_ERR_UNSUPPORTED;
    }
}

}  // namespace fa
