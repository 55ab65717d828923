// Device-side building blocks shared by the attention kernels: vector types, MFMA
// wrappers for gfx950, the transposing LDS reads, and wavefront helpers.
//
// Register layouts used throughout (64-lane wavefront, lane l, col = l % 32, half = l / 32):
//   v_mfma_f32_32x32x16_{bf16,f16}: an A (or B) operand lane holds row (col) `l % 32` and the
//     8 contraction indices 8*half .. 8*half+7; the fp32 result lane holds column `l % 32`
//     and, in register r of 16, row 8*(r/4) + 4*half + r%4.
// Computing the transposed score tile S^T = K Q^T therefore leaves one query per lane
// column with its keys spread over the lane's own registers, and those registers, packed
// to 16 bits, are already a valid B operand for O^T = V^T P^T as long as the V operand
// enumerates keys in the same order -- the gfx950 counterpart of the accumulator-to-operand
// register permutation of the paper's section 3.3 (FP8 layout discussion).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <stdint.h>

namespace fa {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(2))) int i32x2;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;

// f(0), f(1), ..., f(N - 1), each with its number as a type
template <int N, typename F, int I = 0>
static __device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, F, I + 1>(static_cast<F&&>(f));
    }
}

struct bf16_tag {};
struct f16_tag {};

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

template <typename Tag> struct Elem;

template <> struct Elem<bf16_tag> {
    // D = A(32x16) * B(16x32) + C, 16-bit operands packed 8 per lane in a 128-bit carrier
    static __device__ __forceinline__ f32x16 mma(i32x4 a, i32x4 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ int pack2(float lo, float hi) {  // RNE
        f32x2 v = {lo, hi};
        return __builtin_bit_cast(int, __builtin_convertvector(v, bf16x2));
    }
    static __device__ __forceinline__ float to_float(uint16_t bits) {
        return __builtin_bit_cast(float, (uint32_t)bits << 16);
    }
};

template <> struct Elem<f16_tag> {
    static __device__ __forceinline__ f32x16 mma(i32x4 a, i32x4 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ int pack2(float lo, float hi) {  // RNE
        f32x2 v = {lo, hi};
        return __builtin_bit_cast(int, __builtin_convertvector(v, f16x2));
    }
    static __device__ __forceinline__ float to_float(uint16_t bits) {
        return (float)__builtin_bit_cast(_Float16, bits);
    }
};

// A buffer resource as four scalar registers, for loads written as inline assembly (global_to_lds_16B)
struct BufferWords {
    i32x4 w;
};

// The same MFMA written as inline assembly, to choose the half of the register file each operand
// lives in.  A kernel that needs more than 256 registers per lane gets MFMA results in the
// accumulation half by default, where no VALU instruction can read them: a score tile that the
// softmax reads would pay one copy per element.  Here the accumulator is forced into ordinary
// registers and the B operand (touched by MFMA alone) is taken from the accumulation half.
// The compiler's hazard checker cannot see inside: a VALU read of the accumulator must be
// separated from the MFMA that wrote it by mfma_result_wait(), and the first MFMA onto an accumulator
// that was filled with values has to be start(), which keeps the two wait states an MFMA needs behind
// a VALU write of its operands (the compiler may put the copy that fills it directly in front).
template <typename Tag> struct MfmaVgprAcc;
// The _and_load forms also issue a global_to_lds_16B: the MFMA stands between the instruction that sets m0 and the load, in
// place of the wait state that the load needs there.
#define FA_DEFINE_MFMA_VGPR_ACC(TAG, OPCODE)                                                          \
    template <> struct MfmaVgprAcc<TAG> {                                                             \
        static __device__ __forceinline__ void run(f32x16& acc, const i32x4& a, const i32x4& b) {     \
            asm volatile(OPCODE " %0, %1, %2, %0" : "+v"(acc) : "v"(a), "a"(b));                      \
        }                                                                                             \
        static __device__ __forceinline__ void start(f32x16& acc, const i32x4& a, const i32x4& b) {   \
            asm volatile("s_nop 1\n\t" OPCODE " %0, %1, %2, %0" : "+v"(acc) : "v"(a), "a"(b));        \
        }                                                                                             \
        static __device__ __forceinline__ void first(f32x16& acc, const i32x4& a, const i32x4& b) {   \
            asm volatile(OPCODE " %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "a"(b));                      \
        }                                                                                             \
        template <int LDS_OFF>                                                                        \
        static __device__ __forceinline__ void run_and_load(f32x16& acc, const i32x4& a, const i32x4& b, const BufferWords& rsrc, \
                                                            uint32_t lds_base, int byte_off) {        \
            asm volatile("s_add_u32 m0, %3, %4\n\t" OPCODE " %0, %1, %2, %0\n\tbuffer_load_dwordx4 %5, %6, 0 offen lds" \
                         : "+v"(acc) : "v"(a), "a"(b), "s"(lds_base), "n"(LDS_OFF), "v"(byte_off), "s"(rsrc.w) \
                         : "memory", "m0", "scc");                                                    \
        }                                                                                             \
        template <int LDS_OFF>                                                                        \
        static __device__ __forceinline__ void start_and_load(f32x16& acc, const i32x4& a, const i32x4& b, const BufferWords& rsrc, \
                                                              uint32_t lds_base, int byte_off) {      \
            asm volatile("s_add_u32 m0, %3, %4\n\ts_nop 0\n\t" OPCODE " %0, %1, %2, %0\n\tbuffer_load_dwordx4 %5, %6, 0 offen lds" \
                         : "+v"(acc) : "v"(a), "a"(b), "s"(lds_base), "n"(LDS_OFF), "v"(byte_off), "s"(rsrc.w) \
                         : "memory", "m0", "scc");                                                    \
        }                                                                                             \
        template <int LDS_OFF>                                                                        \
        static __device__ __forceinline__ void first_and_load(f32x16& acc, const i32x4& a, const i32x4& b, const BufferWords& rsrc, \
                                                              uint32_t lds_base, int byte_off) {      \
            asm volatile("s_add_u32 m0, %3, %4\n\t" OPCODE " %0, %1, %2, 0\n\tbuffer_load_dwordx4 %5, %6, 0 offen lds" \
                         : "=&v"(acc) : "v"(a), "a"(b), "s"(lds_base), "n"(LDS_OFF), "v"(byte_off), "s"(rsrc.w) \
                         : "memory", "m0", "scc");                                                    \
        }                                                                                             \
    };
FA_DEFINE_MFMA_VGPR_ACC(bf16_tag, "v_mfma_f32_32x32x16_bf16")
FA_DEFINE_MFMA_VGPR_ACC(f16_tag, "v_mfma_f32_32x32x16_f16")
#undef FA_DEFINE_MFMA_VGPR_ACC

// 13 wait states: the 8-pass MFMA needs 11 between its issue and a VALU read of its result, and
// the compiler leaves 12 or more in the code it schedules itself.  The accumulators are operands
// of the statement, so no reader can be scheduled above it; placed after an independent MFMA
// most of the wait passes while the matrix pipe works on that one.
static __device__ __forceinline__ void mfma_result_wait(f32x16& x, f32x16& y) {
    asm volatile("s_nop 12" : "+v"(x), "+v"(y));
}
static __device__ __forceinline__ void mfma_result_wait(f32x16& x) { asm volatile("s_nop 12" : "+v"(x)); }
// The same where at least 12 - STATES instructions stand between.
template <int STATES>
static __device__ __forceinline__ void mfma_result_wait_rest(f32x16& x) { asm volatile("s_nop %1" : "+v"(x) : "n"(STATES - 1)); }

// 32-bit LDS byte address of a __shared__ object, and loads through such an address: a base kept
// in one register with compile-time offsets lets every read use the instruction's immediate
// offset field instead of an address computation of its own.
static __device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)p; }
static __device__ __forceinline__ i32x4 lds_load_16B(uint32_t addr) {
    typedef i32x4 __attribute__((address_space(3))) * lds_vec_ptr;
    return *(lds_vec_ptr)(uintptr_t)addr;
}
static __device__ __forceinline__ float lds_load_4B(uint32_t addr) {
    typedef float __attribute__((address_space(3))) * lds_float_ptr;
    return *(lds_float_ptr)(uintptr_t)addr;
}
static __device__ __forceinline__ f32x4 lds_load_4f(uint32_t addr) {
    typedef f32x4 __attribute__((address_space(3))) * lds_vec_ptr;
    return *(lds_vec_ptr)(uintptr_t)addr;
}

// ds_read_b64_tr_b16: the 16 lanes of a group each point at 4 consecutive 16-bit elements;
// seen as a 4x16 matrix (row r = what lanes 4r..4r+3 point at), lane i of the group
// receives column i.  Used to read a [key][d] tile as the key-contiguous MFMA operand.
static __device__ __forceinline__ i32x2 lds_read_tr16(const void* lds_ptr) {
    typedef s16x4 __attribute__((address_space(3))) * lds_vec_ptr;
    s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_vec_ptr)(uintptr_t)lds_ptr);
    return __builtin_bit_cast(i32x2, v);
}
static __device__ __forceinline__ i32x2 lds_read_tr16(uint32_t lds_addr) {
    typedef s16x4 __attribute__((address_space(3))) * lds_vec_ptr;
    s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_vec_ptr)(uintptr_t)lds_addr);
    return __builtin_bit_cast(i32x2, v);
}

// ds_read_b64_tr_b8: same with bytes; the group's data is an 8x16 byte matrix (row r = what
// lanes 2r, 2r+1 point at) and lane i receives column i.
static __device__ __forceinline__ i32x2 lds_read_tr8(const void* lds_ptr) {
    typedef i32x2 __attribute__((address_space(3))) * lds_vec_ptr;
    return __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_vec_ptr)(uintptr_t)lds_ptr);
}
static __device__ __forceinline__ i32x2 lds_read_tr8(uint32_t lds_addr) {
    typedef i32x2 __attribute__((address_space(3))) * lds_vec_ptr;
    return __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_vec_ptr)(uintptr_t)lds_addr);
}

// v_permlane32_swap exchanges the upper half of its first register with the lower half of
// its second.  Fed two copies of x it yields (x of lanes 0..31 replicated, x of lanes 32..63
// replicated).  The second copy is laundered through an empty asm so the compiler cannot
// treat the two results as one value.
struct HalfPair {
    float lo, hi;  // value of lane (l % 32), value of lane (l % 32) + 32
};
static __device__ __forceinline__ HalfPair both_halves(float x) {
    uint32_t a = __builtin_bit_cast(uint32_t, x);
    uint32_t b = a;
    asm volatile("" : "+v"(b));
    auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    uint32_t r0 = r[0], r1 = r[1];
    asm volatile("" : "+v"(r0), "+v"(r1));
    return {__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1)};
}

static __device__ __forceinline__ float max_both_halves(float x) {
    HalfPair p = both_halves(x);
    return fmaxf(fmaxf(-INFINITY, p.lo), p.hi);  // one three-way maximum; of the two alone, each would be quieted first
}

static __device__ __forceinline__ float sum_both_halves(float x) {
    HalfPair p = both_halves(x);
    return p.lo + p.hi;
}

// Raw buffer access to a caller tensor: reads past `bytes` return zero instead of faulting.
static __device__ __forceinline__ __amdgpu_buffer_rsrc_t make_buffer(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
static __device__ __forceinline__ i32x4 buffer_load_16B(__amdgpu_buffer_rsrc_t rsrc, int byte_off) {
    return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, byte_off, 0, 0));
}

// Asynchronous global -> LDS copy of 16 bytes per lane (buffer load with an LDS destination):
// lane i's bytes land at lds_base + 16 i, lds_base wave-uniform; reads past the resource's size
// store zeros.  Written as inline assembly on purpose: the compiler then does not know that the
// load writes LDS and does not drain all outstanding loads before every later LDS read; the
// caller orders the two with an explicit vmcnt wait and a barrier.
static __device__ __forceinline__ BufferWords make_buffer_words(const void* base, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    BufferWords b;
    b.w = i32x4{(int)(uint32_t)a, (int)(uint32_t)((a >> 32) & 0xFFFF), (int)bytes, 0x00020000};
    return b;
}
// A resource in registers that a vector instruction has written must be five wait states old, which the compiler does not see
// to ahead of inline assembly: where it spills scalar registers and brings the resource back right ahead of a load (the build's
// hazard check says so), RELOADED makes them up.  (Everywhere, that costs the kernels 0 to 3 %.)
template <bool RELOADED = false>
static __device__ __forceinline__ void global_to_lds_16B(const BufferWords& rsrc, uint32_t lds_base, int byte_off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop %3\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(byte_off), "s"(rsrc.w), "n"(RELOADED ? 3 : 0)
                 : "memory", "m0");
}

// The resource `bytes` further on: what was at offset `bytes` is at 0 then, what lies past the end still reads as zero.
// Walking a tensor so costs scalar instructions only, where an offset per load costs a vector one.
static __device__ __forceinline__ void advance(BufferWords& b, int bytes) {
    const uint64_t a = (uint64_t)(uint32_t)b.w[0] | (uint64_t)(uint32_t)b.w[1] << 32;
    const uint64_t n = a + (uint32_t)bytes;
    b.w[0] = (int)(uint32_t)n;
    b.w[1] = (int)(uint32_t)(n >> 32);
    int left = b.w[2];  // (written out: the compiler makes a vector instruction of a saturating difference)
    asm("s_sub_u32 %0, %0, %1\n\ts_cselect_b32 %0, 0, %0" : "+s"(left) : "s"(bytes) : "scc");
    b.w[2] = left;
}

// A wave's private tiles of 32 rows of a 16-bit tensor, staged straight from global memory into LDS that no other wave
// touches: no barriers, only the wave's own vmcnt waits.  A tile is unpadded; 16-byte chunk c of row r sits at
// c ^ swizzle(r), applied through the global address a lane fetches: row reads (16 rows at one chunk) and transposing
// reads (4 rows x 4 chunks) both hit every bank once.
// The lane's LDS addresses are kept, for a tile at `base`; another tile is a compile-time offset in the instruction.  (They
// are opaque: the compiler would add them up again for every read.)
template <int D>
struct WaveTile {
    static constexpr int ROWS = 32, ROWB = D * 2, KS = D / 16, DT = D / 32;
    static constexpr int CPR = D / 8;             // 16-byte chunks per row
    static constexpr int TILE_B = ROWS * ROWB;
    static constexpr int RPI = 1024 / ROWB;       // rows per staging instruction (1 KiB)
    static constexpr int NI = ROWS / RPI;         // staging instructions per tile
    static constexpr int PERIOD = 16 / RPI;       // swizzle(r) has period 16: the rows of so many instructions
    uint32_t base;          // LDS address of the first tile
    int src[NI];            // byte offset within a tile for each staging instruction
    uint32_t row_at[KS];    // row operands: lane (col, half) takes 8 elements from 16 ks + 8 half of row col
    uint32_t tr_at[DT][2];  // transposed operands of rows 0..15; + 16 rows leaves the swizzle as it is

    static __device__ __forceinline__ int swizzle(int r) {
        return D == 64 ? (((r >> 1) & 1) << 2) | ((r >> 2) & 3) : ((r & 3) << 2) | ((r >> 2) & 3);
    }
    // The lane's byte offset within a tile for staging instruction i
    static __device__ __forceinline__ int src_of(int i, int lane) {
        const int r = (i % PERIOD) * RPI + lane / CPR;
        return r * ROWB + ((lane % CPR) ^ swizzle(r)) * 16 + (i / PERIOD) * (PERIOD * 1024);
    }
    // Its offset within a tile of the transposed operand of columns 32 dt .. 32 dt + 31
    static __device__ __forceinline__ uint32_t tr_of(int dt, int hi, int lane) {
        const int half = lane >> 5, tr_row = (lane & 15) >> 2, quad = lane & 3, blk = (lane >> 4) & 1, r = 4 * half + tr_row + 8 * hi;
        return r * ROWB + (((4 * dt + 2 * blk + (quad >> 1)) ^ swizzle(r)) << 4) + 8 * (quad & 1);
    }
    // (src_of and tr_of written out: through the functions the forward's 128-row tiles at d = 128 spill a register)
    __device__ __forceinline__ WaveTile(uint32_t at, int lane) : base(at) {
        const int col = lane & 31, half = lane >> 5, tr_row = (lane & 15) >> 2, quad = lane & 3, blk = (lane >> 4) & 1;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int r = (i % PERIOD) * RPI + lane / CPR;
            src[i] = r * ROWB + ((lane % CPR) ^ swizzle(r)) * 16 + (i / PERIOD) * (PERIOD * 1024);
            asm volatile("" : "+v"(src[i]));
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            row_at[ks] = at + col * ROWB + (((2 * ks + half) ^ swizzle(col)) << 4);
            asm volatile("" : "+v"(row_at[ks]));
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                const int r = 4 * half + tr_row + 8 * hi;
                tr_at[dt][hi] = at + r * ROWB + (((4 * dt + 2 * blk + (quad >> 1)) ^ swizzle(r)) << 4) + 8 * (quad & 1);
                asm volatile("" : "+v"(tr_at[dt][hi]));
            }
    }
    // Instruction i of NI that bring the tile at the resource's start to base + offset (rows past its end arrive as zeros).
    // To be issued one per MFMA step: in a burst, the wave sits about 100 cycles in the issue of each, 64 bytes per clock
    // being what a CU's vector memory path moves.
    __device__ __forceinline__ void request(const BufferWords& rsrc, uint32_t offset, int i) const {
        global_to_lds_16B(rsrc, base + offset + i * 1024, src[i]);
    }
    __device__ __forceinline__ i32x4 row_read(int offset, int ks) const { return lds_load_16B(row_at[ks] + offset); }
    __device__ __forceinline__ i32x4 tr_read(int offset, int slab, int dt) const {
        const int a = offset + slab * 16 * ROWB;
        const i32x2 lo = lds_read_tr16(tr_at[dt][0] + a), hi = lds_read_tr16(tr_at[dt][1] + a);
        return i32x4{lo[0], lo[1], hi[0], hi[1]};
    }
};

static __device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

constexpr int kStreamed = 2;  // the cache policy bit of a raw buffer store that makes it non-temporal

// Stores a wave's 32-row x (32 DT)-column fp32 accumulator tile (MFMA result layout with rows as
// lane columns: lane (col, half) holds row `col`; register r of tile dt is column
// 32 dt + 8 (r / 4) + 4 half + r % 4) as 16-bit elements, scaled by `factor`.  Stored straight from
// that layout every store instruction would touch 32 rows with 16 bytes each; instead the tile
// goes through `patch` (4 KiB of LDS private to the wave), 128 bytes of every row at a time, and
// leaves as whole 128-byte lines: 16-byte chunk c of row r sits at chunk c ^ (r % 8) of the patch.  The stores are marked
// non-temporal (kStreamed): kept in the L2 until the launch ends, the outputs would displace what other workgroups still
// read.  Over 600 drawn launches (forward, FP8 forward, backward with its key blocks' stores so too) 0.98 of the time, 0.81
// at best (d = 256 causal, 488 heads x 128) and none above 1.02; d = 128 causal 512 x 512 75.0 -> 72.8 us, 256 x 512 at d = 64
// 20.8 -> 20.2.  (Written through instead (sc1), small launches take 2 to 3 % longer; the pre-pass's codes, which the next
// launch reads, and the few-workgroup forms' outputs gain nothing.)
// `rsrc` covers the [rows][32 DT] destination; rows at or past its end are dropped by the hardware.
template <typename Tag, int DT>
static __device__ __forceinline__ void store_rows_via_lds(const f32x16 (&acc)[DT], float factor, char* patch,
                                                           __amdgpu_buffer_rsrc_t rsrc, int row0, int lane) {
    static_assert(DT % 2 == 0, "128 bytes of a row are two 32-column tiles");
    using E = Elem<Tag>;
    constexpr int ROWB = DT * 64;  // bytes per destination row
    const int col = lane & 31, half = lane >> 5;
#pragma unroll
    for (int hd = 0; hd < DT / 2; ++hd) {
#pragma unroll
        for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int dt = 2 * hd + d2;
                i32x2 w;
                w[0] = E::pack2(acc[dt][4 * g] * factor, acc[dt][4 * g + 1] * factor);
                w[1] = E::pack2(acc[dt][4 * g + 2] * factor, acc[dt][4 * g + 3] * factor);
                *reinterpret_cast<i32x2*>(patch + col * 128 + (((4 * d2 + g) ^ (col & 7)) << 4) + 8 * half) = w;
            }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 8 * i + (lane >> 3), pc = lane & 7;
            const i32x4 w = *reinterpret_cast<const i32x4*>(patch + r * 128 + (pc << 4));
            __builtin_amdgcn_raw_buffer_store_b128(w, rsrc, (row0 + r) * ROWB + hd * 128 + ((pc ^ (r & 7)) << 4), 0, kStreamed);
        }
    }
}

// The item of workgroup `id` of `total` where every XCD takes a run of consecutive items, whatever the total: ids go to the
// XCDs in turn, and the first total % 8 XCDs get one more.
static __device__ __forceinline__ int xcd_run(int id, int total) {
    const int xcd = id & 7;
    return xcd * (total >> 3) + min(xcd, total & 7) + (id >> 3);
}

// ---------------------------------------------------------------------------------------
// Forward launches divided by keys (FewForward, FewFp8Forward): the pieces that do not depend on the data type.
//
// The head and the 32-query tile of a workgroup.  The tiles of a head share an L2 whatever the number of heads (d = 128, 61
// heads x 252, no mask: 13.5 us where they do not, 8.4 so).  split >= 0: grid (heads x R) x ceil(tiles / R), R = 2^split;
// x / 8 of the ids that land on XCD x % 8 counts through the groups (head, residue of the tile number mod R) of that XCD,
// y through the members of a group; causal: the longest rows first.  split < 0: one id per tile, head by head.
struct KeySplitTile {
    int head, tile, n_tiles;  // tile >= n_tiles: nothing to do
};
static __device__ __forceinline__ KeySplitTile key_split_tile(int N, int split) {
    const int n_t = (N + 31) / 32;
    if (split < 0) {
        const int xcd = blockIdx.x & 7, per = gridDim.x >> 3, rest = gridDim.x & 7;  // the first `rest` XCDs get one more
        const int id = xcd * per + min(xcd, rest) + ((int)blockIdx.x >> 3);
        return {id / n_t, id % n_t, n_t};
    }
    const int group = ((int)blockIdx.x & 7) * ((int)gridDim.x >> 3) + ((int)blockIdx.x >> 3);
    return {group >> split, ((int)blockIdx.y << split) + (group & ((1 << split) - 1)), n_t};
}

// The end of such a workgroup of NT threads: the states (m: reference in log2 units, l: the lane half's row sum, acc: O^T
// accumulator, lane column = query) of its first NW waves, which split the keys of 32 queries, become O and L.  With M the
// largest m and f = 2^(m - M), O = sum f acc / sum f l and L = ln 2 (M + log2 sum f l - bias); fixed order.  Every wave of
// the workgroup calls this; no LDS access or load to LDS may be pending but the caller's own wave's.
template <int D, int NW>
struct KeySplitMerge {
    static constexpr int PSTR = D + 4;  // row stride of the partial outputs (floats)
    static constexpr int kPartial = NW * 32 * PSTR * 4, kLds = kPartial + NW * 32 * 8;
    template <typename Tag, int NT>
    static __device__ __forceinline__ void run(const f32x16 (&acc)[D / 32], float m, float l_half, float bias, char* lds, int wave,
                                               int lane, uint16_t* o_head, float* lse_head, int q0, int N) {
        using E = Elem<Tag>;
        constexpr int CPR = D / 8;
        const int col = lane & 31, half = lane >> 5;
        __syncthreads();
        float* part = reinterpret_cast<float*>(lds);              // [wave][query][PSTR]
        float* state = reinterpret_cast<float*>(lds + kPartial);  // [wave][query][m, l]
        const float l = sum_both_halves(l_half);
        if (wave < NW) {
            if (half == 0) {
                state[(wave * 32 + col) * 2] = m;
                state[(wave * 32 + col) * 2 + 1] = l;
            }
#pragma unroll
            for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 w = {acc[dt][4 * g], acc[dt][4 * g + 1], acc[dt][4 * g + 2], acc[dt][4 * g + 3]};
                    *reinterpret_cast<f32x4*>(part + (wave * 32 + col) * PSTR + dt * 32 + 8 * g + 4 * half) = w;
                }
        }
        __syncthreads();
        for (int c = threadIdx.x; c < 32 * CPR; c += NT) {
            const int r = c / CPR, cc = (c % CPR) * 8;
            float m_all = -INFINITY, l_all = 0.f, f[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, state[(w * 32 + r) * 2]);
            const float m_ref = m_all == -INFINITY ? 0.f : m_all;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                f[w] = fast_exp2(state[(w * 32 + r) * 2] - m_ref);
                l_all += f[w] * state[(w * 32 + r) * 2 + 1];
            }
            float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 y = *reinterpret_cast<const f32x4*>(part + (w * 32 + r) * PSTR + cc + 4 * h);
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[4 * h + e] = __builtin_fmaf(f[w], y[e], x[4 * h + e]);
                }
            const float inv = 1.0f / l_all;
            if (q0 + r < N) {
                i32x4 y;
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = E::pack2(x[2 * e] * inv, x[2 * e + 1] * inv);
                *reinterpret_cast<i32x4*>(o_head + (size_t)(q0 + r) * D + cc) = y;
                if (cc == 0) lse_head[q0 + r] = (m_all + log2f(l_all) - bias) * kLn2;
            }
        }
    }
};

// The chip deals consecutive workgroup ids round-robin to its 8 XCDs, each with a private
// L2.  Remap a linear id so that ids landing on one XCD cover a contiguous range of work
// items (all query tiles of a head share that head's K and V in one L2).
static __device__ __forceinline__ int xcd_contiguous(int id, int total) {
    constexpr int kXcd = 8;
    if (total % kXcd != 0) return id;
    return (id % kXcd) * (total / kXcd) + id / kXcd;
}

// (head, tile) of a workgroup.  Without a mask all tiles of a head cost the same and consecutive ids of an XCD take
// the tiles of one head (above).  Under a causal mask tile 0 is the longest by convention, and workgroups are dealt in
// order of length over all heads: the hardware hands the next one to the first CU that is free, so the last to start
// are the shortest and the CUs finish together.  (Head after head, long tiles of the last heads start when nothing is
// left to fill the other CUs with.)  With a multiple of 8 heads every head still stays on one XCD.
struct WorkItem {
    int head, tile;
};
template <bool CAUSAL>
static __device__ __forceinline__ WorkItem work_item(int block, int total, int n_tiles) {
    if constexpr (CAUSAL) {
        const int n_heads = total / n_tiles;
        return {block % n_heads, block / n_heads};
    } else {
        const int id = xcd_contiguous(block, total);
        return {id / n_tiles, id % n_tiles};
    }
}

// Query tiles of a forward workgroup: `tile` of `head`, then `second` unless it is negative.  A causal launch either
// deals single tiles in order of length (as work_item does; heads along the grid's x, tiles along its y, which spares
// the workgroup two divisions) or, `paired`, tiles i and n_qtiles-1-i one after the other, the longer first: items that
// all cover the same number of key blocks (with an odd tile count the middle tile is an item of its own).  Pairs start
// half as many workgroups, which is the better choice when the items fill whole rounds of the chip (pair_causal_tiles).
// BY_XCD (the 128-row 16-bit tiles): the tiles of a head stay on one XCD also where the number of items or heads is no
// multiple of 8; otherwise they go to all eight, each of which reads the head's K and V.  Items: runs of them per XCD.  Single
// tiles: a row of the grid starts at XCD y heads % 8, so its heads are turned by as much, but for the last heads % 8, whose
// tiles move on from row to row and keep the XCDs even (all tiles of a head on one XCD: 107 heads x 400, d = 64, 16.9 us instead
// of 10.8).  `total` is the number of heads then.  bf16, us, heads x N, spread / kept:
//   no mask  d = 64  85 x 710 22.4 / 20.9, 139 x 648 32.4 / 28.7;  d = 128  85 x 648 33.0 / 28.3, 121 x 896 76.4 / 64.8
//   causal   d = 64  107 x 957 27.0 / 25.4;  d = 128  83 x 1024 40.1 / 33.8, 95 x 1665 113 / 96
// Three of these workgroups share a CU, so more K and V pass through an L2 at a time than with two, and with the tiles spread
// these calls fell behind the 256-row tiles.
struct TileRun {
    int head, tile, second;
    __device__ __forceinline__ int n_pass() const { return second < 0 ? 1 : 2; }
};
template <bool CAUSAL, bool BY_XCD = false>
static __device__ __forceinline__ TileRun query_tiles(int total, int n_qtiles, int paired) {
    const int n_items = CAUSAL ? (n_qtiles + 1) / 2 : n_qtiles;
    const int id = BY_XCD ? xcd_run(blockIdx.x, total) : xcd_contiguous(blockIdx.x, total);
    const bool single = CAUSAL && !paired;
    int single_head = blockIdx.x;
    if constexpr (CAUSAL && BY_XCD)
        if (single_head < (total & ~7)) single_head = (single_head & ~7) | ((single_head + (int)blockIdx.y * total) & 7);
    // (both ways without a branch: with one the code behind it is laid out differently, and pairs took 2.5 % longer at
    // d = 64, 16 x 8192, and d = 128, 256 x 300)
    const int head = single ? single_head : id / n_items, i = single ? (int)blockIdx.y : id - head * n_items;
    return {head, CAUSAL ? n_qtiles - 1 - i : i, CAUSAL && !single && n_qtiles - 1 - i != i ? i : -1};
}

// Measurement builds (-DFA_CLOCK_SPAN): how many shader-clock cycles a launch took on one CU.  A kernel
// declares a ClockSpan as its first statement; workgroups that run on the chosen CU record the earliest
// entry stamp and the latest exit stamp (the shader clock is only comparable within a CU).  The CU is that
// of workgroup 0 of the first launch after the library is loaded, so that launch only chooses and the
// launches after it measure.  Cycles divided by the launch's wall time is the clock the chip actually ran
// at: it lowers the clock under load, so a kernel that needs fewer cycles need not take less time.  Each
// source file that holds measured kernels defines its reader with FA_CLOCK_SPAN_READER(name).  In ordinary
// builds ClockSpan is empty and generates no code.
#ifdef FA_CLOCK_SPAN
static __device__ unsigned long long fa_clock_span_cycles[2] = {~0ull, 0ull};
static __device__ int fa_clock_span_cu = -1;
struct ClockSpan {
    long long t0;
    __device__ __forceinline__ ClockSpan() : t0(__builtin_readcyclecounter()) {}
    __device__ __forceinline__ ~ClockSpan() {
        if (threadIdx.x == 0) {
            // XCC id, then shader engine / shader array / CU from the hardware id register
            const int cu = (int)(((__builtin_amdgcn_s_getreg((31 << 11) | 20) & 15) << 8) |
                                 ((__builtin_amdgcn_s_getreg((31 << 11) | 4) >> 8) & 255));
            if (blockIdx.x == 0 && fa_clock_span_cu < 0) fa_clock_span_cu = cu;
            if (cu == fa_clock_span_cu) {
                atomicMin(&fa_clock_span_cycles[0], (unsigned long long)t0);
                atomicMax(&fa_clock_span_cycles[1], (unsigned long long)__builtin_readcyclecounter());
            }
        }
    }
};
// span[0], span[1]: first entry and last exit stamp since the last call; the call clears them
#define FA_CLOCK_SPAN_READER(name)                                                                              \
    extern "C" int name(unsigned long long* span) {                                                             \
        const unsigned long long init[2] = {~0ull, 0ull};                                                       \
        if (hipDeviceSynchronize() != hipSuccess) return 1;                                                     \
        if (hipMemcpyFromSymbol(span, HIP_SYMBOL(fa::fa_clock_span_cycles), sizeof(init)) != hipSuccess) return 2; \
        return hipMemcpyToSymbol(HIP_SYMBOL(fa::fa_clock_span_cycles), init, sizeof(init)) == hipSuccess ? 0 : 3; \
    }
#else
struct ClockSpan {};
#define FA_CLOCK_SPAN_READER(name)
#endif

}  // namespace fa
