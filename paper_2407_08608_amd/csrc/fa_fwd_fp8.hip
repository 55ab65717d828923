// FP8 (e4m3) forward attention for gfx950 (paper section 3.3).
//
// Same tiling as the 16-bit kernel (Algorithm 1), on v_mfma_f32_32x32x64_f8f6f4: both GEMMs
// contract 64 elements per instruction and a lane holds 32 bytes of an operand.
//   * Block quantisation: a block of S is rescaled by s_Q[i] * s_K[j], folded into the exp2
//     multiplier, so it costs nothing per element.  A V block's scale enters as an offset in
//     the exponent of P~ (the numerator's weights are p * s_V), which costs nothing either.
//   * Layout conformance: V is stored d-contiguous but must be contracted over keys.  The
//     transposing LDS read (ds_read_b64_tr_b8) hands a lane 8 consecutive keys of one column,
//     while the fp32 accumulator of S^T gives a lane-half alternating groups of 4 rows.  The
//     rows of the K operand are therefore permuted (row i of the MFMA reads key pi(i)) so
//     that each lane-half ends up owning two runs of 8 consecutive keys; P~ then goes from
//     accumulator registers to operand registers with conversions only, no cross-lane moves.
//     This is the same idea as the paper's register permutation plus matching V-row
//     permutation, rederived for the gfx950 layouts.
//   * P~ = exp2(s - m_ref + 6) where the reference maximum m_ref is raised only when a block's
//     maximum exceeds it by more than 2 (log2 units), so P~ <= 256 < 448: the bias uses more of
//     e4m3's range, both factors cancel in O / l, and L subtracts the bias again.
#include "fa_device.h"
#include "fa_launch.h"

// Measurement builds only (paper_2407_08608_amd/ablate.py compiles this file with them; the library never
// defines them).  FA_ABLATE removes one part of fa_fwd_fp8_kernel's block to see what the rest costs -- the
// results are wrong on purpose: 1 = no exponentials, 2 = no LDS reads for the second GEMM, 3 = no second GEMM,
// 4 = no softmax arithmetic (scale, exponential, row sum).  FA_PHASE_TRACE stamps the phases of 32 blocks
// of one workgroup of the eight-wave d = 128 instantiation with the shader clock.  FA_STAGED_TILE8 makes the
// launcher pick that instantiation (the register-staged eight-wave tile) where the library runs
// fa_fwd_fp8_async_kernel, which has the same block arithmetic and no such switches.
#ifndef FA_ABLATE
#define FA_ABLATE 0
#endif
#ifdef FA_PHASE_TRACE
__device__ long long fa_phase_trace[8][32][8];
extern "C" int fa_debug_read_phase_trace(void* host) {
    return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(fa_phase_trace), sizeof(fa_phase_trace));
}
#define FA_STAMP(i) do { if (tracing) stamps[i] = __builtin_readcyclecounter(); } while (0)
#define FA_STAMP_AFTER(i, ...) do { if (tracing) { asm volatile("s_nop 0" : __VA_ARGS__); stamps[i] = __builtin_readcyclecounter(); } } while (0)
#else
#define FA_STAMP(i) do { } while (0)
#define FA_STAMP_AFTER(i, ...) do { } while (0)
#endif

namespace fa {

constexpr float kPBias = 6.0f;
constexpr float kLazyLog2 = 2.0f;

static __device__ __forceinline__ f32x16 mma_fp8(i32x8 a, i32x8 b, f32x16 c) {
    // cbsz = blgp = 0: both operands e4m3; scale exponents 127 = 1.0
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
}

// Four values as e4m3 codes, first lowest.  Each conversion writes one half of the word and keeps the other: what the first
// one keeps is overwritten by the second, so the word starts as whatever its register holds (a zero would cost a move).
static __device__ __forceinline__ int pack_e4m3(float a, float b, float c, float d) {
    int word;
    asm volatile("" : "=v"(word));
    word = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, word, false);
    return __builtin_amdgcn_cvt_pk_fp8_f32(c, d, word, true);
}

// key held in MFMA row i of a 32-key tile
static __device__ __forceinline__ int key_of_row(int i) {
    int g = i >> 3, hb = (i >> 2) & 1, r = i & 3;
    return 16 * (g >> 1) + 8 * hb + 4 * (g & 1) + r;
}

// Swizzles of unpadded e4m3 tiles: the 16-byte chunk c of tile row r sits at chunk c ^ k(r) (K, read by rows) or c ^ v(r) (V,
// read transposed) of its LDS row.  256-byte rows fill the 64 banks once: sixteen rows need sixteen different chunk positions
// (K row reads), eight rows x two chunks likewise (V transposing reads).  Two 128-byte rows (four 64-byte rows) share the
// banks, so pairs (fours) of rows share a swizzle value.
template <int D>
struct Fp8Swizzle {
    static __device__ __forceinline__ int k(int r) { return D == 256 ? (r & 15) : D == 128 ? ((r >> 1) & 7) : ((r >> 2) & 3); }
    static __device__ __forceinline__ int v(int r) { return D == 256 ? ((r & 7) << 1) : D == 128 ? (((r >> 1) & 3) << 1) : (((r >> 2) & 1) << 1); }
};

// ---------------------------------------------------------------------------------------
// The FP8 forward where its query tiles would leave most of the chip idle (as FewForward in fa_fwd.hip): a workgroup of NW
// waves owns 32 queries, and NS of the waves split the keys, tiles of 64 dealt in turn, each staged by the wave that works it
// (V beside the scores, K of its next tile beside the products: no barrier), each with a softmax state and an accumulator for
// all columns, merged through the LDS at the end.  The arithmetic of a tile is that of the kernels below.
// (At d = 256 the tiles of eight waves do not fit the LDS: four of them split, the others wait for the merge.)
template <int D, int NW, int NS>
struct FewFp8Forward {
    static constexpr int BK = 64, ROWB = D, TILE = BK * ROWB;  // keys, row bytes and bytes of a tile
    static constexpr int KS = D / 64, DT = D / 32;
    static constexpr int CPR = ROWB / 16, RPI = 1024 / ROWB, NI = TILE / 1024, PERIOD = 16 / RPI;  // (16 rows: both swizzles' period)
    static constexpr int kStages = NS * 2 * TILE;
    static constexpr int kLds = KeySplitMerge<D, NS>::kLds > kStages ? KeySplitMerge<D, NS>::kLds : kStages;

    template <bool CAUSAL, bool SCALED>
    static __device__ __forceinline__ void run(const uint8_t* __restrict__ q, const uint8_t* __restrict__ k, const uint8_t* __restrict__ v,
                                               const float* __restrict__ q_scale, const float* __restrict__ k_scale,
                                               const float* __restrict__ v_scale, uint16_t* __restrict__ o, float* __restrict__ lse,
                                               int N, int split, int n_sblocks, int kv_group, float scale, char* lds) {
        using Swizzle = Fp8Swizzle<D>;
        const int tid = threadIdx.x;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
        const int col = lane & 31, half = lane >> 5;
        const KeySplitTile item = key_split_tile(N, split);
        if (item.tile >= item.n_tiles) return;
        const int bh = item.head, kv_bh = bh / kv_group;
        const int qt = CAUSAL ? item.n_tiles - 1 - item.tile : item.tile;
        const int q0 = qt * 32, n_tiles = CAUSAL ? q0 / BK + 1 : (N + BK - 1) / BK;
        const int row = min(q0 + col, N - 1);    // rows past N compute a copy of row N-1, never stored
        const int limit = CAUSAL ? row : N - 1;  // last visible key

        f32x16 oacc[DT];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
        // m: running (lazily raised) maximum, in log2 units, of the real scores plus log2 of their V block's scale
        float m_run = -INFINITY, l_run = 0.f;

        if (wave < NS) {
            const uint32_t kb = lds_address(lds) + wave * (2 * TILE), vb = kb + TILE;
            // the wave's next tiles (rows past N read as zero)
            BufferWords k_rsrc = make_buffer_words(k + (size_t)kv_bh * N * D, (uint32_t)N * D);
            BufferWords v_rsrc = make_buffer_words(v + (size_t)kv_bh * N * D, (uint32_t)N * D);
            advance(k_rsrc, wave * TILE);
            advance(v_rsrc, wave * TILE);
            int k_src[PERIOD], v_src[PERIOD];  // byte offsets within a tile of the first staging instructions
#pragma unroll
            for (int i = 0; i < PERIOD; ++i) {
                const int r = i * RPI + lane / CPR, c = lane % CPR;
                k_src[i] = r * ROWB + ((c ^ Swizzle::k(r)) << 4);
                v_src[i] = r * ROWB + ((c ^ Swizzle::v(r)) << 4);
            }
            auto request = [&](const BufferWords& rsrc, uint32_t to, const int (&src)[PERIOD], int i) __attribute__((always_inline)) {
                global_to_lds_16B(rsrc, to + i * 1024, src[i % PERIOD] + (i / PERIOD) * (PERIOD * 1024));
            };
            // (a wave without a tile brings rows that nothing reads, or zeros)
#pragma unroll
            for (int i = 0; i < NI; ++i) request(k_rsrc, kb, k_src, i);
            i32x8 qreg[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const uint8_t* p = q + ((size_t)bh * N + row) * D + ks * 64 + half * 32;
                const i32x4 lo = *reinterpret_cast<const i32x4*>(p), hi = *reinterpret_cast<const i32x4*>(p + 16);
                qreg[ks] = i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            }
            float sc_q = scale * kLog2e;
            if constexpr (SCALED) sc_q *= q_scale[(size_t)bh * n_sblocks + q0 / 128];
            // operand addresses: K row key_of_row(col), V rows 8 half + (lane / 2) % 8 (+ 16, 32, 48: the swizzle stays)
            const int krow = key_of_row(col), tr_row = (lane & 15) >> 1, blk = (lane >> 4) & 1;
            uint32_t k_at[KS][2], v_at[DT];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    k_at[ks][j] = kb + krow * ROWB + (((4 * ks + 2 * half + j) ^ Swizzle::k(krow)) << 4);
                    asm volatile("" : "+v"(k_at[ks][j]));
                }
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                v_at[dt] = vb + (8 * half + tr_row) * ROWB + (((2 * dt + blk) ^ Swizzle::v(tr_row)) << 4) + 8 * (lane & 1);
                asm volatile("" : "+v"(v_at[dt]));
            }
            auto k_read = [&](int u) __attribute__((always_inline)) {  // u = (ks, 32-key half of the tile)
                const i32x4 lo = lds_load_16B(k_at[u / 2][0] + (u % 2) * 32 * ROWB), hi = lds_load_16B(k_at[u / 2][1] + (u % 2) * 32 * ROWB);
                return i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            };
            auto v_read = [&](int dt) __attribute__((always_inline)) {
                i32x8 a;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const i32x2 w = lds_read_tr8(v_at[dt] + 16 * x * ROWB);
                    a[2 * x] = w[0];
                    a[2 * x + 1] = w[1];
                }
                return a;
            };
            static_assert(NI == 2 * 2 * KS && NI == 2 * DT, "two staging instructions per MFMA");
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));

            for (int t = wave; t < n_tiles; t += NS) {
                float sk = 1.0f, sv = 1.0f;
                if constexpr (SCALED) {
                    sk = k_scale[(size_t)kv_bh * n_sblocks + t / 2];
                    sv = v_scale[(size_t)kv_bh * n_sblocks + t / 2];
                }
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // K has landed, the last V has been read
                advance(k_rsrc, NS * TILE);
                if (t + NS >= n_tiles) k_rsrc.w[2] = 0;  // past the wave's last tile: zeros that nothing reads
                // S^T = K Q^T (rows permuted by key_of_row)
                f32x16 s[2];
                const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                i32x8 next = k_read(0);
#pragma unroll
                for (int u = 0; u < 2 * KS; ++u) {
                    const i32x8 a = next;
                    if (u + 1 < 2 * KS) next = k_read(u + 1);
                    request(v_rsrc, vb, v_src, 2 * u);
                    request(v_rsrc, vb, v_src, 2 * u + 1);
                    s[u % 2] = mma_fp8(a, qreg[u / 2], u < 2 ? zero : s[u % 2]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (t * BK + BK > N || (CAUSAL && t * BK + BK - 1 > q0)) {
                    int bound = limit - t * BK - 8 * half;  // register r of a 32-key half is key 16 (r / 8) + 8 half + r % 8
                    asm volatile("" : "+v"(bound));
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if (kt * 32 + 16 * (r >> 3) + (r & 7) > bound) s[kt][r] = -INFINITY;
                }
                // reference maximum, P~ as e4m3, row sum: see fa_fwd_fp8_kernel
                float mxp[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) mxp[r & 3] = fmaxf(mxp[r & 3], s[kt][r]);
                const float sc = sc_q * sk;
                float lsv = 0.f;
                if constexpr (SCALED) lsv = __builtin_amdgcn_logf(sv);  // log2
                const float mx = max_both_halves(fmaxf(fmaxf(mxp[0], mxp[1]), fmaxf(mxp[2], mxp[3]))) * sc + lsv;
                const bool raise = mx - m_run > kLazyLog2;
                if (__builtin_amdgcn_ballot_w64(raise) != 0) {
                    const float f = raise ? fast_exp2(m_run - mx) : 1.0f;
                    m_run = raise ? mx : m_run;
                    l_run *= f;
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                        for (int r = 0; r < 16; ++r) oacc[dt][r] *= f;
                }
                const float mb = m_run == -INFINITY ? 0.f : m_run - kPBias - lsv;  // a row of scores of -inf so far: P = 0
                float sc_v = sc;  // a vector-register copy: an FMA with a scalar-register operand issues at a lower rate
                asm volatile("" : "+v"(sc_v));
                float ps[4];
                i32x8 pb;
#pragma unroll
                for (int kt = 0; kt < 2; ++kt) {
                    float p[16];
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        p[r] = fast_exp2(__builtin_fmaf(s[kt][r], sc_v, -mb));
                        ps[r & 3] = kt == 0 && r < 4 ? p[r] : ps[r & 3] + p[r];
                    }
#pragma unroll
                    for (int w = 0; w < 4; ++w) pb[4 * kt + w] = pack_e4m3(p[4 * w], p[4 * w + 1], p[4 * w + 2], p[4 * w + 3]);
                }
                float psum = (ps[0] + ps[1]) + (ps[2] + ps[3]);
                if constexpr (SCALED) psum *= __builtin_amdgcn_rcpf(sv);
                l_run += psum;
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // V has landed, K has been read
                advance(v_rsrc, NS * TILE);
                // O^T += V^T P~^T
                next = v_read(0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const i32x8 a = next;
                    if (dt + 1 < DT) next = v_read(dt + 1);
                    request(k_rsrc, kb, k_src, 2 * dt);
                    request(k_rsrc, kb, k_src, 2 * dt + 1);
                    oacc[dt] = mma_fp8(a, pb, oacc[dt]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the last requests: the LDS is about to be reused
        }
        KeySplitMerge<D, NS>::template run<bf16_tag, NW * 64>(oacc, m_run, l_run, kPBias, lds, wave, lane, o + (size_t)bh * N * D,
                                                              lse + (size_t)bh * N, q0, N);
    }
};

template <int D, int BC, int NW, bool CAUSAL, bool SCALED>
__global__ void __launch_bounds__(NW * 64, D <= 128 ? 2 : 1)
fa_fwd_fp8_kernel(const uint8_t* __restrict__ q, const uint8_t* __restrict__ k, const uint8_t* __restrict__ v,
                  const float* __restrict__ q_scale, const float* __restrict__ k_scale,
                  const float* __restrict__ v_scale, uint16_t* __restrict__ o, float* __restrict__ lse, int N,
                  int n_qtiles, int total_wg, int paired, int n_sblocks, int kv_group, float scale) {
    [[maybe_unused]] ClockSpan clock_span;  // measurement builds only; empty otherwise
    constexpr int NT = NW * 64;
    constexpr int BR = NW * 32;
    constexpr int KSTR = D + 16;  // bytes per LDS row
    constexpr int VSTR = D + 32;
    constexpr int KT = BC / 32;
    constexpr int KS = D / 64;    // MFMA steps along the head dimension
    constexpr int DT = D / 32;
    constexpr int SL = BC / 64;   // MFMA steps along the keys
    constexpr int CPR = D / 16;   // 16-byte chunks per row
    constexpr int CPT = BC * CPR / NT;
    static_assert(BC % 64 == 0 && 128 % BC == 0, "key block must tile the 128-row quantisation block");
    static_assert((BC * CPR) % NT == 0, "tile must divide evenly over the workgroup");

    // K blocks, V blocks, output transposition (4 KiB per wave)
    constexpr int kKLds = 2 * BC * KSTR, kVLds = 2 * BC * VSTR, kTileLds = kKLds + kVLds + NW * 4096;
    static_assert(kKLds % 128 == 0 && kVLds % 128 == 0, "aligned parts");
    constexpr bool kHasFew = NW == 4;  // (the eight-wave instantiations are measurement builds')
    constexpr int kFewLds = kHasFew ? FewFp8Forward<D, 4, 4>::kLds : 0;
    __shared__ __attribute__((aligned(1024))) char lds[kTileLds > kFewLds ? kTileLds : kFewLds];
    if constexpr (kHasFew) {
        if (paired == kFewForward) {
            FewFp8Forward<D, 4, 4>::template run<CAUSAL, SCALED>(q, k, v, q_scale, k_scale, v_scale, o, lse, N, total_wg, n_sblocks, kv_group, scale, lds);
            return;
        }
    }
    uint8_t(*lds_k)[BC * KSTR] = reinterpret_cast<uint8_t(*)[BC * KSTR]>(lds);
    uint8_t(*lds_v)[BC * VSTR] = reinterpret_cast<uint8_t(*)[BC * VSTR]>(lds + kKLds);
    char* lds_o = lds + kKLds + kVLds;

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;

    const TileRun run = query_tiles<CAUSAL>(total_wg, n_qtiles, paired);
    const int bh = run.head;

    const size_t head_off = (size_t)bh * N * D;
    const uint8_t* qh = q + head_off;
    const int kv_bh = bh / kv_group;  // grouped-query: kv_group query heads per K/V head
    const uint8_t* kh = k + (size_t)kv_bh * N * D;
    const uint8_t* vh = v + (size_t)kv_bh * N * D;
#pragma nounroll
    for (int pass = 0; pass < run.n_pass(); ++pass) {
    // every LDS read of the previous pass was followed by a barrier
    const int qt = pass == 0 ? run.tile : run.second;
    const int wave_q0 = qt * BR + wave * 32;

    float sq = 1.0f;
    if constexpr (SCALED) sq = q_scale[(size_t)bh * n_sblocks + min(wave_q0 / 128, n_sblocks - 1)];
    const float sc_q = scale * kLog2e * sq;

    i32x8 qreg[KS];
    {
        int row = min(wave_q0 + col, N - 1);  // rows past N compute a copy of row N-1, never stored
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const uint8_t* p = qh + (size_t)row * D + ks * 64 + half * 32;
            i32x4 lo = *reinterpret_cast<const i32x4*>(p);
            i32x4 hi = *reinterpret_cast<const i32x4*>(p + 16);
            qreg[ks] = i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
    }

    f32x16 oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
    // m: running (lazily raised) maximum, in log2 units, of the real scores plus log2 of their V block's scale
    float m_run = -INFINITY, l_run = 0.f;

    int last_q = min(qt * BR + BR, N) - 1;
    int n_blocks = CAUSAL ? (last_q / BC + 1) : ((N + BC - 1) / BC);

    // a [BC][D] tile of a row-major head is contiguous: chunk c sits at tile offset 16*c; rows past N
    // lie outside the buffer resource and read as zero
    const __amdgpu_buffer_rsrc_t k_rsrc = make_buffer(kh, (uint32_t)N * D);
    const __amdgpu_buffer_rsrc_t v_rsrc = make_buffer(vh, (uint32_t)N * D);
    auto load_tile = [&](__amdgpu_buffer_rsrc_t head, int key0, i32x4 (&regs)[CPT]) {
#pragma unroll
        for (int i = 0; i < CPT; ++i) regs[i] = buffer_load_16B(head, key0 * D + (tid + i * NT) * 16);
    };
    auto store_tile = [&](uint8_t* lds, int stride, const i32x4 (&regs)[CPT]) {
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            int c = tid + i * NT;
            int row = c / CPR, cc = c % CPR;
            *reinterpret_cast<i32x4*>(lds + row * stride + cc * 16) = regs[i];
        }
    };

    i32x4 kpre[CPT], vpre[CPT];
    load_tile(k_rsrc, 0, kpre);
    load_tile(v_rsrc, 0, vpre);
    store_tile(lds_k[0], KSTR, kpre);
    store_tile(lds_v[0], VSTR, vpre);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));  // Q loads complete before the loop
    __syncthreads();

    const int krow = key_of_row(col);  // key (within a 32-key tile) this lane's A row reads
    const int tr_row = (lane & 15) >> 1;
    const int tr_col = 16 * ((lane >> 4) & 1) + 8 * (lane & 1);

    for (int t = 0; t < n_blocks; ++t) {
        const int st = t & 1;
        const int key0 = t * BC;
        const bool more = (t + 1 < n_blocks);
#ifdef FA_PHASE_TRACE
        const bool tracing = D == 128 && NW == 8 && !CAUSAL && blockIdx.x == 300 && t >= 60 && t < 92;
        long long stamps[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#endif
        FA_STAMP(0);
        if (more) {
            load_tile(k_rsrc, key0 + BC, kpre);
            load_tile(v_rsrc, key0 + BC, vpre);
        }
        const bool wave_active = !CAUSAL || key0 <= wave_q0 + 31;
        if (wave_active) {
            float sk = 1.0f, sv_new = 1.0f;
            if constexpr (SCALED) {
                sk = k_scale[(size_t)kv_bh * n_sblocks + key0 / 128];
                sv_new = v_scale[(size_t)kv_bh * n_sblocks + key0 / 128];
            }
            const float sc = sc_q * sk;

            // ---- GEMM0: S^T = K_j Q_i^T (rows permuted by key_of_row)
            f32x16 sacc[KT];
            const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) {
                    const uint8_t* p = lds_k[st] + (kt * 32 + krow) * KSTR + ks * 64 + half * 32;
                    i32x4 lo = *reinterpret_cast<const i32x4*>(p);
                    i32x4 hi = *reinterpret_cast<const i32x4*>(p + 16);
                    i32x8 a = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                    sacc[kt] = mma_fp8(a, qreg[ks], ks == 0 ? zero : sacc[kt]);
                }

            FA_STAMP_AFTER(1, "+v"(sacc[0]), "+v"(sacc[KT - 1]));  // scores done
            const bool need_mask = (key0 + BC > N) || (CAUSAL && key0 + BC - 1 > wave_q0);
            if (need_mask) {
                int qi = wave_q0 + col;
                int limit = CAUSAL ? min(qi, N - 1) : N - 1;
                // register r of lane-half `half` holds key 16 (r / 8) + 8 half + r % 8 of its 32-key tile (the
                // rows of the K operand are permuted); compile-time offsets against one opaque per-lane bound
                int bound = limit - key0 - 8 * half;
                asm volatile("" : "+v"(bound));
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (kt * 32 + 16 * (r >> 3) + (r & 7) > bound) sacc[kt][r] = -INFINITY;
            }

            // ---- online softmax in log2 units of the real scores.  Independent chains for the maximum
            // and the sum: a wave gets few issue slots while its SIMD sibling streams MFMAs, and one
            // long dependent chain would turn every slot missed into a stall.
            float mxp[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};  // (a chain that starts from a score pays to quiet it first)
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) mxp[r & 3] = fmaxf(mxp[r & 3], sacc[kt][r]);
            // V block scales: O = sum_k p_k s_V[j] V^_k / sum_k p_k.  The numerator's weights are
            // 2^(s_k + log2 s_V[j]), so the block's scale is an offset in the exponent of P~ -- no work
            // per element -- and the running maximum is taken over the offset scores: P~ <= 2^(6+2) for
            // every block, and the key that raises the maximum gets P~ = 2^6 exactly.  The row sum needs
            // the weights without the offset: the block's sum divided by s_V[j], once per block.
            float lsv = 0.f;
            if constexpr (SCALED) lsv = __builtin_amdgcn_logf(sv_new);  // log2
            const float mx = max_both_halves(fmaxf(fmaxf(mxp[0], mxp[1]), fmaxf(mxp[2], mxp[3]))) * sc + lsv;
            const bool raise = mx - m_run > kLazyLog2;
            if (__builtin_amdgcn_ballot_w64(raise) != 0) {
                const float f = raise ? fast_exp2(m_run - mx) : 1.0f;
                m_run = raise ? mx : m_run;
                l_run *= f;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[dt][r] *= f;
            }
            FA_STAMP(2);  // mask, row maximum, reference
            const float mb = m_run - kPBias - lsv;
            float sc_v = sc;  // a vector-register copy: an FMA with a scalar-register operand issues at a lower rate
            asm volatile("" : "+v"(sc_v));
            float ps[4];
            i32x8 pb[SL];
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                float p[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
#if FA_ABLATE == 1
                    p[r] = __builtin_fmaf(sacc[kt][r], sc_v, -mb);
#elif FA_ABLATE == 4
                    p[r] = sacc[kt][r];
#else
                    p[r] = fast_exp2(__builtin_fmaf(sacc[kt][r], sc_v, -mb));
#endif
#if FA_ABLATE != 4
                    ps[r & 3] = kt == 0 && r < 4 ? p[r] : ps[r & 3] + p[r];
#endif
                }
#pragma unroll
                for (int w = 0; w < 4; ++w) pb[kt >> 1][4 * (kt & 1) + w] = pack_e4m3(p[4 * w], p[4 * w + 1], p[4 * w + 2], p[4 * w + 3]);
            }
            float psum = (ps[0] + ps[1]) + (ps[2] + ps[3]);
            if constexpr (SCALED) psum *= __builtin_amdgcn_rcpf(sv_new);
            l_run += psum;

            FA_STAMP_AFTER(3, "+v"(pb[0]), "+v"(l_run));  // P~ done
            // ---- GEMM1: O^T += V_j^T P^T
            const uint8_t* vs_base = lds_v[st] + (8 * half + tr_row) * VSTR + tr_col;
#pragma unroll
            for (int sl = 0; sl < SL; ++sl)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    i32x8 a;
#if FA_ABLATE == 2
                    a = qreg[0];
                    asm volatile("" : "+v"(a));
#else
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        i32x2 w = lds_read_tr8(vs_base + (sl * 64 + 16 * u) * VSTR + dt * 32);
                        a[2 * u] = w[0];
                        a[2 * u + 1] = w[1];
                    }
#endif
#if FA_ABLATE == 3
                    asm volatile("" ::"v"(a), "v"(pb[sl]));
#else
                    oacc[dt] = mma_fp8(a, pb[sl], oacc[dt]);
#endif
                }
        }
        FA_STAMP_AFTER(4, "+v"(oacc[0]), "+v"(oacc[DT - 1]));  // products done
        if (more) {
            store_tile(lds_k[st ^ 1], KSTR, kpre);
            store_tile(lds_v[st ^ 1], VSTR, vpre);
        }
        FA_STAMP(5);  // next tiles written to LDS
        __syncthreads();
        FA_STAMP(6);  // barrier passed
#ifdef FA_PHASE_TRACE
        if (tracing && lane == 0)
            for (int i = 0; i < 7; ++i) fa_phase_trace[wave][t - 60][i] = stamps[i];
#endif
    }

    // ---- epilogue: O * s_V / l as bf16 (transposed through a wave-private LDS patch), L
    {
        char* patch = lds_o + wave * 4096;
        const int qi = wave_q0 + col;
        const float l = sum_both_halves(l_run);
        int out_lane = lane;  // opaque: the addresses derived from it are else computed before the loop and kept over it
        asm volatile("" : "+v"(out_lane));
        store_rows_via_lds<bf16_tag, DT>(oacc, 1.0f / l, patch, make_buffer(o + head_off, (uint32_t)N * D * 2),
                                         wave_q0, out_lane);
        if (qi < N && half == 0) lse[(size_t)bh * N + qi] = (m_run + log2f(l) - kPBias) * kLn2;
    }
    }  // passes of a causal pair
}

// ---------------------------------------------------------------------------------------
// Eight waves (two per SIMD), 256 queries per tile, key blocks of 16 KiB (64 keys at d = 256, 128 at d = 128)
// or 8 KiB (128 keys at d = 64): the lock-step tile of fa_fwd_fp8_kernel with the staging taken out of the
// registers.  K and V blocks go
// from global memory straight into two LDS stages per tensor (buffer loads with an LDS destination, one
// block ahead), as unpadded rows whose 16-byte chunk index is XOR-swizzled through the global address a
// lane fetches; both read patterns are free of bank conflicts.  At d = 256 this is what makes two waves
// per SIMD possible at all: an e4m3 Q slab of 32 rows is 32 registers (half of what it is in 16 bits), so
// output accumulator (128), scores (32), Q and P~ fit the 256 registers -- but not together with 16
// staging registers (the register-staged instantiation spills its prefetched tiles).  The arithmetic is
// that of fa_fwd_fp8_kernel, step for step.
template <int D, int BC, bool CAUSAL, bool SCALED>
__global__ void __launch_bounds__(512, 1)
fa_fwd_fp8_async_kernel(const uint8_t* __restrict__ q, const uint8_t* __restrict__ k, const uint8_t* __restrict__ v,
                         const float* __restrict__ q_scale, const float* __restrict__ k_scale,
                         const float* __restrict__ v_scale, uint16_t* __restrict__ o, float* __restrict__ lse, int N,
                         int n_qtiles, int total_wg, int paired, int n_sblocks, int kv_group, float scale) {
    [[maybe_unused]] ClockSpan clock_span;  // measurement builds only; empty otherwise
    constexpr int NW = 8, BR = NW * 32;
    constexpr int NS = 2;            // LDS stages per tensor
    static_assert((D == 256 && BC == 64) || (D == 128 && BC == 128) || (D == 64 && BC == 128),
                  "tiles of 256-, 128- or 64-byte rows, at most 16 KiB");
    constexpr int ROWB = D;          // bytes per tile row
    constexpr int TILE = BC * ROWB;  // bytes per stage
    constexpr int KT = BC / 32, KS = D / 64, DT = D / 32, SL = BC / 64;

    // K stages, then V stages.  The output transposition at the end of a tile reuses the stages (every read
    // of them is behind a barrier by then and no load is in flight).
    using Few = FewFp8Forward<D, NW, D == 256 ? 4 : 8>;
    __shared__ __attribute__((aligned(1024))) char lds_kv[2 * NS * TILE > Few::kLds ? 2 * NS * TILE : Few::kLds];
    if (paired == kFewForward) {
        Few::template run<CAUSAL, SCALED>(q, k, v, q_scale, k_scale, v_scale, o, lse, N, total_wg, n_sblocks, kv_group, scale, lds_kv);
        return;
    }
    char* const lds_k = lds_kv;
    char* const lds_v = lds_kv + NS * TILE;
    static_assert(2 * NS * TILE >= NW * 4096, "output patches must fit the stages");

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;

    const TileRun run = query_tiles<CAUSAL>(total_wg, n_qtiles, paired);
    const int bh = run.head;

    const size_t head_off = (size_t)bh * N * D;
    const uint8_t* qh = q + head_off;
    const int kv_bh = bh / kv_group;  // grouped-query: kv_group query heads per K/V head
    const BufferWords k_rsrc = make_buffer_words(k + (size_t)kv_bh * N * D, (uint32_t)N * D);
    const BufferWords v_rsrc = make_buffer_words(v + (size_t)kv_bh * N * D, (uint32_t)N * D);

    auto k_swz = [](int r) { return Fp8Swizzle<D>::k(r); };
    auto v_swz = [](int r) { return Fp8Swizzle<D>::v(r); };
    // ---- staging: a load instruction fills 1 KiB = RPG rows; wave w loads groups w, w + 8, ... of a tile;
    // lane L fills chunk L % CPR of row L / CPR of its group with the global chunk the swizzle maps there
    constexpr int CPR = ROWB / 16, RPG = 1024 / ROWB;
    const int st_row = RPG * wave + lane / CPR, st_pos = lane % CPR;
    const int k_src = st_row * ROWB + ((st_pos ^ k_swz(st_row)) << 4);  // byte offset within a tile
    const int v_src = st_row * ROWB + ((st_pos ^ v_swz(st_row)) << 4);
    const uint32_t lds_k0 = lds_address(lds_k) + wave * 1024, lds_v0 = lds_address(lds_v) + wave * 1024;
    auto stage = [&](int u) __attribute__((always_inline)) {
        const uint32_t kd = lds_k0 + (u % NS) * TILE, vd = lds_v0 + (u % NS) * TILE;
#pragma unroll
        for (int i = 0; i < TILE / (NW * 1024); ++i) {
            global_to_lds_16B(k_rsrc, kd + i * NW * 1024, k_src + u * TILE + i * NW * 1024);
            global_to_lds_16B(v_rsrc, vd + i * NW * 1024, v_src + u * TILE + i * NW * 1024);
        }
    };
    // this wave's loads have landed and its LDS reads of the block before have returned (the next loads
    // overwrite that block's stage); then everyone's
    auto staged_barrier = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // ---- per-lane operand offsets within a stage (bytes)
    const int krow = key_of_row(col);  // key (within a 32-key tile) this lane's A row reads
    const int tr_row = (lane & 15) >> 1, blk = (lane >> 4) & 1;
    int kofs[KS][2], vofs[DT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int j = 0; j < 2; ++j) kofs[ks][j] = krow * ROWB + (((4 * ks + 2 * half + j) ^ k_swz(krow)) << 4);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
        vofs[dt] = (8 * half + tr_row) * ROWB + (((2 * dt + blk) ^ v_swz(tr_row)) << 4) + 8 * (lane & 1);

#pragma nounroll
    for (int pass = 0; pass < run.n_pass(); ++pass) {
    const int qt = pass == 0 ? run.tile : run.second;
    const int wave_q0 = qt * BR + wave * 32;

    float sq = 1.0f;
    if constexpr (SCALED) sq = q_scale[(size_t)bh * n_sblocks + min(wave_q0 / 128, n_sblocks - 1)];
    const float sc_q = scale * kLog2e * sq;

    i32x8 qreg[KS];
    {
        const int row = min(wave_q0 + col, N - 1);  // rows past N compute a copy of row N-1, never stored
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const uint8_t* p = qh + (size_t)row * D + ks * 64 + half * 32;
            i32x4 lo = *reinterpret_cast<const i32x4*>(p);
            i32x4 hi = *reinterpret_cast<const i32x4*>(p + 16);
            qreg[ks] = i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
    }
    f32x16 oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
    // m: running (lazily raised) maximum, in log2 units, of the real scores plus log2 of their V block's scale
    float m_run = -INFINITY, l_run = 0.f;

    const int last_q = min(qt * BR + BR, N) - 1;
    const int n_blocks = CAUSAL ? (last_q / BC + 1) : ((N + BC - 1) / BC);
    // blocks 0 .. nb_w-1 concern this wave (all of them unless causal)
    int nb_w = CAUSAL ? min(n_blocks, (wave_q0 + 31) / BC + 1) : n_blocks;
    // Opaque also without a mask: with the branch `t < nb_w` folded away the whole block is one scheduling
    // region, the compiler hoists LDS operand reads across the softmax and spills ~40 registers, and every
    // reload waits for the staging loads in flight (they share the vector-memory counter).
    if constexpr (!CAUSAL) asm volatile("" : "+s"(nb_w));

    // every LDS read of the previous pass is done before its stages are overwritten
    if (pass > 0) __syncthreads();
    stage(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));  // Q loads complete before the loop
    staged_barrier();

    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int t = 0; t < n_blocks; ++t) {
        const int key0 = t * BC;
        if (t + 1 < n_blocks) stage(t + 1);
        if (t < nb_w) {
            float sk = 1.0f, sv_new = 1.0f;
            if constexpr (SCALED) {
                sk = k_scale[(size_t)kv_bh * n_sblocks + key0 / 128];
                sv_new = v_scale[(size_t)kv_bh * n_sblocks + key0 / 128];
            }
            const float sc = sc_q * sk;

            // ---- GEMM0: S^T = K_j Q_i^T (rows permuted by key_of_row)
            f32x16 sacc[KT];
            {
                const uint32_t kb = lds_address(lds_k) + (t % NS) * TILE;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt) {
                        const i32x4 lo = lds_load_16B(kb + kofs[ks][0] + kt * 32 * ROWB);
                        const i32x4 hi = lds_load_16B(kb + kofs[ks][1] + kt * 32 * ROWB);
                        const i32x8 a = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                        sacc[kt] = mma_fp8(a, qreg[ks], ks == 0 ? zero : sacc[kt]);
                    }
            }
            if ((key0 + BC > N) || (CAUSAL && key0 + BC - 1 > wave_q0)) {
                const int qi = wave_q0 + col;
                const int limit = CAUSAL ? min(qi, N - 1) : N - 1;
                // register r of lane-half `half` holds key 16 (r / 8) + 8 half + r % 8 of its 32-key tile (the
                // rows of the K operand are permuted); compile-time offsets against one opaque per-lane bound
                int bound = limit - key0 - 8 * half;
                asm volatile("" : "+v"(bound));
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (kt * 32 + 16 * (r >> 3) + (r & 7) > bound) sacc[kt][r] = -INFINITY;
            }

            // ---- reference maximum (see fa_fwd_fp8_kernel: log2 units, V block scale as an exponent offset)
            float mxp[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};  // (a chain that starts from a score pays to quiet it first)
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) mxp[r & 3] = fmaxf(mxp[r & 3], sacc[kt][r]);
            float lsv = 0.f;
            if constexpr (SCALED) lsv = __builtin_amdgcn_logf(sv_new);  // log2
            const float mx = max_both_halves(fmaxf(fmaxf(mxp[0], mxp[1]), fmaxf(mxp[2], mxp[3]))) * sc + lsv;
            const bool raise = mx - m_run > kLazyLog2;
            if (__builtin_amdgcn_ballot_w64(raise) != 0) {
                const float f = raise ? fast_exp2(m_run - mx) : 1.0f;
                m_run = raise ? mx : m_run;
                l_run *= f;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[dt][r] *= f;
            }
            const float mb = m_run - kPBias - lsv;
            float sc_v = sc;  // a vector-register copy: an FMA with a scalar-register operand issues at a lower rate
            asm volatile("" : "+v"(sc_v));

            // ---- P~ = exp2(s sc - mb) as e4m3, and its row sum
            float ps[4];
            i32x8 pb[SL];
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                float p[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    p[r] = fast_exp2(__builtin_fmaf(sacc[kt][r], sc_v, -mb));
                    ps[r & 3] = kt == 0 && r < 4 ? p[r] : ps[r & 3] + p[r];
                }
#pragma unroll
                for (int w = 0; w < 4; ++w) pb[kt >> 1][4 * (kt & 1) + w] = pack_e4m3(p[4 * w], p[4 * w + 1], p[4 * w + 2], p[4 * w + 3]);
            }

            // the sum needs the weights without the V scale's exponent offset
            float psum = (ps[0] + ps[1]) + (ps[2] + ps[3]);
            if constexpr (SCALED) psum *= __builtin_amdgcn_rcpf(sv_new);
            l_run += psum;
            // ---- GEMM1: O^T += V_j^T P~^T
            const uint32_t vb = lds_address(lds_v) + (t % NS) * TILE;
#pragma unroll
            for (int sl = 0; sl < SL; ++sl)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    i32x8 a;
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const i32x2 w = lds_read_tr8(vb + vofs[dt] + (sl * 64 + 16 * x) * ROWB);
                        a[2 * x] = w[0];
                        a[2 * x + 1] = w[1];
                    }
                    oacc[dt] = mma_fp8(a, pb[sl], oacc[dt]);
                }
        }
        if (t + 1 < n_blocks) staged_barrier();
    }

    // ---- epilogue: O * s_V / l as bf16 (transposed through a wave-private LDS patch), L
    __syncthreads();  // every wave is done with the K stages
    {
        char* patch = lds_kv + wave * 4096;
        const int qi = wave_q0 + col;
        const float l = sum_both_halves(l_run);
        int out_lane = lane;  // opaque: the addresses derived from it are else computed before the loop and kept over it
        asm volatile("" : "+v"(out_lane));
        store_rows_via_lds<bf16_tag, DT>(oacc, 1.0f / l, patch, make_buffer(o + head_off, (uint32_t)N * D * 2),
                                         wave_q0, out_lane);
        if (qi < N && half == 0) lse[(size_t)bh * N + qi] = (m_run + log2f(l) - kPBias) * kLn2;
    }
    }  // passes of a causal pair
}

template <int D, int BC, int NW>
static int launch_fp8(const void* q8, const void* k8, const void* v8, const float* qs, const float* ks,
                      const float* vs, void* o, float* lse, int B, int H, int H_kv, int N, float scale, int causal,
                      hipStream_t stream) {
    constexpr int BR = NW * 32;
    int n_qtiles = (N + BR - 1) / BR;
    int n_sblocks = (N + 127) / 128;
    constexpr PairRule kPairs = NW == 4 ? (D == 64 ? PairRule{3, 15.f / 16, kAny, 1.f, 2} : PairRule{2, 7.f / 8, 320, 0.75f, kAny})
                                        : (D == 64 ? PairRule{2, 1.f, kAny, 1.f, 0} : PairRule{1, 0.9f, kAny, 1.f, kAny});
    const bool few = NW == 4 && few_forward_fp8((long)B * H, N, D, causal);
    const int paired = few ? kFewForward : causal && pair_causal_tiles((long)B * H, n_qtiles, kPairs);
    long total = few ? few_split((long)B * H, N) : (long)B * H * (paired ? (n_qtiles + 1) / 2 : n_qtiles);
    if (total > 0x7fffffffL) return FA_ERR_SHAPE;
    const dim3 grid = forward_grid((long)B * H, N, n_qtiles, total, causal, paired), block(NW * 64);
    auto qp = static_cast<const uint8_t*>(q8);
    auto kp = static_cast<const uint8_t*>(k8);
    auto vp = static_cast<const uint8_t*>(v8);
    auto op = static_cast<uint16_t*>(o);
    const bool scaled = qs != nullptr;
#define FA_LAUNCH_FP8(C, S)                                                                                       \
    hipLaunchKernelGGL((fa_fwd_fp8_kernel<D, BC, NW, C, S>), grid, block, 0, stream, qp, kp, vp, qs, ks, vs, op, \
                       lse, N, n_qtiles, (int)total, paired, n_sblocks, H / H_kv, scale)
    if (causal) {
        if (scaled) FA_LAUNCH_FP8(true, true); else FA_LAUNCH_FP8(true, false);
    } else {
        if (scaled) FA_LAUNCH_FP8(false, true); else FA_LAUNCH_FP8(false, false);
    }
#undef FA_LAUNCH_FP8
    return hipGetLastError() == hipSuccess ? FA_OK : FA_ERR_LAUNCH;
}

template <int D, int BC>
static int launch_fp8_async(const void* q8, const void* k8, const void* v8, const float* qs, const float* ks,
                           const float* vs, void* o, float* lse, int B, int H, int H_kv, int N, float scale,
                           int causal, hipStream_t stream) {
    constexpr int BR = 256;
    int n_qtiles = (N + BR - 1) / BR;
    int n_sblocks = (N + 127) / 128;
    // d = 256: short tiles win as pairs a little earlier, above all in the first round (us, pairs / single: 192 x 300 30.0 /
    // 31.0 at a share of 0.75, 448 x 300 59.3 / 63.9 and 112 x 1024 53.9 / 54.7 at 0.88, but 384 x 450 73.9 / 63.9 at 0.75)
    const bool first_round = (long)B * H * ((n_qtiles + 1) / 2) <= 256;
    const float share = D < 256 || n_qtiles > 4 ? 0.9f : n_qtiles > 2 ? (first_round ? 0.875f : 0.9f) : (first_round ? 0.75f : 0.875f);
    const bool few = few_forward_fp8((long)B * H, N, D, causal);
    const int paired = few ? kFewForward
                           : causal && pair_causal_tiles((long)B * H, n_qtiles, D == 64 ? PairRule{2, 1.f, kAny, 1.f, 0} : PairRule{1, share, kAny, 1.f, kAny});
    long total = few ? few_split((long)B * H, N) : (long)B * H * (paired ? (n_qtiles + 1) / 2 : n_qtiles);
    if (total > 0x7fffffffL) return FA_ERR_SHAPE;
    const dim3 grid = forward_grid((long)B * H, N, n_qtiles, total, causal, paired), block(512);
    auto qp = static_cast<const uint8_t*>(q8);
    auto kp = static_cast<const uint8_t*>(k8);
    auto vp = static_cast<const uint8_t*>(v8);
    auto op = static_cast<uint16_t*>(o);
    const bool scaled = qs != nullptr;
#define FA_LAUNCH_FP8_D256(C, S)                                                                                  \
    hipLaunchKernelGGL((fa_fwd_fp8_async_kernel<D, BC, C, S>), grid, block, 0, stream, qp, kp, vp, qs, ks, vs, op, lse, N, \
                       n_qtiles, (int)total, paired, n_sblocks, H / H_kv, scale)
    if (causal) {
        if (scaled) FA_LAUNCH_FP8_D256(true, true); else FA_LAUNCH_FP8_D256(true, false);
    } else {
        if (scaled) FA_LAUNCH_FP8_D256(false, true); else FA_LAUNCH_FP8_D256(false, false);
    }
#undef FA_LAUNCH_FP8_D256
    return hipGetLastError() == hipSuccess ? FA_OK : FA_ERR_LAUNCH;
}

enum class FwdFp8 { kTile4, kTile8, kNone };
static FwdFp8 choose_fp8(int d, int N, int causal) {
    // Short problems keep the 128-row tile of four waves (more workgroups, less waste on the diagonal).  The choice is by
    // N, d and mask alone, so a line lies where no number of heads loses more than noise.  Block-scaled inputs, us, four
    // waves / eight, heads x N:
    //   d = 64   causal:  about 16k tokens, H = 16: N = 2048 70 / 76, 8192 235 / 246, 16384 455 / 475
    //            no mask: about 16k tokens, H = 16: N = 512 36 / 34;  16 x 1150 15.5 / 20.0 but 32 x 1150 22.3 / 20.4
    //   d = 128  causal:  16 x 1408 24.5 / 28.1, 80 x 1408 38.7 / 39.3;  16 x 1500 26.1 / 30.7 but 80 x 1500 42.8 / 39.7;
    //                     16 x 1600 26.6 / 32.2, 64 x 1600 41.2 / 40.1
    //            no mask: 16 x 704 13.5 / 18.0, 48 x 704 19.3 / 18.8;  16 x 770 15.8 / 20.2 but 40 x 770 21.9 / 21.0,
    //                     16 x 1408 24.1 / 28.6 but 28 x 1408 34.5 / 29.2
    // d = 256 has no four-wave tile.
    switch (d) {
        case 64: return causal || N < 512 ? FwdFp8::kTile4 : FwdFp8::kTile8;
        case 128: return N <= (causal ? 1408 : 704) || (causal && odd_row_tiles(N) && N <= 1664) ? FwdFp8::kTile4 : FwdFp8::kTile8;
        case 256: return FwdFp8::kTile8;
        default: return FwdFp8::kNone;
    }
}

int launch_fwd_fp8(const void* q8, const void* k8, const void* v8, const float* q_scale, const float* k_scale,
                   const float* v_scale, void* o, float* lse, int B, int H, int H_kv, int N, int d, float scale, int causal,
                   hipStream_t stream) {
#define FA_FP8_ARGS q8, k8, v8, q_scale, k_scale, v_scale, o, lse, B, H, H_kv, N, scale, causal, stream
    switch (choose_fp8(d, N, causal)) {
        case FwdFp8::kTile4:
            if (d == 64) return launch_fp8<64, 64, 4>(FA_FP8_ARGS);
            return launch_fp8<128, 64, 4>(FA_FP8_ARGS);
        case FwdFp8::kTile8:
#ifdef FA_STAGED_TILE8  // measurement builds: the register-staged eight-wave tile that FA_ABLATE / FA_PHASE_TRACE instrument
            if (d == 64) return launch_fp8<64, 128, 8>(FA_FP8_ARGS);
            if (d == 128) return launch_fp8<128, 128, 8>(FA_FP8_ARGS);
#endif
            if (d == 64) return launch_fp8_async<64, 128>(FA_FP8_ARGS);
            if (d == 128) return launch_fp8_async<128, 128>(FA_FP8_ARGS);
            return launch_fp8_async<256, 64>(FA_FP8_ARGS);
        default: return FA_ERR_UNSUPPORTED;
    }
#undef FA_FP8_ARGS
}

// The name a profiler shows for the kernel launch_fwd_fp8 picks (block-scaled instantiation).
const char* fwd_fp8_kernel_name(int N, int d, int causal) {
    static const char* const names[2][5] = {
        {"fa_fwd_fp8_kernel<64, 64, 4, false, true>", "fa_fwd_fp8_kernel<128, 64, 4, false, true>",
         "fa_fwd_fp8_async_kernel<64, 128, false, true>", "fa_fwd_fp8_async_kernel<128, 128, false, true>",
         "fa_fwd_fp8_async_kernel<256, 64, false, true>"},
        {"fa_fwd_fp8_kernel<64, 64, 4, true, true>", "fa_fwd_fp8_kernel<128, 64, 4, true, true>",
         "fa_fwd_fp8_async_kernel<64, 128, true, true>", "fa_fwd_fp8_async_kernel<128, 128, true, true>",
         "fa_fwd_fp8_async_kernel<256, 64, true, true>"}};
    int idx;
    switch (choose_fp8(d, N, causal)) {
        case FwdFp8::kTile4: idx = d == 64 ? 0 : 1; break;
        case FwdFp8::kTile8: idx = d == 64 ? 2 : d == 128 ? 3 : 4; break;
        default: return nullptr;
    }
    return names[causal ? 1 : 0][idx];
}

}  // namespace fa

FA_CLOCK_SPAN_READER(fa_debug_clock_span_fwd_fp8)
