// Backward attention for gfx950, head dimensions 64, 128 and 256, bf16 / fp16 (paper section 2.1 chain rule,
// Algorithm 3's recomputation of P from L and its D = rowsum(dO o O)).
//
//   dQ pass    : one workgroup per tile of queries (dQ_i on chip).  Its prologue computes D = rowsum(dO o O) of
//                its rows and leaves it in the workspace (or finds it there); loop over key blocks:
//                S^T = K_j Q_i^T, dP^T = V_j dO_i^T, P = exp(S - L), dS = P o (dP - D),
//                dQ_i^T += K_j^T dS^T
//   dK/dV pass : one workgroup per block of 128 keys (64 at d = 256), dK_j, dV_j kept on chip; loop over
//                tiles of 64 queries: S = Q_i K_j^T, dP = dO_i V_j^T, P, dS as above,
//                dV_j += P^T dO_i, dK_j += dS^T Q_i
// (A launch of its own for D read dO once more: 2.7 us of a training step's 34 at B = 2, H = 8, N = 333, d = 64;
// at sizes where the chip's power is the limit the two forms take the same time.)
//
// Algorithm 3 produces dQ inside the dK/dV loop and adds it to HBM with atomics.  Measured on
// MI355X that accumulation (17 GB of fp32 atomic traffic at seqlen 16k) cost about 30 % of the
// pass, so dQ gets its own pass instead: two of the five GEMMs are recomputed, nothing is
// accumulated in HBM, no fp32 dQ buffer or cast pass exists, and the result is deterministic.
//
// Register layouts.  dK/dV pass: S and dP have queries as MFMA rows and keys as columns, so a
// lane owns one key and 16 queries; packed to 16 bits those registers are directly the A
// operand (keys x queries) of the dV and dK products, whose B operands (dO, Q as queries x d)
// come from transposing LDS reads.  dQ pass: the forward kernel's layout -- S^T and dP^T have
// one query per lane column, dS^T packs straight into the B operand of dQ^T += K^T dS^T, and
// K^T is the transposing read of the same LDS tile that fed S^T.
#include <type_traits>

#include "fa_device.h"
#include "fa_launch.h"

namespace fa {


// LDS row stride (elements) of tiles that are read both by rows and transposed: an odd multiple
// of 16 bytes keeps the row reads conflict-free, and the offset from a multiple of 256 bytes
// decides how much the four rows of a transposing read overlap in the banks.  Measured LDS rates
// per CU at d = 128: 304 B gives 211 / 123 B/clk (rows / transposed), 272 B gives 208 / 63, 320 B
// gives 63 / 208.
constexpr int bwd_row_stride(int d) { return d >= 128 ? d + 24 : d + 40; }

// acc + the dot product of 8 packed 16-bit elements, in fp32
template <typename Tag>
static __device__ __forceinline__ float dot8(const i32x4& a, const i32x4& b, float acc) {
    using E = Elem<Tag>;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const uint32_t ua = (uint32_t)a[t], ub = (uint32_t)b[t];
        acc = __builtin_fmaf(E::to_float((uint16_t)(ua & 0xFFFF)), E::to_float((uint16_t)(ub & 0xFFFF)), acc);
        acc = __builtin_fmaf(E::to_float((uint16_t)(ua >> 16)), E::to_float((uint16_t)(ub >> 16)), acc);
    }
    return acc;
}

// 8 consecutive outputs: the sum over NP partial results `stride` floats apart, first to last, times `factor`
template <typename Tag, int NP>
static __device__ __forceinline__ i32x4 sum_parts(const float* p, int stride, float factor) {
    i32x4 out;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        f32x4 s = *reinterpret_cast<const f32x4*>(p + 4 * h);
#pragma unroll
        for (int w = 1; w < NP; ++w) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(p + w * stride + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += x[e];
        }
        out[2 * h] = Elem<Tag>::pack2(s[0] * factor, s[1] * factor);
        out[2 * h + 1] = Elem<Tag>::pack2(s[2] * factor, s[3] * factor);
    }
    return out;
}

// Stores a 32-key x 64-column fp32 accumulator pair (MFMA result layout with keys as rows: lane (col, half), register r
// of tile dt is key 8 (r / 4) + 4 half + r % 4, column 32 dt + col) as 16-bit elements times `factor`.  Straight from
// that layout a store instruction moves two bytes per lane, 128 of them per wave for dK and dV; instead neighbouring
// lanes trade halves (an even lane keeps the even key of a pair, its neighbour the odd one), the tile goes through
// `patch` (4 KiB of LDS private to the wave) as 4-byte words and leaves as whole 128-byte lines.  Rows past the end of
// `rsrc` are dropped by the hardware.  bf16, whole backward, us, two-byte stores / so:
// d = 128 causal B = 64, H = 16, N = 256 228 / 215, B = 32, N = 512 269 / 258, B = 4, N = 4096 952 / 946; d = 256 B = 32, N = 512 630 / 604.
template <typename Tag, int ROWB>
static __device__ __forceinline__ void store_keys_via_lds(const f32x16 (&acc)[2], float factor, char* patch,
                                                          __amdgpu_buffer_rsrc_t rsrc, int key0, int col_byte, int lane) {
    using E = Elem<Tag>;
    const int col = lane & 31, half = lane >> 5, odd = lane & 1;
    const uint32_t sel = odd ? 0x03020706u : 0x05040100u;  // odd key: (neighbour's high, own high); even: (own low, neighbour's low)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const uint32_t w = (uint32_t)E::pack2(acc[dt][r] * factor, acc[dt][r + 1] * factor);
            const uint32_t v = (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0xB1, 0xF, 0xF, true);  // lane ^ 1
            const int key = 8 * (r >> 2) + 4 * half + (r & 3) + odd;
            *reinterpret_cast<uint32_t*>(patch + key * 128 + ((dt * 64 + (col >> 1) * 4) ^ ((key & 4) << 3))) =
                __builtin_amdgcn_perm(v, w, sel);
        }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int key = 8 * i + (lane >> 3), pos = (lane & 7) * 16;
        const i32x4 x = *reinterpret_cast<const i32x4*>(patch + key * 128 + (pos ^ ((key & 4) << 3)));
        __builtin_amdgcn_raw_buffer_store_b128(x, rsrc, (key0 + key) * ROWB + col_byte + pos, 0, kStreamed);
    }
}

// D = rowsum(dO o O) in a launch of its own, where the dK/dV pass cannot wait for the dQ pass to compute it: both passes
// in one launch (fa_bwd_few_kernel), or dQ written over an input of the dK/dV pass; and where a gradient is written over
// O, so that no later launch reads O.
template <typename Tag, int D>
__global__ void __launch_bounds__(256)
fa_bwd_rowsum_kernel(const uint16_t* __restrict__ o, const uint16_t* __restrict__ dout, float* __restrict__ dvec, long rows) {
    constexpr int LPR = D / 8;  // lanes per row, 8 elements each
    const int part = threadIdx.x & (LPR - 1);
    const long row = (long)blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
    float acc = 0.f;
    if (row < rows)
        acc = dot8<Tag>(*reinterpret_cast<const i32x4*>(o + row * D + part * 8),
                        *reinterpret_cast<const i32x4*>(dout + row * D + part * 8), 0.f);
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (row < rows && part == 0) dvec[row] = acc;
}

// ---------------------------------------------------------------------------------------
template <typename Tag, int D, bool CAUSAL>
__global__ void __launch_bounds__(256, 2)
fa_bwd_dkdv_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
              const uint16_t* __restrict__ dout, const float* __restrict__ lse, const float* __restrict__ dvec,
              uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int N,
              int n_kblocks, int total_wg, int kv_group, float scale) {
    [[maybe_unused]] ClockSpan clock_span;  // measurement builds only; empty otherwise
    constexpr int BK = 128;        // keys per workgroup
    constexpr int BQ = 64;         // queries per loop iteration
    constexpr int NT = 256;
    static_assert(D == 64, "two workgroups per CU; wider heads share scores (fa_bwd_dkdv_shared_kernel)");
    constexpr int RSTR = bwd_row_stride(D);
    constexpr int TILE_B = BQ * RSTR * 2;  // bytes per tile
    constexpr int KS = D / 16;
    // MFMA steps by which LDS operand reads lead their use (registers permitting)
    constexpr int KP = 2;
    constexpr int DT = D / 32;
    constexpr int CPR = D / 8;     // 16-byte chunks per row
    constexpr int QCH = BQ * CPR / NT;  // chunks per thread for a Q / dO tile
    using E = Elem<Tag>;

    // tiles 0, 1: Q_i double-buffered; tiles 2, 3: dO_i (a fixed distance from the Q tile of the
    // same parity, so one address register serves both)
    __shared__ __attribute__((aligned(16))) uint16_t lds_t[4][BQ * RSTR];
    constexpr int DO_DIST = 2 * TILE_B;
    __shared__ __attribute__((aligned(16))) float lds_l[2][BQ];
    __shared__ __attribute__((aligned(16))) float lds_d[2][BQ];

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;

    const WorkItem item = work_item<CAUSAL>(blockIdx.x, total_wg, n_kblocks);  // key block 0 has the longest loop
    const int bh = item.head;
    const int key0 = item.tile * BK;

    // bh counts key/value heads; the kv_group query heads that share this one are bh * kv_group + g
    const size_t head_off = (size_t)bh * N * D;
    const uint16_t* kh = k + head_off;
    const uint16_t* vh = v + head_off;
    const float sc = scale * kLog2e;

    // ---- this wave's K and V rows as B operands (lane: key column, 8 head-dim elements)
    i32x4 kreg[KS], vreg[KS];
    const int my_key = key0 + wave * 32 + col;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        i32x4 z = {0, 0, 0, 0};
        kreg[ks] = my_key < N ? *reinterpret_cast<const i32x4*>(kh + (size_t)my_key * D + ks * 16 + half * 8) : z;
        vreg[ks] = my_key < N ? *reinterpret_cast<const i32x4*>(vh + (size_t)my_key * D + ks * 16 + half * 8) : z;
    }
    f32x16 dkacc[DT], dvacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            dkacc[dt][r] = 0.f;
            dvacc[dt][r] = 0.f;
        }

    const int n_qtiles = (N + BQ - 1) / BQ;
    const int it0 = CAUSAL ? key0 / BQ : 0;  // first query tile that can see this key block
    const int tr_row = (lane & 15) >> 2;
    const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    // Masked query tiles come first: every tile when the key block is ragged (keys past N), else
    // the tiles on the causal diagonal.  They get a loop of their own so that the main loop has a
    // single straight-line body.
    const int it_masked_end = key0 + BK > N ? n_qtiles : (CAUSAL ? min(n_qtiles, (key0 + BK - 1) / BQ + 1) : it0);

    // Every query head of the group adds into the same dK_j, dV_j (grouped-query attention: the
    // gradient of a shared key/value head is the sum over the query heads that read it).
#pragma nounroll
    for (int g = 0; g < kv_group; ++g) {
    const size_t qhead = (size_t)bh * kv_group + g;
    const uint16_t* qh = q + qhead * N * D;
    const uint16_t* doh = dout + qhead * N * D;
    const float* lh = lse + qhead * N;
    const float* dh = dvec + qhead * N;

    // Q_i and dO_i tiles are contiguous runs of the row-major tensors; rows past N lie outside the
    // buffer resources and read as zero.
    const __amdgpu_buffer_rsrc_t q_rsrc = make_buffer(qh, (uint32_t)N * D * 2);
    const __amdgpu_buffer_rsrc_t do_rsrc = make_buffer(doh, (uint32_t)N * D * 2);
    i32x4 qpre[QCH], dopre[QCH];
    float lpre = 0.f;  // threads 0..63 carry L, 64..127 carry D
    int lrow = 0;
    // The next tile travels global -> registers (issued at the top of an iteration) -> LDS (at its
    // end).
    auto load_tile = [&](int it) {
#pragma unroll
        for (int j = 0; j < QCH; ++j) {
            qpre[j] = buffer_load_16B(q_rsrc, it * BQ * D * 2 + (tid + j * NT) * 16);
            dopre[j] = buffer_load_16B(do_rsrc, it * BQ * D * 2 + (tid + j * NT) * 16);
        }
    };
    auto load_ld = [&](int it) {
        if (tid < 2 * BQ) {
            // the raw value only: anything computed from it here would make the wave wait for the
            // load on the spot, once per iteration
            lrow = it * BQ + (tid & (BQ - 1));
            lpre = (tid < BQ ? lh : dh)[min(lrow, N - 1)];
        }
    };
    auto store_tile = [&](int st) {
#pragma unroll
        for (int j = 0; j < QCH; ++j) {
            int c = tid + j * NT;
            int row = c / CPR, cc = c % CPR;
            *reinterpret_cast<i32x4*>(lds_t[st] + row * RSTR + cc * 8) = qpre[j];
            *reinterpret_cast<i32x4*>(lds_t[2 + st] + row * RSTR + cc * 8) = dopre[j];
        }
    };
    auto store_ld = [&](int st) {
        // rows past N get L = +inf so that P = exp2(0 - inf) = 0, and D = 0.  D is kept negated:
        // the dP accumulators start from -D_i, so dP - D comes out of the MFMAs
        if (tid < BQ) lds_l[st][tid] = lrow < N ? lpre * kLog2e : INFINITY;
        else if (tid < 2 * BQ) lds_d[st][tid - BQ] = lrow < N ? -lpre : 0.f;
    };

    if (it0 < n_qtiles) {
        load_ld(it0);
        load_tile(it0);
        store_tile(0);
        store_ld(0);
    }
    __syncthreads();

    auto iteration = [&](int it, auto mask_tag) {
        const int st = (it - it0) & 1;
        const int q0 = it * BQ;
        const bool more = it + 1 < n_qtiles;
        if (more) {
            load_tile(it + 1);
            load_ld(it + 1);
        }

        // The SIMD's other wave belongs to another workgroup and is not in step with this one: to count on
        // it alone would leave the matrix pipe idle whenever both run exponentials.  The iteration is
        // therefore software-pipelined by hand over its two 32-query sub-tiles (the intra-warpgroup overlap of the paper's
        // Algorithm 2, applied to the backward pass):
        //   stage 1: S, dP of sub-tile 0                      (MFMA only)
        //   stage 2: S, dP of sub-tile 1  ||  P, dS of sub-tile 0
        //   stage 3: dV, dK += sub-tile 0 ||  P, dS of sub-tile 1
        //   stage 4: dV, dK += sub-tile 1                     (MFMA only)
        // Every step ends in a full scheduling barrier so the interleaving below is what runs, and
        // LDS operand reads lead their MFMAs by KP steps.
        auto body = [&](auto mask_tag) {
            constexpr bool MASK = decltype(mask_tag)::value;
            const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            i32x4 pa[2][2], dsa[2][2];  // [sub-tile][16-query slab]: P^T and dS^T as A operands
            f32x16 sacc[2], pacc[2];

            // This tile's LDS addresses, one register each; every read below adds a compile-time
            // offset that fits the instruction's immediate field.
            // Row reads: lane (col, half) takes 8 elements from 16 ks + 8 half of row col (+ 32 per
            // sub-tile).  Transposing reads: lane takes 4 elements at tr_col of row 4 half + tr_row
            // (+ 8 for the second read, + 16 per slab), 32 elements further per d-tile.
            uint32_t q_rows = lds_address(lds_t[st]) + (col * RSTR + half * 8) * 2;
            uint32_t q_tr = lds_address(lds_t[st]) + ((4 * half + tr_row) * RSTR + tr_col) * 2;
            uint32_t l_rows = lds_address(lds_l[st]) + 16 * half;  // 4 consecutive rows from 4 * half
            uint32_t d_rows = lds_address(lds_d[st]) + 16 * half;
            asm volatile("" : "+v"(q_rows), "+v"(q_tr), "+v"(l_rows), "+v"(d_rows));
            auto row_addr = [&](int u) -> uint32_t {  // step u = (sub-tile, ks) of stages 1 and 2
                const int sub = u / KS, ks = u % KS;
                return q_rows + (sub * 32 * RSTR + ks * 16) * 2;
            };
            auto tr_addr = [&](int u, int hi) -> uint32_t {  // step u = (16-query slab, d-tile) of stages 3 and 4
                const int slab = u / DT, dt = u % DT;
                return q_tr + ((slab * 16 + hi * 8) * RSTR + dt * 32) * 2;
            };

            // L (log2 units) of the lane's query rows, fetched four rows at a time one step before
            // they are needed so that few of them are live at once
            f32x4 l4[2][4];
            auto fetch_l = [&](int sub, int g) { l4[sub][g] = lds_load_4f(l_rows + (sub * 32 + 8 * g) * 4); };
            // dP starts from -D_i: accumulator registers 4g..4g+3 are query rows 8g+4*half..+3
            auto init_dp = [&](int sub) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 t = lds_load_4f(d_rows + (sub * 32 + 8 * g) * 4);
#pragma unroll
                    for (int r = 0; r < 4; ++r) pacc[sub][4 * g + r] = t[r];
                }
            };

            // elements 2c, 2c+1 of a sub-tile: P, dS and one packed register of each.  The two elements
            // are computed in the shadows of two different MFMAs (softmax_elem after each), the pair
            // is packed after the second.
            float pv[8][2], dsv[8][2];  // indexed by the pair's number within its sub-tile
            auto softmax_elem = [&](int sub, int c, int e) {
                const int rr = 2 * c + e, g = rr >> 2, r = rr & 3;
                float p = fast_exp2(__builtin_fmaf(sacc[sub][rr], sc, -l4[sub][g][r]));
                if constexpr (MASK) {
                    const int qi = q0 + sub * 32 + 8 * g + 4 * half + r;
                    const bool masked = my_key >= N || (CAUSAL && my_key > qi);
                    p = masked ? 0.f : p;
                }
                pv[c][e] = p;
                dsv[c][e] = p * pacc[sub][rr];
            };
            auto softmax_pack = [&](int sub, int c) {
                pa[sub][c >> 2][c & 3] = E::pack2(pv[c][0], pv[c][1]);
                dsa[sub][c >> 2][c & 3] = E::pack2(dsv[c][0], dsv[c][1]);
            };

            // ---- stages 1 and 2: S = Q_i K_j^T, dP = dO_i V_j^T
            {
                constexpr int NU = 2 * KS;
                i32x4 aq[KP], ado[KP];
#pragma unroll
                for (int u = 0; u < KP; ++u) {
                    aq[u] = lds_load_16B(row_addr(u));
                    ado[u] = lds_load_16B(row_addr(u) + DO_DIST);
                }
                init_dp(0);
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int sub = u / KS, ks = u % KS;
                    i32x4 a0 = aq[u % KP], a1 = ado[u % KP];
                    if (u + KP < NU) {
                        aq[u % KP] = lds_load_16B(row_addr(u + KP));
                        ado[u % KP] = lds_load_16B(row_addr(u + KP) + DO_DIST);
                    }
                    if (u == KS - 2) init_dp(1);
                    // A wave issues in order and its second MFMA waits for the matrix pipe to take it:
                    // vector work placed after both MFMAs of a step runs in the shadow of the second
                    // one only.  Half of it goes between the two.
                    sacc[sub] = E::mma(a0, kreg[ks], ks == 0 ? zero : sacc[sub]);
                    if (sub == 1) {
                        // the 8 register pairs of sub-tile 0 spread over the KS steps (pair c runs at
                        // step c KS / 8); the L group of a pair is fetched one step before the step
                        // that needs it first
#pragma unroll
                        for (int g = 1; g < 4; ++g)
                            if ((2 * g * KS) / 8 == ks + 1) fetch_l(0, g);
                        if (ks == KS - 1) fetch_l(1, 0);
#pragma unroll
                        for (int c = 0; c < 8; ++c)
                            if ((c * KS) / 8 == ks) softmax_elem(0, c, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    pacc[sub] = E::mma(a1, vreg[ks], pacc[sub]);
                    if (sub == 0 && ks == KS - 1) fetch_l(0, 0);
                    if (sub == 1) {
#pragma unroll
                        for (int c = 0; c < 8; ++c)
                            if ((c * KS) / 8 == ks) {
                                softmax_elem(0, c, 1);
                                softmax_pack(0, c);
                            }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }

            // ---- stages 3 and 4: dV_j += P^T dO_i, dK_j += dS^T Q_i (contract over the tile's queries)
            {
                constexpr int NU = 2 * 2 * DT;  // (sub, slab, d-tile)
                i32x2 dlo[KP], dhi[KP], qlo[KP], qhi[KP];
#pragma unroll
                for (int u = 0; u < KP; ++u) {
                    dlo[u] = lds_read_tr16(tr_addr(u, 0) + DO_DIST);
                    dhi[u] = lds_read_tr16(tr_addr(u, 1) + DO_DIST);
                    qlo[u] = lds_read_tr16(tr_addr(u, 0));
                    qhi[u] = lds_read_tr16(tr_addr(u, 1));
                }
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int sub = u / (2 * DT), s2 = (u / DT) % 2, dt = u % DT;
                    const int w = u % KP;
                    i32x4 b = {dlo[w][0], dlo[w][1], dhi[w][0], dhi[w][1]};
                    i32x4 b2 = {qlo[w][0], qlo[w][1], qhi[w][0], qhi[w][1]};
                    if (u + KP < NU) {
                        dlo[w] = lds_read_tr16(tr_addr(u + KP, 0) + DO_DIST);
                        dhi[w] = lds_read_tr16(tr_addr(u + KP, 1) + DO_DIST);
                        qlo[w] = lds_read_tr16(tr_addr(u + KP, 0));
                        qhi[w] = lds_read_tr16(tr_addr(u + KP, 1));
                    }
                    dvacc[dt] = E::mma(pa[sub][s2], b, dvacc[dt]);
                    constexpr int PP = 8 / (2 * DT);
                    if (sub == 0) {
#pragma unroll
                        for (int g = 1; g < 4; ++g)
                            if ((2 * g) / PP == u + 1) fetch_l(1, g);
#pragma unroll
                        for (int p = 0; p < PP; ++p) softmax_elem(1, u * PP + p, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    dkacc[dt] = E::mma(dsa[sub][s2], b2, dkacc[dt]);
                    if (sub == 0) {
#pragma unroll
                        for (int p = 0; p < PP; ++p) {
                            softmax_elem(1, u * PP + p, 1);
                            softmax_pack(1, u * PP + p);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        body(mask_tag);

        if (more) {
            store_tile(st ^ 1);
            store_ld(st ^ 1);
        }
        __syncthreads();
    };
    int it = it0;
    for (; it < it_masked_end; ++it) iteration(it, std::true_type{});
    for (; it < n_qtiles; ++it) iteration(it, std::false_type{});
    }  // query heads of the group

    // ---- epilogue: dK_j = scale * acc, dV_j = acc, through the tile buffers (every read of them is behind a barrier)
    char* patch = reinterpret_cast<char*>(&lds_t[0][0]) + wave * 4096;
    static_assert(sizeof(lds_t) >= 4 * 4096, "patches must fit");
    store_keys_via_lds<Tag, D * 2>(dkacc, scale, patch, make_buffer(dk + head_off, (uint32_t)N * D * 2), key0 + wave * 32, 0, lane);
    store_keys_via_lds<Tag, D * 2>(dvacc, 1.0f, patch, make_buffer(dv + head_off, (uint32_t)N * D * 2), key0 + wave * 32, 0, lane);
}

// ---------------------------------------------------------------------------------------
// dK/dV pass, head dimensions 128 and 256: four waves, one per SIMD, that share scores.
//
// Bound by the matrix pipes (64 MFMAs of 32 cycles per wave and iteration) if the LDS can feed them: an operand read
// from the LDS serves as many MFMAs as the wave owns 32-key tiles, and the register file holds accumulators for one
// tile of all 128 columns or for two tiles of 64.  So the waves divide the two halves of the work differently:
//   S, dP   : by key tiles and 32-query sub-tiles -- wave (p, g) computes those of its K, V operands (resident: two
//             key tiles at d = 128, one at d = 256) for sub-tile g;
//   dK, dV  : by columns -- a wave accumulates two key tiles x 64 columns, from the P and dS of both sub-tiles.
// P and dS, packed, are already the A operands of the second half (lane = key), so what the waves exchange is raw
// registers, 1 KiB per 32 x 16 piece through the LDS, with one barrier more per iteration.  At d = 128 a row operand and a
// transposed operand serve two MFMAs each (48 LDS operand reads per wave and iteration instead of 96); at d = 256
// the four waves cover all 256 columns from one computation of S and dP (no second workgroup that repeats it: 64
// MFMAs instead of 96 per 32 keys).
//
// Within an iteration (64 queries; "own" = this wave's sub-tile):
//   phase 1  S                               16 MFMAs
//   phase 2  dP                              16 MFMAs  ||  P = exp2(S c - L), packed and sent
//   phase 3  dV += own P dO                            ||  dS = P o (dP - D), packed and sent
//   barrier; the other waves' pieces are requested
//   phase 4  dK += own dS Q, then dV and dK of everything else
// Every step ends in a full scheduling barrier so that the interleaving written here is what runs.
// Measured (bf16, whole backward, one key tile x all columns per wave before): d = 256, B = 2, H = 8, N = 8192 4801 ->
// 3873 us (this pass 3046 -> 2112, 1.04 PFLOP/s of executed MFMAs); d = 128, B = 4, H = 16, N = 4096 causal 1065 ->
// 1029 us.  The chip's power, not a pipe, is what is left at these sizes: without the exponentials, the barrier or the
// row reads the pass gains 1 to 4 %.  Tiles requested two iterations ahead instead of one: no gain.
// Tiles go straight into the LDS (WaveTile's layout): through registers, 16 loads waited for and 16 LDS stores per iteration at
// d = 256 (8 and 8 at d = 128) cost the lone wave more.  Whole backward so, us, before / now: d = 256 16 x 8192 3389 / 3210,
// causal 64 x 2048 566 / 529; d = 128 causal 64 x 4096 925 / 910.
template <typename Tag, int D, bool CAUSAL>
__global__ void __launch_bounds__(256, 1)
fa_bwd_dkdv_shared_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                          const uint16_t* __restrict__ v, const uint16_t* __restrict__ dout,
                          const float* __restrict__ lse, const float* __restrict__ dvec, uint16_t* __restrict__ dk,
                          uint16_t* __restrict__ dv, int N, int n_kblocks, int total_wg, int kv_group, float scale) {
    [[maybe_unused]] ClockSpan clock_span;  // measurement builds only; empty otherwise
    static_assert(D == 128 || D == 256, "d = 64 keeps two workgroups per CU (fa_bwd_dkdv_kernel)");
    using Tile = WaveTile<D>;                 // the layout of a sub-tile in the LDS
    constexpr int BQ = 64;                    // queries per iteration, two sub-tiles
    constexpr int KEYT = D == 128 ? 2 : 1;    // key tiles whose scores a wave computes
    constexpr int NKT = 2 * KEYT;             // key tiles per workgroup
    constexpr int BK = 32 * NKT;              // keys per workgroup
    constexpr int KS = D / 16;                // MFMA steps along the head dimension
    constexpr int TILE_B = 2 * Tile::TILE_B;  // bytes per Q or dO tile
    constexpr int STAGE_B = 2 * TILE_B;       // Q, dO
    constexpr int NREQ = Tile::NI;            // staging instructions of a wave per iteration: half of them for Q
    constexpr int KP = 4;                     // steps by which row operand reads lead their MFMAs
    constexpr int PIECE = 1024;               // bytes of one exchanged operand: 32 keys x 16 queries
    using E = Elem<Tag>;

    __shared__ __attribute__((aligned(1024))) char lds_t[2 * STAGE_B];
    __shared__ __attribute__((aligned(16))) char lds_x[2][NKT * 4 * PIECE];  // P, dS: [key tile][sub-tile][slab]
    __shared__ __attribute__((aligned(16))) float lds_l[2][BQ];
    __shared__ __attribute__((aligned(16))) float lds_d[2][BQ];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;
    const int p = wave >> 1, g = wave & 1;

    // Longest first over all heads (work_item), B = 4, H = 16, N = 4096 causal, with the dQ pass in the same order:
    // whole backward 1016 -> 924 us at d = 128, 578 -> 494 us at d = 64; B = 8, N = 2048: 624 -> 547, 333 -> 273 us.
    const WorkItem item = work_item<CAUSAL>(blockIdx.x, total_wg, n_kblocks);  // key block 0 has the longest loop
    const int bh = item.head;
    const int key0 = item.tile * BK;
    // this wave's accumulators: key tiles acc_tile(0), acc_tile(1), columns col0 .. col0 + 63; tile 0 is one whose
    // scores it computes itself (at d = 128 both are)
    auto acc_tile = [&](int j) { return KEYT == 2 ? 2 * p + j : p ^ j; };
    const int col0 = 64 * (KEYT == 2 ? g : wave);

    // bh counts key/value heads; the kv_group query heads that share this one are bh * kv_group + i
    const size_t head_off = (size_t)bh * N * D;
    float sc = scale * kLog2e;
    asm volatile("" : "+v"(sc));  // in a vector register: an FMA with a scalar operand issues at a lower rate

    // ---- K and V rows of the score tiles as B operands, in the accumulation half of the register file
    i32x4 kreg[KEYT][KS], vreg[KEYT][KS];
    int my_key[KEYT];
#pragma unroll
    for (int i = 0; i < KEYT; ++i) {
        my_key[i] = key0 + (p * KEYT + i) * 32 + col;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const i32x4 z = {0, 0, 0, 0};
            const size_t off = head_off + (size_t)my_key[i] * D + ks * 16 + half * 8;
            kreg[i][ks] = my_key[i] < N ? *reinterpret_cast<const i32x4*>(k + off) : z;
            vreg[i][ks] = my_key[i] < N ? *reinterpret_cast<const i32x4*>(v + off) : z;
        }
    }
#pragma unroll
    for (int i = 0; i < KEYT; ++i)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(kreg[i][ks]), "+a"(vreg[i][ks]));

    f32x16 dkacc[2][2], dvacc[2][2];  // [key tile][32 columns]
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) dkacc[j][dt][r] = dvacc[j][dt][r] = 0.f;

    const int n_qtiles = (N + BQ - 1) / BQ;
    const int it0 = CAUSAL ? key0 / BQ : 0;  // first query tile that can see this key block
    // Addresses: row operands of the own sub-tile, transposed operands of this one and the other (16 rows further, dO and, at d = 256,
    // columns from 128 on of the rows are offsets), in the stage being read, and what the lane fetches of the wave's quarters
    constexpr int RA = KS < 8 ? KS : 8;
    uint32_t row_at[RA], tr_own[2][2], tr_oth[2][2];
    int src[NREQ / 2];
    const uint32_t lds_base = lds_address(lds_t), piece_at = lds_base + wave * (TILE_B / 4);
#pragma unroll
    for (int ks = 0; ks < RA; ++ks) {
        row_at[ks] = lds_base + g * Tile::TILE_B + col * Tile::ROWB + (((2 * ks + half) ^ Tile::swizzle(col)) << 4);
        asm volatile("" : "+v"(row_at[ks]));
    }
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            const uint32_t at = lds_base + Tile::tr_of(col0 / 32 + dt, hi, lane);
            tr_own[dt][hi] = at + g * Tile::TILE_B;
            tr_oth[dt][hi] = at + (g ^ 1) * Tile::TILE_B;
            asm volatile("" : "+v"(tr_own[dt][hi]), "+v"(tr_oth[dt][hi]));
        }
#pragma unroll
    for (int n = 0; n < NREQ / 2; ++n) {
        src[n] = wave * (TILE_B / 4) + Tile::src_of(n, lane);
        asm volatile("" : "+v"(src[n]));
    }
    int st = 0;  // the stage being read
    // Masked query tiles come first: every tile when the key block is ragged (keys past N), else the tiles on the
    // causal diagonal.  They get a loop of their own so that the main loop has a single straight-line body.
    const int it_masked_end = key0 + BK > N ? n_qtiles : (CAUSAL ? min(n_qtiles, (key0 + BK - 1) / BQ + 1) : it0);

    // Barrier for LDS traffic only: the next tile's global loads stay in flight.
    auto lds_barrier = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    // Every query head of the group adds into the same dK_j, dV_j.
#pragma nounroll
    for (int gi = 0; gi < kv_group; ++gi) {
    const size_t qhead = (size_t)bh * kv_group + gi;
    const float* lh = lse + qhead * N;
    const float* dh = dvec + qhead * N;
    // The next tiles to be requested.  Rows past N lie outside the resources and read as zero, so every iteration requests a next
    // tile: the one after the last is zeros that nothing reads.
    BufferWords q_rsrc = make_buffer_words(q + qhead * N * D, (uint32_t)N * D * 2), do_rsrc = make_buffer_words(dout + qhead * N * D, (uint32_t)N * D * 2);
    auto next_tile = [&](int tiles) __attribute__((always_inline)) {
        advance(q_rsrc, tiles * BQ * D * 2);
        advance(do_rsrc, tiles * BQ * D * 2);
    };
    float lpre = 0.f;  // threads 0..63 carry L, 64..127 carry D
    int lrow = 0;
    auto load_ld = [&](int it) __attribute__((always_inline)) {
        if (tid < 2 * BQ) {  // the raw value only: arithmetic on it here would wait for the load on the spot
            lrow = it * BQ + (tid & (BQ - 1));
            lpre = (tid < BQ ? lh : dh)[min(lrow, N - 1)];
        }
    };
    auto store_ld = [&](int st) __attribute__((always_inline)) {
        // rows past N get L = +inf so that P = exp2(0 - inf) = 0, and D = 0.  D is kept negated: the dP
        // accumulators start from -D_i, so dP - D comes out of the MFMAs
        if (tid < BQ) lds_l[st][tid] = lrow < N ? lpre * kLog2e : INFINITY;
        else if (tid < 2 * BQ) lds_d[st][tid - BQ] = lrow < N ? -lpre : 0.f;
    };

    auto landed = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    load_ld(it0);
    next_tile(it0);
#pragma unroll
    for (int n = 0; n < NREQ; ++n)
        global_to_lds_16B(n & 1 ? do_rsrc : q_rsrc, piece_at + st * STAGE_B + (n & 1) * TILE_B + (n >> 1) * 1024, src[n >> 1]);
    next_tile(1);
    store_ld(st);
    landed();

    auto iteration = [&](int it, auto mask_tag) __attribute__((always_inline)) {
        constexpr bool MASK = decltype(mask_tag)::value;
        const int q_first = it * BQ + 32 * g + 4 * half;  // query of score register 0
        uint32_t l_rows = lds_address(lds_l[0]) + st * (BQ * 4) + 128 * g + 16 * half;
        uint32_t d_rows = lds_address(lds_d[0]) + st * (BQ * 4) + 128 * g + 16 * half;
        asm volatile("" : "+v"(l_rows), "+v"(d_rows));
        const uint32_t next = piece_at + (st ^ 1) * STAGE_B;

        f32x16 sacc[KEYT], pacc[KEYT];
        i32x4 pa[KEYT][2], dsa[KEYT][2];  // [key tile][16-query slab] of the own sub-tile, as A operands
        f32x4 l4[4];

        auto await = [&](f32x16 (&x)[KEYT]) __attribute__((always_inline)) {  // results the hazard checker cannot see
            if constexpr (KEYT == 2) mfma_result_wait(x[0], x[1]);
            else mfma_result_wait(x[0]);
        };
        auto row_read = [&](int u) __attribute__((always_inline)) {  // step u of phases 1 (Q) and 2 (dO)
            return lds_load_16B(row_at[u % RA] + (u < KS ? 0 : TILE_B) + (u % KS / RA) * 256);
        };
        auto tr_read = [&](const uint32_t (&at)[2][2], int tensor, int w) __attribute__((always_inline)) {  // w = (slab, 32 columns)
            const int off = (tensor ? 0 : TILE_B) + (w >> 1) * 16 * Tile::ROWB;
            const i32x2 lo = lds_read_tr16(at[w & 1][0] + off), hi = lds_read_tr16(at[w & 1][1] + off);
            return i32x4{lo[0], lo[1], hi[0], hi[1]};
        };
        auto piece = [&](int tensor, int kt, int sub, int slab) __attribute__((always_inline)) {
            return lds_address(lds_x[tensor]) + ((kt * 2 + sub) * 2 + slab) * PIECE + lane * 16;
        };
        auto send = [&](int tensor, int i, int slab, const i32x4& x) __attribute__((always_inline)) {
            typedef i32x4 __attribute__((address_space(3))) * lds_vec_ptr;
            *(lds_vec_ptr)(uintptr_t)piece(tensor, p * KEYT + i, g, slab) = x;
        };

        // ---- phases 1 and 2
        i32x4 ring[KP], bdo[4];
#pragma unroll
        for (int u = 0; u < KP; ++u) ring[u] = row_read(u);
#pragma unroll
        for (int i = 0; i < 4; ++i) l4[i] = lds_load_4f(l_rows + 32 * i);
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // dP starts from -D: registers 4i .. 4i+3 are query rows 8i + 4 half ..
            const f32x4 t = lds_load_4f(d_rows + 32 * i);
#pragma unroll
            for (int j = 0; j < KEYT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) pacc[j][4 * i + r] = t[r];
        }
        load_ld(it + 1);
        __builtin_amdgcn_sched_barrier(0);
        auto probability = [&](int n) __attribute__((always_inline)) {  // score n of 16 KEYT
            const int i = n / 16, rr = n % 16;
            float x = fast_exp2(__builtin_fmaf(sacc[i][rr], sc, -l4[rr >> 2][rr & 3]));
            if constexpr (MASK) {
                const int qi = q_first + 8 * (rr >> 2) + (rr & 3);
                x = (my_key[i] >= N || (CAUSAL && my_key[i] > qi)) ? 0.f : x;
            }
            sacc[i][rr] = x;
            if (rr & 1) pa[i][rr >> 3][(rr >> 1) & 3] = E::pack2(sacc[i][rr - 1], x);
            if ((rr & 7) == 7) send(0, i, rr >> 3, pa[i][rr >> 3]);
        };
        static_for<2 * KS>([&](auto step) __attribute__((always_inline)) {
            constexpr int u = decltype(step)::value, ks = u % KS, n_req = u / 2, to = (n_req & 1) * TILE_B + (n_req >> 1) * 1024;
            static_assert(NREQ == KS, "one request every second step");
            const i32x4 a = ring[u % KP];
            if constexpr (u + KP < 2 * KS) ring[u % KP] = row_read(u + KP);
            else if constexpr (u + KP - 2 * KS < 4) bdo[u + KP - 2 * KS] = tr_read(tr_own, 0, u + KP - 2 * KS);
            const BufferWords& rsrc = n_req & 1 ? do_rsrc : q_rsrc;
            static_for<KEYT>([&](auto tile) __attribute__((always_inline)) {
                constexpr int i = decltype(tile)::value;
                constexpr bool LOAD = u % 2 == 0 && i == 0;
                using M = MfmaVgprAcc<Tag>;
                if constexpr (u < KS) {
                    if constexpr (ks == 0 && LOAD) M::template first_and_load<to>(sacc[i], a, kreg[i][ks], rsrc, next, src[n_req >> 1]);
                    else if constexpr (ks == 0) M::first(sacc[i], a, kreg[i][ks]);
                    else if constexpr (LOAD) M::template run_and_load<to>(sacc[i], a, kreg[i][ks], rsrc, next, src[n_req >> 1]);
                    else M::run(sacc[i], a, kreg[i][ks]);
                } else {
                    if constexpr (ks == 0 && LOAD) M::template start_and_load<to>(pacc[i], a, vreg[i][ks], rsrc, next, src[n_req >> 1]);
                    else if constexpr (ks == 0) M::start(pacc[i], a, vreg[i][ks]);
                    else if constexpr (LOAD) M::template run_and_load<to>(pacc[i], a, vreg[i][ks], rsrc, next, src[n_req >> 1]);
                    else M::run(pacc[i], a, vreg[i][ks]);
                    if constexpr (u == KS && i == KEYT - 1) await(sacc);
                    // 16 KEYT scores over the 16 MFMAs of this phase, none before the wait above
                    constexpr int M0 = KEYT - 1;
                    constexpr int m = ks * KEYT + i;
#pragma unroll
                    for (int n = 0; n < 16 * KEYT; ++n)
                        if (m >= M0 && M0 + (n * (16 - M0)) / (16 * KEYT) == m) probability(n);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        next_tile(1);

        // ---- phase 3: dV of the own piece beside dS
        i32x4 bq[4];
        auto gradient = [&](int n) __attribute__((always_inline)) {
            const int i = n / 16, rr = n % 16;
            pacc[i][rr] *= sacc[i][rr];
            if (rr & 1) dsa[i][rr >> 3][(rr >> 1) & 3] = E::pack2(pacc[i][rr - 1], pacc[i][rr]);
            if ((rr & 7) == 7) send(1, i, rr >> 3, dsa[i][rr >> 3]);
        };
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int i = 0; i < KEYT; ++i) {
                dvacc[i][w & 1] = E::mma(pa[i][w >> 1], bdo[w], dvacc[i][w & 1]);
                if (w == 0 && i == 0) await(pacc);
                if (i == 0) bq[w] = tr_read(tr_own, 1, w);
#pragma unroll
                for (int n = 0; n < 4; ++n) gradient((w * KEYT + i) * 4 + n);
                __builtin_amdgcn_sched_barrier(0);
            }

        lds_barrier();

        // ---- phase 4
        // the other waves' pieces: those of the other sub-tile and, at d = 256, the other key tile's of this one
        i32x4 bo[4], pf[2][2], dsf[2][2], px[2], dsx[2];
        if constexpr (KEYT == 1) {
#pragma unroll
            for (int s = 0; s < 2; ++s) px[s] = lds_load_16B(piece(0, acc_tile(1), g, s));
#pragma unroll
            for (int s = 0; s < 2; ++s) dsx[s] = lds_load_16B(piece(1, acc_tile(1), g, s));
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int j = 0; j < 2; ++j) pf[j][s] = lds_load_16B(piece(0, acc_tile(j), g ^ 1, s));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int i = 0; i < KEYT; ++i) {
                dkacc[i][w & 1] = E::mma(dsa[i][w >> 1], bq[w], dkacc[i][w & 1]);
                if (i == 0) bo[w] = tr_read(tr_oth, 0, w);
                __builtin_amdgcn_sched_barrier(0);
            }
        if constexpr (KEYT == 1) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                dvacc[1][w & 1] = E::mma(px[w >> 1], bdo[w], dvacc[1][w & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                dkacc[1][w & 1] = E::mma(dsx[w >> 1], bq[w], dkacc[1][w & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                dvacc[j][w & 1] = E::mma(pf[j][w >> 1], bo[w], dvacc[j][w & 1]);
                if (j == 0) bq[w] = tr_read(tr_oth, 1, w);
                else if (w < 2) {
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj) dsf[jj][w] = lds_load_16B(piece(1, acc_tile(jj), g ^ 1, w));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                dkacc[j][w & 1] = E::mma(dsf[j][w >> 1], bq[w], dkacc[j][w & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        store_ld(st ^ 1);
        landed();
        const int move = st ? -STAGE_B : STAGE_B;
#pragma unroll
        for (int ks = 0; ks < RA; ++ks) row_at[ks] += move;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                tr_own[dt][hi] += move;
                tr_oth[dt][hi] += move;
            }
        st ^= 1;
    };
    int it = it0;
    for (; it < it_masked_end; ++it) iteration(it, std::true_type{});
    for (; it < n_qtiles; ++it) iteration(it, std::false_type{});
    }  // query heads of the group

    // ---- epilogue: dK_j = scale * acc, dV_j = acc, through the exchange buffers (every read of them is behind the last barrier)
    char* patch = &lds_x[0][0] + wave * 4096;
    static_assert(sizeof(lds_x) >= 4 * 4096, "patches must fit");
    const __amdgpu_buffer_rsrc_t dk_rsrc = make_buffer(dk + head_off, (uint32_t)N * D * 2);
    const __amdgpu_buffer_rsrc_t dv_rsrc = make_buffer(dv + head_off, (uint32_t)N * D * 2);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        store_keys_via_lds<Tag, D * 2>(dkacc[j], scale, patch, dk_rsrc, key0 + acc_tile(j) * 32, col0 * 2, lane);
        store_keys_via_lds<Tag, D * 2>(dvacc[j], 1.0f, patch, dv_rsrc, key0 + acc_tile(j) * 32, col0 * 2, lane);
    }
}

// ---------------------------------------------------------------------------------------
// A wave's private tiles of 32 rows of two tensors (first, second) in two LDS stages (WaveTile).  The addresses are moved from
// stage to stage once per tile: a loop body per stage would save that, but the accumulators then change places
// between the two (64 to 150 register moves a tile, and spills).
template <int D>
struct WaveTiles : WaveTile<D> {
    static_assert(D == 64 || D == 128, "two stages of a wave's tiles must fit a quarter of the LDS");
    using Tile = WaveTile<D>;
    using Tile::TILE_B;
    static constexpr int STAGE_B = 2 * TILE_B;    // first, second
    using Tile::Tile;
    // Instruction n of 2 NI that bring the tiles at the resources' starts into stage st
    static constexpr int NREQ = 2 * Tile::NI;
    static_assert(NREQ == 2 * Tile::KS, "one per MFMA step of the two score products");
    __device__ __forceinline__ void move(int bytes) {
#pragma unroll
        for (int ks = 0; ks < Tile::KS; ++ks) this->row_at[ks] += bytes;
#pragma unroll
        for (int dt = 0; dt < Tile::DT; ++dt) {
            this->tr_at[dt][0] += bytes;
            this->tr_at[dt][1] += bytes;
        }
    }
    __device__ __forceinline__ void request(const BufferWords& first, const BufferWords& second, int st, int n) const {
        Tile::request(n & 1 ? second : first, st * STAGE_B + (n & 1) * TILE_B, n >> 1);
    }
};

// LDS of the kernels below: two stages of four waves' tiles, reused for the partial sums at the end
constexpr int few_lds_bytes(int d) {
    const int staging = 4 * 2 * 2 * 32 * d * 2, partial = 4 * 2 * 32 * (d + 4) * 4;
    return staging > partial ? staging : partial;
}

// ---------------------------------------------------------------------------------------
// dK/dV pass for launches that leave the chip idle (few key/value heads, short sequences), d = 64 and 128.
//
// A workgroup owns 32 keys instead of 128 and its four waves split the queries -- of all query heads that share the
// key/value head -- each with accumulators for all columns; the four partial sums meet in the LDS at the end, in a
// fixed order.  Four times as many workgroups, each with a quarter of the serial chain.  What it costs is operand
// traffic: a Q / dO tile is staged for one wave instead of four and an operand read serves one MFMA, which a chip
// that is mostly idle has to spare.  A wave stages its own tiles (32 queries of Q and dO), so the loop has no barrier.
// One wave to a SIMD issues an instruction every four to five cycles, so what a tile takes is its instructions: 500 became 360 of
// 32 MFMAs.  The mask is put on in a branch that only the tile on the diagonal takes, the next tile of the same head is aimed at
// by two additions, MFMA and staging request share their wait states, and the waits for the score products stand a step
// later.  A tile's first operands are read under the last products of the one before.  Requests go out two to a step of
// the first product: one to a step of both, they came late where many workgroups ask for the same lines.
// Where D is computed here a wave has few tiles, most of them of other heads.  What counts then is the code run once and what
// its requests wait for: the next tile is aimed at in one place, its rows of O follow its staging requests, and dO comes from
// the staged tile.  (With rows of both asked for ahead of the requests and the code at three places, 0.1 to 0.6 us more.)
// bf16, whole backward, us, before the 128-query dQ work beside this / with it / so: d = 64 4 on 1 x 32 4.99 / 5.18 / 4.65, 6 on 1 x 59
// 7.53 / 8.18 / 6.82, 2 x 128 5.57 / 5.43 / 4.90, 16 x 333 causal 9.65 / 9.46 / 8.46; d = 128 16 on 4 x 20 7.31 / 7.70 / 7.04.
// bf16, this pass of d = 128, H = 32 on 4, N = 2048 causal 126 -> 109 us, no mask (whole) 8 on 1 x 2368 143 -> 128.  (Not kept: eight
// waves in pairs that share tiles and trade P and dS through the LDS, which put all of them in step: 177.)
template <typename Tag, int D, bool CAUSAL, bool D_READY>
static __device__ __forceinline__ void dkdv_few(int block, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                const uint16_t* __restrict__ v, const uint16_t* __restrict__ o,
                                                const uint16_t* __restrict__ dout, const float* __restrict__ lse,
                                                const float* __restrict__ dvec, uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int N, int n_heads,
                                                int kv_group, float scale, char* lds, float* lds_ld_all) {
    using Tiles = WaveTiles<D>;
    constexpr int NW = 4, BQ = Tiles::ROWS, BK = 32;
    constexpr int KS = D / 16, DT = D / 32, CPR = D / 8;
    constexpr int KP = 4;                       // steps by which operand reads lead their MFMAs
    constexpr int PSTR = D + 4;                 // row stride of the partial sums (floats)
    static_assert(few_lds_bytes(D) >= NW * 2 * BK * PSTR * 4, "partial sums must fit");
    using E = Elem<Tag>;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;
    // key blocks of equal index one after the other over the heads: under a causal mask the longest come first, and
    // with a multiple of 8 heads all blocks of a head stay on one XCD
    const int bh = block % n_heads;
    const int key0 = (block / n_heads) * BK;
    const size_t head_off = (size_t)bh * N * D;
    const int my_key = key0 + col;
    float sc = scale * kLog2e;
    asm volatile("" : "+v"(sc));

    i32x4 kreg[KS], vreg[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const i32x4 z = {0, 0, 0, 0};
        const size_t off = head_off + (size_t)my_key * D + ks * 16 + half * 8;
        kreg[ks] = my_key < N ? *reinterpret_cast<const i32x4*>(k + off) : z;
        vreg[ks] = my_key < N ? *reinterpret_cast<const i32x4*>(v + off) : z;
    }
    f32x16 dkacc[DT], dvacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) dkacc[dt][r] = dvacc[dt][r] = 0.f;

    float* lds_ld = lds_ld_all + wave * 2 * BQ;  // L (log2 units), then -D, of the wave's tile
    Tiles tiles(lds_address(lds) + wave * 2 * Tiles::STAGE_B, lane);  // Q, dO
    const int n_t = (N + BQ - 1) / BQ, t0 = CAUSAL ? key0 / BQ : 0;

    // ---- this wave's tiles: numbers wave, wave + NW, ... of the group's tiles in order
    const int n_all = kv_group * (n_t - t0), mine = (n_all - wave + NW - 1) / NW;
    int gi = 0, t = t0 + wave;  // the tile aimed at
    float ldpre = 0.f;
    int ldrow = 0;
    const float* ld_head = lse;  // lanes 0..31 carry L, 32..63 carry D
    i32x4 opre[KS];              // without D in the workspace: the lane's half of a row of O
    BufferWords q_rsrc, do_rsrc;
    auto load_rows = [&]() __attribute__((always_inline)) {
        const int row = min(ldrow, N - 1);
        ldpre = ld_head[row];
        if constexpr (!D_READY) {
            const size_t at = ((size_t)bh * kv_group + gi) * N + row;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) opre[ks] = *reinterpret_cast<const i32x4*>(o + at * D + ks * 16 + half * 8);
        }
    };
    auto aim_head = [&]() __attribute__((always_inline)) {  // the next requests: tile t, counted on into the next query heads
        while (t >= n_t) {
            t -= n_t - t0;
            ++gi;
        }
        const size_t qhead = (size_t)bh * kv_group + gi;
        const uint32_t bytes = (uint32_t)N * D * 2;
        q_rsrc = make_buffer_words(q + qhead * N * D, bytes);
        do_rsrc = make_buffer_words(dout + qhead * N * D, bytes);
        advance(q_rsrc, t * Tiles::TILE_B);
        advance(do_rsrc, t * Tiles::TILE_B);
        ldrow = t * BQ + col;
        ld_head = (D_READY && half ? dvec : lse) + qhead * N;
    };
    auto aim_next = [&](bool any) __attribute__((always_inline)) {
        t += NW;
        if (D_READY && __builtin_expect(any & (t < n_t), 1)) {  // the same head, which costs a few instructions only
            advance(q_rsrc, NW * Tiles::TILE_B);
            advance(do_rsrc, NW * Tiles::TILE_B);
            ldrow += NW * BQ;
            load_rows();
        } else if (any) {
            aim_head();
            if constexpr (D_READY) load_rows();
        } else {  // past the last tile: zeros that nothing reads
            q_rsrc.w[2] = do_rsrc.w[2] = 0;
        }
    };
    // L and -D of the tile aimed at, which has landed and which the addresses point at, go where its products find them.  Rows
    // past N get L = +inf so that P = exp2(0 - inf) = 0, and D = 0.  (Keys past N need nothing: what their lanes compute goes
    // to rows of dK and dV that are not stored.)
    const float ld_factor = half ? -1.f : kLog2e, ld_none = half ? 0.f : INFINITY;
    auto put_rows = [&]() __attribute__((always_inline)) {
        float x = ldpre;
        if constexpr (!D_READY) {
            float d_row = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) d_row = dot8<Tag>(opre[ks], tiles.row_read(Tiles::TILE_B, ks), d_row);
            d_row = sum_both_halves(d_row);
            x = half ? d_row : x;
        }
        x *= ld_factor;
        lds_ld[lane] = ldrow < N ? x : ld_none;
    };
    auto row_read = [&](int u) { return tiles.row_read(u < KS ? 0 : Tiles::TILE_B, u % KS); };
    auto tr_read = [&](int u) {  // u = (tensor: dO then Q, slab, dt)
        return tiles.tr_read(u < 2 * DT ? Tiles::TILE_B : 0, (u / DT) % 2, u % DT);
    };
    i32x4 ring[KP];  // the first row operands of a tile are read under the last products of the one before

    // The tile whose first operands are in `ring`, while the tile aimed at is requested into the other stage
    auto tile = [&](int q0, int st, int left) __attribute__((always_inline)) {  // `left`: tiles after this one
        f32x4 l4[4];
        f32x16 sacc, pacc;
        const uint32_t ld = lds_address(lds_ld) + 16 * half;
        const uint32_t next = tiles.base + (st ^ 1) * Tiles::STAGE_B;
        if constexpr (!D_READY) aim_next(left > 0);
        i32x4 tr[KP], pa[2], dsa[2];
        auto probability = [&](int rr) __attribute__((always_inline)) {
            sacc[rr] = fast_exp2(__builtin_fmaf(sacc[rr], sc, -l4[rr >> 2][rr & 3]));
            if (rr & 1) pa[rr >> 3][(rr >> 1) & 3] = E::pack2(sacc[rr - 1], sacc[rr]);
        };
        // S, then dP beside P, which starts one step late: the wait for S has passed by then
        static_for<2 * KS>([&](auto step) __attribute__((always_inline)) {
            constexpr int u = decltype(step)::value;
            const i32x4 a = ring[u % KP];
            if constexpr (u + KP < 2 * KS) ring[u % KP] = row_read(u + KP);
            else tr[u + KP - 2 * KS] = tr_read(u + KP - 2 * KS);
            if constexpr (u < 4) {  // register r of 16 is query row 8 (r / 4) + 4 half + r % 4
                l4[u] = lds_load_4f(ld + 32 * u);
                const f32x4 x = lds_load_4f(ld + 128 + 32 * u);  // dP starts from -D
#pragma unroll
                for (int r = 0; r < 4; ++r) pacc[4 * u + r] = x[r];
            }
            if constexpr (u < KS) global_to_lds_16B(do_rsrc, next + Tiles::TILE_B + u * 1024, tiles.src[u]);
            if constexpr (u == 0) MfmaVgprAcc<Tag>::template first_and_load<u * 1024>(sacc, a, kreg[u], q_rsrc, next, tiles.src[u]);
            else if constexpr (u < KS) MfmaVgprAcc<Tag>::template run_and_load<u * 1024>(sacc, a, kreg[u], q_rsrc, next, tiles.src[u]);
            else if constexpr (u == KS) MfmaVgprAcc<Tag>::start(pacc, a, vreg[u - KS]);
            else MfmaVgprAcc<Tag>::run(pacc, a, vreg[u - KS]);
            if constexpr (!D_READY && u == KS)
                if (left > 0) load_rows();
            if constexpr (u == KS + 1) mfma_result_wait_rest<4>(sacc);
            if constexpr (u > KS) {
                constexpr int i = u - KS - 1;
#pragma unroll
                for (int rr = i * 16 / (KS - 1); rr < (i + 1) * 16 / (KS - 1); ++rr) probability(rr);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if (CAUSAL && __builtin_expect(q0 == key0, 0)) {  // the tile on the diagonal
            const int first_visible = my_key - q0 - 4 * half;  // of the lane's query rows
#pragma unroll
            for (int rr = 0; rr < 16; ++rr) {
                if (8 * (rr >> 2) + (rr & 3) < first_visible) sacc[rr] = 0.f;
                if (rr & 1) pa[rr >> 3][(rr >> 1) & 3] = E::pack2(sacc[rr - 1], sacc[rr]);
            }
        }
        // dV beside dS, which starts one step late likewise, then dK
        constexpr int GE = 16 / (2 * DT);  // gradients per MFMA of the dV group
        static_for<4 * DT>([&](auto step) __attribute__((always_inline)) {
            constexpr int u = decltype(step)::value;
            const i32x4 b = tr[u % KP];
            if constexpr (u + KP < 4 * DT) tr[u % KP] = tr_read(u + KP);
            if constexpr (u == 4 * DT - 2) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the next tile has landed
                tiles.move(st ? -Tiles::STAGE_B : Tiles::STAGE_B);
                if (D_READY || left > 0) put_rows();
            }
            if constexpr (u >= 4 * DT - 2)
#pragma unroll
                for (int i = 0; i < KP / 2; ++i) ring[(u - (4 * DT - 2)) * (KP / 2) + i] = row_read((u - (4 * DT - 2)) * (KP / 2) + i);
            if constexpr (u < 2 * DT) dvacc[u % DT] = E::mma(pa[u / DT], b, dvacc[u % DT]);
            else dkacc[u % DT] = E::mma(dsa[(u - 2 * DT) / DT], b, dkacc[u % DT]);
            if constexpr (u == 1) mfma_result_wait_rest<1>(pacc);
            if constexpr (u >= 1 && u <= 2 * DT)
#pragma unroll
                for (int n = 0; n < GE; ++n) {
                    const int rr = (u - 1) * GE + n;
                    pacc[rr] *= sacc[rr];
                    if (rr & 1) dsa[rr >> 3][(rr >> 1) & 3] = E::pack2(pacc[rr - 1], pacc[rr]);
                }
            if constexpr (D_READY && u == 4 * DT - 1) aim_next(left > 1);
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    if (mine > 0) {
        aim_head();
        load_rows();
#pragma unroll
        for (int n = 0; n < Tiles::NREQ; ++n) tiles.request(q_rsrc, do_rsrc, 0, n);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(kreg[ks]), "+a"(vreg[ks]));
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        put_rows();
#pragma unroll
        for (int u = 0; u < KP; ++u) ring[u] = row_read(u);
        int q0 = t * BQ;
        if constexpr (D_READY) aim_next(mine > 1);
        for (int n = 0, st = 0; n < mine; ++n, st ^= 1) {
            const int q0_next = t * BQ;
            tile(q0, st, mine - 1 - n);
            q0 = D_READY ? q0_next : t * BQ;
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the zeros of the last request: the LDS is about to be reused

    // ---- sum of the four waves' parts, wave 0 first
    __syncthreads();
    float* part = reinterpret_cast<float*>(lds);  // [wave][dK, dV][key][PSTR]
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float* p = part + (wave * 2 * BK + 8 * (r >> 2) + 4 * half + (r & 3)) * PSTR + dt * 32 + col;
            p[0] = dkacc[dt][r];
            p[BK * PSTR] = dvacc[dt][r];
        }
    __syncthreads();
#pragma nounroll
    for (int i = 0; i < 2 * BK * CPR / 256; ++i) {
        const int c = tid + i * 256, row = c / CPR, cc = (c % CPR) * 8;  // row: keys of dK, then of dV
        const int key = key0 + row % BK;
        const i32x4 w = sum_parts<Tag, NW>(part + row * PSTR + cc, 2 * BK * PSTR, row < BK ? scale : 1.0f);
        if (key < N) *reinterpret_cast<i32x4*>((row < BK ? dk : dv) + head_off + (size_t)key * D + cc) = w;
    }
}

// The dQ pass for such launches: the same division the other way round.  A workgroup
// owns 32 queries and its four waves split the keys (tiles of 32, staged by the wave that works them), each with a dQ
// accumulator; the four partial sums meet in the LDS at the end, in a fixed order.
// bf16, B = 1, H = 4, N = 1024: whole backward 54 -> 27 us at d = 128, 33 -> 18 us at d = 64.
template <typename Tag, int D, bool CAUSAL, bool D_READY>
static __device__ __forceinline__ void dq_few(int block, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                              const uint16_t* __restrict__ v, const uint16_t* __restrict__ o,
                                              const uint16_t* __restrict__ dout, const float* __restrict__ lse,
                                              float* __restrict__ dvec, uint16_t* __restrict__ dq, int N,
                                              int n_heads, int kv_group, float scale, char* lds) {
    using Tiles = WaveTiles<D>;
    constexpr int NW = 4, BQ = 32, BK = Tiles::ROWS;
    constexpr int KS = D / 16, DT = D / 32, CPR = D / 8;
    constexpr int KP = 4;        // steps by which operand reads lead their MFMAs
    constexpr int PSTR = D + 4;  // row stride of the partial sums (floats)
    using E = Elem<Tag>;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;
    // tiles of equal index one after the other over the heads (all of a head on one XCD when their number is a
    // multiple of 8); causal: the longest rows first
    const int bh = block % n_heads;
    const int n_t = (N + BK - 1) / BK;
    const int qt = CAUSAL ? n_t - 1 - block / n_heads : block / n_heads;
    const int q0 = qt * BQ;
    const int row = min(q0 + col, N - 1);  // rows past N compute a copy of row N-1, never stored
    const int limit = CAUSAL ? row : N - 1;  // last visible key
    const size_t head_off = (size_t)bh * N * D;
    const size_t kv_off = (size_t)(bh / kv_group) * N * D;
    float sc = scale * kLog2e;
    asm volatile("" : "+v"(sc));
    // the wave's next tiles (rows past N read as zero)
    BufferWords k_rsrc = make_buffer_words(k + kv_off, (uint32_t)N * D * 2), v_rsrc = make_buffer_words(v + kv_off, (uint32_t)N * D * 2);
    advance(k_rsrc, wave * Tiles::TILE_B);
    advance(v_rsrc, wave * Tiles::TILE_B);
    Tiles tiles(lds_address(lds) + wave * 2 * Tiles::STAGE_B, lane);  // K, V

    const int n_tiles = CAUSAL ? qt + 1 : n_t;
#pragma unroll
    for (int n = 0; n < Tiles::NREQ; ++n) tiles.request(k_rsrc, v_rsrc, 0, n);

    i32x4 qreg[KS], doreg[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const size_t off = head_off + (size_t)row * D + ks * 16 + half * 8;
        qreg[ks] = *reinterpret_cast<const i32x4*>(q + off);
        doreg[ks] = *reinterpret_cast<const i32x4*>(dout + off);
    }
    float d_row = 0.f;  // D = rowsum(dO o O)
    if constexpr (D_READY) {
        d_row = dvec[(size_t)bh * N + row];
    } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            d_row = dot8<Tag>(*reinterpret_cast<const i32x4*>(o + head_off + (size_t)row * D + ks * 16 + half * 8), doreg[ks], d_row);
        d_row = sum_both_halves(d_row);
        if (wave == 0 && half == 0 && q0 + col < N) dvec[(size_t)bh * N + q0 + col] = d_row;
    }
    const float l2 = lse[(size_t)bh * N + row] * kLog2e;
    f32x16 acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[dt][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qreg[ks]), "+a"(doreg[ks]));

    int st = 0;
    for (int t = wave; t < n_tiles; t += NW, st ^= 1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this tile has landed
        advance(k_rsrc, NW * Tiles::TILE_B);
        advance(v_rsrc, NW * Tiles::TILE_B);
        i32x4 ring[KP];
#pragma unroll
        for (int u = 0; u < KP; ++u) ring[u] = tiles.row_read(0, u);
        const uint32_t next = tiles.base + (st ^ 1) * Tiles::STAGE_B;
        auto issue = [&](auto step, f32x16& c, const i32x4& a, const i32x4& b) __attribute__((always_inline)) {
            // past this workgroup's last tile the requests bring rows (or zeros) that nothing reads
            constexpr int u = decltype(step)::value, to = (u & 1) * Tiles::TILE_B + (u >> 1) * 1024;
            const BufferWords& rsrc = u & 1 ? v_rsrc : k_rsrc;
            if constexpr (u == 0) MfmaVgprAcc<Tag>::template first_and_load<to>(c, a, b, rsrc, next, tiles.src[u >> 1]);
            else if constexpr (u == KS) MfmaVgprAcc<Tag>::template start_and_load<to>(c, a, b, rsrc, next, tiles.src[u >> 1]);
            else MfmaVgprAcc<Tag>::template run_and_load<to>(c, a, b, rsrc, next, tiles.src[u >> 1]);
        };
        f32x16 sacc, pacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) pacc[r] = -d_row;  // dP - D comes out of the MFMAs
        i32x4 tr[KP], dsb[2];
        // S^T, then dP^T beside P, which starts one step late: the wait for S has passed by then
        static_for<2 * KS>([&](auto step) __attribute__((always_inline)) {
            constexpr int u = decltype(step)::value;
            const i32x4 a = ring[u % KP];
            if constexpr (u + KP < 2 * KS) ring[u % KP] = tiles.row_read(u + KP < KS ? 0 : Tiles::TILE_B, (u + KP) % KS);
            else tr[u + KP - 2 * KS] = tiles.tr_read(0, (u + KP - 2 * KS) / DT, (u + KP - 2 * KS) % DT);
            if constexpr (u < KS) issue(step, sacc, a, qreg[u]);
            else issue(step, pacc, a, doreg[u - KS]);
            if constexpr (u == KS + 1) mfma_result_wait_rest<7>(sacc);
            if constexpr (u > KS) {
                constexpr int i = u - KS - 1;
#pragma unroll
                for (int r = i * 16 / (KS - 1); r < (i + 1) * 16 / (KS - 1); ++r) sacc[r] = fast_exp2(__builtin_fmaf(sacc[r], sc, -l2));
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if (__builtin_expect(t == n_t - 1 || (CAUSAL && t == qt), 0)) {  // keys past N (K = 0, but their P may be anything) and keys after the query
            const int bound = limit - t * BK - 4 * half;                 // key 8 (r / 4) + r % 4 of the lane's half is visible up to here
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + (r & 3) > bound) sacc[r] = 0.f;
        }
        mfma_result_wait(pacc);
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 8 * s2 + 2 * e;
                dsb[s2][e] = E::pack2(sacc[r] * pacc[r], sacc[r + 1] * pacc[r + 1]);
            }
        // dQ^T += K^T dS^T
#pragma unroll
        for (int u = 0; u < 2 * DT; ++u) {
            const i32x4 a = tr[u % KP];
            if (u + KP < 2 * DT) tr[u % KP] = tiles.tr_read(0, (u + KP) / DT, (u + KP) % DT);
            acc[u % DT] = E::mma(a, dsb[u / DT], acc[u % DT]);
            __builtin_amdgcn_sched_barrier(0);
        }
        tiles.move(st ? -Tiles::STAGE_B : Tiles::STAGE_B);
    }

    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the last request: the LDS is about to be reused

    // ---- sum of the four waves' parts, wave 0 first
    __syncthreads();
    float* part = reinterpret_cast<float*>(lds);  // [wave][query][PSTR]
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 w = {acc[dt][4 * g], acc[dt][4 * g + 1], acc[dt][4 * g + 2], acc[dt][4 * g + 3]};
            *reinterpret_cast<f32x4*>(part + (wave * BQ + col) * PSTR + dt * 32 + 8 * g + 4 * half) = w;
        }
    __syncthreads();
#pragma nounroll
    for (int c = tid; c < BQ * CPR; c += 256) {
        const int r = c / CPR, cc = (c % CPR) * 8;
        const i32x4 w = sum_parts<Tag, NW>(part + r * PSTR + cc, BQ * PSTR, scale);
        if (q0 + r < N) *reinterpret_cast<i32x4*>(dq + head_off + (size_t)(q0 + r) * D + cc) = w;
    }
}

// The dQ pass with 128 queries to a workgroup, 32 to each of its four waves, which walk all the keys together: every tile of
// K and V is staged once for the four of them, three tiles ahead into a ring, one barrier to a tile.  The last product
// comes one tile late, beside the next tile's dS; without that, 128 queries took 68.3 us where these take 63.5 and 32 queries 96.6
// (bf16, D and this pass, d = 128, H = 32 on 4, N = 2048 causal).
template <typename Tag, int D, bool CAUSAL, bool D_READY>
static __device__ __forceinline__ void dq_rows(int block, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                               const uint16_t* __restrict__ v, const uint16_t* __restrict__ o,
                                               const uint16_t* __restrict__ dout, const float* __restrict__ lse,
                                               float* __restrict__ dvec, uint16_t* __restrict__ dq, int N,
                                               int n_heads, int kv_group, float scale, char* lds) {
    using Tiles = WaveTiles<D>;
    // (five stages would do for this lead and a product that comes a tile late; eight are there for the key blocks' tiles anyway, and
    // the ring's remainder by eight is one instruction)
    constexpr int NW = 4, BR = 32 * NW, BK = Tiles::ROWS, STAGES = 8, LEAD = 3;
    constexpr int KS = D / 16, DT = D / 32;
    constexpr int KP = D == 128 ? 8 : 4;      // steps by which operand reads lead their MFMAs
    constexpr int PER = Tiles::NREQ / NW;     // staging instructions of a wave per tile
    static_assert(few_lds_bytes(D) >= STAGES * Tiles::STAGE_B, "the ring must fit");
    using E = Elem<Tag>;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;
    const int bh = block % n_heads;
    const int n_t = (N + BK - 1) / BK, n_q = (N + BR - 1) / BR;
    const int qt = CAUSAL ? n_q - 1 - block / n_heads : block / n_heads;  // the longest rows first
    const int q0 = qt * BR + wave * 32;
    const int row = min(q0 + col, N - 1);  // rows past N compute a copy of row N-1, never stored
    const int limit = CAUSAL ? row : N - 1;  // last visible key
    const size_t head_off = (size_t)bh * N * D;
    const size_t kv_off = (size_t)(bh / kv_group) * N * D;
    float sc = scale * kLog2e;
    asm volatile("" : "+v"(sc));
    // the next tile to be requested (rows past N, and tiles past the last one, read as zero)
    BufferWords k_rsrc = make_buffer_words(k + kv_off, (uint32_t)N * D * 2), v_rsrc = make_buffer_words(v + kv_off, (uint32_t)N * D * 2);
    Tiles tiles(lds_address(lds), lane);  // K, V
    int src[PER / 2];                     // of the wave's pieces of a tile
#pragma unroll
    for (int i = 0; i < PER / 2; ++i) {
        src[i] = Tiles::src_of(wave * (PER / 2) + i, lane);
        asm volatile("" : "+v"(src[i]));
    }
    const uint32_t piece = tiles.base + wave * (PER / 2) * 1024;
    auto request = [&](int st, int n) __attribute__((always_inline)) {  // instruction n of PER
        global_to_lds_16B(n & 1 ? v_rsrc : k_rsrc, piece + st * Tiles::STAGE_B + (n & 1) * Tiles::TILE_B + (n >> 1) * 1024, src[n >> 1]);
    };
    auto next_tile = [&]() __attribute__((always_inline)) {
        advance(k_rsrc, Tiles::TILE_B);
        advance(v_rsrc, Tiles::TILE_B);
    };

    const int n_tiles = CAUSAL ? min((qt + 1) * NW, n_t) : n_t;
#pragma unroll
    for (int st = 0; st < LEAD; ++st) {
#pragma unroll
        for (int n = 0; n < PER; ++n) request(st, n);
        next_tile();
    }

    i32x4 qreg[KS], doreg[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const size_t off = head_off + (size_t)row * D + ks * 16 + half * 8;
        qreg[ks] = *reinterpret_cast<const i32x4*>(q + off);
        doreg[ks] = *reinterpret_cast<const i32x4*>(dout + off);
    }
    float d_row = 0.f;  // D = rowsum(dO o O)
    if constexpr (D_READY) {
        d_row = dvec[(size_t)bh * N + row];
    } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            d_row = dot8<Tag>(*reinterpret_cast<const i32x4*>(o + head_off + (size_t)row * D + ks * 16 + half * 8), doreg[ks], d_row);
        d_row = sum_both_halves(d_row);
        if (half == 0 && q0 + col < N) dvec[(size_t)bh * N + q0 + col] = d_row;
    }
    const float l2 = lse[(size_t)bh * N + row] * kLog2e;
    f32x16 acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[dt][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qreg[ks]), "+a"(doreg[ks]));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // from here on the wave's requests are all that the counter counts

    auto arrive = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((LEAD - 1) * PER) : "memory");  // the wave's pieces of the next tile have landed
        __builtin_amdgcn_s_barrier();  // everyone's have, and the tile before this one is done with
        asm volatile("" ::: "memory");
    };
    const int own_tiles = CAUSAL ? min(n_tiles, qt * NW + wave + 1) : n_tiles;  // that concern the wave
    i32x4 ring[KP], ds[2];  // the next tile's first row operands; dS^T of the tile before, whose product comes one tile late
    arrive();
#pragma unroll
    for (int u = 0; u < KP; ++u) ring[u] = tiles.row_read(0, u);
    auto tr_read = [&](int u) { return tiles.tr_read(0, u / DT, u % DT); };
    int st = 0, t = 0, tr_move = 0;
    auto tile = [&](auto first_tile) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_tile)::value;
        const uint32_t next = piece + (st + LEAD) % STAGES * Tiles::STAGE_B;
        const int row_move = st == STAGES - 1 ? -(STAGES - 1) * Tiles::STAGE_B : Tiles::STAGE_B;
        f32x16 sacc, pacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) pacc[r] = -d_row;  // dP - D comes out of the MFMAs
        i32x4 tr[KP], ds_new[2];
        // S^T, then dP^T beside P, which starts one step late: the wait for S has passed by then
        static_for<2 * KS>([&](auto step) __attribute__((always_inline)) {
            constexpr int u = decltype(step)::value;
            const i32x4 a = ring[u % KP];
            if constexpr (u + KP < 2 * KS) ring[u % KP] = tiles.row_read(u + KP < KS ? 0 : Tiles::TILE_B, (u + KP) % KS);
            else if constexpr (!FIRST) tr[u + KP - 2 * KS] = tr_read(u + KP - 2 * KS);
            f32x16& c = u < KS ? sacc : pacc;
            const i32x4& b = u < KS ? qreg[u % KS] : doreg[u % KS];
            constexpr int EVERY = 2 * KS / PER, n = u / EVERY, to = (n & 1) * Tiles::TILE_B + (n >> 1) * 1024;
            const BufferWords& rsrc = n & 1 ? v_rsrc : k_rsrc;
            if constexpr (u == 0) MfmaVgprAcc<Tag>::template first_and_load<to>(c, a, b, rsrc, next, src[n >> 1]);
            else if constexpr (u == KS) MfmaVgprAcc<Tag>::template start_and_load<to>(c, a, b, rsrc, next, src[n >> 1]);
            else if constexpr (u % EVERY == 0) MfmaVgprAcc<Tag>::template run_and_load<to>(c, a, b, rsrc, next, src[n >> 1]);
            else MfmaVgprAcc<Tag>::run(c, a, b);
            if constexpr (u == KS + 1) mfma_result_wait_rest<7>(sacc);
            if constexpr (u > KS) {
                constexpr int i = u - KS - 1;
#pragma unroll
                for (int r = i * 16 / (KS - 1); r < (i + 1) * 16 / (KS - 1); ++r) sacc[r] = fast_exp2(__builtin_fmaf(sacc[r], sc, -l2));
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if (__builtin_expect(t == n_t - 1 || (CAUSAL && t * BK == q0), 0)) {  // keys past N (K = 0, but their P may be anything) and keys after the query
            const int bound = limit - t * BK - 4 * half;                      // key 8 (r / 4) + r % 4 of the lane's half is visible up to here
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + (r & 3) > bound) sacc[r] = 0.f;
        }
        // dQ^T += K^T dS^T of the tile before beside this one's dS, and at the end the next tile's first operands
        static_for<2 * DT>([&](auto step) __attribute__((always_inline)) {
            constexpr int u = decltype(step)::value;
            i32x4 a = {};
            if constexpr (!FIRST) {
                a = tr[u % KP];
                if constexpr (u + KP < 2 * DT) tr[u % KP] = tr_read(u + KP);
            }
            if constexpr (u == 2 * DT - KP) {
                next_tile();
                arrive();
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) tiles.row_at[ks] += row_move;
                if constexpr (!FIRST)
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) {
                        tiles.tr_at[dt][0] += tr_move;
                        tiles.tr_at[dt][1] += tr_move;
                    }
            }
            if constexpr (u >= 2 * DT - KP) ring[u - (2 * DT - KP)] = tiles.row_read(0, u - (2 * DT - KP));
            if constexpr (!FIRST) acc[u % DT] = E::mma(a, ds[u / DT], acc[u % DT]);
            if constexpr (u == 1) {
                if constexpr (FIRST) mfma_result_wait(pacc);
                else mfma_result_wait_rest<8>(pacc);
            }
            if constexpr (u > 0)
#pragma unroll
                for (int r = (u - 1) * 16 / (2 * DT - 1); r < u * 16 / (2 * DT - 1); ++r) {
                    pacc[r] *= sacc[r];
                    if (r & 1) ds_new[r >> 3][(r >> 1) & 3] = E::pack2(pacc[r - 1], pacc[r]);
                }
            __builtin_amdgcn_sched_barrier(0);
        });
        ds[0] = ds_new[0];
        ds[1] = ds_new[1];
        tr_move = row_move;
        st = (st + 1) % STAGES;
        ++t;
    };
    tile(std::true_type{});
    while (t < own_tiles) tile(std::false_type{});
#pragma unroll
    for (int u = 0; u < 2 * DT; ++u) acc[u % DT] = E::mma(tr_read(u), ds[u / DT], acc[u % DT]);
    for (; t < n_tiles; ++t) {  // the others' last tiles
#pragma unroll
        for (int n = 0; n < PER; ++n) request((st + LEAD) % STAGES, n);
        next_tile();
        arrive();
        st = (st + 1) % STAGES;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the last requests: the LDS is about to be reused
    __syncthreads();
    store_rows_via_lds<Tag, DT>(acc, scale, lds + wave * 4096, make_buffer(dq + head_off, (uint32_t)N * D * 2), q0, lane);
}

// One launch for the dK/dV pass or for both: n_dkdv workgroups take 32 keys each, the others 32 or 128 queries each
// (choose_bwd_form).  With both in one launch the dQ work fills the CUs that the shorter key blocks of a causal dK/dV pass leave
// idle.  (dQ alone comes here where it has to follow the dK/dV pass.)
// D_READY: D is in the workspace already; otherwise both kinds compute it for the rows they work on (the dK/dV kind
// once per tile; bwd_own_row_sums says when).
constexpr int kDqRows = 1, kDqFirst = 2;  // dq_form: 128 queries to a workgroup; dQ work ahead of the key blocks
template <typename Tag, int D, bool CAUSAL, bool D_READY>
__global__ void __launch_bounds__(256, D == 64 ? 2 : 1)
fa_bwd_few_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                  const uint16_t* __restrict__ o, const uint16_t* __restrict__ dout, const float* __restrict__ lse,
                  float* __restrict__ dvec, uint16_t* __restrict__ dq, uint16_t* __restrict__ dk,
                  uint16_t* __restrict__ dv, int N, int n_dkdv, int dq_form, int n_heads, int kv_group, float scale) {
    [[maybe_unused]] ClockSpan clock_span;  // measurement builds only; empty otherwise
    __shared__ __attribute__((aligned(1024))) char lds[few_lds_bytes(D)];
    __shared__ __attribute__((aligned(16))) float lds_ld[4 * 64];
    const int n_dq = gridDim.x - n_dkdv, block = blockIdx.x;
    const bool dq_first = dq_form & kDqFirst, is_dq = dq_first ? block < n_dq : block >= n_dkdv;
    const int id = block - (is_dq == dq_first ? 0 : is_dq ? n_dkdv : n_dq);
    if (!is_dq)
        dkdv_few<Tag, D, CAUSAL, D_READY>(id, q, k, v, o, dout, lse, dvec, dk, dv, N, n_heads / kv_group, kv_group, scale, lds, lds_ld);
    else if (dq_form & kDqRows)
        dq_rows<Tag, D, CAUSAL, D_READY>(id, q, k, v, o, dout, lse, dvec, dq, N, n_heads, kv_group, scale, lds);
    else
        dq_few<Tag, D, CAUSAL, D_READY>(id, q, k, v, o, dout, lse, dvec, dq, N, n_heads, kv_group, scale, lds);
}

// ---------------------------------------------------------------------------------------
// dQ pass: the forward kernel's structure with dO alongside Q and K^T in place of V^T.
template <typename Tag, int D, int BC, int NW, bool CAUSAL>
__global__ void __launch_bounds__(NW * 64, 2)
fa_bwd_dq_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                 const uint16_t* __restrict__ o, const uint16_t* __restrict__ dout, const float* __restrict__ lse,
                 float* __restrict__ dvec, uint16_t* __restrict__ dq, int N, int n_qtiles, int total_wg, int kv_group, float scale) {
    [[maybe_unused]] ClockSpan clock_span;  // measurement builds only; empty otherwise
    constexpr int NT = NW * 64;
    constexpr int BR = NW * 32;
    constexpr int RSTR = bwd_row_stride(D);  // K tile: row reads and transposed reads
    constexpr int VSTR = D + 8;              // V tile: row reads only
    constexpr int KT = BC / 32;
    constexpr int KS = D / 16;
    constexpr int DT = D / 32;
    constexpr int SL = BC / 16;
    constexpr int CPR = D / 8;
    constexpr int CPT = BC * CPR / NT;
    static_assert((BC * CPR) % NT == 0, "tile must divide evenly over the workgroup");
    using E = Elem<Tag>;

    __shared__ __attribute__((aligned(16))) uint16_t lds_k[2][BC * RSTR];
    __shared__ __attribute__((aligned(16))) uint16_t lds_v[2][BC * VSTR];

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;

    const WorkItem item = work_item<CAUSAL>(blockIdx.x, total_wg, n_qtiles);
    const int bh = item.head;
    const int qt = CAUSAL ? n_qtiles - 1 - item.tile : item.tile;  // the last rows see the most keys

    const size_t head_off = (size_t)bh * N * D;
    const size_t kv_off = (size_t)(bh / kv_group) * N * D;  // grouped-query: kv_group query heads per K/V head
    const uint16_t* kh = k + kv_off;
    const uint16_t* vh = v + kv_off;
    const int wave_q0 = qt * BR + wave * 32;
    const int qi = wave_q0 + col;
    const int qrow = min(qi, N - 1);  // rows past N compute a copy of row N-1, never stored
    const float sc = scale * kLog2e;

    i32x4 qreg[KS], doreg[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        qreg[ks] = *reinterpret_cast<const i32x4*>(q + head_off + (size_t)qrow * D + ks * 16 + half * 8);
        doreg[ks] = *reinterpret_cast<const i32x4*>(dout + head_off + (size_t)qrow * D + ks * 16 + half * 8);
    }
    const float l2 = lse[(size_t)bh * N + qrow] * kLog2e;
    // D = rowsum(dO o O): the two lanes of a row hold its dO between them, so O is read in the same pieces.  The
    // dK/dV pass, launched after this one, reads D from the workspace.  o == nullptr: D is there already.
    float dq_row = 0.f;
    if (o) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            dq_row = dot8<Tag>(*reinterpret_cast<const i32x4*>(o + head_off + (size_t)qrow * D + ks * 16 + half * 8), doreg[ks], dq_row);
        }
        dq_row = sum_both_halves(dq_row);
        if (half == 0 && qi < N) dvec[(size_t)bh * N + qi] = dq_row;
    } else {
        dq_row = dvec[(size_t)bh * N + qrow];
    }
    constexpr bool NEG_D_START = D == 64;
    f32x16 negd;
#pragma unroll
    for (int r = 0; r < 16; ++r) negd[r] = -dq_row;

    f32x16 acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[dt][r] = 0.f;

    int last_q = min(qt * BR + BR, N) - 1;
    int n_blocks = CAUSAL ? (last_q / BC + 1) : ((N + BC - 1) / BC);

    const __amdgpu_buffer_rsrc_t k_rsrc = make_buffer(kh, (uint32_t)N * D * 2);
    const __amdgpu_buffer_rsrc_t v_rsrc = make_buffer(vh, (uint32_t)N * D * 2);
    i32x4 kpre[CPT], vpre[CPT];
    auto load_tile = [&](int key0) {
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            kpre[i] = buffer_load_16B(k_rsrc, key0 * D * 2 + (tid + i * NT) * 16);
            vpre[i] = buffer_load_16B(v_rsrc, key0 * D * 2 + (tid + i * NT) * 16);
        }
    };
    auto store_tile = [&](int st) {
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            int c = tid + i * NT;
            int row = c / CPR, cc = c % CPR;
            *reinterpret_cast<i32x4*>(lds_k[st] + row * RSTR + cc * 8) = kpre[i];
            *reinterpret_cast<i32x4*>(lds_v[st] + row * VSTR + cc * 8) = vpre[i];
        }
    };
    load_tile(0);
    store_tile(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]), "+v"(doreg[ks]));  // loads done before the loop
    __syncthreads();

    const int tr_row = (lane & 15) >> 2;
    const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);

    for (int t = 0; t < n_blocks; ++t) {
        const int st = t & 1;
        const int key0 = t * BC;
        const bool more = (t + 1 < n_blocks);
        // a wave whose queries all precede this block has nothing to add (causal)
        const bool wave_active = !CAUSAL || key0 <= wave_q0 + 31;
        if (more) load_tile(key0 + BC);

        if (wave_active) {
            // ---- S^T = K_j Q_i^T and dP^T = V_j dO_i^T
            f32x16 sacc[KT], pacc[KT];
            const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            const int kbase = col * RSTR + half * 8, vbase = col * VSTR + half * 8;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) {
                    i32x4 ak = *reinterpret_cast<const i32x4*>(lds_k[st] + kbase + kt * 32 * RSTR + ks * 16);
                    i32x4 av = *reinterpret_cast<const i32x4*>(lds_v[st] + vbase + kt * 32 * VSTR + ks * 16);
                    sacc[kt] = E::mma(ak, qreg[ks], ks == 0 ? zero : sacc[kt]);
                    // where registers allow, dP starts from -D (a lane owns one query, so D is one value per
                    // lane, kept as a 16-register constant): dP - D comes out of the MFMAs
                    pacc[kt] = E::mma(av, doreg[ks], ks == 0 ? (NEG_D_START ? negd : zero) : pacc[kt]);
                }

            // ---- P = exp(S - L), dS = P o (dP - D), packed as the B operand of the dQ product
            // keys past N, and keys after the query when causal, get S = -inf (P = 0): one uniform branch per
            // block, not a select per element in every block
            const bool need_mask = (key0 + BC > N) || (CAUSAL && key0 + BC - 1 > wave_q0);
            const int limit = CAUSAL ? min(qi, N - 1) : N - 1;  // last visible key
            if (need_mask) {
                // compile-time key offsets against one per-lane bound (kept opaque: the compiler otherwise
                // hoists 32 per-element key indices out of the block loop into registers of their own)
                int bound = limit - key0 - 4 * half;
                asm volatile("" : "+v"(bound));
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (kt * 32 + 8 * (r >> 2) + (r & 3) > bound) sacc[kt][r] = -INFINITY;
            }
            i32x4 dsb[SL];
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                float ds[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float p = fast_exp2(__builtin_fmaf(sacc[kt][r], sc, -l2));
                    ds[r] = NEG_D_START ? p * pacc[kt][r] : p * (pacc[kt][r] - dq_row);
                }
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    i32x4 w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[e] = E::pack2(ds[8 * s2 + 2 * e], ds[8 * s2 + 2 * e + 1]);
                    dsb[2 * kt + s2] = w;
                }
            }

            // ---- dQ_i^T += K_j^T dS^T
            const uint16_t* kt_base = lds_k[st] + (4 * half + tr_row) * RSTR + tr_col;
#pragma unroll
            for (int sl = 0; sl < SL; ++sl)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const uint16_t* p0 = kt_base + (sl * 16) * RSTR + dt * 32;
                    i32x2 lo = lds_read_tr16(p0);
                    i32x2 hi = lds_read_tr16(p0 + 8 * RSTR);
                    i32x4 a = {lo[0], lo[1], hi[0], hi[1]};
                    acc[dt] = E::mma(a, dsb[sl], acc[dt]);
                }
        }

        if (more) store_tile(st ^ 1);
        __syncthreads();
    }

    // dQ_i = scale * acc.  Every LDS read of the loop was followed by a barrier, so the K and V
    // buffers are free: each wave takes 4 KiB of them to transpose its tile into whole 128-byte lines.
    static_assert(sizeof(lds_k) >= NW / 2 * 4096 && sizeof(lds_v) >= NW / 2 * 4096, "patches must fit");
    char* patch = (wave < NW / 2 ? reinterpret_cast<char*>(&lds_k[0][0]) : reinterpret_cast<char*>(&lds_v[0][0])) +
                  (wave % (NW / 2)) * 4096;
    store_rows_via_lds<Tag, DT>(acc, scale, patch, make_buffer(dq + head_off, (uint32_t)N * D * 2), wave_q0, lane);
}

// ---------------------------------------------------------------------------------------
// dQ pass at head dimension 256: four waves, one per SIMD (the 128-register accumulator and the Q, dO operands fill the
// register file), so only the wave's own instruction stream can keep its matrix pipe busy.  Per 64-key block:
//   S^T   32 MFMAs  ||  dP accumulators set to -D, requests of the next block
//   dP^T  32 MFMAs  ||  P = exp2(S c - L), requests of the next block
//   dQ^T  32 MFMAs  ||  dS of the second key tile
// LDS operand reads lead their MFMAs by KP steps, across the phases (read in the step that used them, they cost the
// wave the LDS latency 96 times per block).  S and dP are produced by MfmaVgprAcc into ordinary registers, Q, dO and
// dQ live in the accumulation half; every step ends in a full scheduling barrier, so the order written here is what runs.
// bf16, whole backward, us, before / so: B = 2, H = 8, N = 8192 3858 / 3452 (this pass 1834 / ~1410, 1.17 PFLOP/s of
// executed MFMAs), causal 2020 / 1809; B = 8, H = 8, N = 2048 causal 650 / 579.  Blocks straight into the LDS instead of through 16
// registers, with 16 loads waited for and 16 LDS stores per wave: 3197 / 3147, 526 / 518.
template <typename Tag, bool CAUSAL>
__global__ void __launch_bounds__(256, 1)
fa_bwd_dq_d256_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                      const uint16_t* __restrict__ o, const uint16_t* __restrict__ dout, const float* __restrict__ lse,
                      float* __restrict__ dvec, uint16_t* __restrict__ dq, int N, int n_qtiles, int total_wg,
                      int kv_group, float scale) {
    [[maybe_unused]] ClockSpan clock_span;  // measurement builds only; empty otherwise
    constexpr int D = 256, BC = 64, BR = 128;
    using Tile = WaveTile<D>;                // the layout of 32 rows in the LDS; a block is two of them
    constexpr int BLOCK_B = 2 * Tile::TILE_B;  // a block of K or V
    constexpr int STAGE_B = 2 * BLOCK_B;     // K, V
    constexpr int KS = D / 16, DT = D / 32;
    constexpr int KP = 4;
    using E = Elem<Tag>;
    __shared__ __attribute__((aligned(1024))) char lds[2 * STAGE_B];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;
    const WorkItem item = work_item<CAUSAL>(blockIdx.x, total_wg, n_qtiles);
    const int bh = item.head;
    const int qt = CAUSAL ? n_qtiles - 1 - item.tile : item.tile;  // the last rows see the most keys

    const size_t head_off = (size_t)bh * N * D;
    const size_t kv_off = (size_t)(bh / kv_group) * N * D;  // grouped-query: kv_group query heads per K/V head
    const int wave_q0 = qt * BR + wave * 32;
    const int qi = wave_q0 + col;
    const int qrow = min(qi, N - 1);  // rows past N compute a copy of row N-1, never stored
    const int limit = CAUSAL ? qrow : N - 1;  // last visible key
    float sc = scale * kLog2e;
    asm volatile("" : "+v"(sc));  // in a vector register: an FMA with a scalar operand issues at a lower rate

    // the next block to be requested (keys past N, and blocks past the last one, read as zero), a quarter by each wave
    BufferWords k_rsrc = make_buffer_words(k + kv_off, (uint32_t)N * D * 2), v_rsrc = make_buffer_words(v + kv_off, (uint32_t)N * D * 2);
    auto next_block = [&]() __attribute__((always_inline)) {
        advance(k_rsrc, BLOCK_B);
        advance(v_rsrc, BLOCK_B);
    };
    // Addresses: row and transposed operands in the stage being read (V, the second 32 keys, 16 keys and columns from 128 on are
    // offsets), and what the lane fetches
    const uint32_t lds_base = lds_address(lds), piece = lds_base + wave * (BLOCK_B / 4);
    uint32_t row_at[KS / 2], tr_at[DT / 2][2];
    int src[8];
#pragma unroll
    for (int ks = 0; ks < KS / 2; ++ks) {
        row_at[ks] = lds_base + col * Tile::ROWB + (((2 * ks + half) ^ Tile::swizzle(col)) << 4);
        asm volatile("" : "+v"(row_at[ks]));
    }
#pragma unroll
    for (int dt = 0; dt < DT / 2; ++dt)
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            tr_at[dt][hi] = lds_base + Tile::tr_of(dt, hi, lane);
            asm volatile("" : "+v"(tr_at[dt][hi]));
        }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        src[i] = wave * (BLOCK_B / 4) + Tile::src_of(i, lane);
        asm volatile("" : "+v"(src[i]));
    }
#pragma unroll
    for (int n = 0; n < 16; ++n) global_to_lds_16B(n & 1 ? v_rsrc : k_rsrc, piece + (n & 1) * BLOCK_B + (n >> 1) * 1024, src[n >> 1]);
    next_block();

    i32x4 qreg[KS], doreg[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const size_t off = head_off + (size_t)qrow * D + ks * 16 + half * 8;
        qreg[ks] = *reinterpret_cast<const i32x4*>(q + off);
        doreg[ks] = *reinterpret_cast<const i32x4*>(dout + off);
    }
    float d_row = 0.f;  // D = rowsum(dO o O), or (o == nullptr) from the workspace
    if (o) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            d_row = dot8<Tag>(*reinterpret_cast<const i32x4*>(o + head_off + (size_t)qrow * D + ks * 16 + half * 8), doreg[ks], d_row);
        d_row = sum_both_halves(d_row);
        if (half == 0 && qi < N) dvec[(size_t)bh * N + qi] = d_row;
    } else {
        d_row = dvec[(size_t)bh * N + qrow];
    }
    const float l2 = lse[(size_t)bh * N + qrow] * kLog2e;
    f32x16 acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[dt][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qreg[ks]), "+a"(doreg[ks]));
    auto landed = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    landed();

    int st = 0;
    auto block = [&](int t, auto mask_tag) __attribute__((always_inline)) {
        constexpr bool MASK = decltype(mask_tag)::value;
        const uint32_t next = piece + (st ^ 1) * STAGE_B;
        int bound = limit - t * BC - 4 * half;  // last visible key of the lane's half of a tile
        asm volatile("" : "+v"(bound));
        // step u of the two score products: (tensor, 16 columns, 32-key tile), the two tiles' chains alternating
        auto row_read = [&](int u) __attribute__((always_inline)) {
            const int ks = (u % (2 * KS)) / 2, kt = u & 1;
            return lds_load_16B(row_at[ks % (KS / 2)] + (u < 2 * KS ? 0 : BLOCK_B) + kt * Tile::TILE_B + (ks / (KS / 2)) * 256);
        };
        auto tr_read = [&](int w) __attribute__((always_inline)) {  // step w of the dQ product: (16 keys, 32 columns)
            const int dt = w % DT, off = (w / DT) * 16 * Tile::ROWB + (dt / (DT / 2)) * 256;
            const i32x2 lo = lds_read_tr16(tr_at[dt % (DT / 2)][0] + off), hi = lds_read_tr16(tr_at[dt % (DT / 2)][1] + off);
            return i32x4{lo[0], lo[1], hi[0], hi[1]};
        };
        f32x16 sacc[2], pacc[2];
        i32x4 ring[KP], tr[KP], dsb[4];
#pragma unroll
        for (int u = 0; u < KP; ++u) ring[u] = row_read(u);
        __builtin_amdgcn_sched_barrier(0);
        static_for<4 * KS>([&](auto step) __attribute__((always_inline)) {
            constexpr int u = decltype(step)::value, ks = (u % (2 * KS)) / 2, kt = u & 1;
            constexpr int n_req = u / 4, to = (n_req & 1) * BLOCK_B + (n_req >> 1) * 1024;  // 16 requests, one every fourth step
            const i32x4 a = ring[u % KP];
            if constexpr (u + KP < 4 * KS) ring[u % KP] = row_read(u + KP);
            else tr[u + KP - 4 * KS] = tr_read(u + KP - 4 * KS);
            f32x16& c = u < 2 * KS ? sacc[kt] : pacc[kt];
            const i32x4& b = u < 2 * KS ? qreg[ks] : doreg[ks];
            const BufferWords& rsrc = n_req & 1 ? v_rsrc : k_rsrc;
            using M = MfmaVgprAcc<Tag>;
            if constexpr (u == 0) M::template first_and_load<to>(c, a, b, rsrc, next, src[n_req >> 1]);
            else if constexpr (u == 1) M::first(c, a, b);
            else if constexpr (u == 2 * KS) M::template start_and_load<to>(c, a, b, rsrc, next, src[n_req >> 1]);
            else if constexpr (u == 2 * KS + 1) M::start(c, a, b);
            else if constexpr (u % 4 == 0) M::template run_and_load<to>(c, a, b, rsrc, next, src[n_req >> 1]);
            else M::run(c, a, b);
            if (u < 16) pacc[0][u] = pacc[1][u] = -d_row;  // dP - D comes out of the MFMAs
            if (u == 2 * KS) mfma_result_wait(sacc[0], sacc[1]);
            if (u >= 2 * KS) {
                const int n = u - 2 * KS, i = n >> 4, r = n & 15;
                float x = fast_exp2(__builtin_fmaf(sacc[i][r], sc, -l2));
                if constexpr (MASK) x = i * 32 + 8 * (r >> 2) + (r & 3) > bound ? 0.f : x;
                sacc[i][r] = x;
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        next_block();
        mfma_result_wait(pacc[0], pacc[1]);
        auto gradient = [&](int i, int r) __attribute__((always_inline)) {  // a pair of scores becomes a register of dS
            dsb[2 * i + (r >> 3)][(r >> 1) & 3] = E::pack2(sacc[i][r] * pacc[i][r], sacc[i][r + 1] * pacc[i][r + 1]);
        };
#pragma unroll
        for (int r = 0; r < 16; r += 2) gradient(0, r);
#pragma unroll
        for (int w = 0; w < 4 * DT; ++w) {
            const i32x4 a = tr[w % KP];
            if (w + KP < 4 * DT) tr[w % KP] = tr_read(w + KP);
            acc[w % DT] = E::mma(a, dsb[w / DT], acc[w % DT]);
            if (w < 16 && !(w & 1)) gradient(1, w);
            __builtin_amdgcn_sched_barrier(0);
        }
        landed();
        const int move = st ? -STAGE_B : STAGE_B;
#pragma unroll
        for (int ks = 0; ks < KS / 2; ++ks) row_at[ks] += move;
#pragma unroll
        for (int dt = 0; dt < DT / 2; ++dt) {
            tr_at[dt][0] += move;
            tr_at[dt][1] += move;
        }
        st ^= 1;
    };
    const int last_q = min(qt * BR + BR, N) - 1;
    const int n_blocks = CAUSAL ? last_q / BC + 1 : (N + BC - 1) / BC;
    // blocks that need no mask: all their keys exist and (causal) precede every row of the workgroup
    const int n_plain = min(n_blocks, CAUSAL ? min(qt * BR + 1, N) / BC : N / BC);
    int t = 0;
    for (; t < n_plain; ++t) block(t, std::false_type{});
    for (; t < n_blocks; ++t) block(t, std::true_type{});

    // dQ_i = scale * acc, transposed into whole 128-byte lines through the stages (every read and write of them is behind the last
    // barrier)
    store_rows_via_lds<Tag, DT>(acc, scale, lds + wave * 4096, make_buffer(dq + head_off, (uint32_t)N * D * 2), wave_q0, lane);
}

// ---------------------------------------------------------------------------------------
size_t bwd_workspace_bytes(int B, int H, int N, int d) {
    (void)d;
    size_t rows = (size_t)B * H * N;
    return (rows * sizeof(float) + 15) & ~(size_t)15;  // D = rowsum(dO o O)
}

// Whether two runs of bytes share memory.
inline bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + b_bytes && y < x + a_bytes;
}

template <typename Tag, int D>
static int launch_bwd_t(const void* q, const void* k, const void* v, const void* o, const float* lse,
                        const void* dout, void* dq, void* dk, void* dv, void* workspace, int B, int H, int H_kv,
                        int N, float scale, int causal, hipStream_t stream) {
    float* dvec = static_cast<float*>(workspace);
    auto u16 = [](const void* p) { return static_cast<const uint16_t*>(p); };
    // every size check comes before the first launch: a call that fails has enqueued nothing
    constexpr int kKeys = D == 256 ? 64 : 128;  // keys per workgroup of the dK/dV pass
    const int n_kblocks = (N + kKeys - 1) / kKeys;
    const long total = (long)B * H_kv * n_kblocks;
    constexpr int kRows = D == 256 ? 128 : 256;  // queries per workgroup of the dQ pass (d = 256: a wave needs a SIMD to itself)
    const long total_q = (long)B * H * ((N + kRows - 1) / kRows);
    if (total > 0x7fffffffL || total_q > 0x7fffffffL) return FA_ERR_SHAPE;

    // Two launches, the dQ pass first: it also writes D, which the dK/dV pass reads.  Or both passes in one, in their
    // few-workgroup forms, behind a launch for D or not.
    auto dqp = [&](auto kernel, int rows, bool d_ready) {  // `rows`: queries, and threads / 2, of a workgroup
        const int tiles = (N + rows - 1) / rows, items = B * H * tiles;
        hipLaunchKernelGGL(kernel, dim3((unsigned)items), dim3(rows * 2), 0, stream, u16(q), u16(k), u16(v),
                           d_ready ? nullptr : u16(o), u16(dout), lse, dvec, static_cast<uint16_t*>(dq), N, tiles, items,
                           H / H_kv, scale);
    };
    // workgroups of 32 or 128 queries / of 32 keys, when a pass is to use them
    const BwdForm form = D > 128 ? kBwdLarge : choose_bwd_form((long)B * H, (long)B * H_kv, N, D, causal);
    const bool one_launch = form == kBwdOne32 || form == kBwdOneRows;
    const int dq_form = form == kBwdOneRows ? kDqRows | (bwd_rows_first(H / H_kv, causal) ? kDqFirst : 0) : 0;
    const int few_rows = dq_form & kDqRows ? 128 : 32;
    const long dq_few = one_launch ? (long)B * H * ((N + few_rows - 1) / few_rows) : 0;
    const long dkdv_few = form != kBwdLarge ? (long)B * H_kv * ((N + 31) / 32) : 0;
    auto few = [&](long n_dkdv, long n_dq, bool d_ready) {
        if constexpr (D <= 128) {
            auto run = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3((unsigned)(n_dkdv + n_dq)), dim3(256), 0, stream, u16(q), u16(k), u16(v),
                                   u16(o), u16(dout), lse, dvec, static_cast<uint16_t*>(dq),
                                   static_cast<uint16_t*>(dk), static_cast<uint16_t*>(dv), N, (int)n_dkdv, dq_form, B * H, H / H_kv, scale);
            };
            if (d_ready) causal ? run(fa_bwd_few_kernel<Tag, D, true, true>) : run(fa_bwd_few_kernel<Tag, D, false, true>);
            else causal ? run(fa_bwd_few_kernel<Tag, D, true, false>) : run(fa_bwd_few_kernel<Tag, D, false, false>);
        }
    };
    auto row_sums = [&]() {
        const long rows = (long)B * H * N;
        constexpr int kRowsPerWg = 256 / (D / 8);
        hipLaunchKernelGGL((fa_bwd_rowsum_kernel<Tag, D>), dim3((unsigned)((rows + kRowsPerWg - 1) / kRowsPerWg)), dim3(256), 0,
                           stream, u16(o), u16(dout), dvec, rows);
        return hipGetLastError() == hipSuccess;
    };
    auto dq_pass = [&](bool d_ready) {
        if constexpr (D == 256) {
            causal ? dqp(fa_bwd_dq_d256_kernel<Tag, true>, 128, d_ready) : dqp(fa_bwd_dq_d256_kernel<Tag, false>, 128, d_ready);
        } else if (dq_few) {
            few(0, dq_few, d_ready);
        } else if (N <= bwd_short_rows(D, causal)) {
            causal ? dqp(fa_bwd_dq_kernel<Tag, D, 32, 4, true>, 128, d_ready) : dqp(fa_bwd_dq_kernel<Tag, D, 32, 4, false>, 128, d_ready);
        } else {
            causal ? dqp(fa_bwd_dq_kernel<Tag, D, 64, 8, true>, 256, d_ready) : dqp(fa_bwd_dq_kernel<Tag, D, 64, 8, false>, 256, d_ready);
        }
        return hipGetLastError() == hipSuccess;
    };
    auto dkdv = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)total), dim3(256), 0, stream, u16(q), u16(k), u16(v), u16(dout), lse,
                           dvec, static_cast<uint16_t*>(dk), static_cast<uint16_t*>(dv), N, n_kblocks, (int)total,
                           H / H_kv, scale);
    };
    auto dkdv_pass = [&]() {
        if (dkdv_few) few(dkdv_few, 0, true);
        else if constexpr (D == 64) causal ? dkdv(fa_bwd_dkdv_kernel<Tag, D, true>) : dkdv(fa_bwd_dkdv_kernel<Tag, D, false>);
        else causal ? dkdv(fa_bwd_dkdv_shared_kernel<Tag, D, true>) : dkdv(fa_bwd_dkdv_shared_kernel<Tag, D, false>);
        return hipGetLastError() == hipSuccess;
    };

    // A gradient may be written over O, wholly or in part: D is then computed in full before anything is written
    const size_t q_bytes = (size_t)B * H * N * D * 2, kv_bytes = (size_t)B * H_kv * N * D * 2;
    const bool over_o = overlap(dq, q_bytes, o, q_bytes) || overlap(dk, kv_bytes, o, q_bytes) || overlap(dv, kv_bytes, o, q_bytes);
    bool ok;
    if (overlap(dq, q_bytes, q, q_bytes) || overlap(dq, q_bytes, dout, q_bytes)) {
        // dQ written over Q or dO: a workgroup of the dQ pass reads these at its own rows before it writes them, but
        // the dK/dV pass reads all of them and has to come first.  (dK or dV may be over O then: D is not computed again.)
        ok = row_sums() && dkdv_pass() && dq_pass(true);
    } else if (one_launch) {
        const bool own = !over_o && bwd_own_row_sums((long)B * H, (long)B * H_kv, N, D);
        ok = own || row_sums();
        if (ok) {
            few(dkdv_few, dq_few, !own);
            ok = hipGetLastError() == hipSuccess;
        }
    } else {
        ok = (!over_o || row_sums()) && dq_pass(over_o) && dkdv_pass();
    }
    return ok ? FA_OK : FA_ERR_LAUNCH;
}

int launch_bwd(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dout,
               void* dq, void* dk, void* dv, void* workspace, int B, int H, int H_kv, int N, int d, float scale,
               int causal, int dtype, hipStream_t stream) {
#define FA_BWD_CASE(TAG, DD) \
    return launch_bwd_t<TAG, DD>(q, k, v, o, lse, dout, dq, dk, dv, workspace, B, H, H_kv, N, scale, causal, stream)
    if (dtype == FA_BF16 && d == 128) FA_BWD_CASE(bf16_tag, 128);
    if (dtype == FA_BF16 && d == 64) FA_BWD_CASE(bf16_tag, 64);
    if (dtype == FA_F16 && d == 128) FA_BWD_CASE(f16_tag, 128);
    if (dtype == FA_F16 && d == 64) FA_BWD_CASE(f16_tag, 64);
    if (dtype == FA_BF16 && d == 256) FA_BWD_CASE(bf16_tag, 256);
    if (dtype == FA_F16 && d == 256) FA_BWD_CASE(f16_tag, 256);
#undef FA_BWD_CASE
    return FA_ERR_UNSUPPORTED;
}

}  // namespace fa

FA_CLOCK_SPAN_READER(fa_debug_clock_span_bwd)
