// Forward attention kernels for gfx950: 16-bit (bf16 / fp16) MFMA path and the fp32 path.
//
// One workgroup owns a tile of BR = NW * 32 * RQ query rows of one (batch, head) and walks
// the key/value blocks of that head (paper Algorithm 1: T_r query tiles on the grid, T_c
// key blocks in the inner loop).  Per block: S^T = K_j Q_i^T on MFMA, online softmax with
// running row maximum m and row sum l, O^T += V_j^T P^T on MFMA, O rescaled by
// exp(m_old - m_new); epilogue O / l and L = m + log l.  K_j and V_j are staged in the LDS, the next block's while the
// current one is being computed (the role the producer warpgroup plays in the paper).
#include <type_traits>

#include "fa_device.h"
#include "fa_launch.h"

// Measurement builds only (paper_2407_08608_amd/ablate.py compiles this file with it; the library never defines
// it): FA_ABLATE_PP removes one part of fa_fwd_pingpong_kernel's block to see what the rest costs -- results
// wrong on purpose: 1 = no exponentials, 2 = no LDS reads of V operands, 3 = no LDS reads of K operands,
// 4 = no softmax arithmetic at all (P~ = packed scores).
#ifndef FA_ABLATE_PP
#define FA_ABLATE_PP 0
#endif

namespace fa {

constexpr float kLazyLog2 = 8.0f;
// fa_fwd_pingpong_kernel: a block whose per-lane sum of P~ exceeds this moves the row's reference (2^14:
// every P~ of a block that stays below it fits fp16 with room to spare)
constexpr float kRaiseAbove = 16384.0f;

// ---------------------------------------------------------------------------------------
// The forward where its query tiles would leave most of the chip idle (few heads, short sequences): FewForward.
//
// A workgroup owns 32 queries instead of 128 or 256 and its NW waves split the keys, tiles of 32 dealt in turn, each with
// a softmax state and an output accumulator for all columns; the states meet in the LDS at the end, in a fixed order:
// with M the largest of their references and f = exp(m - M), O = sum f O / sum f l and L = M + log sum f l.  Four to
// eight times as many workgroups, each with a quarter to an eighth of the serial chain.  A wave stages its own tiles
// (WaveTile), so the loop has no barrier; what that costs is traffic (K and V come to a CU once per 32 queries), which a
// chip that is mostly idle has to spare.  V of a tile is requested beside its score MFMAs, K of the wave's next tile beside
// its products, each into the one stage that its last reader has left: a second stage per tensor gains nothing with one
// workgroup on a CU and costs the second workgroup (d = 128 causal, 32 heads x 512: 12.8 us with two stages, 10.0 with one).
template <int D, int NW>
struct FewForward {
    using Tile = WaveTile<D>;
    static constexpr int KS = D / 16, DT = D / 32, KP = 4;
    static constexpr int kStages = NW * 2 * Tile::TILE_B;
    static constexpr int kLds = KeySplitMerge<D, NW>::kLds > kStages ? KeySplitMerge<D, NW>::kLds : kStages;

    template <typename Tag, bool CAUSAL>
    static __device__ __forceinline__ void run(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                               const uint16_t* __restrict__ v, uint16_t* __restrict__ o,
                                               float* __restrict__ lse, int N, int split, int kv_group, float scale, char* lds) {
        using E = Elem<Tag>;
        const int tid = threadIdx.x;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
        const int col = lane & 31, half = lane >> 5;
        const KeySplitTile item = key_split_tile(N, split);
        if (item.tile >= item.n_tiles) return;
        const int bh = item.head, n_t = item.n_tiles, tile_no = item.tile;
        const int qt = CAUSAL ? n_t - 1 - tile_no : tile_no;
        const int q0 = qt * 32, n_tiles = CAUSAL ? qt + 1 : n_t;
        const int row = min(q0 + col, N - 1);    // rows past N compute a copy of row N-1, never stored
        const int limit = CAUSAL ? row : N - 1;  // last visible key
        const size_t head_off = (size_t)bh * N * D, kv_off = (size_t)(bh / kv_group) * N * D;
        const Tile tile(lds_address(lds) + wave * (2 * Tile::TILE_B), lane);
        constexpr int kK = 0, kV = Tile::TILE_B;  // the two tiles
        // the wave's next tiles (rows past N read as zero)
        BufferWords k_rsrc = make_buffer_words(k + kv_off, (uint32_t)N * D * 2), v_rsrc = make_buffer_words(v + kv_off, (uint32_t)N * D * 2);
        advance(k_rsrc, wave * Tile::TILE_B);
        advance(v_rsrc, wave * Tile::TILE_B);

        // (a wave without a tile brings rows that nothing reads, or zeros)
#pragma unroll
        for (int i = 0; i < Tile::NI; ++i) tile.request(k_rsrc, kK, i);
        i32x4 qreg[KS];  // Q^T as the B operand
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            qreg[ks] = *reinterpret_cast<const i32x4*>(q + head_off + (size_t)row * D + ks * 16 + half * 8);
        f32x16 acc[DT];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[dt][r] = 0.f;
        float m_run = -INFINITY, l_run = 0.f;  // reference (raw scores) and this half's row sum of P~
        const float sc = scale * kLog2e;
        float sc_v = sc;  // a vector-register copy: an FMA with a scalar-register operand issues at a lower rate
        asm volatile("" : "+v"(sc_v));
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));

        for (int t = wave; t < n_tiles; t += NW) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // K has landed
            advance(k_rsrc, NW * Tile::TILE_B);
            if (t + NW >= n_tiles) k_rsrc.w[2] = 0;  // past the wave's last tile: zeros that nothing reads
            i32x4 ring[KP], tr[KP];
#pragma unroll
            for (int u = 0; u < KP; ++u) ring[u] = tile.row_read(kK, u);
            __builtin_amdgcn_sched_barrier(0);
            // S^T = K Q^T
            f32x16 s = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < KS; ++u) {
                const i32x4 a = ring[u % KP];
                if (u + KP < KS) ring[u % KP] = tile.row_read(kK, u + KP);
                tile.request(v_rsrc, kV, u);
                s = E::mma(a, qreg[u], s);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (t * 32 + 32 > N || (CAUSAL && t == qt)) {
                int bound = limit - t * 32 - 4 * half;  // key 8 (r / 4) + r % 4 of the lane's half is visible up to here
                asm volatile("" : "+v"(bound));
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (8 * (r >> 2) + (r & 3) > bound) s[r] = -INFINITY;
            }
            // the reference is the first tile's row maximum and rises when a tile's exceeds it by more than 2^kLazyLog2
            float mx[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
            for (int r = 0; r < 16; ++r) mx[r & 3] = fmaxf(mx[r & 3], s[r]);
            const float m_new = max_both_halves(fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3])));
            const bool raise = (m_new - m_run) * sc > kLazyLog2;
            if (__builtin_amdgcn_ballot_w64(raise) != 0) {
                const float corr = raise ? fast_exp2((m_run - m_new) * sc) : 1.0f;
                m_run = raise ? m_new : m_run;
                l_run *= corr;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    if constexpr (D == 256) asm volatile("" : "+a"(acc[dt]));  // (copied out of the accumulation half here, not in every tile)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[dt][r] *= corr;
                    if constexpr (D == 256) asm volatile("" : "+a"(acc[dt]));
                }
            }
            const float mb = m_run == -INFINITY ? 0.f : m_run * sc;  // a row of scores of -inf so far: P = 0
            float ps[4];
            i32x4 pb[2];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                s[r] = fast_exp2(__builtin_fmaf(s[r], sc_v, -mb));
                ps[r & 3] = r < 4 ? s[r] : ps[r & 3] + s[r];
                if (r & 1) pb[r >> 3][(r >> 1) & 3] = E::pack2(s[r - 1], s[r]);
            }
            l_run += (ps[0] + ps[1]) + (ps[2] + ps[3]);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // V has landed
            advance(v_rsrc, NW * Tile::TILE_B);
#pragma unroll
            for (int u = 0; u < KP; ++u) tr[u] = tile.tr_read(kV, u / DT, u % DT);
            __builtin_amdgcn_sched_barrier(0);
            // O^T += V^T P^T
#pragma unroll
            for (int u = 0; u < 2 * DT; ++u) {
                const i32x4 a = tr[u % KP];
                if (u + KP < 2 * DT) tr[u % KP] = tile.tr_read(kV, (u + KP) / DT, (u + KP) % DT);
                tile.request(k_rsrc, kK, u);
                acc[u % DT] = E::mma(a, pb[u / DT], acc[u % DT]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the last requests: the LDS is about to be reused

        KeySplitMerge<D, NW>::template run<Tag, NW * 64>(acc, m_run * sc, l_run, 0.f, lds, wave, lane, o + head_off, lse + (size_t)bh * N, q0, N);
    }
};

// (not in the eight-wave tile at d = 128, which only a forced schedule takes)
template <int D, int NW>
constexpr bool kHasFew = D == 64 || NW == 4;

// The lane, counted anew: a register less over a loop that has none to spare, for what comes before and after it.
static __device__ __forceinline__ int lane_again() {
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(lane));
    return lane;
}

// The K and V tiles of fa_fwd_16bit_kernel, BC rows each, brought by all its waves from global memory straight into the LDS:
// no staging registers and no LDS writes.  They are laid out as a WaveTile is.  Row and column operands differ from one
// another by a bit pattern in the chunk number alone, so a lane keeps one address per tensor and the rest is an exclusive or.
// Two stages for K; two for V where they cost no workgroup on the CU, else one: at d = 128 and four waves 48 KiB instead of
// 64, three workgroups on a CU (and three waves' worth of registers) instead of two.
template <int D, int BC, int NW>
struct SharedTiles {
    static constexpr int ROWB = D * 2, CPR = D / 8, RPI = 1024 / ROWB;  // (as in WaveTile)
    static constexpr int TILE_B = BC * ROWB;
    static constexpr int NI = TILE_B / 1024 / NW;           // staging instructions of a wave for a tile
    static constexpr int VS = D == 128 && NW == 4 ? 1 : 2;  // stages of V
    static constexpr int kV = 2 * TILE_B, kLds = (2 + VS) * TILE_B;
    uint32_t mine;       // LDS address of what this wave brings of a tile at the start
    int src[NI];         // byte offset within a tile for each staging instruction
    uint32_t row0, tr0;  // this stage's operands: K row `col`, elements 8 half...; V rows 4 half + tr_row, transposed

    __device__ __forceinline__ SharedTiles(uint32_t at, int wave, int lane) : mine(at + wave * (NI * 1024)) {
        const int col = lane & 31, half = lane >> 5, tr_row = (lane & 15) >> 2, quad = lane & 3, blk = (lane >> 4) & 1;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int r = (wave * NI + i) * RPI + lane / CPR;
            src[i] = r * ROWB + ((lane % CPR) ^ WaveTile<D>::swizzle(r)) * 16;
            asm volatile("" : "+v"(src[i]));
        }
        row0 = at + col * ROWB + ((half ^ WaveTile<D>::swizzle(col)) << 4);
        const int r = 4 * half + tr_row;
        tr0 = at + kV + r * ROWB + (((2 * blk + (quad >> 1)) ^ WaveTile<D>::swizzle(r)) << 4) + 8 * (quad & 1);
        asm volatile("" : "+v"(row0), "+v"(tr0));
    }
    // Instruction i of the wave's NI that bring the tile at the resource's start to `offset` (rows past its end: zeros).
    __device__ __forceinline__ void request(const BufferWords& rsrc, uint32_t offset, int i) const {
        global_to_lds_16B<D == 128 && NW == 8>(rsrc, mine + offset + i * 1024, src[i]);
    }
    __device__ __forceinline__ void other_stage(int step) {
        row0 += step;
        if constexpr (VS == 2) tr0 += step;
        asm volatile("" : "+v"(row0), "+v"(tr0));
    }
    __device__ __forceinline__ i32x4 row_read(int kt, int ks) const { return lds_load_16B((row0 ^ (ks << 5)) + kt * 32 * ROWB); }
    __device__ __forceinline__ i32x4 tr_read(int slab, int dt) const {
        const uint32_t a = tr0 ^ (dt << 6);
        const i32x2 lo = lds_read_tr16(a + slab * 16 * ROWB), hi = lds_read_tr16((a ^ 32) + (slab * 16 + 8) * ROWB);
        return i32x4{lo[0], lo[1], hi[0], hi[1]};
    }
};

// The query tiles of a workgroup, its keys walked by all waves together.
template <typename Tag, int D, int BC, int NW, int RQ, int PD, bool CAUSAL>
static __device__ __forceinline__ void shared_tiles_forward(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                            const uint16_t* __restrict__ v, uint16_t* __restrict__ o,
                                                            float* __restrict__ lse, int N, int n_qtiles, int total_wg, int paired,
                                                            int kv_group, float scale, char* lds) {
    constexpr int BR = NW * 32 * RQ;
    constexpr int KT = BC / 32;   // 32-key score tiles per block
    constexpr int KS = D / 16;    // MFMA steps along the head dimension
    constexpr int DT = D / 32;    // 32-column output tiles
    constexpr int SL = BC / 16;   // 16-key MFMA steps along the keys
    using E = Elem<Tag>;
    using Tiles = SharedTiles<D, BC, NW>;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;

    const TileRun run = query_tiles<CAUSAL, NW == 4>(total_wg, n_qtiles, paired);
    const int bh = run.head;

    const size_t head_off = (size_t)bh * N * D;
    const size_t kv_off = (size_t)(bh / kv_group) * N * D;  // grouped-query: kv_group query heads per K/V head
    const uint16_t* qh = q + head_off;
    const uint16_t* kh = k + kv_off;
    const uint16_t* vh = v + kv_off;

    const float sc = scale * kLog2e;  // exp(scale*s - scale*m) = exp2(sc*s - sc*m)
    float sc_v = sc;  // a vector-register copy: an FMA with a scalar-register operand issues at a lower rate
    asm volatile("" : "+v"(sc_v));
    Tiles tiles(lds_address(lds), wave, lane);
    int step = Tiles::TILE_B;  // from the stage being read to the other one
    // Where a wave issues its requests: beside the score MFMAs at d = 128 (in a burst it sits about 100 cycles in each: 48 heads
    // x 512 16.9 us, so 15.5), at once at d = 64, which has fewer of them and gains from the compiler's order of the operand
    // reads, that requests between them would pin (causal 160 x 2048 104 us at once, 107 between).
    constexpr bool kSpread = D == 128;
    // all but the last `n` requests of every wave have arrived, and no wave reads any more what it read before
    auto landed = [&](auto n) __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(decltype(n)::value) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

#pragma nounroll
    for (int pass = 0; pass < run.n_pass(); ++pass) {
    // every LDS read of the previous pass was followed by a barrier
    const int qt = pass == 0 ? run.tile : run.second;
    const int wave_q0 = qt * BR + wave * (32 * RQ);
    const int lane_now = lane_again(), col = lane_now & 31, half = lane_now >> 5;
    BufferWords k_rsrc = make_buffer_words(kh, (uint32_t)N * D * 2), v_rsrc = make_buffer_words(vh, (uint32_t)N * D * 2);
    const int stage0 = step > 0 ? 0 : Tiles::TILE_B;
    // Q ahead of the first tiles, or behind: its loads wait for the requests to be issued.  bf16, us, heads x N, behind / ahead:
    // d = 64 four waves, no mask 296 x 99 6.85 / 6.40, 348 x 116 7.72 / 7.40, 512 x 512 51.5 / 51.7;  causal 296 x 99 7.29 / 7.15
    // but 128 x 512 11.2 / 11.6;  eight waves 24 x 2048 41.5 / 42.1;  d = 128 level
    constexpr bool kQFirst = D == 64 && NW == 4 && !CAUSAL;
    if constexpr (!kQFirst) {
#pragma unroll
        for (int i = 0; i < Tiles::NI; ++i) {
            tiles.request(k_rsrc, stage0, i);
            if constexpr (Tiles::VS == 2) tiles.request(v_rsrc, Tiles::kV + stage0, i);
        }
    }

    // Q_i^T as the B operand, resident in registers for the whole loop
    static_assert(RQ == 1 && PD == 0, "one 32-row slab per wave");
    i32x4 qreg[KS];
    {
        int row = min(wave_q0 + col, N - 1);  // rows past N compute a copy of row N-1, never stored
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            qreg[ks] = *reinterpret_cast<const i32x4*>(qh + (size_t)row * D + ks * 16 + half * 8);
    }
    if constexpr (kQFirst) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < Tiles::NI; ++i) {
            tiles.request(k_rsrc, stage0, i);
            if constexpr (Tiles::VS == 2) tiles.request(v_rsrc, Tiles::kV + stage0, i);
        }
    }

    f32x16 oacc[DT];
    float m_run = 0.f, l_run = 0.f;  // reference (log2 units of the scaled scores; set by block 0) and row sum of P~
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;

    // key blocks this workgroup must visit
    int last_q = min(qt * BR + BR, N) - 1;
    int n_blocks = CAUSAL ? (last_q / BC + 1) : ((N + BC - 1) / BC);

    // (pins the Q loads' completion here: the compiler's waits for them would otherwise sit inside the loop)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));
    landed(std::integral_constant<int, 0>{});

    for (int t = 0; t < n_blocks; ++t) {
        const int key0 = t * BC;
        const bool more = (t + 1 < n_blocks);
        // K of the next block, and V of the next block or, where it has one stage, of this one; V goes first
        advance(k_rsrc, Tiles::TILE_B);
        if (!more) k_rsrc.w[2] = 0;  // past the last block: zeros that nothing reads
        if constexpr (Tiles::VS == 2) {
            advance(v_rsrc, Tiles::TILE_B);
            if (!more) v_rsrc.w[2] = 0;
        }
        const int k_to = step > 0 ? Tiles::TILE_B : 0, v_to = Tiles::kV + (Tiles::VS == 2 ? k_to : 0);
        auto request = [&](int i) __attribute__((always_inline)) {
            if (i < Tiles::NI) tiles.request(v_rsrc, v_to, i);
            else if (i < 2 * Tiles::NI) tiles.request(k_rsrc, k_to, i - Tiles::NI);
        };

        // a wave whose queries all precede this block has nothing to add (causal)
        const bool wave_active = !CAUSAL || key0 <= wave_q0 + 32 * RQ - 1;
        // (opaque: as the other arm of the branch below, this makes the accumulators change registers in every block)
        int all_now = __builtin_amdgcn_readfirstlane(kSpread && wave_active ? 0 : 1);
        asm volatile("" : "+s"(all_now));
        if (!kSpread || (CAUSAL && all_now != 0))
#pragma unroll
            for (int i = 0; i < 2 * Tiles::NI; ++i) request(i);
        i32x4 pb[SL];
        if (wave_active) {
            // ---- GEMM0: S^T = K_j Q_i^T, then the mask: keys past N, and keys after the query when causal
            f32x16 sacc[KT];
            const bool need_mask = (key0 + BC > N) || (CAUSAL && key0 + BC - 1 > wave_q0);
            auto scores = [&](auto first) __attribute__((always_inline)) {
                const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                if constexpr (kSpread && decltype(first)::value) {
                    static_assert(!kSpread || 2 * Tiles::NI <= KS, "a request per step");
                    i32x4 next[KT];
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt) next[kt] = tiles.row_read(kt, 0);
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                        for (int kt = 0; kt < KT; ++kt) {
                            const i32x4 a = next[kt];
                            if (ks + 1 < KS) next[kt] = tiles.row_read(kt, ks + 1);
                            if (kt == 0) request(ks);
                            sacc[kt] = E::mma(a, qreg[ks], ks == 0 ? zero : sacc[kt]);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                } else {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                        for (int kt = 0; kt < KT; ++kt) sacc[kt] = E::mma(tiles.row_read(kt, ks), qreg[ks], ks == 0 ? zero : sacc[kt]);
                }
                if (need_mask) {
                    const int qi = wave_q0 + col;
                    const int limit = CAUSAL ? min(qi, N - 1) : N - 1;  // last visible key
                    // compile-time key offsets against one opaque per-lane bound: a compare and a select per
                    // score, no index arithmetic
                    int bound = limit - key0 - 4 * half;
                    asm volatile("" : "+v"(bound));
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if (kt * 32 + 8 * (r >> 2) + (r & 3) > bound) sacc[kt][r] = -INFINITY;
                }
            };
            // The row's reference m (log2 units of the scaled scores) becomes the maximum of the block in
            // `sacc` for the lanes that ask for it; O and l follow.
            auto move_reference = [&](bool wanted, auto first_block) __attribute__((always_inline)) {
                float mxp[4] = {sacc[0][0], sacc[0][1], sacc[0][2], sacc[0][3]};
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) mxp[r & 3] = fmaxf(mxp[r & 3], sacc[kt][r]);
                const float m_new = max_both_halves(fmaxf(fmaxf(mxp[0], mxp[1]), fmaxf(mxp[2], mxp[3]))) * sc;
                if constexpr (decltype(first_block)::value) {  // O and l are still zero: only m changes
                    m_run = m_new;
                } else {
                    const float corr = wanted ? fast_exp2(m_run - m_new) : 1.0f;
                    m_run = wanted ? m_new : m_run;
                    l_run *= corr;
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                        for (int r = 0; r < 16; ++r) oacc[dt][r] *= corr;
                }
            };
            // P~ = exp2(s c - m) packed as the operand for GEMM1; returns this lane's part of the row sum
            auto probabilities = [&]() __attribute__((always_inline)) {
                float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) {
                    float p[16];
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        p[r] = fast_exp2(__builtin_fmaf(sacc[kt][r], sc_v, -m_run));
                        ps[r & 3] += p[r];
                    }
#pragma unroll
                    for (int s2 = 0; s2 < 2; ++s2) {
                        i32x4 w;
#pragma unroll
                        for (int i = 0; i < 4; ++i) w[i] = E::pack2(p[8 * s2 + 2 * i], p[8 * s2 + 2 * i + 1]);
                        pb[2 * kt + s2] = w;
                    }
                }
                return (ps[0] + ps[1]) + (ps[2] + ps[3]);
            };

            // ---- online softmax (Algorithm 1: m, P~, l) without a row maximum per block.  The reference m
            // is block 0's true row maximum and afterwards moves only when a block's row sum of P~ --
            // computed anyway -- exceeds kRaiseAbove: below that every P~ of the block is below it too (also
            // as a 16-bit value of the fp16 path), the reference cancels in O / l, and L = m + log2 l
            // either way.  A block that does exceed it (scores that rose by more than 14 in log2 units
            // since the reference was set: rare) is computed again from the K tile, which is still in
            // LDS, with its own maximum as the new reference.
            scores(std::true_type{});
            if (t == 0) move_reference(true, std::true_type{});
            float blk = probabilities();
            const bool over = max_both_halves(blk) > kRaiseAbove;
            if (__builtin_amdgcn_ballot_w64(over) != 0) {
                scores(std::false_type{});
                move_reference(over, std::false_type{});
                blk = probabilities();
            }
            l_run += blk;
        }
        if constexpr (Tiles::VS == 1) {  // V of this block; K of the next stays on its way
            landed(std::integral_constant<int, Tiles::NI>{});
            advance(v_rsrc, Tiles::TILE_B);
        }
        if (wave_active) {
            // ---- GEMM1: O^T += V_j^T P^T
#pragma unroll
            for (int sl = 0; sl < SL; ++sl)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) oacc[dt] = E::mma(tiles.tr_read(sl, dt), pb[sl], oacc[dt]);
        }
        tiles.other_stage(step);
        step = -step;
        landed(std::integral_constant<int, 0>{});
    }

    // ---- epilogue: O / l, L = m + log l.  Every LDS read of the loop was followed by a barrier,
    // so the K and V buffers are free: each wave takes 4 KiB of them to transpose its output tile.
    {
        static_assert(Tiles::kLds >= NW * 4096, "patches must fit");
        char* patch = lds + wave * 4096;
        const int out_lane = lane_again(), qi = wave_q0 + (out_lane & 31);
        const float l = sum_both_halves(l_run);
        store_rows_via_lds<Tag, DT>(oacc, 1.0f / l, patch, make_buffer(o + head_off, (uint32_t)N * D * 2), wave_q0,
                                    out_lane);
        if (qi < N && out_lane < 32) lse[(size_t)bh * N + qi] = (m_run + log2f(l)) * kLn2;
    }
    if (pass + 1 < run.n_pass()) __syncthreads();  // the next pass's first tile overwrites the patches
    }  // passes of a causal pair
}

template <typename Tag, int D, int BC, int NW, int RQ, int PD, bool CAUSAL>
// (512 threads: the four-wave tiles also run FewForward with eight waves.  The second launch bound is waves per SIMD.
// bf16, us, heads x N, against tiles staged through registers and written to the LDS, two workgroups of the d = 128 form on a CU
// instead of three and three of the four-wave d = 64 form instead of four:
// d = 128 causal 512 x 512 67.1 -> 63.7, 160 x 512 24.7 -> 20.7, 160 x 1400 112 -> 95.6; no mask 512 x 512 92.2 -> 75.8,
// 48 x 512 16.3 -> 15.5.
// d = 64 causal 160 x 1024 38.1 -> 33.2, 512 x 512 38.7 -> 35.6; no mask 64 x 4096 277 -> 269, 512 x 512 49.8 -> 45.6.)
__global__ void __launch_bounds__(512, D == 64 ? 4 : NW == 4 ? 3 : 2)
fa_fwd_16bit_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                    const uint16_t* __restrict__ v, uint16_t* __restrict__ o, float* __restrict__ lse,
                    int N, int n_qtiles, int total_wg, int paired, int kv_group, float scale) {
    [[maybe_unused]] ClockSpan clock_span;  // measurement builds only; empty otherwise
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    // (the shared tiles come first: behind the code of the key splits the smallest calls took 0.05 to 0.1 us longer, d = 64 causal
    // 32 x 64 3.93 us instead of 3.86, d = 128 4.95 instead of 4.87, and more scalar registers were spilled)
    if (__builtin_expect(paired < kFewForward, 1)) {
        shared_tiles_forward<Tag, D, BC, NW, RQ, PD, CAUSAL>(q, k, v, o, lse, N, n_qtiles, total_wg, paired, kv_group, scale, lds);
        return;
    }
    if constexpr (NW == 4) {
        if (paired == kFewForward8) {
            FewForward<D, 8>::template run<Tag, CAUSAL>(q, k, v, o, lse, N, total_wg, kv_group, scale, lds);
            return;
        }
    }
    if constexpr (kHasFew<D, NW>) FewForward<D, NW>::template run<Tag, CAUSAL>(q, k, v, o, lse, N, total_wg, kv_group, scale, lds);
}

// ---------------------------------------------------------------------------------------
// Head dimension 256: four waves, one per SIMD.
//
// The output accumulator of 32 query rows (128 registers per lane) and the 64 registers of Q_i
// leave room for one wave per SIMD, so nothing but the wave's own instruction stream can keep
// the matrix pipe busy while the exponentials run.  The loop is therefore software-pipelined
// across key blocks the way the paper's Algorithm 2 (section 3.2) pipelines within a warpgroup:
// the scores of block t+1 are produced while the exponentials of block t run,
//   stage A: S(t+1)^T = K(t+1) Q^T     ||  reference maximum for S(t) (raised lazily; rarely a rescale
//                                          of O and l), P~(t) = exp2(S(t) - m), row sums
//   stage B: O^T += V(t)^T P~(t)^T     ||  mask and row maxima of S(t+1)
// so both score tiles are live at once (the paper's extra S_next registers), K runs one block
// ahead of V through the LDS buffers, and the only rescale of O sits at the head of stage A,
// whose MFMAs do not touch O.  O and Q live in the accumulation half of the register file, which MFMA
// alone can address; the score tiles are produced by MfmaVgprAcc into ordinary registers, where
// the softmax reads them without a copy per score.  Every step ends in a full scheduling
// barrier, so the interleaving written here is what runs, and LDS operand reads lead their
// MFMAs by KP steps.  The block after the last one is computed like any other and comes out
// fully masked (32 MFMAs per tile that add nothing).
// What it is bound by: one wave to a SIMD issues an instruction every four to five cycles (about 470 for the 64 MFMAs of a block),
// and the LDS.  bf16, us, heads x N, with blocks staged through registers / straight into the LDS: causal 64 x 2048 182 / 164,
// 16 x 8192 572 / 507; no mask 16 x 16384 4104 / 3780 (1.16 PFLOP/s), 24 x 1000 36.9 / 31.8.  Not kept: read leads of six and eight steps
// (155 -> 158, 162), all requests in the first 16 steps (166), the second tile's first K block and Q requested before the first output.
template <typename Tag, bool CAUSAL>
__global__ void __launch_bounds__(256, 1)
fa_fwd_d256_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                   uint16_t* __restrict__ o, float* __restrict__ lse, int N, int n_qtiles, int total_wg,
                   int paired, int kv_group, float scale) {
    [[maybe_unused]] ClockSpan clock_span;  // measurement builds only; empty otherwise
    constexpr int D = 256, BC = 64, BR = 128;
    constexpr int KS = D / 16, DT = D / 32, KP = 4;
    using E = Elem<Tag>;
    using Tile = WaveTile<D>;                // the layout of 32 rows in the LDS; a block is two of them
    constexpr int BLOCK_B = 2 * Tile::TILE_B;  // K and V have two stages each

    constexpr int kLds = FewForward<D, 4>::kLds > 4 * BLOCK_B ? FewForward<D, 4>::kLds : 4 * BLOCK_B;
    __shared__ __attribute__((aligned(1024))) char lds[kLds];
    static_assert(FewForward<D, 4>::kLds <= kLds, "both divisions of the work use it");
    if (paired == kFewForward) {
        FewForward<D, 4>::template run<Tag, CAUSAL>(q, k, v, o, lse, N, total_wg, kv_group, scale, lds);
        return;
    }
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;

    const TileRun run = query_tiles<CAUSAL>(total_wg, n_qtiles, paired);
    const int bh = run.head;

    const size_t head_off = (size_t)bh * N * D;
    const size_t kv_off = (size_t)(bh / kv_group) * N * D;
    const uint16_t* qh = q + head_off;
    const float sc = scale * kLog2e;
    // Addresses: row operands of K, transposed operands of V in the first stages (columns from 128 on, 16 rows and the second
    // stage further are offsets), and where the lane fetches the wave's quarter of a block
    const uint32_t k_at = lds_address(lds), v_at = k_at + 2 * BLOCK_B, piece = k_at + wave * (BLOCK_B / 4);
    uint32_t row_at[KS / 2], tr_at[DT / 2][2];
    int src[8];
#pragma unroll
    for (int ks = 0; ks < KS / 2; ++ks) {
        row_at[ks] = k_at + col * Tile::ROWB + (((2 * ks + half) ^ Tile::swizzle(col)) << 4);
        asm volatile("" : "+v"(row_at[ks]));
    }
#pragma unroll
    for (int dt = 0; dt < DT / 2; ++dt)
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            tr_at[dt][hi] = v_at + Tile::tr_of(dt, hi, lane);
            asm volatile("" : "+v"(tr_at[dt][hi]));
        }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        src[i] = wave * (BLOCK_B / 4) + Tile::src_of(i, lane);
        asm volatile("" : "+v"(src[i]));
    }

#pragma nounroll
    for (int pass = 0; pass < run.n_pass(); ++pass) {
    const int qt = pass == 0 ? run.tile : run.second;
    const int wave_q0 = qt * BR + wave * 32;
    const int limit = CAUSAL ? min(wave_q0 + col, N - 1) : N - 1;  // last key this lane's query sees

    // the next blocks of K and V to be requested (rows past N, and blocks past the last one, read as zero)
    BufferWords k_rsrc = make_buffer_words(k + kv_off, (uint32_t)N * D * 2), v_rsrc = make_buffer_words(v + kv_off, (uint32_t)N * D * 2);
#pragma unroll
    for (int i = 0; i < 8; ++i) global_to_lds_16B(k_rsrc, piece + i * 1024, src[i]);
    advance(k_rsrc, BLOCK_B);

    // Q_i^T as the B operand of S^T = K Q^T, resident for the whole loop
    i32x4 qreg[KS];
    {
        const int row = min(wave_q0 + col, N - 1);  // rows past N compute a copy of row N-1, never stored
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            qreg[ks] = *reinterpret_cast<const i32x4*>(qh + (size_t)row * D + ks * 16 + half * 8);
    }
    f32x16 oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f, mb = 0.f;

    const int last_q = min(qt * BR + BR, N) - 1;
    const int n_blocks = CAUSAL ? (last_q / BC + 1) : ((N + BC - 1) / BC);

    // ---- pieces shared by the prologue and the loop
    float mxp[4];
    auto need_mask = [&](int t) { return (t * BC + BC > N) || (CAUSAL && t * BC + BC - 1 > wave_q0); };
    auto mask_block = [&](int t, f32x16 (&s)[2]) {  // keys past N, and keys after the query when causal
        // compile-time key offsets against one per-lane bound (kept opaque: the compiler otherwise gives the
        // 32 per-element key indices registers of their own)
        int bound = limit - t * BC - 4 * half;
        asm volatile("" : "+v"(bound));
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (kt * 32 + 8 * (r >> 2) + (r & 3) > bound) s[kt][r] = -INFINITY;
    };
    auto max_part = [&](f32x16 (&s)[2], int part) {  // registers 8 part .. 8 part + 7 of the 32
#pragma unroll
        for (int i = 8 * part; i < 8 * part + 8; ++i)
            mxp[i & 3] = i < 4 ? s[0][i] : fmaxf(mxp[i & 3], s[i >> 4][i & 15]);
    };
    // K rows for S^T (A operand) in stage ST, 32 steps (kt, ks); the scores land in ordinary registers
    auto row_read = [&](int st, int u) { return lds_load_16B(row_at[u % (KS / 2)] + st * BLOCK_B + (u / KS) * Tile::TILE_B + (u % KS / (KS / 2)) * 256); };

    // Staging, global -> LDS without registers (global_to_lds_16B), a quarter of a block by each wave.  A block's K and V
    // are 64 KiB, half of what the CU's vector memory path moves in the time of the block's MFMAs:
    // issued in one burst the loads make every wave sit in its own issue for over a thousand
    // cycles.  They are spread over the steps of stage A, one every second step: K(t+2) replaces K(t), V(t+1) replaces V(t-1),
    // both last read in block t-1, and both are there at the barrier that ends block t.
    auto blocks_landed = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // the Q loads complete here and Q moves to the accumulation half
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qreg[ks]));
    blocks_landed();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        global_to_lds_16B(v_rsrc, piece + 2 * BLOCK_B + i * 1024, src[i]);
        global_to_lds_16B(k_rsrc, piece + BLOCK_B + i * 1024, src[i]);
    }
    advance(k_rsrc, BLOCK_B);
    advance(v_rsrc, BLOCK_B);

    // ---- prologue: S(0) and its reference maximum (O and l are still zero: nothing to rescale)
    f32x16 sa[2], sb[2];
    {
        i32x4 ring[KP];
#pragma unroll
        for (int u = 0; u < KP; ++u) ring[u] = row_read(0, u);
#pragma unroll
        for (int u = 0; u < 2 * KS; ++u) {
            const i32x4 a = ring[u % KP];
            if (u + KP < 2 * KS) ring[u % KP] = row_read(0, u + KP);
            if (u % KS == 0) MfmaVgprAcc<Tag>::first(sa[u / KS], a, qreg[0]);
            else MfmaVgprAcc<Tag>::run(sa[u / KS], a, qreg[u % KS]);
            __builtin_amdgcn_sched_barrier(0);
        }
        mfma_result_wait(sa[0], sa[1]);
        if (need_mask(0)) mask_block(0, sa);
#pragma unroll
        for (int part = 0; part < 4; ++part) max_part(sa, part);
        m_run = max_both_halves(fmaxf(fmaxf(mxp[0], mxp[1]), fmaxf(mxp[2], mxp[3])));
        mb = m_run * sc;
    }
    blocks_landed();

    // ---- one key block: `cur` holds S(t), `nxt` receives S(t+1); ST = t % 2
    auto block = [&](auto stage, int t, f32x16 (&cur)[2], f32x16 (&nxt)[2]) __attribute__((always_inline)) {
        constexpr int ST = decltype(stage)::value;
        i32x4 pb[4];  // P~(t)^T as B operands, 16 keys each
        float psum = 0.f;

        // ---- stage A
        {
            i32x4 ring[KP];
#pragma unroll
            for (int u = 0; u < KP; ++u) ring[u] = row_read(ST ^ 1, u);
            static_for<2 * KS>([&](auto step) __attribute__((always_inline)) {
                constexpr int u = decltype(step)::value, ks = u % KS, n = u / 2;
                constexpr int to = (n & 1 ? 2 + (ST ^ 1) : ST) * BLOCK_B + (n >> 1) * 1024;
                const i32x4 a = ring[u % KP];
                if constexpr (u + KP < 2 * KS) ring[u % KP] = row_read(ST ^ 1, u + KP);
                f32x16& s = nxt[u / KS];
                const BufferWords& rsrc = n & 1 ? v_rsrc : k_rsrc;
                if constexpr (ks == 0) MfmaVgprAcc<Tag>::template first_and_load<to>(s, a, qreg[ks], rsrc, piece, src[n >> 1]);
                else if constexpr (u % 2 == 0) MfmaVgprAcc<Tag>::template run_and_load<to>(s, a, qreg[ks], rsrc, piece, src[n >> 1]);
                else MfmaVgprAcc<Tag>::run(s, a, qreg[ks]);
                if constexpr (u == 0) {
                    // Reference maximum for S(t) from the row maxima taken beside the previous block's
                    // products: raised only when they exceed it by more than 2^kLazyLog2 (P~ <= 2^kLazyLog2
                    // otherwise and the factor cancels in O / l).  Every product of the previous block has
                    // been issued, and the MFMAs of this stage write the score registers only, so the rare
                    // rescale of O is in order here.  (Block 0: the prologue has set the reference; no rise.)
                    const float mx = max_both_halves(fmaxf(fmaxf(mxp[0], mxp[1]), fmaxf(mxp[2], mxp[3])));
                    const bool raise = (mx - m_run) * sc > kLazyLog2;
                    if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {
                        const float corr = raise ? fast_exp2((m_run - mx) * sc) : 1.0f;
                        m_run = raise ? mx : m_run;
                        l_run *= corr;
#pragma unroll
                        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                            for (int r = 0; r < 16; ++r) oacc[dt][r] *= corr;
                    }
                    mb = m_run * sc;
                }
#pragma unroll
                for (int c = 0; c < 16; ++c)
                    if (2 + (c * 30) / 16 == u) {  // pair c of the 16: two scores of S(t) become one packed register of P~
                        const int kt = c / 8, j = c % 8;
                        const float p0 = fast_exp2(__builtin_fmaf(cur[kt][2 * j], sc, -mb));
                        const float p1 = fast_exp2(__builtin_fmaf(cur[kt][2 * j + 1], sc, -mb));
                        psum += p0 + p1;
                        pb[2 * kt + (j >> 2)][j & 3] = E::pack2(p0, p1);
                    }
                __builtin_amdgcn_sched_barrier(0);
            });
            advance(k_rsrc, BLOCK_B);
            advance(v_rsrc, BLOCK_B);
            l_run += psum;
        }

        // ---- stage B
        {
            constexpr int NU = 4 * DT;  // (16-key slab, d-tile)
            auto v_addr = [&](int u, int hi) -> uint32_t {
                return tr_at[u % (DT / 2)][hi] + ST * BLOCK_B + (u / DT) * 16 * Tile::ROWB + (u % DT / (DT / 2)) * 256;
            };
            i32x2 lo[KP], hi[KP];
#pragma unroll
            for (int u = 0; u < KP; ++u) {
                lo[u] = lds_read_tr16(v_addr(u, 0));
                hi[u] = lds_read_tr16(v_addr(u, 1));
            }
            const bool mask_next = need_mask(t + 1);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int sl = u / DT, dt = u % DT;
                const i32x4 a = {lo[u % KP][0], lo[u % KP][1], hi[u % KP][0], hi[u % KP][1]};
                if (u + KP < NU) {
                    lo[u % KP] = lds_read_tr16(v_addr(u + KP, 0));
                    hi[u % KP] = lds_read_tr16(v_addr(u + KP, 1));
                }
                oacc[dt] = E::mma(a, pb[sl], oacc[dt]);
                if (u == 0) mfma_result_wait(nxt[0], nxt[1]);  // written by MFMAs the hazard checker cannot see
                if (u == 1 && __builtin_expect(mask_next, 0)) mask_block(t + 1, nxt);
                if (u >= 2 && u < 6) max_part(nxt, u - 2);
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        blocks_landed();
    };

    for (int t = 0; t < n_blocks; t += 2) {
        block(std::integral_constant<int, 0>{}, t, sa, sb);
        if (t + 1 < n_blocks) block(std::integral_constant<int, 1>{}, t + 1, sb, sa);
    }

    // ---- epilogue: O / l, L = m + log l, through a 4 KiB LDS patch per wave (the last barrier of
    // the loop has passed, so the K buffers are free)
    {
        char* patch = lds + wave * 4096;
        const int qi = wave_q0 + col;
        const float l = sum_both_halves(l_run);
        int out_lane = lane;  // opaque: the addresses derived from it are else computed before the loop, and spilled over it
        asm volatile("" : "+v"(out_lane));
        store_rows_via_lds<Tag, DT>(oacc, 1.0f / l, patch, make_buffer(o + head_off, (uint32_t)N * D * 2), wave_q0, out_lane);
        if (qi < N && half == 0) lse[(size_t)bh * N + qi] = (m_run * sc + log2f(l)) * kLn2;
    }
    if (pass + 1 < run.n_pass()) __syncthreads();  // the next pass's first tile overwrites the patches
    }  // passes of a causal pair
}

// ---------------------------------------------------------------------------------------
// Eight-wave ping-pong variant (head dimension 128).
//
// An eight-wave workgroup puts two waves on every SIMD (waves w and w + 4).  If all of them run
// a block's steps in the same order they stay in lock-step: both waves of a SIMD issue MFMAs
// together and then both do softmax together, so the matrix pipe idles during every softmax --
// the problem the paper's ping-pong scheduling (section 3.1) solves with named barriers between
// two warpgroups.  Here the waves form two groups, one wave of each per SIMD, and every
// iteration has two half-steps separated by workgroup barriers:
//
//     iteration t          half-step 1                   half-step 2
//        group A     MFMA stream(t)                 softmax(t), operand prefetch
//        group B     softmax(t-1), prefetch         MFMA stream(t)
//
//     stream(t) = O^T += V(t-1)^T P~(t-1)^T  followed by  S(t)^T = K(t) Q^T
//
// so that one wave of each SIMD always has MFMA work while the other has VALU work.  Group A
// carries P~ from one iteration to the next, group B carries S.  A stream is one sequence of
// (LDS operand read, MFMA) units whose reads run P units ahead of their use through a register
// ring; the first P reads are issued before the barrier that precedes the stream, so they
// complete while the wave waits there.
//
// Staging: K and V blocks go from global memory straight into a ring of NS LDS stages
// (buffer loads with an LDS destination: no staging registers, no LDS store instructions), issued
// two to three iterations before their first use.  Such a load writes 64 lanes x 16 bytes
// contiguously, so the tiles are stored unpadded (256 bytes per row) and bank conflicts are
// avoided by an XOR swizzle of the 16-byte chunk index instead, applied through the *global*
// address each lane fetches:  K: chunk ^ (row % 16)  (16 lanes read 16 rows at one chunk),
// V: chunk ^ 4 (row % 4)  (a transposing read covers 4 rows x 4 chunks).
template <typename Tag, int BC, int P, bool CAUSAL>
__global__ void __launch_bounds__(512, 2)
fa_fwd_pingpong_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                       const uint16_t* __restrict__ v, uint16_t* __restrict__ o, float* __restrict__ lse,
                       int N, int n_qtiles, int total_wg, int paired, int kv_group, float scale) {
    [[maybe_unused]] ClockSpan clock_span;  // measurement builds only; empty otherwise
    constexpr int D = 128;
    constexpr int BR = 256;
    constexpr int NS = 4;              // LDS stages per tensor
    constexpr int ROWB = D * 2;        // bytes per tile row
    constexpr int TILE = BC * ROWB;    // bytes per stage
    constexpr int KT = BC / 32;
    constexpr int KS = D / 16;
    constexpr int DT = D / 32;
    constexpr int SL = BC / 16;
    constexpr int N1 = SL * DT;  // MFMA units of the second GEMM
    constexpr int N0 = KS * KT;  // MFMA units of the first GEMM
    static_assert(BC == 64, "the staging pattern below covers 64-row tiles with two loads per wave");
    using E = Elem<Tag>;

    __shared__ __attribute__((aligned(1024))) char lds[2 * NS * TILE + 8 * 4096];
    static_assert(FewForward<D, 8>::kLds <= sizeof(lds), "both divisions of the work use it");
    if (paired == kFewForward) {
        FewForward<D, 8>::template run<Tag, CAUSAL>(q, k, v, o, lse, N, total_wg, kv_group, scale, lds);
        return;
    }
    char *lds_k = lds, *lds_v = lds + NS * TILE, *lds_o = lds + 2 * NS * TILE;  // lds_o: output transposition, 4 KiB per wave

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;
    // the two waves of a SIMD take adjacent 32-row slabs of the query tile
    const int group = wave >> 2;
    const int slab = (wave & 3) * 2 + group;

    const TileRun run = query_tiles<CAUSAL>(total_wg, n_qtiles, paired);
    const int bh = run.head;

    const size_t head_off = (size_t)bh * N * D;
    const uint16_t* qh = q + head_off;
    int wave_q0 = 0;  // first query row of this wave in the current pass
    const float sc = scale * kLog2e;
    float sc_v = sc;  // a vector-register copy: an FMA with a scalar-register operand issues at a lower rate
    asm volatile("" : "+v"(sc_v));

    i32x4 qreg[KS];
    f32x16 oacc[DT];
    float m_run = 0.f, l_run = 0.f;  // reference (log2 units of the scaled scores) and row sum of P~

    // ---- staging: wave w loads rows 4w .. 4w+3 and 32+4w .. 32+4w+3 of a tile (1 KiB each)
    const size_t kv_off = (size_t)(bh / kv_group) * N * D;  // grouped-query: kv_group query heads per K/V head
    const BufferWords k_rsrc = make_buffer_words(k + kv_off, (uint32_t)N * D * 2);
    const BufferWords v_rsrc = make_buffer_words(v + kv_off, (uint32_t)N * D * 2);
    const int st_row = 4 * wave + (lane >> 4), st_pos = lane & 15;
    const int k_src = st_row * ROWB + ((st_pos ^ (st_row & 15)) << 4);        // byte offset within a tile
    const int v_src = st_row * ROWB + ((st_pos ^ ((st_row & 3) << 2)) << 4);
    const uint32_t lds_k0 = (uint32_t)(uintptr_t)lds_k + wave * 1024, lds_v0 = (uint32_t)(uintptr_t)lds_v + wave * 1024;
    // Block u of K and block u2 of V.  Blocks past the end lie outside the buffer resources and
    // read as zeros, so every iteration issues the same four loads and the vmcnt waits below can
    // count on that.
    auto stage_k = [&](int u) __attribute__((always_inline)) {
        const uint32_t kd = lds_k0 + (u & (NS - 1)) * TILE;
        global_to_lds_16B(k_rsrc, kd, k_src + u * TILE);
        global_to_lds_16B(k_rsrc, kd + 8 * 1024, k_src + u * TILE + 32 * ROWB);
    };
    auto stage_v = [&](int u) __attribute__((always_inline)) {
        const uint32_t vd = lds_v0 + (u & (NS - 1)) * TILE;
        global_to_lds_16B(v_rsrc, vd, v_src + u * TILE);
        global_to_lds_16B(v_rsrc, vd + 8 * 1024, v_src + u * TILE + 32 * ROWB);
    };
    auto stage = [&](int u, int u2) __attribute__((always_inline)) {
        stage_k(u);
        stage_v(u2);
    };

    // ---- per-lane operand offsets within a stage (bytes)
    const int tr_row = (lane & 15) >> 2, quad = lane & 3, blk = (lane >> 4) & 1;
    int kofs[KS], vofs[DT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kofs[ks] = col * ROWB + (((2 * ks + half) ^ (col & 15)) << 4);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
        vofs[dt] = (4 * half + tr_row) * ROWB + (((4 * dt + 2 * blk + (quad >> 1)) ^ (tr_row << 2)) << 4) + 8 * (quad & 1);

    f32x16 sacc[KT];
    i32x4 pb[SL];
    i32x4 ring[P];

    // Unit u of stream(t): the second GEMM's units (if DO1) then the first GEMM's (if DO0).
    auto read_unit = [&](auto do1, int t, int u) __attribute__((always_inline)) {
        constexpr int n1 = decltype(do1)::value ? N1 : 0;
        if (u < n1) {
#if FA_ABLATE_PP == 2
            asm volatile("" : "+v"(ring[u % P]));
#else
            const int sl = u / DT, dt = u % DT;
            const char* p0 = lds_v + ((t - 1) & (NS - 1)) * TILE + vofs[dt] + sl * 16 * ROWB;
            i32x2 lo = lds_read_tr16(p0);
            i32x2 hi = lds_read_tr16(p0 + 8 * ROWB);
            ring[u % P] = i32x4{lo[0], lo[1], hi[0], hi[1]};
#endif
        } else {
#if FA_ABLATE_PP == 3
            asm volatile("" : "+v"(ring[u % P]));
#else
            const int ks = (u - n1) / KT, kt = (u - n1) % KT;
            ring[u % P] = *reinterpret_cast<const i32x4*>(lds_k + (t & (NS - 1)) * TILE + kofs[ks] + kt * 32 * ROWB);
#endif
        }
    };
    auto prefill = [&](auto do1, auto do0, int t) __attribute__((always_inline)) {
        constexpr int NU = (decltype(do1)::value ? N1 : 0) + (decltype(do0)::value ? N0 : 0);
#pragma unroll
        for (int u = 0; u < (P < NU ? P : NU); ++u) read_unit(do1, t, u);
    };
    auto run_stream = [&](auto do1, auto do0, int t) __attribute__((always_inline)) {
        constexpr int n1 = decltype(do1)::value ? N1 : 0;
        constexpr int NU = n1 + (decltype(do0)::value ? N0 : 0);
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const i32x4 a = ring[u % P];
            if (u + P < NU) read_unit(do1, t, u + P);
            if (u < n1) {
                const int sl = u / DT, dt = u % DT;
                oacc[dt] = E::mma(a, pb[sl], oacc[dt]);
            } else {
                const int ks = (u - n1) / KT, kt = (u - n1) % KT;
                sacc[kt] = E::mma(a, qreg[ks], ks == 0 ? zero : sacc[kt]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // mask block t (keys past N; keys after the query when causal), then the online softmax of
    // Algorithm 1 (m, P~, l); P~ leaves packed as the B operand of the second GEMM
    auto softmax = [&](int t) __attribute__((always_inline)) {
        const int key0 = t * BC;
        if ((key0 + BC > N) || (CAUSAL && key0 + BC - 1 > wave_q0)) {
            const int qi = wave_q0 + col;
            const int limit = CAUSAL ? min(qi, N - 1) : N - 1;  // last visible key
            // compile-time key offsets against one opaque per-lane bound: a compare and a select per score
            int bound = limit - key0 - 4 * half;
            asm volatile("" : "+v"(bound));
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (kt * 32 + 8 * (r >> 2) + (r & 3) > bound) sacc[kt][r] = -INFINITY;
        }
        // Every step below is a batch of independent instructions: a wave gets few issue slots
        // while its SIMD sibling streams MFMAs, and dependent chains (fma -> exp, sum) would turn
        // each slot missed into a stall.
        //
        // No row maximum is taken per block.  Scores are referred to a per-row reference m (log2
        // units) that is the true row maximum of block 0 and afterwards moves only when a block's
        // P~ grow large: x = s c - m stays in the score registers, P~ = exp2(x) goes to the operand
        // registers, and the block's row sum -- needed anyway -- is the overflow detector.  While it
        // stays below kRaiseAbove every P~ of the block is below it too (also the 16-bit P~ of the
        // fp16 path); otherwise the reference is moved to this block's true maximum, O and l are
        // rescaled and the block's P~ recomputed from x.  The reference cancels in O / l and L is
        // m + log2 l either way, so the result is that of Algorithm 1 with any reference.
#if FA_ABLATE_PP != 4
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) sacc[kt][r] = __builtin_fmaf(sacc[kt][r], sc_v, -m_run);
#endif
        __builtin_amdgcn_sched_barrier(0);
        float blk = 0.f;
        auto probabilities = [&]() __attribute__((always_inline)) {
            float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                float e[16];
#pragma unroll
#if FA_ABLATE_PP == 1 || FA_ABLATE_PP == 4
                for (int r = 0; r < 16; ++r) e[r] = sacc[kt][r];
#else
                for (int r = 0; r < 16; ++r) e[r] = fast_exp2(sacc[kt][r]);
#endif
#if FA_ABLATE_PP != 4
#pragma unroll
                for (int r = 0; r < 16; ++r) ps[r & 3] += e[r];
#endif
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    i32x4 w;
#pragma unroll
                    for (int i = 0; i < 4; ++i) w[i] = E::pack2(e[8 * s2 + 2 * i], e[8 * s2 + 2 * i + 1]);
                    pb[2 * kt + s2] = w;
                }
            }
            blk = (ps[0] + ps[1]) + (ps[2] + ps[3]);
        };
        probabilities();
        const bool first = t == 0;
        const bool raise = first || max_both_halves(blk) > kRaiseAbove;
        if (first || __builtin_amdgcn_ballot_w64(raise) != 0) {
            float mxp[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) mxp[c] = sacc[0][c];
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) mxp[r & 3] = fmaxf(mxp[r & 3], sacc[kt][r]);
            const float mx = max_both_halves(fmaxf(fmaxf(mxp[0], mxp[1]), fmaxf(mxp[2], mxp[3])));
            const float delta = raise ? mx : 0.f;
            const float corr = fast_exp2(-delta);
            m_run += delta;
            l_run *= corr;
            if (!first) {
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[dt][r] *= corr;
            }
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) sacc[kt][r] -= delta;
            probabilities();
        }
        l_run += blk;
        // P~ must exist in registers here: the compiler is otherwise free to sink the exponentials
        // past the next barrier, next to the MFMAs that consume them
#pragma unroll
        for (int i = 0; i < SL; ++i) asm volatile("" : "+v"(pb[i]));
    };

    // Workgroup barrier that leaves the staging loads in flight.  LDS reads issued before it (the
    // operand prefetch) may still be outstanding; their results are only used after it anyway.
    auto barrier = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // Iteration t issues K(t+3) and V(t+2) (four loads per wave); before the barrier that ends
    // half-step 1 of iteration t a wave makes sure its loads of iteration t-2 have landed: K(t+1)
    // and V(t), first read by the prefetch at the end of this iteration.
    auto mid_barrier = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        barrier();
    };

    const std::true_type yes{};
    const std::false_type no{};

#pragma nounroll
    for (int pass = 0; pass < run.n_pass(); ++pass) {
    const int qt = pass == 0 ? run.tile : run.second;
    wave_q0 = qt * BR + slab * 32;
    {
        int row = min(wave_q0 + col, N - 1);  // rows past N compute a copy of row N-1, never stored
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            qreg[ks] = *reinterpret_cast<const i32x4*>(qh + (size_t)row * D + ks * 16 + half * 8);
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
    m_run = 0.f;  // set from block 0's row maximum by its softmax
    l_run = 0.f;
    const int last_q = min(qt * BR + BR, N) - 1;
    const int n_blocks = CAUSAL ? (last_q / BC + 1) : ((N + BC - 1) / BC);
    // blocks 0 .. nb_w-1 concern this wave (all of them unless causal)
    const int nb_w = CAUSAL ? min(n_blocks, (wave_q0 + 31) / BC + 1) : n_blocks;
    // every wave's staging loads of the previous pass have landed (each waited for its own
    // before its epilogue) and every LDS read of that pass is done
    if (pass > 0) barrier();

    // ---- prologue: K(0), K(1), K(2), V(0), V(1) staged and visible before the first iteration
    stage(0, 0);
    stage(1, 1);
    stage_k(2);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));  // Q loads complete before the loop
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    barrier();

    if (group == 0) {
        prefill(no, yes, 0);
        // stream(t) was prefetched at the end of the previous iteration
        auto iteration = [&](int t, auto do1, auto do0, auto next1, auto next0) __attribute__((always_inline)) {
            stage(t + 3, t + 2);
            run_stream(do1, do0, t);
            mid_barrier();
            if constexpr (decltype(do0)::value) softmax(t);
            prefill(next1, next0, t + 1);
            barrier();
        };
        // stream shapes over t: (no,yes) at 0; (yes,yes) for 1..nb_w-1; (yes,no) at nb_w; nothing after
        if (nb_w > 1) iteration(0, no, yes, yes, yes);
        else iteration(0, no, yes, yes, no);
        for (int t = 1; t + 1 < nb_w; ++t) iteration(t, yes, yes, yes, yes);
        if (nb_w > 1) iteration(nb_w - 1, yes, yes, yes, no);
        iteration(nb_w, yes, no, no, no);
        for (int t = nb_w + 1; t <= n_blocks; ++t) iteration(t, no, no, no, no);
    } else {
        auto iteration = [&](int t, auto do1, auto do0) __attribute__((always_inline)) {
            stage(t + 3, t + 2);
            prefill(do1, do0, t);
            if constexpr (decltype(do1)::value) softmax(t - 1);
            mid_barrier();
            run_stream(do1, do0, t);
            barrier();
        };
        iteration(0, no, yes);
        for (int t = 1; t < nb_w; ++t) iteration(t, yes, yes);
        iteration(nb_w, yes, no);
        for (int t = nb_w + 1; t <= n_blocks; ++t) iteration(t, no, no);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // staging loads past the last block: nothing may land after the end

    // ---- epilogue: O / l, L = m + log l
    {
        const int qi = wave_q0 + col;
        const float l = sum_both_halves(l_run);
        store_rows_via_lds<Tag, DT>(oacc, 1.0f / l, lds_o + wave * 4096, make_buffer(o + head_off, (uint32_t)N * D * 2),
                                    wave_q0, lane);
        if (qi < N && half == 0) lse[(size_t)bh * N + qi] = (m_run + log2f(l)) * kLn2;
    }
    }  // passes of a causal pair
}

// ---------------------------------------------------------------------------------------
// fp32 path (d = 64) on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: fp32 operands, products and sums).
//
// Bound by that instruction: 64 cycles for 4 KFLOP per SIMD, 157 TFLOP/s for the chip, against which the softmax of
// a 32 x 32 score tile (64 MFMAs) is about a tenth.  Requests in fp32 are mostly small, so the tile is chosen to
// put work on every SIMD: a workgroup owns 64 query rows in two slabs of 32, and the four waves of a slab split
// the keys (wave `split` takes the 32-key tiles split, split + 4, ...) with a softmax state each; the four states are
// merged through the LDS at the end, in a fixed order.  That quarters the serial chain of tiles and puts two waves on
// each SIMD, one's softmax under the other's MFMAs.  Each wave stages its own tiles straight into LDS of its own, V
// beside the score MFMAs and the next K beside the products: without a barrier the two waves of a SIMD drift apart and
// stay there.  (Staged by the workgroup, 128 keys at a time behind a barrier, both waves of a SIMD did their softmax
// together: B = 2, H = 8, N = 1000 42.3 us, 36.6 so, most of it from the 110 vector instructions
// per tile that offsets, addresses and needless rescales took: the matrix instruction leaves the vector pipe little room.)
//   S^T = K Q^T: step i contracts head-dim elements {i, 32 + i}, so a lane's operands are 32 consecutive floats of a
//     row, four MFMAs to a 16-byte LDS read.
//   O^T += V^T P^T: score register r of a lane is key 8 (r / 4) + 4 half + r % 4, so the register itself is the B
//     operand of the step that contracts this pair of keys; A is V read down a column.
//   The tiles are unpadded rows of 256 bytes, 16-byte chunk c of row r at c ^ swizzle(r): sixteen rows at one chunk hit
//     every bank once (K), and so do the halves of two rows four apart (V).
template <int D, int BC, bool CAUSAL>
__global__ void __launch_bounds__(512, 2)
fa_fwd_f32_kernel(const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                  float* __restrict__ o, float* __restrict__ lse, int N, int n_qtiles, int total_wg, int first_head,
                  int kv_group, float scale) {
    static_assert(D == 64 && BC == 32, "one 32-key score tile per step, two 32-column output tiles");
    constexpr int NT = 512, SLABS = 2, SPLITS = 4;
    constexpr int BR = 32 * SLABS;    // query rows per workgroup
    constexpr int ROWB = D * 4, TILE = BC * ROWB;  // bytes of a row and of a tile
    constexpr int PSTR = D + 4;       // row stride of the partial outputs (floats)
    constexpr int NI = TILE / 1024;   // staging instructions per tile (four rows each)
    constexpr int KP = 2, VP = 4;     // steps by which operand reads lead their MFMAs
    __shared__ __attribute__((aligned(1024))) char lds[SLABS * SPLITS * 2 * TILE];
    __shared__ float lds_m[SPLITS][BR], lds_l[SPLITS][BR];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31, half = lane >> 5;
    const int slab = wave & 1, split = wave >> 1;

    const WorkItem item = work_item<CAUSAL>(blockIdx.x, total_wg, n_qtiles);
    const int bh = first_head + item.head, qt = CAUSAL ? n_qtiles - 1 - item.tile : item.tile;  // the last rows see the most keys
    const size_t head_off = (size_t)bh * N * D;
    const size_t kv_off = (size_t)(bh / kv_group) * N * D;  // grouped-query: kv_group query heads per K/V head
    const int q0 = qt * BR + slab * 32;                     // first row of this wave's slab
    const int row = min(q0 + col, N - 1);                   // rows past N compute a copy of row N-1, never stored
    const int limit = CAUSAL ? row : N - 1;                 // last visible key
    const int n_tiles = CAUSAL ? min(q0 / BC + 1, (N + BC - 1) / BC) : (N + BC - 1) / BC;
    const float sc = scale * kLog2e;

    // the wave's next tiles (rows past N read as zero)
    BufferWords k_rsrc = make_buffer_words(k + kv_off, (uint32_t)N * D * 4), v_rsrc = make_buffer_words(v + kv_off, (uint32_t)N * D * 4);
    advance(k_rsrc, split * TILE);
    advance(v_rsrc, split * TILE);
    auto swizzle = [](int r) { return (r & 3) | ((r >> 3) & 1) << 2 | ((r >> 2) & 1) << 3; };
    const uint32_t kb = lds_address(lds) + wave * (2 * TILE), vb = kb + TILE;
    int src[NI];  // byte offset within a tile
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int r = 4 * i + (lane >> 4);
        src[i] = r * ROWB + ((lane & 15) ^ swizzle(r)) * 16;
    }
    auto request = [&](const BufferWords& rsrc, uint32_t to, int i) __attribute__((always_inline)) {
        global_to_lds_16B(rsrc, to + i * 1024, src[i]);
    };
#pragma unroll
    for (int i = 0; i < NI; ++i) request(k_rsrc, kb, i);

    f32x4 qreg[D / 8];  // Q^T as the B operand: lane (row, half) holds elements 32 half .. 32 half + 31
#pragma unroll
    for (int j = 0; j < D / 8; ++j)
        qreg[j] = *reinterpret_cast<const f32x4*>(q + head_off + (size_t)row * D + half * (D / 2) + 4 * j);
    f32x16 acc[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    // LDS addresses of the operands, opaque: they are else computed again in every tile.  K: chunk 8 half + j of row col.
    // V: columns col and col + 32 of rows 8 (r / 4) + 4 half + r % 4, r < 8 (16 rows on the swizzle is the same).
    uint32_t k_at[D / 8], v_at[8][2];
#pragma unroll
    for (int j = 0; j < D / 8; ++j) {
        k_at[j] = kb + col * ROWB + (((8 * half + j) ^ swizzle(col)) << 4);
        asm volatile("" : "+v"(k_at[j]));
    }
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
            const int key = 8 * (r >> 2) + 4 * half + (r & 3);
            v_at[r][dt] = vb + key * ROWB + ((((col >> 2) + 8 * dt) ^ swizzle(key)) << 4) + 4 * (col & 3);
            asm volatile("" : "+v"(v_at[r][dt]));
        }
    float sc_v = sc;  // a vector-register copy: an FMA with a scalar-register operand issues at a lower rate
    asm volatile("" : "+v"(sc_v));
#pragma unroll
    for (int j = 0; j < D / 8; ++j) asm volatile("" : "+v"(qreg[j]));

    for (int t = split; t < n_tiles; t += SPLITS) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // K has landed, the last V has been read
        advance(k_rsrc, SPLITS * TILE);
        if (t + SPLITS >= n_tiles) k_rsrc.w[2] = 0;  // past the wave's last tile: zeros that nothing reads
        const int key0 = t * BC;
        f32x16 s;
        f32x4 ring[KP];  // operand reads lead their MFMAs
#pragma unroll
        for (int j = 0; j < KP; ++j) ring[j] = __builtin_bit_cast(f32x4, lds_load_16B(k_at[j]));
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < D / 8; ++j) {
            const f32x4 a = ring[j % KP];
            if (j + KP < D / 8) ring[j % KP] = __builtin_bit_cast(f32x4, lds_load_16B(k_at[j + KP]));
            request(v_rsrc, vb, j);
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], qreg[j][e], s, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        static_assert(NI == D / 8, "one request per operand read, one per pair of products");
        if (key0 + BC > N || (CAUSAL && key0 + BC - 1 > q0)) {
            const int bound = limit - key0 - 4 * half;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + (r & 3) > bound) s[r] = -INFINITY;
        }
        float mx[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
        for (int r = 0; r < 16; ++r) mx[r & 3] = fmaxf(mx[r & 3], s[r]);
        const float m_new = max_both_halves(fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3])));
        // the reference rises when a tile's maximum exceeds it by more than 2^kLazyLog2 (the factor cancels in O / l)
        const bool raise = (m_new - m_run) * sc > kLazyLog2;
        if (__builtin_amdgcn_ballot_w64(raise) != 0) {
            const float corr = raise ? fast_exp2((m_run - m_new) * sc) : 1.0f;
            m_run = raise ? m_new : m_run;
            l_run *= corr;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[0][r] *= corr;
                acc[1][r] *= corr;
            }
        }
        const float mb = m_run == -INFINITY ? 0.f : m_run * sc;  // a row of scores of -inf so far: P = 0
        float ps[4];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = fast_exp2(__builtin_fmaf(s[r], sc_v, -mb));
            ps[r & 3] = r < 4 ? s[r] : ps[r & 3] + s[r];
        }
        l_run += (ps[0] + ps[1]) + (ps[2] + ps[3]);
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // V has landed, K has been read
        advance(v_rsrc, SPLITS * TILE);
        auto v_read = [&](int r, int dt) __attribute__((always_inline)) { return lds_load_4B(v_at[r & 7][dt] + (r >> 3) * 16 * ROWB); };
        float v0[VP], v1[VP];
#pragma unroll
        for (int r = 0; r < VP; ++r) {
            v0[r] = v_read(r, 0);
            v1[r] = v_read(r, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float a0 = v0[r % VP], a1 = v1[r % VP];
            if (r + VP < 16) {
                v0[r % VP] = v_read(r + VP, 0);
                v1[r % VP] = v_read(r + VP, 1);
            }
            if (r & 1) request(k_rsrc, kb, r >> 1);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, s[r], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, s[r], acc[1], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the last requests: the LDS is about to be reused

    // ---- merge the four key splits of a row: with M the largest of their maxima and f = exp(m - M),
    // L = M + log sum f l and O = sum f O / sum f l
    const float l = sum_both_halves(l_run);
    if (half == 0) {
        lds_m[split][slab * 32 + col] = m_run;
        lds_l[split][slab * 32 + col] = l;
    }
    __syncthreads();
    float m_all = -INFINITY, l_all = 0.f;
#pragma unroll
    for (int w = 0; w < SPLITS; ++w) m_all = fmaxf(m_all, lds_m[w][slab * 32 + col]);
    const float m_ref = m_all == -INFINITY ? 0.f : m_all;  // a row whose every score is -inf: l = 0, L = -inf
#pragma unroll
    for (int w = 0; w < SPLITS; ++w)
        l_all += lds_l[w][slab * 32 + col] * fast_exp2((lds_m[w][slab * 32 + col] - m_ref) * sc);
    const float f = fast_exp2((m_run - m_ref) * sc) / l_all;
    // the tiles are free: [split][row][d] partial outputs, already scaled
    static_assert(sizeof(lds) >= SPLITS * BR * PSTR * sizeof(float), "partial outputs must fit");
    float* part = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 w = {acc[dt][4 * g] * f, acc[dt][4 * g + 1] * f, acc[dt][4 * g + 2] * f, acc[dt][4 * g + 3] * f};
            *reinterpret_cast<f32x4*>(part + (split * BR + slab * 32 + col) * PSTR + dt * 32 + 8 * g + 4 * half) = w;
        }
    if (split == 0 && half == 0 && q0 + col < N) lse[(size_t)bh * N + q0 + col] = (m_all * sc + log2f(l_all)) * kLn2;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < BR * D / 4 / NT; ++i) {
        const int c = tid + i * NT, r = c / (D / 4), cc = (c % (D / 4)) * 4;
        if (qt * BR + r < N) {
            f32x4 w = *reinterpret_cast<const f32x4*>(part + r * PSTR + cc);
#pragma unroll
            for (int sp = 1; sp < SPLITS; ++sp) {
                const f32x4 x = *reinterpret_cast<const f32x4*>(part + (sp * BR + r) * PSTR + cc);
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] += x[e];
            }
            *reinterpret_cast<f32x4*>(o + head_off + (size_t)(qt * BR + r) * D + cc) = w;
        }
    }
}

// fp32, N <= 32: one wave does a head by itself, straight from and to memory -- the score tile's operands, a row of K and
// of Q per lane, need no sharing, and V read down a column is 128 contiguous bytes per half wave.  Neither LDS nor a barrier,
// so the chip holds as many waves as the registers allow; bound by latency with few heads and by memory with many.
// The kernel above stages 128 keys for 64 rows of which all but 32 are padding here.  No mask, us, the kernel above / one
// thread per row and scalar FMAs / this one: 8192 heads N = 1 153 / 94 / 24, N = 16 171 / 123 / 31, N = 32 181 / 168 / 67
// (4.0 TB/s); 512 heads N = 32 12.4 / 27.1 / 6.3; 1 head N = 32 6.3 / 24.2 / 5.3.
template <bool CAUSAL>
__global__ void __launch_bounds__(256, 4)
fa_fwd_f32_short_kernel(const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                        float* __restrict__ o, float* __restrict__ lse, int N, int n_heads, int kv_group, float scale) {
    constexpr int D = 64;
    const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
    const int bh = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (bh >= n_heads) return;
    const size_t head_off = (size_t)bh * N * D;
    const size_t kv_off = (size_t)(bh / kv_group) * N * D;  // grouped-query: kv_group query heads per K/V head
    const int row = min(col, N - 1);                        // rows past N compute a copy of row N-1, never stored
    const float sc = scale * kLog2e;
    const __amdgpu_buffer_rsrc_t k_rsrc = make_buffer(k + kv_off, (uint32_t)N * D * 4);  // rows past N read as zero
    const __amdgpu_buffer_rsrc_t v_rsrc = make_buffer(v + kv_off, (uint32_t)N * D * 4);

    // S^T = K Q^T: step i contracts head-dim elements {i, 32 + i}
    f32x4 kreg[D / 8], qreg[D / 8];
#pragma unroll
    for (int j = 0; j < D / 8; ++j) {
        kreg[j] = __builtin_bit_cast(f32x4, buffer_load_16B(k_rsrc, (col * D + half * (D / 2) + 4 * j) * 4));
        qreg[j] = *reinterpret_cast<const f32x4*>(q + head_off + (size_t)row * D + half * (D / 2) + 4 * j);
    }
    float vreg[16][2];  // score register r is key 8 (r / 4) + 4 half + r % 4
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
            vreg[r][dt] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                              v_rsrc, ((8 * (r >> 2) + 4 * half + (r & 3)) * D + dt * 32 + col) * 4, 0, 0));
    f32x16 s, acc[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = acc[0][r] = acc[1][r] = 0.f;
#pragma unroll
    for (int j = 0; j < D / 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kreg[j][e], qreg[j][e], s, 0, 0, 0);

    const int bound = (CAUSAL ? row : N - 1) - 4 * half;  // last visible key of the lane's half
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if (8 * (r >> 2) + (r & 3) > bound) s[r] = -INFINITY;
        m = fmaxf(m, s[r]);
    }
    m = max_both_halves(m);
    const float mb = m == -INFINITY ? 0.f : m * sc;  // every score -inf: P = 0
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        s[r] = fast_exp2(__builtin_fmaf(s[r], sc, -mb));
        l += s[r];
    }
    l = sum_both_halves(l);
    // O^T = V^T P^T
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vreg[r][dt], s[r], acc[dt], 0, 0, 0);

    if (col >= N) return;
    const float inv = 1.0f / l;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 w = {acc[dt][4 * g] * inv, acc[dt][4 * g + 1] * inv, acc[dt][4 * g + 2] * inv, acc[dt][4 * g + 3] * inv};
            *reinterpret_cast<f32x4*>(o + head_off + (size_t)col * D + dt * 32 + 8 * g + 4 * half) = w;
        }
    if (half == 0) lse[(size_t)bh * N + col] = (m * sc + log2f(l)) * kLn2;
}

// ---------------------------------------------------------------------------------------
template <typename Tag, int D, int BC, int NW, int RQ, int PD>
static int launch_16bit(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int H_kv, int N,
                        float scale, int causal, bool few, hipStream_t stream) {
    constexpr int BR = NW * 32 * RQ;
    int n_qtiles = (N + BR - 1) / BR;
    constexpr PairRule kPairs = NW == 4 ? (D == 64 ? PairRule{3, 15.f / 16, 384, 0.8f, 4} : PairRule{2, 7.f / 8, 256, 0.75f, kAny})
                                        : (D == 64 ? PairRule{2, 1.f, kAny, 1.f, 0} : PairRule{1, 7.f / 8, kAny, 1.f, kAny});
    const int few_waves = few && NW == 4 ? few_forward_waves((long)B * H, N, D, causal) : NW;
    const int paired = few_waves != NW ? kFewForward8 : few ? kFewForward : causal && pair_causal_tiles((long)B * H, n_qtiles, kPairs);
    long total = few ? few_split((long)B * H, N) : (long)B * H * (paired ? (n_qtiles + 1) / 2 : n_qtiles);
    if (total > 0x7fffffffL) return FA_ERR_SHAPE;
    const dim3 grid = forward_grid((long)B * H, N, n_qtiles, total, causal, few ? kFewForward : paired), block(few_waves * 64);
    if (causal && !paired) total = (long)B * H;  // (query_tiles)
    int lds = SharedTiles<D, BC, NW>::kLds;
    if constexpr (kHasFew<D, NW>)
        if (few) lds = few_waves == 8 ? FewForward<D, 8>::kLds : FewForward<D, 4>::kLds;
    auto qp = static_cast<const uint16_t*>(q);
    auto kp = static_cast<const uint16_t*>(k);
    auto vp = static_cast<const uint16_t*>(v);
    auto op = static_cast<uint16_t*>(o);
    if (causal)
        hipLaunchKernelGGL((fa_fwd_16bit_kernel<Tag, D, BC, NW, RQ, PD, true>), grid, block, lds, stream, qp, kp, vp,
                           op, lse, N, n_qtiles, (int)total, paired, H / H_kv, scale);
    else
        hipLaunchKernelGGL((fa_fwd_16bit_kernel<Tag, D, BC, NW, RQ, PD, false>), grid, block, lds, stream, qp, kp, vp,
                           op, lse, N, n_qtiles, (int)total, paired, H / H_kv, scale);
    return hipGetLastError() == hipSuccess ? FA_OK : FA_ERR_LAUNCH;
}

template <typename Tag>
static int launch_pingpong(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int H_kv, int N,
                           float scale, int causal, bool few, hipStream_t stream) {
    constexpr int BR = 256, BC = 64, P = 4;
    int n_qtiles = (N + BR - 1) / BR;
    const int paired = few ? kFewForward : causal && pair_causal_tiles((long)B * H, n_qtiles, PairRule{1, 27.f / 32, kAny, 1.f, kAny});
    long total = few ? few_split((long)B * H, N) : (long)B * H * (paired ? (n_qtiles + 1) / 2 : n_qtiles);
    if (total > 0x7fffffffL) return FA_ERR_SHAPE;
    const dim3 grid = forward_grid((long)B * H, N, n_qtiles, total, causal, paired), block(512);
    auto qp = static_cast<const uint16_t*>(q);
    auto kp = static_cast<const uint16_t*>(k);
    auto vp = static_cast<const uint16_t*>(v);
    auto op = static_cast<uint16_t*>(o);
    if (causal)
        hipLaunchKernelGGL((fa_fwd_pingpong_kernel<Tag, BC, P, true>), grid, block, 0, stream, qp, kp, vp, op, lse, N,
                           n_qtiles, (int)total, paired, H / H_kv, scale);
    else
        hipLaunchKernelGGL((fa_fwd_pingpong_kernel<Tag, BC, P, false>), grid, block, 0, stream, qp, kp, vp, op, lse, N,
                           n_qtiles, (int)total, paired, H / H_kv, scale);
    return hipGetLastError() == hipSuccess ? FA_OK : FA_ERR_LAUNCH;
}

template <typename Tag>
static int launch_d256(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int H_kv, int N,
                       float scale, int causal, bool few, hipStream_t stream) {
    constexpr int BR = 128;
    int n_qtiles = (N + BR - 1) / BR;
    const int paired = few ? kFewForward : causal && pair_causal_tiles((long)B * H, n_qtiles, PairRule{1, 7.f / 8, 128, 0.7f, kAny});
    long total = few ? few_split((long)B * H, N) : (long)B * H * (paired ? (n_qtiles + 1) / 2 : n_qtiles);
    if (total > 0x7fffffffL) return FA_ERR_SHAPE;
    const dim3 grid = forward_grid((long)B * H, N, n_qtiles, total, causal, paired), block(256);
    auto qp = static_cast<const uint16_t*>(q);
    auto kp = static_cast<const uint16_t*>(k);
    auto vp = static_cast<const uint16_t*>(v);
    auto op = static_cast<uint16_t*>(o);
    if (causal)
        hipLaunchKernelGGL((fa_fwd_d256_kernel<Tag, true>), grid, block, 0, stream, qp, kp, vp, op, lse, N, n_qtiles,
                           (int)total, paired, H / H_kv, scale);
    else
        hipLaunchKernelGGL((fa_fwd_d256_kernel<Tag, false>), grid, block, 0, stream, qp, kp, vp, op, lse, N, n_qtiles,
                           (int)total, paired, H / H_kv, scale);
    return hipGetLastError() == hipSuccess ? FA_OK : FA_ERR_LAUNCH;
}

// Kernel choice, by N, d and mask alone (fa_fwd_kernel_name promises that, so a line lies where no number of heads loses
// more than noise, though many win on its other side):
//   d = 128: the eight-wave ping-pong kernel (256 query rows) for long sequences, 128-row workgroups of four waves for
//     short ones, which fill the chip better and waste less of a tile on the diagonal.
//   d = 64: eight waves share each K/V block (256 rows, two waves per SIMD), four waves for short problems.
//   d = 256: the 128-register output accumulator allows only one wave per SIMD; fa_fwd_d256_kernel
//     pipelines the softmax of one block under the score MFMAs of the next inside that wave.
// us, 128 / 256 rows, heads x N, each in the better order of work:
//   d = 64   causal:  16 x 2560 36.0 / 45.8, 64 x 2560 70.4 / 75.5, 32 x 4096 89.8 / 94.5, 48 x 6144 261 / 273;
//                     16 x 8192 172 / 177, 24 x 8192 226 / 238, 8 x 16384 329 / 333
//            no mask: 16 x 700 12.3 / 15.4, 139 x 648 30.1 / 30.0, 40 x 896 18.9 / 20.3, 256 x 896 71.6 / 79.8;
//                     32 x 1024 18.4 / 22.2, 512 x 1024 170 / 178 but 128 x 1024 46.1 / 45.1
//   d = 128  causal:  16 x 1920 43.5 / 46.1, 64 x 1920 86.7 / 89.0, 112 x 1920 127 / 175;  16 x 2048 46.9 / 50.3, 48 x 2048 68.4 / 70.6
//            no mask: 85 x 648 30.0 / 31.9, 129 x 704 49.5 / 54.6, 16 x 768 17.9 / 21.7, 64 x 768 29.3 / 29.2, 256 x 896 118 / 152;
//                     32 x 960 26.1 / 30.2, 512 x 1024 270 / 341 but 48 x 960 32.7 / 32.2
//   Of 740 shapes without a mask and 4500 causal ones within the lines none took over 2 % longer than with the lines at 640 keys
//   (causal: 2048 and 1408) and the tiles of that time; beyond them most numbers of heads still win, a few lose up to 3 %.
enum class Fwd16 { kTile4, kTile8, kPingPong, kD256, kNone };
static Fwd16 choose_16bit(int d, int N, int causal) {
    switch (d) {
        case 64: return N <= (causal ? 6144 : 896) ? Fwd16::kTile4 : Fwd16::kTile8;
        case 128: return N <= (causal ? 1920 : 896) ? Fwd16::kTile4 : Fwd16::kPingPong;
        case 256: return Fwd16::kD256;
        default: return Fwd16::kNone;
    }
}

template <typename Tag>
static int dispatch_16bit(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int H_kv, int N,
                          int d, float scale, int causal, int schedule, hipStream_t stream) {
    if (schedule != FA_SCHED_AUTO) {
        // forced kernel choice for the scheduling ablation (section 4.2's table, re-done on this chip)
        if (d != 128) return FA_ERR_UNSUPPORTED;
        switch (schedule) {
            case FA_SCHED_LOCKSTEP_4W:
                return launch_16bit<Tag, 128, 64, 4, 1, 0>(q, k, v, o, lse, B, H, H_kv, N, scale, causal, false, stream);
            case FA_SCHED_LOCKSTEP_8W:
                return launch_16bit<Tag, 128, 128, 8, 1, 0>(q, k, v, o, lse, B, H, H_kv, N, scale, causal, false, stream);
            case FA_SCHED_PINGPONG: return launch_pingpong<Tag>(q, k, v, o, lse, B, H, H_kv, N, scale, causal, false, stream);
            default: return FA_ERR_SHAPE;
        }
    }
    const bool few = few_forward((long)B * H, N, d, causal);
    switch (choose_16bit(d, N, causal)) {
        case Fwd16::kTile4:
            if (d == 64) return launch_16bit<Tag, 64, 64, 4, 1, 0>(q, k, v, o, lse, B, H, H_kv, N, scale, causal, few, stream);
            return launch_16bit<Tag, 128, 64, 4, 1, 0>(q, k, v, o, lse, B, H, H_kv, N, scale, causal, few, stream);
        case Fwd16::kTile8: return launch_16bit<Tag, 64, 64, 8, 1, 0>(q, k, v, o, lse, B, H, H_kv, N, scale, causal, few, stream);
        case Fwd16::kPingPong: return launch_pingpong<Tag>(q, k, v, o, lse, B, H, H_kv, N, scale, causal, few, stream);
        case Fwd16::kD256: return launch_d256<Tag>(q, k, v, o, lse, B, H, H_kv, N, scale, causal, few, stream);
        default: return FA_ERR_UNSUPPORTED;
    }
}

// The name a profiler shows for the kernel dispatch_16bit picks (FA_SCHED_AUTO).
const char* fwd_16bit_kernel_name(bool f16, int N, int d, int causal) {
    static const char* const names[2][2][5] = {
        {{"fa_fwd_16bit_kernel<bf16_tag, 64, 64, 4, 1, 0, false>", "fa_fwd_16bit_kernel<bf16_tag, 128, 64, 4, 1, 0, false>",
          "fa_fwd_16bit_kernel<bf16_tag, 64, 64, 8, 1, 0, false>", "fa_fwd_pingpong_kernel<bf16_tag, 64, 4, false>",
          "fa_fwd_d256_kernel<bf16_tag, false>"},
         {"fa_fwd_16bit_kernel<bf16_tag, 64, 64, 4, 1, 0, true>", "fa_fwd_16bit_kernel<bf16_tag, 128, 64, 4, 1, 0, true>",
          "fa_fwd_16bit_kernel<bf16_tag, 64, 64, 8, 1, 0, true>", "fa_fwd_pingpong_kernel<bf16_tag, 64, 4, true>",
          "fa_fwd_d256_kernel<bf16_tag, true>"}},
        {{"fa_fwd_16bit_kernel<f16_tag, 64, 64, 4, 1, 0, false>", "fa_fwd_16bit_kernel<f16_tag, 128, 64, 4, 1, 0, false>",
          "fa_fwd_16bit_kernel<f16_tag, 64, 64, 8, 1, 0, false>", "fa_fwd_pingpong_kernel<f16_tag, 64, 4, false>",
          "fa_fwd_d256_kernel<f16_tag, false>"},
         {"fa_fwd_16bit_kernel<f16_tag, 64, 64, 4, 1, 0, true>", "fa_fwd_16bit_kernel<f16_tag, 128, 64, 4, 1, 0, true>",
          "fa_fwd_16bit_kernel<f16_tag, 64, 64, 8, 1, 0, true>", "fa_fwd_pingpong_kernel<f16_tag, 64, 4, true>",
          "fa_fwd_d256_kernel<f16_tag, true>"}}};
    int idx;
    switch (choose_16bit(d, N, causal)) {
        case Fwd16::kTile4: idx = d == 64 ? 0 : 1; break;
        case Fwd16::kTile8: idx = 2; break;
        case Fwd16::kPingPong: idx = 3; break;
        case Fwd16::kD256: idx = 4; break;
        default: return nullptr;
    }
    return names[f16 ? 1 : 0][causal ? 1 : 0][idx];
}

int launch_fwd_bf16(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int H_kv, int N, int d,
                    float scale, int causal, int schedule, hipStream_t stream) {
    return dispatch_16bit<bf16_tag>(q, k, v, o, lse, B, H, H_kv, N, d, scale, causal, schedule, stream);
}

int launch_fwd_f16(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int H_kv, int N, int d,
                   float scale, int causal, int schedule, hipStream_t stream) {
    return dispatch_16bit<f16_tag>(q, k, v, o, lse, B, H, H_kv, N, d, scale, causal, schedule, stream);
}

int launch_fwd_f32(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int H_kv, int N, int d,
                   float scale, int causal, hipStream_t stream) {
    if (d != 64) return FA_ERR_UNSUPPORTED;
    constexpr int BR = 64;
    int n_qtiles = (N + BR - 1) / BR;
    long total = (long)B * H * n_qtiles;
    if (total > 0x7fffffffL) return FA_ERR_SHAPE;
    auto qp = static_cast<const float*>(q);
    auto kp = static_cast<const float*>(k);
    auto vp = static_cast<const float*>(v);
    auto op = static_cast<float*>(o);
    const long heads = (long)B * H;
    if (f32_short(N)) {
        const dim3 waves((unsigned)((heads + 3) / 4));
        if (causal)
            hipLaunchKernelGGL(fa_fwd_f32_short_kernel<true>, waves, dim3(256), 0, stream, qp, kp, vp, op, lse, N, (int)heads, H / H_kv, scale);
        else
            hipLaunchKernelGGL(fa_fwd_f32_short_kernel<false>, waves, dim3(256), 0, stream, qp, kp, vp, op, lse, N, (int)heads, H / H_kv, scale);
        return hipGetLastError() == hipSuccess ? FA_OK : FA_ERR_LAUNCH;
    }
    // HIP takes fewer than 2^32 threads along a grid's x: beyond that, as many heads at a time as fit
    constexpr int kThreads = 512;
    const long most = ((1L << 32) - 1) / kThreads / n_qtiles;
    for (long head = 0; head < heads; head += most) {
        const int items = (int)((heads - head < most ? heads - head : most) * n_qtiles);
        if (causal)
            hipLaunchKernelGGL((fa_fwd_f32_kernel<64, 32, true>), dim3((unsigned)items), dim3(kThreads), 0, stream, qp, kp, vp, op, lse, N,
                               n_qtiles, items, (int)head, H / H_kv, scale);
        else
            hipLaunchKernelGGL((fa_fwd_f32_kernel<64, 32, false>), dim3((unsigned)items), dim3(kThreads), 0, stream, qp, kp, vp, op, lse, N,
                               n_qtiles, items, (int)head, H / H_kv, scale);
        if (hipGetLastError() != hipSuccess) return FA_ERR_LAUNCH;
    }
    return FA_OK;
}

}  // namespace fa

FA_CLOCK_SPAN_READER(fa_debug_clock_span_fwd)
