// Block-structured linear  y = x W + b  (+ s (x A_k) B_k)  with fused epilogues (Sec. 3.1), bf16 with fp32 accumulators.
// (Small calls, fp32, and contractions or widths that do not fit these tiles: gemm_ks.hip.)
//
// The low-rank expand (x A_k) B_k is one more K step of the same MFMA per 16 ranks, fed with the
// shrink output S and the adapter's Bt slab, so W + A_k B_k is never formed and the base product of
// an input block is shared by all the row-blocks that fan out of it.
#include "rowtile.h"

#include <utility>

namespace {

// ------------------------------------------------------------------ bf16 MFMA, K % 64 == 0 and N % 8 == 0
// BM x BN x 64 tiles, v_mfma_f32_32x32x16_bf16.
//
// Loads: global_load_lds_dwordx4 -- each wave instruction drops 64 x 16 bytes (8 tile rows of 64 elements)
// straight into LDS, so up to NS k-tiles are in flight per workgroup without costing registers.  The lane that
// fills position p of row r fetches chunk p ^ ((r >> 1) & 7): a swizzle that keeps 16-byte reads free of bank
// conflicts for 8 or 16 lanes per LDS cycle, without padding.  Waits are counted by hand (vmcnt = loads of
// the k-tiles still allowed in flight) and the barrier is a bare s_barrier, because a fenced barrier would
// drain every outstanding load.
//
// Main loop: fragments are read a 16-column step ahead of their MFMAs, across the barrier too, and nothing in it makes the compiler wait for more
// than the reads it needs (no scalar load outstanding, no branch around a load).  Reads, wait and MFMAs of a step one after the other left the
// matrix unit idle for a read's latency in every step: 22655 x 3072 -> 768 166 us (256 x 128 tiles; now 146), 50432 x 768 -> 2304 514 k cycles at
// 2.10 GHz (256 x 256; now 479 k).  The second gains 3 % of time for 7 % of cycles: the clock follows the power, 2.02 GHz now.
//
// The product is accumulated transposed (Wt fragment as the A operand) so that a lane ends up with four
// consecutive output columns of one row; the epilogue adds the low-rank expand as one more MFMA K step per
// 16 ranks, stages fp32 rows through LDS with 16-byte writes and stores whole 128/256-byte row segments,
// adding bias, residual and position rows with vector loads.
//
// Tile order: workgroup ids are dealt round-robin to the 8 XCDs, so id % 8 picks the XCD.  The tiles, ordered by panel of
// PANEL column tiles, then row tile, then column tile, are cut into eight equal runs, one per XCD: an XCD works on one
// W panel at a time (it stays in that XCD's 4 MB L2 instead of all of W streaming past every row tile) and the XCDs
// finish together (a ninth of a round more on one XCD is a whole round more for the kernel).

template <typename F, int... I> __device__ __forceinline__ void static_for_each(F f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>()), ...); }
template <int N, typename F> __device__ __forceinline__ void static_for(F f) { static_for_each(f, std::make_integer_sequence<int, N>()); }

// BM x BN tile, WM x WN waves, each wave (BM/WM) x (BN/WN) = (MI*32) x (NJ*32); NS LDS stages of 64 k-columns.
// EK, the epilogue: 0 = subtile by subtile (fp32 output with residual / position rows, or one column subtile per wave);
// 1, 2 = row-wise for bf16 output (two column subtiles per wave): 2 when the host knows that a wave's region touches at most two
// input blocks and every output block has one low-rank term of at most 16 ranks (all operands of a pass prefetched), 1 otherwise;
// 3 = the same conditions and prefetching as 2 for fp32 output with a residual (no position rows), staged 32 rows at a time.
// In a kernel of two tiles the compiler merges their loads and loses sight of the bases being uniform.
template <bool TWO, typename T> __device__ __forceinline__ const T *uniform(const T *p)
{
    if (!TWO) return p;
    const uintptr_t v = (uintptr_t)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return (const T *)((uintptr_t)hi << 32 | lo);
}

// One tile (TWO: the kernel has one of another size too): rows t0 .. of block xb (of the run of rows over all blocks, of which Tlim exist: xb = 0), columns n0 ..
template <int BM, int BN, int WM, int WN, int NS, int EK, bool TWO>
__device__ __forceinline__ void dma_tile(const GemmArgs &g, const bool flat, const int Tlim, const int xb, const int t0, const int n0)
{
    constexpr int BK = 64, NW = WM * WN;
    constexpr int MI = BM / WM / 32, NJ = BN / WN / 32;   // 32 x 32 subtiles per wave
    constexpr int A_EL = BM * BK, B_EL = BN * BK, STAGE_EL = A_EL + B_EL;
    constexpr int NC = NJ * 8;                             // 16-byte chunks per staged fp32 row (NJ*32 columns)
    constexpr int AG = BM / 8 / NW, BG = BN / 8 / NW;      // 8-row groups (1 KB each) per wave and stage
    constexpr int NLD = AG + BG;                           // loads per wave and stage
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0 && (NS - 1) * NLD <= 63, "tile / wave layout");
    static_assert(NW * 32 * NC * 16 <= NS * STAGE_EL * 2, "staging must fit in the tile ring");
    extern __shared__ __attribute__((aligned(16))) bf16_t dsmem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN, lm = lane & 31, lh = lane >> 5;
    const bf16_t *A = (const bf16_t *)g.A + (size_t)xb * g.T * g.K;
    const bf16_t *Wt = (const bf16_t *)g.Wt;

    // rows past the end of the block / of W are clamped: their products land in accumulator rows / columns that
    // are never stored
    const int lr = lane >> 3;   // row inside an 8-row group; lane & 7 = position inside the row
    unsigned ga[AG], gb[BG];                               // bytes (the host has checked that they fit)
#pragma unroll
    for (int i = 0; i < AG; ++i) {
        const int row = (wave * AG + i) * 8 + lr;
        ga[i] = 2u * (unsigned)(min(t0 + row, g.T - 1) * g.K + (((lane & 7) ^ ((row >> 1) & 7)) << 3));
    }
#pragma unroll
    for (int i = 0; i < BG; ++i) {
        const int row = (wave * BG + i) * 8 + lr;
        gb[i] = 2u * (unsigned)(min(n0 + row, g.N - 1) * g.K + (((lane & 7) ^ ((row >> 1) & 7)) << 3));
    }
    const int nk = g.K / BK;
    const unsigned ring = __builtin_amdgcn_readfirstlane(lds_addr_of(dsmem));
    auto issue_one = [&](int kt, int s, auto load) {        // one of the NLD loads of this wave for k-tile kt into stage s; past the last
        constexpr int l = decltype(load)::value, i = l < AG ? l : l - AG;       // k-tile it moves nothing, so that the waits count the same
        const int go = nk - kt;                                                 // loads everywhere
        const unsigned st = ring + s * (STAGE_EL * 2);
        if constexpr (l < AG) glds16_if(uniform<TWO>(A + (size_t)kt * BK), ga[i], st + (wave * AG + i) * 1024, go);
        else glds16_if(uniform<TWO>(Wt + (size_t)kt * BK), gb[i], st + A_EL * 2 + (wave * BG + i) * 1024, go);
    };

    // Row-wise epilogue (two column subtiles per wave, bf16 output): the accumulators start from the bias, so no output block
    // has to add it later.  It comes through LDS with the tiles: the compiler would wait for all of them before it used a register load.
    constexpr bool RW = EK > 0;
    static_assert(!RW || NJ == 2, "row-wise epilogue: two column subtiles per wave");
    float *const bias_s = (float *)(dsmem + NS * STAGE_EL);
    if constexpr (RW) {
        if (g.bias && wave == 0 && lane < BN / 4) glds16_s(g.bias, 4u * (unsigned)min(n0 + 4 * lane, g.N - 4), ring + NS * STAGE_EL * 2);
    }

    // The tile loads need nothing but the tile coordinates, so they go out first; the fan-out offsets and the adapter id are
    // read while they fly.  A tile whose block has no output drains its loads and leaves.
#pragma unroll
    for (int s = 0; s < NS; ++s) static_for<NLD>([&](auto l) { issue_one(s, s, l); });
    int ob0 = xb, ob1 = xb + 1;
    if (g.out_off && !flat) { ob0 = g.out_off[xb]; ob1 = g.out_off[xb + 1]; }
    if (ob0 >= ob1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }

    // operands of the low-rank expand for ranks [s0, s0 + 16) of output block ob: S rows of this wave's MI row
    // subtiles and Bt rows of its NJ column subtiles (rows past T / columns past N are clamped or zero: they only
    // feed results that are never stored)
    const bf16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
    auto load_fs = [&](bf16x8(&fs)[MI], int ob, int s0) {
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int t = min(t0 + wm * MI * 32 + i * 32 + lm, g.T - 1);
            fs[i] = *(const bf16x8 *)((const bf16_t *)g.S + ((size_t)ob * g.T + t) * g.RP + s0 + lh * 8);
        }
    };
    auto load_fw = [&](bf16x8(&fw)[NJ], int k_ad, int s0) {
        const bf16_t *Bt = (const bf16_t *)g.Bt + (size_t)k_ad * g.N * g.r;
        const int j0 = s0 + lh * 8;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int bcol = n0 + wn * NJ * 32 + j * 32 + lm;
            bf16x8 f = zero8;
            if (bcol < g.N) {
                const bf16_t *p = Bt + (size_t)bcol * g.r + j0;
                if ((g.r & 7) == 0) {
                    if (j0 + 8 <= g.r) f = *(const bf16x8 *)p;
                } else {
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        if (j0 + q < g.r) f[q] = p[q];
                }
            }
            fw[j] = f;
        }
    };
    // small tiles have registers to spare: fetch the first output block's expand operands now, so that their
    // latency hides behind the main loop.  They are younger than the prologue's tile loads, so the in-order load
    // counter used below can only over-wait (by these few loads), never under-wait.
    constexpr bool EARLY = MI * NJ <= 4;
    const bool has_lora = g.S && g.adapter_of_out;
    bf16x8 fs0[MI], fw0[NJ];
    int k_ad0 = -1;
    if (EARLY && has_lora && !flat && !g.set_off) {
        k_ad0 = g.adapter_of_out[ob0];
        if (k_ad0 >= 0) { load_fs(fs0, ob0, 0); load_fw(fw0, k_ad0, 0); }
    }

    // Row-wise epilogue: which input blocks this wave's (MI * 32)-row region touches, their fan-out and the adapters of the first
    // two passes.  Every one of these is a chain of dependent loads and each link a full memory round trip under load, so the
    // fan-out offsets are requested here, the adapter ids inside the main loop once the offsets have arrived, and nothing is
    // waited for before the loop has run.
    constexpr int RROWS = MI * 32, RCOLS = NJ * 32;
    static_assert(!RW || NW * RROWS * RCOLS <= NS * STAGE_EL, "bf16 staging must fit in the tile ring");
    int R0 = 0, Rend = 0, Tblk = 1, bbA = 0, bbZ = 0, baseA = 0, tB = 0, oA0 = 0, oA1 = 0, oB0 = 0, oB1 = 0, maxfan = 0;
    int oA0v = 0, oA1v = 0, oB0v = 0, oB1v = 0;               // as loaded (per lane, all lanes equal)
    int kA = -1, kB = -1, kAv = -1, kBv = -1, kAnv = -1, kBnv = -1;   // adapters of the current pass; as loaded: current / next pass
    bool two = true, hasB = false;
    if constexpr (RW) {
        R0 = t0 + wm * RROWS; Rend = min(R0 + RROWS, Tlim);
        if (R0 < Rend) {
            Tblk = flat ? g.Tb : g.T;                         // rows of a block: stride of S and of the output blocks
            bbA = flat ? __builtin_amdgcn_readfirstlane(R0 / Tblk) : xb; bbZ = flat ? __builtin_amdgcn_readfirstlane((Rend - 1) / Tblk) : xb;
            baseA = flat ? bbA * Tblk : 0; tB = baseA + Tblk;  // first row (tile coordinates) of blocks bbA and bbA + 1
            two = bbZ - bbA <= 1; hasB = bbZ > bbA;
            // fan-out of the region's first and last input block (with more than two blocks: looked up per block in the epilogue)
            oA0v = g.out_off ? g.out_off[bbA] : bbA; oA1v = g.out_off ? g.out_off[bbA + 1] : bbA + 1;
            oB0v = g.out_off ? g.out_off[bbZ] : bbZ; oB1v = g.out_off ? g.out_off[bbZ + 1] : bbZ + 1;
        }
    }
    auto fanout_arrived = [&]() {
        oA0 = __builtin_amdgcn_readfirstlane(oA0v); oA1 = __builtin_amdgcn_readfirstlane(oA1v);
        oB0 = __builtin_amdgcn_readfirstlane(oB0v); oB1 = __builtin_amdgcn_readfirstlane(oB1v);
        maxfan = R0 < Rend ? max(oA1 - oA0, oB1 - oB0) : 0;
    };
    auto request_ids = [&](int pp, int &kav, int &kbv) {       // adapters of pass pp for blocks A and B (-1: nothing to add)
        kav = kbv = -1;
        if (!has_lora || pp >= maxfan) return;
        // (as vector loads: an outstanding scalar load would make the compiler wait for all LDS reads at once in the main loop)
        int ia, ib;
        asm("v_mov_b32 %0, %1" : "=v"(ia) : "s"(oA0 + pp));
        asm("v_mov_b32 %0, %1" : "=v"(ib) : "s"(oB0 + pp));
        if (oA0 + pp < oA1) kav = g.adapter_of_out[ia];
        if (hasB && oB0 + pp < oB1) kbv = g.adapter_of_out[ib];
    };

    // fragment rows are wm*MI*32 + i*32 + lm and wn*NJ*32 + j*32 + lm: (row >> 1) & 7 == (lm >> 1) & 7 for all
    const int fa0 = (wm * MI * 32 + lm) * BK, fb0 = A_EL + (wn * NJ * 32 + lm) * BK, sw = (lm >> 1) & 7;
    // Fragments are read one 16-column step ahead of their MFMAs, the first ones of the next k-tile too: the wait for it and the barrier stand
    // before the last step's MFMAs, when every wave has read all of the current k-tile, so its stage can be refilled from there on.
    bf16x8 fa[2][MI], fb[2][NJ];
    auto read_frags = [&](int buf, const bf16_t *tile, int kk) {
        const int ko = ((2 * kk + lh) ^ sw) << 3;
#pragma unroll
        for (int i = 0; i < MI; ++i) fa[buf][i] = *(const bf16x8 *)(tile + fa0 + i * 32 * BK + ko);
#pragma unroll
        for (int j = 0; j < NJ; ++j) fb[buf][j] = *(const bf16x8 *)(tile + fb0 + j * 32 * BK + ko);
    };
    rl_wait_barrier<(NS - 1) * NLD>();
    read_frags(0, dsmem, 0);
    f32x16 acc[MI][NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            f32x4 bq = {0.f, 0.f, 0.f, 0.f};
            if (RW && g.bias) bq = *(const f32x4 *)(bias_s + wn * NJ * 32 + j * 32 + 8 * q + 4 * lh);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] = bq[e];
        }
    if constexpr (EK >= 2) {                                  // (younger than every tile load in flight: the counted waits over-wait at most)
        fanout_arrived();
        request_ids(0, kAv, kBv);
        request_ids(1, kAnv, kBnv);
    }
    int st = 0;                                               // stage of k-tile it
    auto step = [&](auto first, int it) {                     // (k-tile 0 apart: a branch around loads would cost the reads' counted waits)
        const int st_prev = st == 0 ? NS - 1 : st - 1, st_next = st == NS - 1 ? 0 : st + 1;
        const bf16_t *cur = dsmem + st * STAGE_EL;
        static_for<4>([&](auto kk_) {
            constexpr int kk = decltype(kk_)::value, NM = MI * NJ, PER = (NLD + 2) / 3, part = (kk + 1) & 3;
            if constexpr (kk < 3) read_frags((kk + 1) & 1, cur, kk + 1);
            else {
                rl_wait_barrier<(NS - 2) * NLD>();            // k-tile it + 1 has landed, the younger ones may stay in flight
                read_frags(0, dsmem + st_next * STAGE_EL, 0);
            }
            // The refill of the stage that is free, spread over this step and the next two, between the MFMAs.  Issued as one
            // burst the loads hold the wave at the issue stage until the L2 path has taken them, and the MFMAs behind them
            // start that much later.
            __builtin_amdgcn_sched_barrier(0);
            static_for<NM>([&](auto m_) {
                constexpr int m = decltype(m_)::value, from = part * PER + m * PER / NM, to = part * PER + (m + 1) * PER / NM;
                static_for<NLD>([&](auto l) {
                    if constexpr (part < 3 && l() >= from && l() < to) {
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (kk == 3) issue_one(it + NS, st, l);
                        else if constexpr (!decltype(first)::value) issue_one(it - 1 + NS, st_prev, l);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                });
                acc[m / NJ][m % NJ] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[kk & 1][m % NJ], fa[kk & 1][m / NJ], acc[m / NJ][m % NJ], 0, 0, 0);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        st = st_next;
    };
    step(std::true_type(), 0);
    for (int it = 1; it < nk; ++it) step(std::false_type(), it);
    __syncthreads();   // all loads that move something have landed (the last wait leaves none but those switched off) and all waves are done with the tiles

    // ---- row-wise epilogue (bf16 output, two column subtiles per wave).  Per pass p the wave produces, for every row of its
    // (MI * 32) x 64 region, the p-th output block of that row's input block: base product (+ bias, in the accumulators) + the
    // low-rank terms of that output block, GELU, rounding to bf16 -- all in accumulator layout -- then the whole region goes through
    // the wave's own LDS area once (8-byte writes, 16-byte reads, chunks swizzled by row & 7) and leaves as 128-byte row segments,
    // eight rows per store instruction.  A 32-row subtile that straddles two input blocks adds each block's term with the
    // other block's S rows zeroed, so block boundaries cost one more MFMA, not one more trip through LDS.
    if constexpr (RW) {
        bf16_t *stg16 = dsmem + wave * (RROWS * RCOLS);
        if (R0 >= Rend) return;
        if constexpr (EK == 1) {
            fanout_arrived();
            if (!two)
                for (int bb = bbA + 1; bb < bbZ; ++bb) maxfan = max(maxfan, g.out_off ? g.out_off[bb + 1] - g.out_off[bb] : 1);
        }
        const bool gelu = g.mode == EPI_GELU;
        const bf16_t *Sg = (const bf16_t *)g.S;
        const int r8 = lane >> 3, ch = lane & 7;
        const int col = n0 + wn * RCOLS + ch * 8;
        const bool col_ok = col < g.N;

        // one column subtile of results (accumulator layout, fp32) -> GELU -> bf16 -> the wave's staging rows [32 i, 32 i + 32)
        auto stage1 = [&](const f32x16 &cj, int i, int j) {
            const int srow = 32 * i + lm;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 v = {cj[4 * q], cj[4 * q + 1], cj[4 * q + 2], cj[4 * q + 3]};
                if (gelu) v = gelu_poly4(v);
                const bf16x4 w = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
                *(bf16x4 *)(stg16 + srow * RCOLS + ((((j * 4 + q) ^ (srow & 7)) << 3) + 4 * lh)) = w;
            }
        };
        // rows of pass p: staging -> global, 8 rows x 128 bytes per instruction
        auto store_rows = [&](int p) {
            const int obA = (two && oA0 + p < oA1) ? oA0 + p : -1, obB = (two && hasB && oB0 + p < oB1) ? oB0 + p : -1;
#pragma unroll 2
            for (int q = 0; q < RROWS / 8; ++q) {
                const int row = 8 * q + r8, t = R0 + row;
                int ob, trow;
                if (EK == 2 || two) {
                    const bool inB = t >= tB;
                    ob = inB ? obB : obA;
                    trow = t - (inB ? tB : baseA);
                } else {                                      // more than two input blocks in the region: looked up per row
                    const int bb = min(t, Rend - 1) / Tblk;
                    trow = t - bb * Tblk;
                    const int o0 = g.out_off ? g.out_off[bb] : bb, o1 = g.out_off ? g.out_off[bb + 1] : bb + 1;
                    ob = o0 + p < o1 ? o0 + p : -1;
                }
                if (t >= Rend || ob < 0 || !col_ok) continue;
                const bf16x8 v = *(const bf16x8 *)(stg16 + row * RCOLS + ((ch ^ r8) << 3));
                *(bf16x8 *)((bf16_t *)g.out + ((long)ob * g.Tout + g.t_off + trow) * g.N + col) = v;
            }
        };

        if constexpr (EK >= 2) {
            // The host has checked: a region touches at most two input blocks, one low-rank term per output block, rank 8 or 16
            // in one 16-rank step.  All operands of a pass -- the Bt fragments of the two adapters, one S fragment per subtile and
            // one more for the subtile that straddles the block boundary -- are requested together, those of pass p + 1 before
            // the rows of pass p are stored and the adapter ids of pass p + 2 with them: a pass never waits for more than what
            // is left of one round trip.  (Bt columns past N and ranks past r are read from clamped addresses: the former
            // feed columns that are never stored, the latter meet the zero padding of S.)
            bf16x8 fwA[NJ], fwB[NJ], fs1[MI], fs2 = zero8;
            auto request_operands = [&](int pp, int ka, int kb) {
                const int j0 = min(lh * 8, g.r - 8);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const size_t bcol = (size_t)min(n0 + wn * RCOLS + j * 32 + lm, g.N - 1);
                    if (ka >= 0) fwA[j] = *(const bf16x8 *)((const bf16_t *)g.Bt + ((size_t)ka * g.N + bcol) * g.r + j0);
                    if (kb >= 0) fwB[j] = *(const bf16x8 *)((const bf16_t *)g.Bt + ((size_t)kb * g.N + bcol) * g.r + j0);
                }
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    const int tw = R0 + 32 * i;
                    const bool inB = tw >= tB;                    // the subtile's first block
                    if ((inB ? kb : ka) >= 0 && tw < Rend) {
                        const int trow = min(max(tw + lm - (inB ? tB : baseA), 0), Tblk - 1);
                        fs1[i] = *(const bf16x8 *)(Sg + ((size_t)((inB ? oB0 : oA0) + pp) * Tblk + trow) * 16 + lh * 8);
                    }
                    if (!inB && tw + 32 > tB && tB < Rend && kb >= 0) {   // straddles the boundary: block B's rows of this subtile
                        const int trow = min(max(tw + lm - tB, 0), Tblk - 1);
                        fs2 = *(const bf16x8 *)(Sg + ((size_t)(oB0 + pp) * Tblk + trow) * 16 + lh * 8);
                    }
                }
            };
            kA = __builtin_amdgcn_readfirstlane(kAv); kB = __builtin_amdgcn_readfirstlane(kBv);
            request_operands(0, kA, kB);
            // results of subtile i, column subtile j of the current pass: accumulators + the low-rank term(s)
            auto result = [&](int i, int j, int tw) {
                const bool inB = tw >= tB, both = !inB && tw + 32 > tB && tB < Rend && kB >= 0;
                const bf16x8 f1 = (inB || lm < tB - tw) ? fs1[i] : zero8;   // rows of the other block add nothing
                const bf16x8 f2 = lm >= tB - tw ? fs2 : zero8;
                f32x16 cj = acc[i][j];
                if (inB) {
                    if (kB >= 0) cj = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fwB[j], f1, cj, 0, 0, 0);
                } else {
                    if (kA >= 0) cj = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fwA[j], f1, cj, 0, 0, 0);
                    if (both) cj = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fwB[j], f2, cj, 0, 0, 0);
                }
                return cj;
            };
            if constexpr (EK == 2) {
                for (int p = 0; p < maxfan; ++p) {
#pragma unroll
                    for (int i = 0; i < MI; ++i) {
                        const int tw = R0 + 32 * i;
                        if (tw >= Rend) break;
#pragma unroll
                        for (int j = 0; j < NJ; ++j) stage1(result(i, j, tw), i, j);   // one column subtile at a time: 16 live result registers
                    }
                    kA = __builtin_amdgcn_readfirstlane(kAnv); kB = __builtin_amdgcn_readfirstlane(kBnv);
                    if (p + 1 < maxfan) {
                        request_operands(p + 1, kA, kB);
                        request_ids(p + 2, kAnv, kBnv);
                    }
                    store_rows(p);
                }
            } else {
                // fp32 output with a residual: 32 rows at a time through the wave's 8 KB of LDS (16-byte chunks swizzled by row & 15),
                // whole 256-byte row segments out, 4 rows per store.  The residual rows of a subtile are requested before its MFMAs
                // and without per-lane conditions (rows past the end read a clamped row and are dropped at the store).
                float *stg32 = (float *)dsmem + wave * (32 * RCOLS);
                const int rrow = lane >> 4, rch = lane & 15;
                const int col4 = n0 + wn * RCOLS + rch * 4;
                const bool col4_ok = col4 < g.N;
                const int cfix = col4_ok ? col4 : g.N - 4;
                for (int p = 0; p < maxfan; ++p) {
                    const int obA = oA0 + p < oA1 ? oA0 + p : -1, obB = (hasB && oB0 + p < oB1) ? oB0 + p : -1;
                    const int rbA = (g.res && obA >= 0) ? (g.res_block_of_out ? g.res_block_of_out[obA] : obA) : 0;
                    const int rbB = (g.res && obB >= 0) ? (g.res_block_of_out ? g.res_block_of_out[obB] : obB) : 0;
                    // where row 0 of the tile's coordinates would lie in block A and in block B; rows [lo, lo + span) are stored
                    auto row0 = [&](long blk, int base) { return (blk * g.Tout + g.t_off - base) * g.N; };
                    const long rA = row0(rbA, baseA), rB = row0(rbB, tB), wA = row0(max(obA, 0), baseA), wB = row0(max(obB, 0), tB);
                    const int lo = obA >= 0 ? R0 : tB, hi = obB >= 0 ? Rend : min(Rend, tB);
                    const unsigned span = col4_ok ? max(hi - lo, 0) : 0;
                    int trow0 = R0 + rrow;
                    asm volatile("" : "+v"(trow0));           // (or the rows' offsets are worked out ahead of the passes and kept)
                    constexpr int RQ = MI > 2 ? 4 : 8;        // residual loads in flight (with four row subtiles per wave eight do not fit beside the accumulators)
#pragma unroll
                    for (int i = 0; i < MI; ++i) {
                        const int tw = R0 + 32 * i;
                        if (tw >= Rend) break;
                        f32x4 rv[RQ];
                        auto request_res = [&](int q) {
                            const int t = min(trow0 + 32 * i + 4 * q, Rend - 1);
                            const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
                            rv[q % RQ] = g.res ? *(const f32x4 *)(g.res + (t >= tB ? rB : rA) + (long)t * g.N + cfix) : z4;
                        };
                        auto finish_row = [&](int q) {
                            const int row = 4 * q + rrow, t = trow0 + 32 * i + 4 * q;
                            const f32x4 v = *(const f32x4 *)(stg32 + row * RCOLS + ((rch ^ (row & 15)) << 2)) + rv[q % RQ];
                            if ((unsigned)(t - lo) < span) *(f32x4 *)((float *)g.out + (t >= tB ? wB : wA) + (long)t * g.N + col4) = v;
                        };
#pragma unroll
                        for (int q = 0; q < RQ; ++q) request_res(q);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int j = 0; j < NJ; ++j) {
                            const f32x16 cj = result(i, j, tw);
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const f32x4 v = {cj[4 * q], cj[4 * q + 1], cj[4 * q + 2], cj[4 * q + 3]};
                                *(f32x4 *)(stg32 + lm * RCOLS + (((j * 8 + 2 * q + lh) ^ (lm & 15)) << 2)) = v;
                            }
                        }
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            if (q == RQ) __builtin_amdgcn_sched_barrier(0);
                            finish_row(q);
                            if (q + RQ < 8) request_res(q + RQ);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    kA = __builtin_amdgcn_readfirstlane(kAnv); kB = __builtin_amdgcn_readfirstlane(kBnv);
                    if (p + 1 < maxfan) {
                        request_operands(p + 1, kA, kB);
                        request_ids(p + 2, kAnv, kBnv);
                    }
                }
            }
        } else {
            for (int p = 0; p < maxfan; ++p) {
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    const int tw = R0 + 32 * i;
                    if (tw >= Rend) break;
                    f32x16 c[NJ];
#pragma unroll
                    for (int j = 0; j < NJ; ++j) c[j] = acc[i][j];
                    if (has_lora) {
                        const int twe = min(tw + 32, Rend);
                        const int b_lo = flat ? tw / Tblk : xb, b_hi = flat ? (twe - 1) / Tblk : xb;
                        for (int bb = b_lo; bb <= b_hi; ++bb) {
                            const int o0 = g.out_off ? g.out_off[bb] : bb, o1 = g.out_off ? g.out_off[bb + 1] : bb + 1;
                            const int ob = o0 + p;
                            if (ob >= o1) continue;
                            const int rb0 = flat ? bb * Tblk : 0;
                            const int lo = max(rb0 - tw, 0), hi = min(rb0 + Tblk - tw, 32);   // rows [lo, hi) of the subtile lie in block bb
                            const int trow = min(max(tw + lm - rb0, 0), Tblk - 1);
                            const int sb0 = g.set_off ? g.set_off[ob] : ob, sb1 = g.set_off ? g.set_off[ob + 1] : ob + 1;
                            for (int sb = sb0; sb < sb1; ++sb) {
                                const int k_ad = g.adapter_of_out[sb];
                                if (k_ad < 0) continue;
                                for (int s0 = 0; s0 < g.RP; s0 += 16) {
                                    bf16x8 fsb = *(const bf16x8 *)(Sg + ((size_t)sb * Tblk + trow) * g.RP + s0 + lh * 8);
                                    if (lm < lo || lm >= hi) fsb = zero8;
                                    bf16x8 fwb[NJ];
                                    load_fw(fwb, k_ad, s0);
#pragma unroll
                                    for (int j = 0; j < NJ; ++j) c[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fwb[j], fsb, c[j], 0, 0, 0);
                                }
                            }
                        }
                    }
#pragma unroll
                    for (int j = 0; j < NJ; ++j) stage1(c[j], i, j);
                }
                store_rows(p);
            }
        }
        return;
    }

    // ---- epilogue, wave by wave and 32 rows at a time: no workgroup barrier is needed because each wave stages
    // through its own LDS region and the LDS executes one wave's instructions in order.
    // acc[i][j][e] = C[row wm*MI*32 + i*32 + lm][col wn*NJ*32 + j*32 + 8*(e/4) + 4*lh + e%4]
    float *stg = (float *)dsmem + wave * (32 * NC * 4);   // 32 rows x NC chunks of 4 floats; chunk ch of row r at ch ^ swz(r)
    auto swz = [](int r) { return NC == 16 ? (r & 15) : ((r >> 1) & 7); };

    // read-back mapping: NC consecutive lanes cover one row segment; each pass covers 64 / NC rows
    constexpr int RPP = 64 / NC;
    const int rch = lane % NC, rrow = lane / NC;
    const int col = n0 + wn * NJ * 32 + rch * 4;
    const bool col_ok = col < g.N;
    f32x4 bias4 = {0.f, 0.f, 0.f, 0.f};
    if (g.bias && col_ok) bias4 = *(const f32x4 *)(g.bias + col);
    const bool gelu = g.mode == EPI_GELU;

    // one 32-row subtile of one output block: c -> LDS -> global.  Row 0 of the subtile is row trow0 of the block (negative
    // when the block starts inside the subtile); rows [lo, hi) of the subtile are stored.
    auto emit = [&](f32x16(&c)[NJ], int ob, int rb, int trow0, int lo, int hi) {
        const long obase = ((long)ob * g.Tout + g.t_off + trow0) * g.N + col;
        const float *res = (g.mode == EPI_RESID && g.res) ? g.res + ((long)rb * g.Tout + g.t_off + trow0) * g.N + col : nullptr;
        const float *pos = (g.mode == EPI_RESID && g.pos) ? g.pos + (long)(g.t_off + trow0) * g.N + col : nullptr;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ch = j * 8 + 2 * q + lh;
                const f32x4 v = {c[j][4 * q], c[j][4 * q + 1], c[j][4 * q + 2], c[j][4 * q + 3]};
                *(f32x4 *)(stg + lm * (NC * 4) + ((ch ^ swz(lm)) << 2)) = v;
            }
        // LDS -> global
        if (g.mode == EPI_RESID) {
            float *out = (float *)g.out + obase;
#pragma unroll 2
            for (int q = 0; q < 32 / RPP; ++q) {
                const int row = q * RPP + rrow;
                if (row < lo || row >= hi || !col_ok) continue;
                f32x4 v = *(const f32x4 *)(stg + row * (NC * 4) + ((rch ^ swz(row)) << 2)) + bias4;
                if (res) v += *(const f32x4 *)(res + (long)row * g.N);
                if (pos) v += *(const f32x4 *)(pos + (long)row * g.N);
                *(f32x4 *)(out + (long)row * g.N) = v;
            }
        } else {
            bf16_t *out = (bf16_t *)g.out + obase;
#pragma unroll 2
            for (int q = 0; q < 32 / RPP; ++q) {
                const int row = q * RPP + rrow;
                if (row < lo || row >= hi || !col_ok) continue;
                f32x4 v = *(const f32x4 *)(stg + row * (NC * 4) + ((rch ^ swz(row)) << 2)) + bias4;
                if (gelu) {
#pragma unroll
                    for (int z = 0; z < 4; ++z) v[z] = gelu_poly(v[z]);
                }
                const bf16x4 w = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
                *(bf16x4 *)(out + (long)row * g.N) = w;
            }
        }
    };

    if (flat) {
        // Row tiles that ignore block boundaries.  The 32 rows of a subtile lie in one block or (a block being at least 32
        // rows, else in several) in consecutive ones: block by block, every row-block that fans out of it gets its own
        // expand, fed with the S rows of that row-block only, and stores its rows of the subtile.
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int tw = t0 + wm * MI * 32 + i * 32;     // first row of this 32-row subtile
            if (tw >= Tlim) break;
            int lo = 0;
            for (int bb = tw / g.Tb; lo < 32 && bb * g.Tb < Tlim; ++bb) {   // (blocks past the true count have no valid ids)
                const int trow0 = tw - bb * g.Tb;
                const int hi = min(32, g.Tb - trow0);                       // rows [lo, hi) of the subtile belong to block bb
                const int o0 = g.out_off ? g.out_off[bb] : bb, o1 = g.out_off ? g.out_off[bb + 1] : bb + 1;
                for (int ob = o0; ob < o1; ++ob) {
                    const int rb = (g.mode == EPI_RESID && g.res) ? (g.res_block_of_out ? g.res_block_of_out[ob] : ob) : 0;
                    f32x16 c[NJ];
#pragma unroll
                    for (int j = 0; j < NJ; ++j) c[j] = acc[i][j];
                    const int sb0 = g.set_off ? g.set_off[ob] : ob, sb1 = g.set_off ? g.set_off[ob + 1] : ob + 1;
                    for (int sb = sb0; has_lora && sb < sb1; ++sb) {     // one low-rank term, or all the terms summed on this block
                        const int k_ad = g.adapter_of_out[sb];
                        if (k_ad < 0) continue;
                        const int t = min(max(trow0 + lm, 0), g.Tb - 1);
                        for (int s0 = 0; s0 < g.RP; s0 += 16) {
                            bf16x8 fsb = *(const bf16x8 *)((const bf16_t *)g.S + ((size_t)sb * g.Tb + t) * g.RP + s0 + lh * 8);
                            if (lm < lo || lm >= hi) fsb = zero8;
                            bf16x8 fwb[NJ];
                            load_fw(fwb, k_ad, s0);
#pragma unroll
                            for (int j = 0; j < NJ; ++j) c[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fwb[j], fsb, c[j], 0, 0, 0);
                        }
                    }
                    emit(c, ob, rb, trow0, lo, hi);
                }
                lo = hi;
            }
        }
        return;
    }

    if (g.set_off) {
        // several low-rank terms summed on one output block: operands fetched term by term, one subtile at a time
        for (int ob = ob0; ob < ob1; ++ob) {
            const int rb = (g.mode == EPI_RESID && g.res) ? (g.res_block_of_out ? g.res_block_of_out[ob] : ob) : 0;
            const int sb0 = g.set_off[ob], sb1 = g.set_off[ob + 1];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const int tw = t0 + wm * MI * 32 + i * 32;
                if (tw >= g.T) break;
                f32x16 c[NJ];
#pragma unroll
                for (int j = 0; j < NJ; ++j) c[j] = acc[i][j];
                for (int sb = sb0; has_lora && sb < sb1; ++sb) {
                    const int k_ad = g.adapter_of_out[sb];
                    if (k_ad < 0) continue;
                    const int t = min(tw + lm, g.T - 1);
                    for (int s0 = 0; s0 < g.RP; s0 += 16) {
                        const bf16x8 fsb = *(const bf16x8 *)((const bf16_t *)g.S + ((size_t)sb * g.T + t) * g.RP + s0 + lh * 8);
                        bf16x8 fwb[NJ];
                        load_fw(fwb, k_ad, s0);
#pragma unroll
                        for (int j = 0; j < NJ; ++j) c[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fwb[j], fsb, c[j], 0, 0, 0);
                    }
                }
                emit(c, ob, rb, tw, 0, min(32, g.T - tw));
            }
        }
        return;
    }

    for (int ob = ob0; ob < ob1; ++ob) {
        const int k_ad = has_lora ? g.adapter_of_out[ob] : -1;
        const int rb = (g.mode == EPI_RESID && g.res) ? (g.res_block_of_out ? g.res_block_of_out[ob] : ob) : 0;
        bf16x8 fs[MI], fw[NJ];
        if (k_ad >= 0) {
            if (EARLY && ob == ob0) {
#pragma unroll
                for (int i = 0; i < MI; ++i) fs[i] = fs0[i];
#pragma unroll
                for (int j = 0; j < NJ; ++j) fw[j] = fw0[j];
            } else {
                if (EARLY) { load_fs(fs, ob, 0); load_fw(fw, k_ad, 0); }
            }
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int tw = t0 + wm * MI * 32 + i * 32;     // first row of this 32-row subtile
            if (tw >= g.T) break;
            f32x16 c[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) c[j] = acc[i][j];
            if (k_ad >= 0) {
                // low-rank expand: one more MFMA K step per 16 ranks
                if (!EARLY) {   // large tiles are short of registers: operands are fetched one subtile at a time
                    const int t = min(tw + lm, g.T - 1);
                    fs[i] = *(const bf16x8 *)((const bf16_t *)g.S + ((size_t)ob * g.T + t) * g.RP + lh * 8);
                    load_fw(fw, k_ad, 0);
                }
#pragma unroll
                for (int j = 0; j < NJ; ++j) c[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[j], fs[i], c[j], 0, 0, 0);
                for (int s0 = 16; s0 < g.RP; s0 += 16) {
                    bf16x8 fs2[MI], fw2[NJ];
                    load_fs(fs2, ob, s0);
                    load_fw(fw2, k_ad, s0);
#pragma unroll
                    for (int j = 0; j < NJ; ++j) c[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw2[j], fs2[i], c[j], 0, 0, 0);
                }
            }
            emit(c, ob, rb, tw, 0, min(32, g.T - tw));
        }
    }
}

// TAIL: the rows past the full rounds on 128 x 128 tiles of the same eight waves, four stages of them in the large tiles' ring (gemm_tiles.h)
template <int BM, int BN, int WM, int WN, int NS, int EK> struct DmaKernel {
    static constexpr bool TAIL = EK > 0 && has_tail(BM, BN, EK == 3 ? EPI_RESID : EPI_STORE, true);
    static constexpr int THREADS = 64 * WM * WN, RING = NS * (BM + BN) * 128, BIAS = EK > 0 ? BN * 4 : 0;
    static constexpr int TAIL_LDS = TAIL ? 4 * (128 + 128) * 128 + 128 * 4 : 0;
    static constexpr int LDS = RING + BIAS > TAIL_LDS ? RING + BIAS : TAIL_LDS;
};

template <int BM, int BN, int WM, int WN, int NS, int EK>
__global__ __launch_bounds__(64 * WM * WN, (BM * BN >= 256 * 256 || NS * (BM + BN) * 128 > 80 * 1024) ? 1 : 2)
void gemm_bf16_dma_kernel(const GemmArgs g, int tiles_m, int tiles_n)
{
    constexpr int PANEL = panel_tiles(BN);
    // The eight runs are cut from the tiles that exist: the grid is sized for the caller's bound on the blocks, which can be
    // half as many again as the true count, and the tiles past it would all fall on the last XCDs (config 3 with room for 3
    // adapters on each of 64 frames: five of eight XCDs busy, 178 us per qkv or fc1 launch instead of 131).  The workgroups left over exit at once.
    const bool flat = g.Tb > 0;                            // one run of rows over all blocks: xb = 0, t0 = first row of the tile
    const int n_bound = flat ? g.nb : g.n_in;
    const int n_true = g.n_in_dev ? __builtin_amdgcn_readfirstlane(min(*g.n_in_dev, n_bound)) : n_bound;
    const int Tlim = flat ? n_true * g.Tb : g.T;           // rows that exist
    const int xcd = blockIdx.x & 7;                        // workgroups are dealt round-robin to the XCDs
    constexpr bool TAIL = DmaKernel<BM, BN, WM, WN, NS, EK>::TAIL;
    const int large = TAIL && flat ? large_tile_rows(Tlim, g.N, BM, BN) : Tlim;
    int j = blockIdx.x >> 3, mt, tn;
    const bool has = xcd_tile(xcd, j, flat ? (large + BM - 1) / BM : n_true * tiles_m, tiles_n, PANEL, mt, tn);
    if constexpr (TAIL) {
        if (!has) {
            if (large < Tlim && xcd_tile(xcd, j, (Tlim - large + 127) / 128, (g.N + 127) / 128, panel_tiles(128), mt, tn))
                dma_tile<128, 128, 4, 2, 4, EK, true>(g, true, Tlim, 0, large + mt * 128, tn * 128);
            return;
        }
    } else {
        if (!has) return;
    }
    const int xb = mt / tiles_m;
    dma_tile<BM, BN, WM, WN, NS, EK, TAIL>(g, flat, Tlim, xb, (mt - xb * tiles_m) * BM, tn * BN);
}

}  // namespace

template <int BM, int BN, int WM, int WN, int NS> static void launch_dma(const GemmArgs &g, hipStream_t st);

template <int BM, int BN, int WM, int WN, int NS, int EK>
static void launch_dma_ek(const GemmArgs &g, hipStream_t st)
{
    using K = DmaKernel<BM, BN, WM, WN, NS, EK>;
    auto kern = gemm_bf16_dma_kernel<BM, BN, WM, WN, NS, EK>;
    if (K::LDS > 64 * 1024) {
        static bool attr_set = false;   // raising the dynamic LDS limit is a per-kernel, process-wide setting
        if (!attr_set) {
            (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, K::LDS);
            attr_set = true;
        }
    }
    const int tiles_m = (g.T + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    const long run = xcd_workgroups((long)g.n_in * tiles_m * tiles_n, K::TAIL && g.Tb, !g.n_in_dev, g.T, g.N, BM, BN);
    POLY_LAUNCH_SHMEM(POLY_STAGE_GEMM, kern, dim3((unsigned)(8 * run)), dim3(K::THREADS), K::LDS, st, g, tiles_m, tiles_n);
}

template <int BM, int BN, int WM, int WN, int NS>
static void launch_dma(const GemmArgs &g, hipStream_t st)
{
    if constexpr (BN / WN == 64) {
        // a wave's region of BM / WM rows touches at most two input blocks when a block is at least that long (or when tiles
        // stay inside blocks: Tb == 0)
        const bool two_blocks = g.Tb == 0 || g.Tb >= BM / WM;
        const bool prefetchable = two_blocks && !g.set_off && (!g.S || (g.RP == 16 && g.r % 8 == 0));
        if (g.mode != EPI_RESID) {
            if (prefetchable) launch_dma_ek<BM, BN, WM, WN, NS, 2>(g, st);
            else launch_dma_ek<BM, BN, WM, WN, NS, 1>(g, st);
            return;
        }
        if (prefetchable && !g.pos) { launch_dma_ek<BM, BN, WM, WN, NS, 3>(g, st); return; }
    }
    launch_dma_ek<BM, BN, WM, WN, NS, 0>(g, st);
}

static long product_tiles(const GemmArgs &g, int bm, int bn) { return product_tiles(g.n_in, g.T, g.N, bm, bn); }

static int launch_gemm_dma(const GemmArgs &g, GemmCount count, hipStream_t st)
{
    if (g.pos) {                                           // patch embedding: row tiles inside blocks, an epilogue that fetches nothing ahead
        if (g.N % 128 == 0) launch_dma<128, 128, 2, 2, 2>(g, st);
        else if (product_tiles(g, 128, 64) < 256) launch_dma<64, 64, 2, 2, 4>(g, st);    // (147 tiles of 128 x 64: 14.3 us, as 64 x 64 9 us)
        else launch_dma<128, 64, 2, 2, 2>(g, st);
        return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
    }
    const float terms = g.out_off || g.set_off ? (float)count.terms / (g.Tb ? g.nb : g.n_in) : 1.f;
    switch (cheapest_tile({g.n_in, g.T, g.Tb, g.K, g.N, g.S ? g.RP : 0, g.r, g.mode, g.out_off ? terms : 1.f, terms, g.set_off != nullptr,
                           !g.n_in_dev || count.known})) {
    case TILE_128x64: launch_dma<128, 64, 4, 1, 2>(g, st); break;
    case TILE_128x128: launch_dma<128, 128, 4, 2, 2>(g, st); break;
    case TILE_256x128: launch_dma<256, 128, 4, 2, 3>(g, st); break;
    case TILE_256x256: launch_dma<256, 256, 2, 4, 2>(g, st); break;
    case TILE_64x64: launch_dma<64, 64, 2, 2, 4>(g, st); break;
    case TILE_128x64_TALL: launch_dma<128, 64, 2, 2, 2>(g, st); break;
    default: launch_dma<128, 128, 2, 2, 2>(g, st);
    }
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

int launch_gemm(const GemmArgs &g, GemmCount count, int dtype, hipStream_t st)
{
    if (g.n_in <= 0 || g.T <= 0) return POLY_OK;
    const bool bf16 = dtype == POLY_BF16;
    if (g.K % (bf16 ? 8 : 4) != 0 || (g.S && g.RP % 16 != 0)) return POLY_EINVAL;
    const long rows = (long)g.n_in * g.T;
    if (bf16 && ((long)g.N * g.K > 0x7fffffffL || (long)g.T * g.K > 0x7fffffffL)) return POLY_EINVAL;
    // input blocks stored back to back and nothing but the output block indexed by the row inside a block: the row
    // tiles run over all input blocks as one (a 197-row block fills only 77 % of a 256-row tile of its own)
    GemmArgs gf = g;
    if (g.Tout == g.T && g.t_off == 0 && !g.pos && g.n_in > 1 && g.T % 256 != 0 && rows <= 0x7fffffffL &&
        (!bf16 || (rows * g.K <= 0x7fffffffL && rows * g.N <= 0x7fffffffL))) {
        gf.Tb = g.T; gf.nb = g.n_in;
        gf.T = (int)rows; gf.n_in = 1;          // (Tout stays the block length: it places the output blocks)
    }
    if (!bf16 || g.K % 64 != 0 || g.N % 8 != 0 || !gemm_aligned(g)) return launch_gemm_ks(gf, dtype, st);
    if (g.T == 1 && g.S && one_row_split(rows, g.N, g.K, g.RP, g.out_off != nullptr, g.set_off != nullptr)) return launch_gemm_ks(gf, dtype, st);
    // A long contraction on fewer 128 x 128 tiles than half the CUs is split over the waves (gemm_ks.hip) where tiles of 32 x 64 get a CU each, and
    // above a contraction of 1024 also where tiles of 64 x 64 do.  us per product of the 768-wide backbone, split / tiles of 64 x 64 on a shared ring /
    // 128 x 128 (rows x K -> N):
    //   197 x 768 -> 2304  7.6 / 7.0 / 11.9    591 x 768 -> 768   9.3 / 9.1 / 14.6    591 x 3072 -> 768   14.6 / 18.0 / 38.8
    //   197 x 768 -> 3072  9.0 / 7.4 / 13.4    985 x 768 -> 768  10.7 / 9.2 / 14.9    1182 x 3072 -> 768  19.0 / 19.2 / 39.1
    //   591 x 768 -> 2304 16.9 / 9.8 / 12.3    1576 x 768 -> 768 17.8 / 11.0 / 15.0   1576 x 3072 -> 768  32.4 / 25.3 / 39.0
    //   591 x 768 -> 3072 18.0 / 10.9 / 13.7   985 x 768 -> 2304 23.8 / 14.7 / 12.6 (144 tiles of 128 x 128)
    if (g.K >= 512 && product_tiles(gf, 128, 128) < 128 && (product_tiles(gf, 32, 64) <= 256 || (g.K > 1024 && product_tiles(gf, 64, 64) <= 256)))
        return launch_gemm_ks(gf, dtype, st);
    return launch_gemm_dma(gf, count, st);
}
