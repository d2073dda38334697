// Everything of a pre-LN transformer layer that works row by row, for narrow models (D <= 192), in one kernel
// on tiles of 64 token rows:
//
//   A   x' = res + o Wp + bp + s (o Ap_k) Bp_k                       attention output projection, Sec. 3.1 form
//   B   x'' = x' + b2 + GELU(LayerNorm2(x') W1 + b1) W2              feed-forward block (no low-rank branch here)
//   C   qkv = LayerNorm1'(x'') Wq + bq + s (.. Aq_k) Bq_k            qkv linear of the NEXT layer (optional)
//
// (LAYER = false: C alone, on rows read from memory: the first layer's qkv and the one where frames fan out into row-blocks.)
// Only softmax attention needs whole blocks, so a layer is two launches, and x', the hidden activation and the LayerNorm outputs never leave the
// chip.  Without adapters the rows of all blocks are tiled as one run: 333 blocks of 197 rows are 1026 tiles, five rounds of 256 CUs, where tiles
// that end with their block are 1332, six rounds.
//
// Eight waves (kh, wc), two per SIMD, all of which compute and request the weights they multiply:
//   product with D outputs (proj, W2)  wave (kh, wc): 16 KT columns of all 64 rows for half kh of the contraction; the halves meet once, at the end of
//                                      A and of B, through LDS (exchange), and from there on wave (kh, wc) owns row half kh of its columns: the
//                                      residual stream is 24 fp32 registers of a lane and never a tile in LDS.
//   product with D inputs (W1, Wq)     wave w: 16 of 128 columns of all 64 rows, whose operands stay in registers (96 of them).
// A wave thus multiplies weights that no other wave needs: each byte of them passes the CU's load path and LDS once, into a slot of the wave's
// own (two of 6 KB), refilled as soon as it has been read, with no barrier between.  What is left to share are the hidden columns: one barrier per 128.
//
// Bounds, for DeiT-tiny (885 KB of weights per tile), in cycles of a 57 k-cycle launch of 248 tiles: start and the first loads 8.5 k, proj + exchange +
// shrink 6 k, the two LayerNorms 7 k, the six chunks of the feed-forward block 21 k, qkv 11 k.  A chunk takes 3.35 k: LDS is busy for about 2.6 k of
// it (96 KB of weights in and out, GELU lookups at 6.3 cycles per instruction, hidden columns), the matrix units 1.54 k; without the stream it takes
// 2.4 k, without the lookups 2.6 k.  32.8 us per launch with one wave for the stream and three for the second product became 30.4 us (62 blocks of 197
// rows, rank 8), 156 us became 118 us (333 blocks, no adapters).  Tried and dropped: weights in a ring shared by all waves with a barrier per 24 KB
// (31 us; its steps wait for each other), the same with the two row halves a barrier apart, one multiplying while the other reads (32 us), tiles of 96
// and 128 rows (registers spill), the GELU as a polynomial (the same: fewer lookups, more issue slots).
#include "poly_dev.h"
#include "rowtile.h"

#include <type_traits>

namespace {

constexpr int LY_THREADS = 512;
constexpr int LY_TILE = 8192;       // bytes of a [64][64] bf16 tile in LDS: 128 bytes a row, its 16-byte pieces permuted
constexpr int LY_TILES = 4;         // of activations
constexpr int LY_MAX_DM = 768;
constexpr int LY_GELU = (GELU_TAB_ENTRIES + 1) & ~1;    // (what lies behind is read in 16-byte pieces)
constexpr int LY_AT_STRIDE = 200;   // elements per rank row of At_k in LDS (192 + 8: rows start 4 banks apart)

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) char *lds_ptr;

// sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48 that share a token row, in every one of them
__device__ __forceinline__ float quad16_sum(float v)
{
    unsigned p = __builtin_bit_cast(unsigned, v);
    const u32x2 a = __builtin_amdgcn_permlane32_swap(p, p, false, false);
    const unsigned a0 = a[0], a1 = a[1];
    p = __builtin_bit_cast(unsigned, __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1));
    const u32x2 b = __builtin_amdgcn_permlane16_swap(p, p, false, false);
    const unsigned b0 = b[0], b1 = b[1];
    return __builtin_bit_cast(float, b0) + __builtin_bit_cast(float, b1);
}

template <int KT, bool LAYER, bool QKV>
__global__ __launch_bounds__(LY_THREADS, 2) void rowlayer_kernel(const RowLayerArgs a, const int flat_rows)
{
    constexpr int D = 64 * KT, Nq = 3 * D, NQ = (Nq + 127) / 128;
    constexpr int CT = KT;                                 // column tiles of 16 per wave of a product with D columns
    constexpr int SLOT = KT * 2048;                        // bytes of a slot: 16 rows of D columns, or 16 CT rows of 64 columns
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char *As = lds;                                        // activations: KT tiles [64][64] bf16; two pairs of tiles for the hidden columns, and for qkv
    char *Ws = lds + LY_TILES * LY_TILE;                   // two slots per wave
    float *b1_s = (float *)(Ws + 16 * SLOT);               // [Dm]
    float *bq_s = b1_s + LY_MAX_DM;                        // [3 D]
    float *bp_s = bq_s + Nq;                               // [D]
    float *b2_s = bp_s + D;                                // [D]
    float *gb2_s = b2_s + D;                               // LayerNorm2 gain [D], shift [D]
    float *gbq_s = gb2_s + 2 * D;                          // LayerNorm1' gain, shift
    float *gelu_s = gbq_s + 2 * D;
    f32x2 *stat_s = (f32x2 *)(gelu_s + 2 * LY_GELU);       // [64][4]: mean and squared deviations of a wave's columns of a row
    s16x4 *sh_s = (s16x4 *)stat_s;                         // in C: shrink output, [4][64 lanes]
    bf16_t *at_s = (bf16_t *)(stat_s + 64 * 4);            // At_k of the phase, [16][LY_AT_STRIDE]
    bf16_t *bt_s = at_s + 16 * LY_AT_STRIDE;               // Bt_k of A, [D][r]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = wave >> 2, wc = wave & 3, lm = lane & 15, lg = lane >> 4, lr = lane >> 3;
    const int Dm = a.Dm, nc = LAYER ? (Dm + 127) >> 7 : 0;

    // ---- this tile's rows
    int ob = 0, t0;
    size_t row0;                                           // of the output
    int rows;
    if (flat_rows) {
        t0 = blockIdx.x * 64;
        row0 = t0;
        rows = min(64, flat_rows - t0);
    } else {
        const int tiles = (a.T + 63) / 64;
        ob = blockIdx.x / tiles;
        t0 = (blockIdx.x % tiles) * 64;
        row0 = (size_t)ob * a.T + t0;
        rows = min(64, a.T - t0);
    }
    const int n_out = a.n_out_dev ? min(*a.n_out_dev, a.n_out) : a.n_out;
    const int k_ad = a.adapter_of_out ? a.adapter_of_out[ob] : -1;      // (meaningless past n_out)
    size_t xrow0 = row0;
    if (a.res_block_of_out) {                              // (the map has entries for the blocks that exist only)
        if (ob >= n_out) return;
        xrow0 = (size_t)a.res_block_of_out[ob] * a.T + t0;
    }

    // ---- the stream of weights, into slots of the wave that multiplies them: 8 rows x 128 bytes per instruction, the swizzle of the LDS rows applied
    // on the global side.
    const unsigned slot0 = __builtin_amdgcn_readfirstlane(lds_addr_of(Ws)) + wave * (2 * SLOT);     // N slot, then K slot
    const unsigned piece = (unsigned)(((lane & 7) ^ (lr >> 1)) << 4);                               // of rows lr; of rows 8 + lr: ^ 64
    const unsigned off_d = (unsigned)lr * (D * 2) + piece, off_m = (unsigned)lr * (Dm * 2) + piece;
    // 16 rows of a matrix with D columns from row `row`
    auto issue_n1 = [&](const bf16_t *W, int row, unsigned slot, int j) {
        const bf16_t *base = W + (size_t)(row + 8 * (j & 1)) * D + 64 * (j >> 1);
        glds16_s(base, off_d ^ (64 * (j & 1)), slot + j * 1024);
    };
    auto issue_n = [&](const bf16_t *W, int row, unsigned slot) {
#pragma unroll
        for (int j = 0; j < 2 * KT; ++j) issue_n1(W, row, slot, j);
    };
    // W2: rows 16 CT wc .., 64 columns from column `col`
    auto issue_k1 = [&](int col, int j) { glds16_s(a.W2t + (size_t)(16 * CT * wc + 8 * j) * Dm + col, off_m ^ (64 * (j & 1)), slot0 + SLOT + j * 1024); };
    // first row of W1 / first column of W2 that this wave multiplies of chunk c (the last chunk may be half a one: what lies past it is not used)
    auto row_n = [&](int c) { return min(128 * c + 16 * wave, Dm - 16); };
    auto col_k = [&](int c) { return min(128 * c + 64 * kh, Dm - 64); };
    auto row_q = [&](int q) { return 128 * q + 16 * (128 * q + 128 <= Nq ? wave : wc); };
    auto slot_q = [&](int q) { return slot0 + (q & 1 ? 0 : SLOT); };

    // ---- prologue: everything is requested at once, in the order in which it is needed
    if (LAYER) {
        const char *src = (const char *)(a.o + row0 * D);
#pragma unroll
        for (int t = 0; t < KT; ++t) {                     // rows 8 wave .. + 7 of each tile
            const unsigned p = (unsigned)(((lane & 7) ^ ((wave & 1) * 4 + (lr >> 1))) << 4);
            glds16_s(src + t * 128, (unsigned)min(8 * wave + lr, rows - 1) * (D * 2) + p, __builtin_amdgcn_readfirstlane(lds_addr_of(As)) + t * LY_TILE + wave * 1024);
        }
        // Wp: rows 16 CT wc .., columns 64 t + 32 kh .. + 31 as [16 CT][32], 16 rows x 64 bytes per instruction
        const unsigned vo = (unsigned)(lane >> 2) * (D * 2) + (((lane & 3) ^ ((lane >> 4) & 3)) << 4);
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                glds16_s(a.Wpt + (size_t)(16 * CT * wc + 16 * ct) * D + 64 * t + 32 * kh, vo, slot0 + (t * CT + ct) * 1024);
    } else {
        issue_n(a.Wqt, row_q(0), slot_q(0));
        issue_n(a.Wqt, row_q(1), slot_q(1));
    }
    // vectors -> LDS, 64 floats per instruction (any alignment of a float), shared out by wave
    auto vec = [&](const float *src, int from, int to, const float *dst) {
        for (int i = from; i < to; i += 64) glds4(src + i + lane, __builtin_amdgcn_readfirstlane(lds_addr_of(dst)) + i * 4);
    };
    if (LAYER) {
        if (wave == 0) vec(a.b1, 0, Dm >> 1 & ~63, b1_s);
        if (wave == 1) vec(a.b1, Dm >> 1 & ~63, Dm, b1_s);
        if (wave == 2) { vec(a.bp, 0, D, bp_s); vec(a.b2, 0, D, b2_s); }
        if (wave == 3) { vec(a.ln2_g, 0, D, gb2_s); vec(a.ln2_b, 0, D, gb2_s + D); }
    }
    if (QKV) {
        if (wave == 4) { vec(a.lnq_g, 0, D, gbq_s); vec(a.lnq_b, 0, D, gbq_s + D); }
        if (wave >= 5) vec(a.bq, (wave - 5) * D, (wave - 4) * D, bq_s);
    }
    // the residual stream of the row half kh: row lm of tile rt, columns 16 CT wc + 16 ct + 4 lg + {0..3}
    const int wrow = 32 * kh, wcol = 16 * CT * wc + 4 * lg;
    const bool none = flat_rows ? (long)t0 >= (long)n_out * a.T : ob >= n_out;
    if (none) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }
    if (flat_rows) rows = min(rows, (int)((long)n_out * a.T - t0));
    const bool lora_p = LAYER && a.Apt && k_ad >= 0, lora_q = QKV && a.Aqt && k_ad >= 0;
    const int r = a.r;
    // At_k [r][D] -> at_s, a rank row per instruction; Bt_k [D][r] -> bt_s, as it is
    auto issue_at = [&](const bf16_t *At_k) {
        for (int rk = wave; rk < r; rk += 8)
            if (lane < D / 8) glds16(At_k + rk * D + lane * 8, __builtin_amdgcn_readfirstlane(lds_addr_of(at_s + rk * LY_AT_STRIDE)));
    };
    // rank lm (repeated past r: such ranks meet zeros of Bt_k), columns 32 k + 8 lg + {0..7}
    auto at_frag = [&](int k) { return *(const bf16x8 *)(at_s + min(lm, r - 1) * LY_AT_STRIDE + 32 * k + 8 * lg); };
    // column n of Bt_k [.][r], ranks 4 lg + {0..3} (r is a multiple of 4; zero where the rank does not exist)
    auto bt_frag = [&](const bf16_t *Bt_k, int n) { return *(const s16x4 *)(Bt_k + n * r + min(4 * lg, r - 4)); };
    // four ranks of a lane as a step of 32, the other four zeros on both sides (v_mfma_f32_16x16x16_bf16 takes several times as long)
    auto wide = [](s16x4 v) { return __builtin_bit_cast(bf16x8, __builtin_shufflevector(v, s16x4{0, 0, 0, 0}, 0, 1, 2, 3, 4, 5, 6, 7)); };
    auto bt_operand = [&](s16x4 v) { return 4 * lg < r ? v : s16x4{0, 0, 0, 0}; };
    if (lora_p) {
        issue_at(a.Apt + (size_t)k_ad * r * D);
        const char *Bt_k = (const char *)(a.Bpt + (size_t)k_ad * D * r);
        const int n16 = D * r / 8;                         // 16-byte pieces
        for (int i = wave * 64; i < n16; i += 512)
            if (i + lane < n16) glds16(Bt_k + (i + lane) * 16, __builtin_amdgcn_readfirstlane(lds_addr_of(bt_s)) + i * 16);
    }
    if (!LAYER && lora_q) issue_at(a.Aqt + (size_t)k_ad * r * D);
    f32x4 x[CT][2];
    auto load_x = [&]() {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                x[ct][rt] = *(const f32x4 *)(a.res + xrow0 * D + (unsigned)(min(wrow + 16 * rt + lm, rows - 1) * D + wcol + 16 * ct));
    };
    if (!LAYER) load_x();
    const bf16_t *Bq_k = QKV && lora_q ? a.Bqt + (size_t)k_ad * Nq * r : nullptr;
    if (LAYER) {                                           // Phi table of the GELU
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = tid + LY_THREADS * j;
            if (i < GELU_TAB_ENTRIES) *(f32x2 *)(gelu_s + 2 * i) = gelu_tab_entry(i);
        }
    }

    // ---- operands.  A fragment is 16 rows x 32 contraction columns: lane (lm, lg) holds columns 8 lg .. + 7 of row lm, the 16-byte piece
    // (4 kk + lg) ^ (row >> 1 & 7) of a 128-byte row.
    const int fo0 = lm * 128 + ((lg ^ ((lm >> 1) & 7)) << 4), fo1 = fo0 ^ 64;
    lds_ptr act[2], wn[2];                                 // [k & 1]: rows of activations, rows of a slot
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        act[k] = (lds_ptr)(As + (k ? fo1 : fo0));
        wn[k] = (lds_ptr)(Ws + wave * (2 * SLOT) + (k ? fo1 : fo0));
        asm("" : "+v"(act[k]));
        asm("" : "+v"(wn[k]));
    }
    auto rd = [&](lds_ptr p, int off) { return *(const __attribute__((address_space(3))) bf16x8 *)(p + off); };
    auto act_frag = [&](int tile, int rt, int kk) { return rd(act[kk], tile * LY_TILE + rt * 2048); };
    bf16x8 fa[2 * KT][4];                                  // the resident rows as the B operand of the transposed product
    auto load_fa = [&]() {
#pragma unroll
        for (int k = 0; k < 2 * KT; ++k)
#pragma unroll
            for (int rt = 0; rt < 4; ++rt) fa[k][rt] = act_frag(k >> 1, rt, k & 1);
    };
    // s (x At_k): ranks 4 lg + {0..3} of row lm, the operand of the expand as it is
    auto shrink_out = [&](f32x4 c) {
        const bf16x4 o = {(bf16_t)(a.scale * c[0]), (bf16_t)(a.scale * c[1]), (bf16_t)(a.scale * c[2]), (bf16_t)(a.scale * c[3])};
        return __builtin_bit_cast(s16x4, o);
    };
    // 4 columns 16 cg + 4 lg + {0..3} (cg < 4) of row 16 rt + lm -> a [64][64] tile
    auto put = [&](char *tile, int cg, int rt, f32x4 v) {
        const bf16x4 o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
        *(bf16x4 *)(tile + (16 * rt + lm) * 128 + (((2 * cg + (lg >> 1)) ^ ((lm >> 1) & 7)) << 4) + 8 * (lg & 1)) = o;
    };
    // The sums over the two halves of the contraction meet: a wave hands the row half that is not its own to the wave with the same columns, through
    // its own N slot, and adds what it is handed.
    auto exchange = [&](f32x4 (&acc)[CT][4], f32x4 (&own)[CT][2]) {
        f32x4 *mine = (f32x4 *)(Ws + wave * (2 * SLOT)) + lane;
        const f32x4 *theirs = (const f32x4 *)(Ws + (wave ^ 4) * (2 * SLOT)) + lane;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                mine[(ct * 2 + rt) * 64] = kh ? acc[ct][rt] : acc[ct][2 + rt];
                own[ct][rt] = kh ? acc[ct][2 + rt] : acc[ct][rt];
            }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) own[ct][rt] += theirs[(ct * 2 + rt) * 64];
    };
    // LayerNorm (fp32 statistics, centred second moments of 16 CT columns each, put together by Chan's rule) of x -> bf16 tiles at As -> fragments.
    // Behind the first barrier every wave is done with what it read before: `between` runs there.
    auto layernorm = [&](const float *gb_s, auto between) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            float t = 0.f;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) t += (x[ct][rt][0] + x[ct][rt][1]) + (x[ct][rt][2] + x[ct][rt][3]);
            const float m = quad16_sum(t) * (1.0f / (16 * CT));
            float q = 0.f;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int z = 0; z < 4; ++z) { const float d = x[ct][rt][z] - m; q = fmaf(d, d, q); }
            q = quad16_sum(q);
            if (lg == 0) stat_s[(wrow + 16 * rt + lm) * 4 + wc] = f32x2{m, q};
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        between();
        f32x4 g[CT], b[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) { g[ct] = *(const f32x4 *)(gb_s + wcol + 16 * ct); b[ct] = *(const f32x4 *)(gb_s + D + wcol + 16 * ct); }
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            const int row = wrow + 16 * rt + lm;
            const f32x4 s0 = *(const f32x4 *)(stat_s + row * 4), s1 = *(const f32x4 *)(stat_s + row * 4 + 2);
            const float mean = 0.25f * ((s0[0] + s0[2]) + (s1[0] + s1[2]));
            const float d0 = s0[0] - mean, d1 = s0[2] - mean, d2 = s1[0] - mean, d3 = s1[2] - mean;
            const float q = (s0[1] + s0[3]) + (s1[1] + s1[3]) + (16 * CT) * ((d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3));
            const float inv = rsqrtf(q * (1.0f / D) + a.eps), nmi = -mean * inv;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                bf16x4 o;
#pragma unroll
                for (int z = 0; z < 4; ++z) o[z] = (bf16_t)fmaf(fmaf(x[ct][rt][z], inv, nmi), g[ct][z], b[ct][z]);   // ((x - mean) inv) g + b
                const int col = wcol + 16 * ct;
                *(bf16x4 *)(As + (col >> 6) * LY_TILE + row * 128 + ((((col & 63) >> 3) ^ ((lm >> 1) & 7)) << 4) + 2 * (col & 4)) = o;
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        load_fa();
    };
    constexpr int NS = 4 * KT;                             // MFMAs of a segment
    // a segment: every MFMA is followed by a share of the other work
    auto segment = [&](auto mfma, auto side) {
#pragma unroll
        for (int n = 0; n < NS; ++n) {
            mfma(n);
            side(n);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // pieces 0 .. count - 1 over the slots [first, last) of a segment
    auto share = [&](int n, int first, int last, int count, auto piece) {
#pragma unroll
        for (int j = 0; j < count; ++j)
            if (n == first + j * (last - first) / count) piece(j);
    };

    if (LAYER) {
        // ============================================================ A: x' = res + o Wp + bp + lora
        f32x4 y[CT][4];
        rl_wait_barrier<0>();                              // o, Wp, At_k, Bt_k and the vectors
        {
            const lds_ptr wp = (lds_ptr)(Ws + wave * (2 * SLOT) + lm * 64 + ((lg ^ ((lm >> 2) & 3)) << 4));
            bf16x8 w[KT][CT], h[KT][4];
#pragma unroll
            for (int t = 0; t < KT; ++t) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) w[t][ct] = rd(wp, (t * CT + ct) * 1024);
#pragma unroll
                for (int rt = 0; rt < 4; ++rt) h[t][rt] = rd(kh ? act[1] : act[0], t * LY_TILE + rt * 2048);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int j = 0; j < 2 * CT; ++j) issue_k1(col_k(0), j);
            load_x();                                      // (16 rows x 64 bytes an instruction hold the load path up: not in front of the first product)
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int rt = 0; rt < 4; ++rt)
                        y[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t][ct], h[t][rt], t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : y[ct][rt], 0, 0, 0);
        }
        {
            f32x4 own[CT][2];
            exchange(y, own);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const f32x4 b = *(const f32x4 *)(bp_s + wcol + 16 * ct);
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) x[ct][rt] += own[ct][rt] + b;
            }
        }
        if (lora_p) {
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 2 * KT; ++k) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at_frag(k), rd(act[k & 1], (k >> 1) * LY_TILE + wrow * 128 + rt * 2048), c, 0, 0, 0);
                const s16x4 fs = shrink_out(c);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) x[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wide(bt_operand(bt_frag(bt_s, 16 * CT * wc + 16 * ct + lm))), wide(fs), x[ct][rt], 0, 0, 0);
            }
        }
        layernorm(gb2_s, [&]() { issue_n(a.W1t, row_n(0), slot0); });
        // The second product of B adds to x' + b2 on half 0 of its contraction in every row, so that a row's bits do not depend on its place in the tile: the
        // waves of half 1 hand their rows over, in LDS that is in no use until the second chunk (tile 3, and what LayerNorm and A are done with).  0.3 us of a
        // launch of 248 tiles (twelve of them and the rest of 32 frames of 224 x 224, 62 blocks: 498 / 502 us; through the weight slots, before the first of
        // W1 is requested, 504).
        auto handed = [&](int ct, int rt) {
            const int i = ct * 2 + rt;
            return (f32x4 *)((i < 2 ? As + 3 * LY_TILE + i * 4096 : (char *)stat_s + (i - 2) * 4096) + wc * 1024) + lane;
        };
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const f32x4 b = *(const f32x4 *)(b2_s + wcol + 16 * ct), z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                if (kh) *handed(ct, rt) = x[ct][rt] + b;
                y[ct][rt] = kh ? z : x[ct][rt] + b;
                y[ct][2 + rt] = z;
            }
        }

        // ============================================================ B: x'' = x' + b2 + GELU(LayerNorm2(x') W1 + b1) W2
        bf16x8 wN[2 * KT], wK[2][CT], hk[2][4];
        f32x4 h[4];
        float xc[4];
        f32x2 en[4];
        const unsigned gelu_a = lds_addr_of(gelu_s);
        auto fetch_n1 = [&](int j) { wN[j] = rd(wn[j & 1], (j >> 1) * 2048); };
        auto fetch_w1 = [&](int kk, int j) { wK[kk][j] = rd(wn[kk], SLOT + j * 2048); };
        auto fetch_h1 = [&](int kk, int buf, int rt) { hk[kk][rt] = rd(act[kk], buf * (2 * LY_TILE) + kh * LY_TILE + rt * 2048); };
        auto mfma_n = [&](int n, int rt0, f32x4 b) {       // rows of two tiles
            const int k = n / 2, rt = rt0 + n % 2;
            h[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wN[k], fa[k][rt], k == 0 ? b : h[rt], 0, 0, 0);
        };
        auto mfma_k = [&](int n, int kk) {
            const int ct = n / 4, rt = n % 4;
            y[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wK[kk][ct], hk[kk][rt], y[ct][rt], 0, 0, 0);
        };
        // GELU of one row tile: four lookups, then (fin) the results
        auto look = [&](int rt, int j) { gelu_look(h[rt][j], gelu_a, xc[j], en[j]); };
        auto fin = [&](int rt, int buf) { put(As + buf * (2 * LY_TILE) + kh * LY_TILE, wc, rt, gelu_tab4(h[rt], xc, en)); };
        auto gelu_side = [&](int n, int rt0, int buf) {    // of two row tiles in a segment of NS slots
            share(n, 0, NS / 4, 4, [&](int j) { look(rt0, j); });
            if (n == NS / 2 - 1) fin(rt0, buf);
            share(n, NS / 2, 3 * NS / 4, 4, [&](int j) { look(rt0 + 1, j); });
            if (n == NS - 1) fin(rt0 + 1, buf);
        };
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int j = 0; j < 2 * KT; ++j) fetch_n1(j);
        auto chunk = [&](int c, auto FIRST) {              // first product of chunk c, second of chunk c - 1
            constexpr bool first = decltype(FIRST)::value;
            const int buf = c & 1;
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");     // hidden columns of chunk c - 1 are there; wN is in registers
            const f32x4 b = *(const f32x4 *)(b1_s + min(128 * c + 16 * wave, Dm - 16) + 4 * lg);
            if (c + 1 < nc) issue_n(a.W1t, row_n(c + 1), slot0);
            if (first && !kh) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt) y[ct][2 + rt] = *handed(ct, rt);
            }
            segment([&](int n) { mfma_n(n, 0, b); }, [&](int n) {});
            segment([&](int n) { mfma_n(n, 2, b); },
                    [&](int n) {
                        gelu_side(n, 0, buf);
                        if (!first) {
                            share(n, 0, NS / 2, 4, [&](int j) { fetch_h1(0, buf ^ 1, j); });
                            if (n == NS / 2) {
                                if (c + 1 < nc) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * KT) : "memory");
                                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                            }
                            share(n, NS / 2, NS, CT, [&](int j) { fetch_w1(0, j); });
                        }
                    });
            if (first) {
#pragma unroll
                for (int n = 0; n < NS; ++n) gelu_side(n, 2, buf);
            } else {
                segment([&](int n) { mfma_k(n, 0); },
                        [&](int n) {
                            gelu_side(n, 2, buf);
                            share(n, 0, NS / 2, 4, [&](int j) { fetch_h1(1, buf ^ 1, j); });
                            share(n, NS / 2, NS - 1, CT, [&](int j) { fetch_w1(1, j); });
                        });
            }
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            if (first) {
                if (c + 1 < nc) {
#pragma unroll
                    for (int j = 0; j < 2 * KT; ++j) fetch_n1(j);
                }
            } else {
                segment([&](int n) { mfma_k(n, 1); },
                        [&](int n) {
                            share(n, 0, NS, 2 * CT, [&](int j) { issue_k1(col_k(c), j); });
                            if (c + 1 < nc) share(n, 0, NS - 1, 2 * KT, [&](int j) { fetch_n1(j); });
                        });
            }
        };
        chunk(0, std::true_type{});
#pragma unroll 1
        for (int c = 1; c < nc; ++c) chunk(c, std::false_type{});
        {                                                  // second product of the last chunk; where that is half a chunk, the second half has nothing
            const int buf = (nc - 1) & 1;
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
                for (int j = 0; j < 4; ++j) fetch_h1(kk, buf, j);
#pragma unroll
                for (int j = 0; j < CT; ++j) fetch_w1(kk, j);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (QKV) issue_n(a.Wqt, row_q(0), slot_q(0));
            if (lora_q) issue_at(a.Aqt + (size_t)k_ad * r * D);
            if (!kh || !(Dm & 64)) {
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                    for (int n = 0; n < NS; ++n) mfma_k(n, kk);
            }
        }
        exchange(y, x);
    }
    auto store_x = [&](int e) {                            // piece e of x''
        const int rt = e / CT, ct = e % CT, row = wrow + 16 * rt + lm;
        if (row < rows) *(f32x4 *)(a.x_out + (row0 + row) * D + wcol + 16 * ct) = x[ct][rt];
    };
    if (!QKV) {
#pragma unroll
        for (int e = 0; e < 2 * CT; ++e) store_x(e);
        return;
    }

    // ================================================================ C: qkv = LayerNorm1'(x'') Wq + bq + lora
    layernorm(gbq_s, [&]() { if (LAYER) issue_n(a.Wqt, row_q(1), slot_q(1)); });
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // Q(0), Q(1), At_k
    s16x4 fs[4];
    if (lora_q) {                                          // one row tile per wave, to every wave
        asm volatile("s_barrier" ::: "memory");
        f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 2 * KT; ++k) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at_frag(k), rd(act[k & 1], (k >> 1) * LY_TILE + wc * 2048), c, 0, 0, 0);
        if (!kh) sh_s[wc * 64 + lane] = shrink_out(c);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int rt = 0; rt < 4; ++rt) fs[rt] = sh_s[rt * 64 + lane];
    }
    char *out = (char *)a.qkv_out + row0 * Nq * 2;
    f32x4 sv[2];
    // the columns of a round, staged in tiles 2 (q & 1) .., leave as whole rows of them
    auto stage_read = [&](int q) {
        const int pr = 128 * q + 128 <= Nq ? 16 : 8;       // 16-byte pieces of a row
#pragma unroll
        for (int j = 0; j < pr / 8; ++j) {
            const int idx = tid + LY_THREADS * j, row = idx / pr, p = idx % pr;
            sv[j] = *(const f32x4 *)(As + (2 * (q & 1) + (p >> 3)) * LY_TILE + row * 128 + (((p & 7) ^ ((row >> 1) & 7)) << 4));
        }
    };
    auto store = [&](int q) {
        const int pr = 128 * q + 128 <= Nq ? 16 : 8;
#pragma unroll
        for (int j = 0; j < pr / 8; ++j) {
            const int idx = tid + LY_THREADS * j, row = idx / pr, p = idx % pr;
            if (row < rows) *(f32x4 *)(out + (size_t)row * Nq * 2 + q * 256 + p * 16) = sv[j];
        }
    };
    bf16x8 W[2][2 * KT];
    auto fetch = [&](int q, int j) { W[q & 1][j] = rd(wn[j & 1], (q & 1 ? 0 : SLOT) + (j >> 1) * 2048); };
#pragma unroll
    for (int j = 0; j < 2 * KT; ++j) fetch(0, j);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const bool full = 128 * q + 128 <= Nq;
        const int col = row_q(q);
        s16x4 b2 = {0, 0, 0, 0};
        if (lora_q) b2 = bt_frag(Bq_k, col + lm);
        if (q + 2 < NQ) issue_n(a.Wqt, row_q(q + 2), slot_q(q + 2));    // W[q & 1] is in registers
        const f32x4 b = *(const f32x4 *)(bq_s + col + 4 * lg);
        f32x4 acc[4];
        auto mfma = [&](int n, int rt0) {
            const int k = n / 2, rt = rt0 + n % 2;
            acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[q & 1][k], fa[k][rt], k == 0 ? b : acc[rt], 0, 0, 0);
        };
        auto next = [&](int n) {                           // the operands of the next round
            if (q + 1 == NQ) return;
            if (n == 0 && q > 0) {                         // (behind it: at least two stores of the last round, in a tile that has all its rows)
                constexpr int ahead = 2 * KT;
                const bool two = rows == 64 && (LAYER || q > 2);
                if (q + 2 < NQ) {
                    if (two) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(ahead + 2) : "memory");
                    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(ahead) : "memory");
                } else {
                    if (two) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
                    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                }
            }
            share(n, 0, NS - 2, 2 * KT, [&](int j) { fetch(q + 1, j); });
        };
        if (full) {
            segment([&](int n) { mfma(n, 0); }, next);
            segment([&](int n) { mfma(n, 2); }, [&](int n) {
                if (n == 0 && q > 1) store(q - 2);
                if (LAYER && n == NS - 1) {
#pragma unroll
                    for (int e = 0; e < 2 * CT; ++e)
                        if (e / 2 == q) store_x(e);
                }
            });
        } else {                                           // half a round: 64 columns, every wave 16 of them for its row half
            if (kh) {
#pragma unroll
                for (int n = 0; n < NS; ++n) mfma(n, 2);
                acc[0] = acc[2];
                acc[1] = acc[3];
            } else {
#pragma unroll
                for (int n = 0; n < NS; ++n) mfma(n, 0);
            }
            if (q > 1) store(q - 2);
        }
        if (lora_q) {
            const bf16x8 w = wide(bt_operand(b2));
            if (full) {
#pragma unroll
                for (int rt = 0; rt < 4; ++rt) acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, wide(fs[rt]), acc[rt], 0, 0, 0);
            } else {
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, wide(kh ? fs[2 + rt] : fs[rt]), acc[rt], 0, 0, 0);
            }
        }
        // the columns of round q - 1 are staged, those of round q - 2 have been read; the operands of the next round are in registers
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (q > 0) stage_read(q - 1);
#pragma unroll
        for (int rt = 0; rt < (full ? 4 : 2); ++rt)
            put(As + (2 * (q & 1) + (full ? kh : 0)) * LY_TILE, wc, full ? rt : 2 * kh + rt, acc[rt]);
    }
    store(NQ - 2);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    stage_read(NQ - 1);
    store(NQ - 1);
}

template <int KT, bool LAYER, bool QKV> int launch_t(const RowLayerArgs &a, hipStream_t st)
{
    constexpr int D = 64 * KT;
    constexpr int END = 64 * 4 * 8 + 16 * LY_AT_STRIDE * 2 + D * 16 * 2, HANDED = (2 * KT - 2) * 4096;   // from stat_s on
    constexpr int LDS = LY_TILES * LY_TILE + 16 * KT * 2048 + (LY_MAX_DM + 3 * D + 2 * D + 4 * D) * 4 + LY_GELU * 8 + (END > HANDED ? END : HANDED);
    static_assert(LDS <= 160 * 1024, "LDS budget");
    auto kern = rowlayer_kernel<KT, LAYER, QKV>;
    if (LDS > 64 * 1024) {
        static bool attr_set = false;   // raising the dynamic LDS limit is a per-kernel, process-wide setting
        if (!attr_set) {
            if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS) != hipSuccess) return POLY_EHIP;
            attr_set = true;
        }
    }
    const bool flat = !a.adapter_of_out && !a.res_block_of_out;
    const int flat_rows = flat ? a.n_out * a.T : 0;
    const int grid = flat ? (flat_rows + 63) / 64 : a.n_out * ((a.T + 63) / 64);
    POLY_LAUNCH_SHMEM(POLY_STAGE_GEMM, kern, dim3((unsigned)grid), dim3(LY_THREADS), LDS, st, a, flat_rows);
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

template <int KT> int launch_kt(const RowLayerArgs &a, hipStream_t st)
{
    if (!a.o) return launch_t<KT, false, true>(a, st);
    return a.qkv_out ? launch_t<KT, true, true>(a, st) : launch_t<KT, true, false>(a, st);
}

}  // namespace

// D, Dm: model and hidden width; r: adapter rank of the proj / qkv linears that carry adapters (0 = none)
bool rowlayer_supported(int D, int Dm, int r)
{
    if (!((D == 64 || D == 128 || D == 192) && Dm >= 128 && Dm % 64 == 0 && Dm <= LY_MAX_DM)) return false;
    return r == 0 || (r >= 4 && r <= 16 && r % 4 == 0);
}

int launch_rowlayer(const RowLayerArgs &a, hipStream_t st)
{
    if (a.n_out <= 0 || a.T <= 0) return POLY_OK;
    const bool lora = (a.o && a.Apt) || (a.qkv_out && a.Aqt);
    if (!rowlayer_supported(a.D, a.Dm, lora ? a.r : 0)) return POLY_EINVAL;
    switch (a.D / 64) {
    case 1: return launch_kt<1>(a, st);
    case 2: return launch_kt<2>(a, st);
    default: return launch_kt<3>(a, st);
    }
}
