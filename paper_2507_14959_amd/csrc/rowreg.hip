// The row-wise part of a layer of a model 192 wide (rowlayer.hip: A proj, B feed-forward, C qkv of the next layer) for many rows: 32 rows in the registers
// of each of four or eight waves.
//
// rowlayer.hip gives a CU 64 rows at a time, and every 64 rows pull the layer's 885 KB of weights through its LDS and pass their activations from wave to
// wave there.  Here a wave owns its rows from the first product to the last: the residual stream is the accumulator of proj and of the second product of B
// (96 registers), a LayerNorm is a sum over a lane's own registers and one exchange with the lane that has the other half of the row, its result becomes
// the operand of the next product by a swap of lane halves (operand()), and so do the hidden columns.  LDS holds weights (and, for stores by whole lines, a
// wave's 4 KB): a ring of four units of 24 KB that all waves load and all waves read, a barrier per two of them.
//
// In B a wave works in steps of 32 hidden columns, and the GELU of a step runs on the vector unit under the products of its neighbours.  Four waves are one
// per SIMD: 3.2 k cycles per 64 hidden columns, bounded by the instructions a lone wave issues (one per 5 to 6 cycles; 1.54 k of MFMA).  Eight waves take
// 4.5 k for twice the rows (3.07 k of MFMA; 3.7 k without GELU and without reading the weights again).  A launch of all three parts, 197-token blocks
// without adapters: 128 blocks 54.6 us as 394 tiles of 64 rows in two rounds, 39 us as 197 tiles of 128; 320 blocks 116 us in four rounds, 76 us as 247
// tiles of 256.  Of the 76 us 11 are spent on the first loads (75 MB that all CUs want at once, 6.8 TB/s) and 25 behind B on stores of 125 MB beside the
// qkv products; the 30 to 36 of B run at the clock that the power leaves (cycle counter against the constant clock: 1.75 to 1.9 GHz, 2.3 before B; 256 tiles
// of 128 rows 2.0 to 2.1, 197 of them 2.3 to 2.4).
//
// Rows are tiled as one run over all blocks, with adapters too: a wave's rows lie in one block or two (a block has 32 or more), and a wave in two blocks
// computes both low-rank terms and takes each row's own.  The attention output and, between two of these launches, the residual stream lie in the order of
// the registers (poly_dev.h), so that a wave reads and writes them 1 KB at a time.
//
// Tried and dropped: five, six or seven waves (the SIMDs with two waves set the pace: as slow as eight); a wave's GELU as a block that alternates with the
// other wave's products (the same time, but nothing under it where there is one wave per SIMD); the GELU as a polynomial (5.6 k cycles per 64 columns).
#include "poly_dev.h"
#include "row_waves.h"
#include "rowtile.h"

#include <type_traits>

namespace {

constexpr int RR_SLOTS = 4;         // of the ring of weights
constexpr int RR_UNIT = 24576;      // bytes of one: three tiles [64][64]
constexpr int RR_STAGE = 4096;      // bytes of a wave's staging area: 32 rows x 128 bytes
constexpr int RR_GELU = (GELU_TAB_ENTRIES + 1) & ~1;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) char *lds_ptr;

__device__ __forceinline__ unsigned pack2(float a, float b)
{
    const bf16x2 v = {(bf16_t)a, (bf16_t)b};
    return __builtin_bit_cast(unsigned, v);
}
// Columns 8 q + 4 lh + {0..3} (q = 0, 1) of a lane's row, as a product leaves them, -> columns 8 lh + {0..7}, as the next one takes them
__device__ __forceinline__ bf16x8 operand(f32x4 q0, f32x4 q1)
{
    const u32x2 a = __builtin_amdgcn_permlane32_swap(pack2(q0[0], q0[1]), pack2(q1[0], q1[1]), false, false);
    const u32x2 b = __builtin_amdgcn_permlane32_swap(pack2(q0[2], q0[3]), pack2(q1[2], q1[3]), false, false);
    const u32x4 v = {a[0], b[0], a[1], b[1]};
    return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ float halves_sum(float v)      // over the two lanes of a row
{
    const unsigned p = __builtin_bit_cast(unsigned, v);
    const u32x2 a = __builtin_amdgcn_permlane32_swap(p, p, false, false);
    const unsigned a0 = a[0], a1 = a[1];
    return __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1);
}
__device__ __forceinline__ f32x4 quad(const f32x16 &v, int q) { return f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]}; }

template <int W, bool LAYER, bool QKV, bool LORA>
__global__ __launch_bounds__(64 * W, 2) void rowreg_kernel(const RowLayerArgs a)
{
    constexpr int D = RR_D, KT = D / 64, NJ = D / 32, KS = D / 16, Nq = 3 * D, NQ = Nq / 64, UNIT = RR_UNIT;
    static_assert(UNIT == KT * 8192, "a unit is a tile per 64 columns");
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char *stage = lds + RR_SLOTS * UNIT;
    float *b1_s = (float *)(stage + W * RR_STAGE);         // [Dm]
    float *bq_s = b1_s + RR_MAX_DM;                        // [3 D]
    float *bp_s = bq_s + Nq;                               // [D]
    float *b2_s = bp_s + D;                                // [D]
    float *gb2_s = b2_s + D;                               // LayerNorm2 gain [D], shift [D]
    float *gbq_s = gb2_s + 2 * D;                          // LayerNorm1' gain, shift
    float *gelu_s = gbq_s + 2 * D;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 31, lh = lane >> 5, lr = lane >> 3;
    const int Dm = a.Dm, nc = LAYER ? Dm >> 6 : 0;
    const int n_out = a.n_out_dev ? min(*a.n_out_dev, a.n_out) : a.n_out;
    const int total = n_out * a.T;
    if (a.row_first + (int)blockIdx.x * 32 * W >= total) return;
    const int row0 = a.row_first + (blockIdx.x * W + wave) * 32;
    const int rows = min(max(total - row0, 0), 32);        // none in the last waves of the last tile: they load weights and compute what is not stored
    const bool full = rows == 32;

    // ---- the ring of weights.  A unit is KT tiles [64][64]: 64 rows of a matrix with D columns (N), or all D rows of 64 columns (K).
    const unsigned ring = __builtin_amdgcn_readfirstlane(lds_addr_of(lds));
    // Of the eight pieces of a tile (8 rows, 1 KB, an instruction) a wave loads piece `wave`, of four waves piece `wave` + 4 too.
    constexpr int PW = 8 / W, PU = KT * PW;                // pieces of a wave per tile and per unit
    const unsigned swz = (unsigned)(((lane & 7) ^ (4 * (wave & 1) + (lr >> 1))) << 4);
    const unsigned off_d = (unsigned)lr * (D * 2) + swz, off_m = (unsigned)lr * (Dm * 2) + swz;
    auto slot = [&](int pos) { return ring + (pos & RR_SLOTS - 1) * UNIT + wave * 1024; };
    const bf16_t *const w1 = a.W1t + (size_t)(8 * wave) * D, *const w2 = a.W2t + (size_t)(8 * wave) * Dm, *const wq = a.Wqt + (size_t)(8 * wave) * D;
    auto issue_n = [&](const bf16_t *w, int pos) {         // w: first row of the unit for this wave
#pragma unroll
        for (int i = 0; i < PU; ++i) glds16_s(w + 64 * (i / PW) + 32 * (i % PW) * D, off_d, slot(pos) + i / PW * 8192 + i % PW * 4096);
    };
    auto issue_k = [&](const bf16_t *w, int ld, unsigned off, int pos) {
#pragma unroll
        for (int i = 0; i < PU; ++i) glds16_s(w + (size_t)(64 * (i / PW) + 32 * (i % PW)) * ld, off, slot(pos) + i / PW * 8192 + i % PW * 4096);
    };
    // positions in the order of use: P0 .., N0, K0, N1, K1, .., K(nc - 1), Q0 ..
    const int pos_n0 = KT, pos_q0 = LAYER ? KT + 2 * nc : 0;
    auto issue_first = [&](int p) {                        // of the first KT + 3 positions
        if (!LAYER) issue_n(wq + (size_t)(64 * p) * D, p);
        else if (p < KT) issue_k(a.Wpt + (size_t)(8 * wave) * D + 64 * p, D, off_d, p);
        else if (p == KT) issue_n(w1, p);
        else if (p == KT + 1) issue_k(w2, Dm, off_m, p);
        else issue_n(w1 + (size_t)64 * D, p);
    };
    auto issue_q = [&](int q) { issue_n(wq + (size_t)(64 * q) * D, pos_q0 + q); };

    // ---- prologue: everything is requested at once
#pragma unroll
    for (int p = 0; p < RR_SLOTS; ++p) issue_first(p);
    auto vec = [&](const float *src, int from, int to, const float *dst) {
        for (int i = from; i < to; i += 64) glds4(src + i + lane, __builtin_amdgcn_readfirstlane(lds_addr_of(dst)) + i * 4);
    };
    if (LAYER) {
        if (wave == 0) vec(a.b1, 0, Dm, b1_s);
        if (wave == 1) { vec(a.bp, 0, D, bp_s); vec(a.b2, 0, D, b2_s); vec(a.ln2_g, 0, D, gb2_s); vec(a.ln2_b, 0, D, gb2_s + D); }
    }
    if (QKV) {
        if (wave == 2) { vec(a.lnq_g, 0, D, gbq_s); vec(a.lnq_b, 0, D, gbq_s + D); }
        if (wave == W - 1) vec(a.bq, 0, Nq, bq_s);
    }

    // The rows of this wave: block bA up to row tB of them, block bA + 1 from there on (with adapters or a map a block has at least 32 rows).  A wave
    // without rows reads the last ones there are; the maps have entries for the blocks that exist only.
    const int lrow = min(row0 + lm, total - 1), group = min(row0, total - 1) >> 5;
    const int bA = min(row0, total - 1) / a.T, tB = rows > 0 ? (bA + 1) * a.T - row0 : 32;
    const bool hasB = tB < rows;
    int kA = 0, kB = 0;
    if (LORA) {
        kA = a.adapter_of_out[bA];
        if (hasB) kB = a.adapter_of_out[bA + 1];
    }
    const bool lora_p = LORA && LAYER && a.Apt, lora_q = LORA && QKV && a.Aqt;
    bf16x8 fa[KS];                                         // rows as the operand of a product over D
    if (LAYER) {
        const bf16_t *o = a.o + (size_t)group * (32 * D) + lane * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s) fa[s] = *(const bf16x8 *)(o + s * 512);
    }
    f32x16 x[NJ];                                          // the residual stream: columns 32 j + 8 q + 4 lh + {0..3} of row lm
    {
        const float *src = a.res + (size_t)group * (32 * D) + lane * 4;
        int step = 256;                                    // from q to q + 1
        if (!a.res_fragments) {
            size_t xrow = lrow;
            if (a.res_block_of_out) {
                const int inB = hasB && lrow - row0 >= tB;
                const int mA = a.res_block_of_out[bA], mB = hasB ? a.res_block_of_out[bA + 1] : 0;
                xrow = (size_t)(inB ? mB : mA) * a.T + (lrow - (bA + inB) * a.T);
            }
            src = a.res + xrow * D + 4 * lh;
            step = 8;
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 v = *(const f32x4 *)(src + (j * 4 + q) * step);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[j][4 * q + e] = v[e];
            }
    }
    if (LAYER) {                                           // Phi table of the GELU
#pragma unroll 1
        for (int i = tid; i < GELU_TAB_ENTRIES; i += 64 * W) *(f32x2 *)(gelu_s + 2 * i) = gelu_tab_entry(i);
    }

    // s (rows At_k), the operand of the expand, from At_k requested earlier.  Rows of the other block get this block's term too and leave it: theirs may
    // not come near this adapter's values.
    const int r = a.r;
    const bool inB = lm >= tB;
    constexpr int NA = LORA ? KS : 1;
    auto request_at = [&](bf16x8(&at)[NA], const bf16_t *At, int k) {
        const bf16_t *At_k = At + (size_t)k * r * D + min(lm, r - 1) * D + 8 * lh;
        if constexpr (LORA) {
#pragma unroll
            for (int s = 0; s < KS; ++s) at[s] = *(const bf16x8 *)(At_k + 16 * s);
        }
    };
    auto shrink = [&](const bf16x8(&at)[NA]) {
        f32x16 c;
#pragma unroll
        for (int e = 0; e < 16; ++e) c[e] = 0.f;
        if constexpr (LORA) {
#pragma unroll
            for (int s = 0; s < KS; ++s) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at[s], fa[s], c, 0, 0, 0);
        }
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        return operand(a.scale * quad(c, 0), r > 8 ? a.scale * quad(c, 1) : z);
    };
    // ranks 8 lh .. + 7 of column n of Bt_k [.][r] (of 8 ranks: the second half meets zeros)
    const int off_r = r > 8 ? 8 * lh : 0;
    auto bt = [&](const bf16_t *Bt_k, int n) { return *(const bf16x8 *)(Bt_k + n * r + off_r); };
    bf16x8 at0[NA];
    if (lora_p) request_at(at0, a.Apt, kA);
    if (!LAYER && lora_q) request_at(at0, a.Aqt, kA);

    // ---- operands out of the ring: 32 rows x 16 columns, lane (lm, lh) columns 8 lh .. + 7 of row lm
    const unsigned wf = lm * 128 + ((lh ^ ((lm >> 1) & 7)) << 4);
    lds_ptr wk[4];
    auto unit = [&](int pos) {
        unsigned f = wf;
        asm volatile("" : "+v"(f));                        // (kept as one register instead of four)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) wk[kk] = (lds_ptr)(lds + (pos & RR_SLOTS - 1) * UNIT + (f ^ (kk << 5)));
    };
    auto rd = [&](int tile, int half, int kk) { return *(const __attribute__((address_space(3))) bf16x8 *)(wk[kk] + tile * 8192 + half * 4096); };
    auto frag_k = [&](int n) { return rd((n % NJ) >> 1, n & 1, n / NJ); };     // weights of product n of a K unit (NJ is even), of an N unit
    auto frag_n = [&](int n) { return rd(n >> 3, n & 1, (n >> 1) & 3); };
    constexpr int PF = 6, NP = 8 * KT;                     // weights are read PF products ahead; products of a unit
    bf16x8 w[PF];
    auto mul_k = [&](int n, const bf16x8 *f) { x[n % NJ] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[n % PF], f[n / NJ], x[n % NJ], 0, 0, 0); };
    auto bias = [&](f32x16(&y)[2], const float *b) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 v = *(const f32x4 *)(b + 32 * i + 8 * q + 4 * lh);
#pragma unroll
                for (int e = 0; e < 4; ++e) y[i][4 * q + e] = v[e];
            }
    };
    auto product_n = [&](f32x16(&y)[2], auto side) {       // the 64 columns of the unit at wk, on top of y
#pragma unroll
        for (int i = 0; i < PF; ++i) w[i] = frag_n(i);
#pragma unroll
        for (int n = 0; n < NP; ++n) {
            __builtin_amdgcn_sched_barrier(0);
            y[n & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[n % PF], fa[n >> 1], y[n & 1], 0, 0, 0);
            if (n + PF < NP) w[n % PF] = frag_n(n + PF);
            side(n);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // (the barriers for the scheduler, here and below: left alone it reads all of a vector ahead and has no registers left)
    auto add_bias = [&](const float *b) {
        f32x4 v[2][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[0][q] = *(const f32x4 *)(b + 8 * q + 4 * lh);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            __builtin_amdgcn_sched_barrier(0);
            if (j + 1 < NJ) {
#pragma unroll
                for (int q = 0; q < 4; ++q) v[(j + 1) & 1][q] = *(const f32x4 *)(b + 32 * (j + 1) + 8 * q + 4 * lh);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) x[j][4 * q + e] += v[j & 1][q][e];
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // LayerNorm (fp32 statistics, centred second moment) of the rows -> fa
    auto layernorm = [&](const float *gb) {
        float t[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) t[e & 3] += x[j][e];
        const float mean = halves_sum((t[0] + t[1]) + (t[2] + t[3])) * (1.0f / D);
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) { const float d = x[j][e] - mean; v[e & 3] = fmaf(d, d, v[e & 3]); }
        const float inv = rsqrtf(halves_sum((v[0] + v[1]) + (v[2] + v[3])) * (1.0f / D) + a.eps), nmi = -mean * inv;
        f32x4 g[2][2], b[2][2];
        auto fetch = [&](int s) {
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                g[s & 1][z] = *(const f32x4 *)(gb + 16 * s + 8 * z + 4 * lh);
                b[s & 1][z] = *(const f32x4 *)(gb + D + 16 * s + 8 * z + 4 * lh);
            }
        };
        fetch(0);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            __builtin_amdgcn_sched_barrier(0);
            if (s + 1 < KS) fetch(s + 1);
            f32x4 y[2];
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int e = 0; e < 4; ++e) y[z][e] = fmaf(fmaf(x[s >> 1][8 * (s & 1) + 4 * z + e], inv, nmi), g[s & 1][z][e], b[s & 1][z][e]);   // ((x - mean) inv) g + b
            fa[s] = operand(y[0], y[1]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    char *const st = stage + wave * RR_STAGE;
    const int sr = lane >> 3, sp = lane & 7;               // row and 16-byte piece of eight staged rows that a lane moves
    auto store_x = [&]() {
        if (a.out_fragments) {
            float *dst = a.x_out + (size_t)group * (32 * D) + lane * 4;
            if (lm < rows) {
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) *(f32x4 *)(dst + (j * 4 + q) * 256) = quad(x[j], q);
            }
        } else {
            float *dst = a.x_out + (size_t)row0 * D + 4 * sp;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
#pragma unroll
                for (int q = 0; q < 4; ++q) *(f32x4 *)(st + lm * 128 + (((2 * q + lh) ^ (lm & 7)) << 4)) = quad(x[j], q);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = 8 * q + sr;
                    const f32x4 v = *(const f32x4 *)(st + row * 128 + ((sp ^ (row & 7)) << 4));
                    if (row < rows) *(f32x4 *)(dst + (size_t)row * D + 32 * j) = v;
                }
            }
        }
    };

    rl_wait_barrier<0>();
    if (LAYER) {
        // ============================================================ A: x' = res + o Wp + bp + lora
        bf16x8 fs[2], bp[NJ];
        if (lora_p) {
            fs[0] = shrink(at0);
        }
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            unit(t);
#pragma unroll
            for (int i = 0; i < PF; ++i) w[i] = frag_k(i);
#pragma unroll
            for (int n = 0; n < NP; ++n) {
                __builtin_amdgcn_sched_barrier(0);
                mul_k(n, fa + 4 * t);
                if (n + PF < NP) w[n % PF] = frag_k(n + PF);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        auto request_bp = [&](int k) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) bp[j] = bt(a.Bpt + (size_t)k * D * r, 32 * j + lm);
        };
        if (lora_p) request_bp(kA);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int p = RR_SLOTS; p < KT + 3; ++p) issue_first(p);
        add_bias(bp_s);
        if (lora_p) {
            if (hasB) {
                bf16x8 at[NA];
                request_at(at, a.Apt, kB);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const f32x16 y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bp[j], fs[0], x[j], 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 16; ++e) x[j][e] = inB ? x[j][e] : y[e];
                }
                fs[1] = shrink(at);
                request_bp(kB);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const f32x16 y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bp[j], fs[1], x[j], 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 16; ++e) x[j][e] = inB ? y[e] : x[j][e];
                }
            } else {
#pragma unroll
                for (int j = 0; j < NJ; ++j) x[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bp[j], fs[0], x[j], 0, 0, 0);
            }
        }
        layernorm(gb2_s);

        // ============================================================ B: x'' = x' + b2 + GELU(LayerNorm2(x') W1 + b1) W2
        add_bias(b2_s);
        // In steps of 32 hidden columns: while the GELU of step s runs on the vector unit, the matrix unit adds step s - 1 to x and makes the columns of
        // step s + 1.  A chunk of the ring: steps 2 c + 1 and 2 c + 2, K(c) and N(c + 1).
        const unsigned gelu_a = lds_addr_of(gelu_s);
        bf16x8 hb[2][2];                                   // [step & 1]
        // weights of the n-th product of a step whose columns are half `i` of their units: even ones of x, odd ones of the next columns
        auto frag_s = [&](int n, int i) {
            const int m = n >> 1;
            if (n & 1) return *(const __attribute__((address_space(3))) bf16x8 *)(wk[m & 3] + UNIT + (m >> 2) * 8192 + i * 4096);
            return *(const __attribute__((address_space(3))) bf16x8 *)(wk[2 * i + m / NJ] + (m % NJ >> 1) * 8192 + (m & 1) * 4096);
        };
        float xc[4];
        f32x2 en[4];
        f32x4 gy[2];
        auto look = [&](const f32x16 &v, int e) { gelu_look(v[e], gelu_a, xc[e & 3], en[e & 3]); };
        auto fin = [&](const f32x16 &v, int e, bf16x8(&o)[2]) {
            gy[e >> 2 & 1][e & 3] = v[e] * fmaf(xc[e & 3], en[e & 3][1], en[e & 3][0]);
            if ((e & 7) == 7) o[e >> 3] = operand(gy[0], gy[1]);
        };
        auto bias32 = [&](f32x16 &v, const float *b) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 t = *(const f32x4 *)(b + 8 * q + 4 * lh);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * q + e] = t[e];
            }
        };
        // step: GELU of `cur` -> out; x += prev * K; next = columns of N
        constexpr int PS = 4;
        auto step = [&](auto I, const f32x16 &cur, bf16x8(&out)[2], const bf16x8(&prev)[2], f32x16 &next, const float *b, auto last, auto side) {
            constexpr int i = decltype(I)::value, M = 4 * NJ;       // 2 NJ of x and as many of the next columns
            constexpr bool end = decltype(last)::value;
#pragma unroll
            for (int n = 0; n < PS; ++n)
                if (!end || !(n & 1)) w[n] = frag_s(n, i);
            if (!end) bias32(next, b);
#pragma unroll
            for (int n = 0; n < M; ++n) {
                __builtin_amdgcn_sched_barrier(0);
                const int m = n >> 1;
                if (!(n & 1)) x[m % NJ] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[n % PS], prev[m / NJ], x[m % NJ], 0, 0, 0);
                else if (!end) next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[n % PS], fa[m], next, 0, 0, 0);
                if (n + PS < M && (!end || !(n & 1))) w[n % PS] = frag_s(n + PS, i);
#pragma unroll
                for (int e = 0; e < 16; ++e) {              // value e: looked up in slot e (M - 6) / 16, finished four values on
                    if (e >= 4 && n == e * (M - 6) / 16) fin(cur, e - 4, out);
                    if (n == e * (M - 6) / 16) look(cur, e);
                }
                if (n >= M - 4) fin(cur, 12 + n - (M - 4), out);
                side(n);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        f32x16 h0, h1;
        {                                                  // columns of steps 0 and 1, GELU of step 0
            unit(pos_n0);
            bias32(h0, b1_s);
            bias32(h1, b1_s + 32);
            constexpr int M = 2 * KS;
            auto frag = [&](int n) { return *(const __attribute__((address_space(3))) bf16x8 *)(wk[(n >> 1) & 3] + (n >> 3) * 8192 + (n & 1) * 4096); };
#pragma unroll
            for (int n = 0; n < PF; ++n) w[n] = frag(n);
#pragma unroll
            for (int n = 0; n < M; ++n) {
                __builtin_amdgcn_sched_barrier(0);
                if (n & 1) h1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[n % PF], fa[n >> 1], h1, 0, 0, 0);
                else h0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[n % PF], fa[n >> 1], h0, 0, 0, 0);
                if (n + PF < M) w[n % PF] = frag(n + PF);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 20; ++e) {
                if (e >= 4) fin(h0, e - 4, hb[0]);
                if (e < 16) look(h0, e);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        using std::integral_constant;
        integral_constant<int, 0> half0;
        integral_constant<int, 1> half1;
#pragma unroll 1
        for (int c = 0; c < nc - 1; ++c) {
            const int pos = pos_n0 + 1 + 2 * c;            // K(c); N(c + 1) behind it
            rl_wait_barrier<0>();                          // both are there, and the two before them are no longer read
            // K(c + 1) and N(c + 2), past the end Q(0), into the slots of those two, a load between every few products
            const bool b_n = c + 2 < nc;
            const bf16_t *base_a = w2 + 64 * (c + 1), *base_b = b_n ? w1 + (size_t)(64 * (c + 2)) * D : wq;
            const int go_b = QKV || b_n;
            const unsigned slot_a = slot(pos + 2), slot_b = slot(pos + 3);
            auto share = [&](int n, auto load) {
#pragma unroll
                for (int i = 0; i < PU; ++i)
                    if (n == 1 + i * (4 * NJ - 2) / PU) load(i / PW, i % PW);
            };
            unit(pos);
            step(half0, h1, hb[1], hb[0], h0, b1_s + 64 * (c + 1), std::false_type{}, [&](int n) {
                share(n, [&](int t, int p) { glds16_s(base_a + (size_t)(64 * t + 32 * p) * Dm, off_m, slot_a + t * 8192 + p * 4096); });
            });
            step(half1, h0, hb[0], hb[1], h1, b1_s + 64 * (c + 1) + 32, std::false_type{}, [&](int n) {
                share(n, [&](int t, int p) { glds16_if(base_b + 64 * t + 32 * p * D, off_d, slot_b + t * 8192 + p * 4096, go_b); });
            });
        }
        {                                                  // the last chunk
            rl_wait_barrier<0>();
            const int pos = pos_q0 - 1;
            if (QKV) { issue_q(1); issue_q(2); }
            unit(pos);
            step(half0, h1, hb[1], hb[0], h0, b1_s, std::true_type{}, [](int) {});
#pragma unroll
            for (int m = 0; m < 2 * NJ; ++m)
                x[m % NJ] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_s(2 * m, 1), hb[1][m / NJ], x[m % NJ], 0, 0, 0);
        }
    }

    if (LAYER && !QKV) store_x();
    if (QKV) {
        if (LAYER) {                                       // K(nc - 1) is no longer read
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            issue_q(3);
        }
        bf16x8 at1[NA];
        if (LAYER && lora_q) request_at(at1, a.Aqt, kA);
        layernorm(gbq_s);
        if (LAYER) rl_wait_barrier<0>();                   // Q(0) .. Q(3)
        bf16x8 fsA, fsB, wA[2], wB[2];
        auto request_bt = [&](int q) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                wA[i] = bt(a.Bqt + (size_t)kA * Nq * r, 64 * q + 32 * i + lm);
                if (hasB) wB[i] = bt(a.Bqt + (size_t)kB * Nq * r, 64 * q + 32 * i + lm);
            }
        };
        if (lora_q) {
            fsA = shrink(LAYER ? at1 : at0);
            request_bt(0);
        }
        if (LAYER) store_x();
        if (lora_q && hasB) {
            bf16x8 at[NA];
            request_at(at, a.Aqt, kB);
            fsB = shrink(at);
        }
        char *const out = (char *)(a.qkv_out + (size_t)row0 * Nq) + sp * 16;
        // 64 columns of unit q; what is done with those of the unit before stands between the products
        auto columns = [&](f32x16(&y)[2], int q, auto side) {
            unit(pos_q0 + q);
            bias(y, bq_s + 64 * q);
            product_n(y, side);
            if (lora_q) {
                if (hasB) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const f32x16 v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wB[i], fsB, y[i], 0, 0, 0);
                        y[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wA[i], fsA, y[i], 0, 0, 0);
#pragma unroll
                        for (int e = 0; e < 16; ++e) y[i][e] = inB ? v[e] : y[i][e];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 2; ++i) y[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wA[i], fsA, y[i], 0, 0, 0);
                }
                request_bt(min(q + 1, NQ - 1));
            }
        };
        f32x4 sv[4];
        auto finish = [&](int n, const f32x16(&y)[2], int q) {         // the n-th of the steps that round, stage and store the columns of unit q
            if (n < 8) {
                const int i = n >> 2, g = n & 3;
                const u32x2 v = {pack2(y[i][4 * g], y[i][4 * g + 1]), pack2(y[i][4 * g + 2], y[i][4 * g + 3])};
                *(u32x2 *)(st + lm * 128 + ((n ^ (lm & 7)) << 4) + 8 * lh) = v;
            } else if (n < 12) {
                const int row = 8 * (n - 8) + sr;
                sv[n - 8] = *(const f32x4 *)(st + row * 128 + ((sp ^ (row & 7)) << 4));
            } else if (n < 16) {
                const int row = 8 * (n - 12) + sr;
                if (row < rows) *(f32x4 *)(out + (size_t)row * (Nq * 2) + q * 128) = sv[n - 12];
            }
        };
        f32x16 h[2], h1[2];
#pragma unroll 1
        for (int q = 0; q < NQ; q += 2) {
            if (q > 0) {
                // Q(q) and Q(q + 1) have landed, and the two before them are no longer read.  Behind their loads, where every store is issued: the stores of two units
                if (q < RR_SLOTS) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                else if (full) rl_wait_barrier<8>();
                else rl_wait_barrier<0>();
                if (q + 2 < NQ) issue_q(q + 2);
                if (q + 3 < NQ) issue_q(q + 3);
                columns(h, q, [&](int n) { finish(n, h1, q - 1); });
            } else columns(h, q, [](int) {});
            if (q + 1 < NQ) columns(h1, q + 1, [&](int n) { finish(n, h, q); });
        }
#pragma unroll
        for (int n = 0; n < 16; ++n) finish(n, NQ & 1 ? h : h1, NQ - 1);
    }
}

template <int W, bool LAYER, bool QKV, bool LORA> int launch_t(const RowLayerArgs &a, long rows, hipStream_t st)
{
    constexpr int D = RR_D;
    constexpr int LDS = RR_SLOTS * RR_UNIT + W * RR_STAGE + (RR_MAX_DM + 3 * D + 2 * D + 4 * D) * 4 + RR_GELU * 8;
    static_assert(LDS <= 160 * 1024, "LDS budget");
    auto kern = rowreg_kernel<W, LAYER, QKV, LORA>;
    static bool attr_set = false;       // raising the dynamic LDS limit is a per-kernel, process-wide setting
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS) != hipSuccess) return POLY_EHIP;
        attr_set = true;
    }
    POLY_LAUNCH_SHMEM(POLY_STAGE_GEMM, kern, dim3((unsigned)((rows + 32 * W - 1) / (32 * W))), dim3(64 * W), LDS, st, a);
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

template <int W> int launch_w(const RowLayerArgs &a, long rows, hipStream_t st)      // rows: from a.row_first on
{
    const bool lora = (a.o && a.Apt) || (a.qkv_out && a.Aqt);
    if (!a.o) return lora ? launch_t<W, false, true, true>(a, rows, st) : launch_t<W, false, true, false>(a, rows, st);
    if (!a.qkv_out) return lora ? launch_t<W, true, false, true>(a, rows, st) : launch_t<W, true, false, false>(a, rows, st);
    return lora ? launch_t<W, true, true, true>(a, rows, st) : launch_t<W, true, true, false>(a, rows, st);
}

}  // namespace

int launch_rowreg(const RowLayerArgs &a, int waves, hipStream_t st)
{
    if (a.n_out <= 0 || a.T <= 0) return POLY_OK;
    const bool lora = (a.o && a.Apt) || (a.qkv_out && a.Aqt);
    if (a.D != RR_D || a.Dm < 128 || a.Dm % 64 || a.Dm > RR_MAX_DM || (lora && a.r != 8 && a.r != 16) || ((lora || a.res_block_of_out) && a.T < 32)) return POLY_EINVAL;
    const long rows = (long)a.n_out * a.T, full = waves == ROWREG_BOTH ? rowreg_full(rows) : waves == 8 ? rows : 0;
    RowLayerArgs rest = a;
    rest.row_first = (int)full;
    if (full > 0) { const int rc = launch_w<8>(a, full, st); if (rc != POLY_OK) return rc; }
    return full < rows ? launch_w<4>(rest, rows - full, st) : POLY_OK;
}
