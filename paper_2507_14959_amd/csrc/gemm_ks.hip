// The linears of small calls and of single precision: y = x W + b (+ s (x A_k) B_k) on tiles of 32 or 64 rows and columns, the
// contraction split over the four waves of a workgroup.
//
// What bounds a product of a few hundred rows is not arithmetic: a grid of 128 x 128 tiles leaves most of the 256 CUs idle, and
// the busy ones wait for K / 64 round trips of an LDS ring that all their waves share through a barrier.  Here
//  - tiles are small, so that the weights and rows a CU has to pull through its load path (30-50 bytes per clock) are few and the
//    grid covers the chip;
//  - wave w takes the k-tiles w, w + 4, .. (128 bytes of every row each) of the whole tile through a ring of its own: up to three
//    of its k-tiles are in flight, there is no barrier in the loop, and a 768-long contraction is three steps;
//  - the four partial sums meet in LDS once, in fixed order (the same for every tile size of this file; the kernels that larger calls
//    take sum in other orders), and each wave finishes one 32 x 32 subtile: low-rank expand, bias, GELU or residual;
//  - the chain offsets -> adapter ids -> operands of the expand, and the residual rows, are requested before the loop.
// v_mfma_f32_32x32x16_bf16, or v_mfma_f32_32x32x2_f32 (true single precision: twice the rate of the vector ALU without packed
// operations).  A lane's 16 bytes are 8 or 4 consecutive contraction elements of one row; both operands use the same order.
//
// 3 frames (591 rows) through the 768-wide backbone: proj and fc2 30 us each with 128 x 128 tiles, 16 us here, 1338 -> 906 us per
// forward.  fp32 (68-119 rows, K = 192 and 768) 49 us per product on the vector ALU, 7 to 9 us here.
#include "poly_dev.h"
#include "rowtile.h"

namespace {

template <typename T> struct Elt;
template <> struct Elt<bf16_t> {
    static constexpr int V = 8;                            // elements per 16 bytes
    typedef bf16x8 frag;
    static __device__ __forceinline__ f32x16 mma(frag w, frag x, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, x, c, 0, 0, 0); }
    static __device__ __forceinline__ f32x4 gelu4(f32x4 v) { return gelu_poly4(v); }
};
template <> struct Elt<float> {
    static constexpr int V = 4;
    typedef f32x4 frag;
    static __device__ __forceinline__ f32x16 mma(frag w, frag x, f32x16 c)
    {
#pragma unroll
        for (int z = 0; z < 4; ++z) c = __builtin_amdgcn_mfma_f32_32x32x2f32(w[z], x[z], c, 0, 0, 0);
        return c;
    }
    static __device__ __forceinline__ f32x4 gelu4(f32x4 v) { return f32x4{gelu_erf(v[0]), gelu_erf(v[1]), gelu_erf(v[2]), gelu_erf(v[3])}; }
};

// a value that every lane of the wave reads from the same address, written by an earlier launch: through the scalar cache, whose
// counter is not the one the tile loads wait on
__device__ __forceinline__ int uload(const int *p) { return *(const int __attribute__((address_space(4))) *)(uintptr_t)p; }

constexpr int KS_NSMAX = 3;

// MI x NI subtiles of 32 x 32 per tile.  ns: ring stages per wave.  SHRINK: S = scale * x At_k^T (weights of the output block's own
// adapter, row tiles inside blocks, columns past the rank zero) instead of a linear with shared weights.  AL: every pointer is on a
// 16-byte boundary; else the operands are fetched and the results stored element by element (the addresses the caller gave need no more
// than the alignment of an element; loads to LDS need 16 bytes).
// PATCH: the rows are the patches of a frame, gathered by the loads (PatchRows).
template <typename T, int MI, int NI, bool SHRINK, bool AL, bool PATCH>
__device__ __forceinline__ void gemm_ks_tile(const GemmArgs &g, int tiles_m, int tiles_n, int ns, const PatchRows &pr)
{
    typedef Elt<T> E;
    typedef typename E::frag frag;
    constexpr int V = E::V, BK = 8 * V, BM = 32 * MI, BN = 32 * NI;
    constexpr int STAGE = (BM + BN) * 128, NLD = (BM + BN) / 8;      // bytes / loads (8 rows x 128 bytes) per stage
    constexpr int NF = MI * NI;                                       // subtiles, finished by waves 0 .. NF - 1
    static_assert(NF <= 4, "one subtile per wave at most");
    extern __shared__ __attribute__((aligned(16))) char ks_lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lm = lane & 31, lh = lane >> 5;
    const bool flat = g.Tb > 0;                            // one run of rows over all input blocks
    const int n_bound = flat ? g.nb : g.n_in;
    const int n_true = g.n_in_dev ? min(uload(g.n_in_dev), n_bound) : n_bound;
    const int Tlim = flat ? n_true * g.Tb : g.T, Tblk = flat ? g.Tb : g.T;
    const int mtot = flat ? (Tlim + BM - 1) / BM : n_true * tiles_m;
    // the tiles that exist are cut into eight equal runs, one per XCD: of columns with all their rows when there are more columns
    // than rows (a column's weights come to one L2 only), else of rows with all their columns
    int mt, tn;
    {
        const int xcd = blockIdx.x & 7;
        const long total = (long)mtot * tiles_n, lo = total * xcd / 8, hi = total * (xcd + 1) / 8, L = lo + (blockIdx.x >> 3);
        if (L >= hi) return;
        if (mtot <= tiles_n) { tn = (int)(L / mtot); mt = (int)(L - (long)tn * mtot); }
        else { mt = (int)(L / tiles_n); tn = (int)(L - (long)mt * tiles_n); }
    }
    const int blk = flat ? 0 : mt / tiles_m, t0 = (flat ? mt : mt - blk * tiles_m) * BM, n0 = tn * BN;
    int xb = blk, k_own = -1;                              // input block; SHRINK: adapter whose weights this tile uses
    if (SHRINK) {
        k_own = uload(g.adapter_of_out + blk);
        if (g.res_block_of_out) xb = uload(g.res_block_of_out + blk);
        if (k_own < 0) return;
    }
    const int nw = SHRINK ? g.r : g.N;                     // weight rows
    const T *A = (const T *)g.A + ((size_t)xb * g.T + (PATCH ? 0 : t0)) * g.K;    // (a frame has as many elements as its patches)
    const T *W = (const T *)g.Wt + ((size_t)(SHRINK ? k_own * g.r : 0) + n0) * g.K;

    // ---- k-tiles of this wave: wave, wave + 4, ..  A lane loads 16 bytes: row 8 g + lane / 8 of a tile, position lane % 8; the
    // 128-byte rows are stored with their chunks swizzled by (row >> 1) & 7.  Rows past the end repeat the last one (their
    // results are never stored); chunks past K are read from the row's last chunk and masked below.
    const int nk = (g.K + BK - 1) / BK, steps = (nk - wave + 3) >> 2;
    const unsigned rowb = (unsigned)g.K * sizeof(T);
    const int lr = lane >> 3, c0 = (lane & 7) ^ (lr >> 1), c1 = c0 ^ 4;
    const int tail = g.K - (nk - 1) * BK;                  // elements in the last k-tile
    const int adj0 = min(c0, tail / V - 1) - c0, adj1 = min(c1, tail / V - 1) - c1;
    char *ring = ks_lds + wave * ns * STAGE;
    unsigned patch0[PATCH ? BM / 8 : 1];                   // first byte of this lane's patches
    if constexpr (PATCH) {
#pragma unroll
        for (int q = 0; q < BM / 8; ++q) patch0[q] = patch_start(pr, min(t0 + 8 * q + lr, Tlim - 1), sizeof(T));
    }
    // 16 bytes of this lane's: to LDS at lds + 16 lane
    auto fetch = [&](const char *base, unsigned off, char *lds) {
        if constexpr (AL) {
            glds16_s(base, off, __builtin_amdgcn_readfirstlane(lds_addr_of(lds)));
        } else {
            const T *src = (const T *)(base + off);
            frag v;
#pragma unroll
            for (int z = 0; z < V; ++z) v[z] = src[z];
            *(frag *)(lds + lane * 16) = v;
        }
    };
    auto issue = [&](int i) {
        const int kt = wave + 4 * i;
        const bool last = kt == nk - 1;                    // uniform
        char *st = ring + (i % ns) * STAGE;
        const unsigned e0 = (unsigned)(c0 + (last ? adj0 : 0)) * 16, e1 = (unsigned)(c1 + (last ? adj1 : 0)) * 16;
        if constexpr (PATCH) {
            const unsigned p0 = patch_piece(pr, 8 * kt + e0 / 16), p1 = patch_piece(pr, 8 * kt + e1 / 16);
#pragma unroll
            for (int q = 0; q < BM / 8; ++q) fetch((const char *)A, patch0[q] + ((q & 1) ? p1 : p0), st + q * 1024);
        } else {
#pragma unroll
            for (int q = 0; q < BM / 8; ++q)
                fetch((const char *)A + (size_t)kt * 128, (unsigned)min(8 * q + lr, Tlim - 1 - t0) * rowb + ((q & 1) ? e1 : e0), st + q * 1024);
        }
#pragma unroll
        for (int q = 0; q < BN / 8; ++q)
            fetch((const char *)W + (size_t)kt * 128, (unsigned)min(8 * q + lr, nw - 1 - n0) * rowb + ((q & 1) ? e1 : e0), st + (BM / 8 + q) * 1024);
    };
    const int npro = min(ns, steps);
    for (int i = 0; i < npro; ++i) issue(i);

    // ---- what the finishing waves will need: the first output block of their subtile's first input block, its first low-rank
    // term and its residual rows, requested now
    const int fi = wave / NI, fj = wave % NI;              // this wave's subtile
    const int tw = t0 + 32 * fi, nc = n0 + 32 * fj;        // its first row (in the run or the block) and column
    const bool fin = wave < NF && tw < Tlim && nc < g.N;
    const int b_lo = flat ? tw / Tblk : xb;
    const bool has_lora = !SHRINK && g.S && g.adapter_of_out, vec = AL && g.N % 4 == 0;
    const int rch = lane & 7, rrow = lane >> 3;            // read-back mapping: 8 lanes x 16 bytes cover a row of the subtile
    const int col = nc + 4 * rch;
    // Short blocks: up to three or more lie in a subtile.  Where every input block is its own output block with one term (`own`), the subtile is
    // finished as one run of rows, with what its first PB blocks need requested here (block by block that was a round trip or two for each).
    // Single precision on 4 frames of 17 tokens, us per product, before / after: 192 -> 576 12.5 / 8.6, 192 -> 768 10.6 / 6.6, 768 -> 192 10.1 / 8.1.
    // (At most 256 registers: more, and the accumulators move to and from a second file: 3 % of the 768-wide backbone on 3 frames.)
    constexpr int PB = 3;
    const bool own = flat && !g.out_off && !g.set_off && vec;
    int pre_k[PB] = {-1, -1, -1};
    frag pre_s[16 / (2 * V)], pre_w[PB][16 / (2 * V)];     // operands of ranks [0, 16) of the first term (own: of every row, of PB blocks)
    f32x4 pre_r[4];
    int ob_pre = -1;
    const frag zero = {};
    auto load_s = [&](int sb, int t, int s0) { return *(const frag *)((const T *)g.S + ((size_t)sb * Tblk + t) * g.RP + s0 + lh * V); };
    auto load_w = [&](int k_ad, int s0) {                  // Bt rows of this subtile's columns
        const int c = min(nc + lm, g.N - 1), j0 = s0 + lh * V;
        const T *p = (const T *)g.Bt + ((size_t)k_ad * g.N + c) * g.r;
        frag f = zero;
        if (AL && g.r % V == 0) {
            f = *(const frag *)(p + min(j0, g.r - V));
            if (j0 + V > g.r) f = zero;
        } else {
#pragma unroll
            for (int q = 0; q < V; ++q)
                if (j0 + q < g.r) f[q] = p[j0 + q];
        }
        return f;
    };
    auto load_res = [&](f32x4(&v)[4], int ob, int trow0, int rows) {
        const int rb = g.res_block_of_out ? uload(g.res_block_of_out + ob) : ob;
        const float *src = g.res + ((size_t)rb * g.Tout + g.t_off) * g.N + min(col, g.N - 4);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = *(const f32x4 *)(src + (long)min(max(trow0 + 8 * q + rrow, 0), rows - 1) * g.N);
    };
    f32x4 bias4 = {0.f, 0.f, 0.f, 0.f};
    if (!SHRINK && fin && g.bias && vec) bias4 = *(const f32x4 *)(g.bias + min(col, g.N - 4));
    if (!SHRINK && fin && own) {
        ob_pre = b_lo;
        if (has_lora) {
            const int b_hi = (min(tw + 32, Tlim) - 1) / Tblk;
#pragma unroll
            for (int b = 0; b < PB; ++b)
                if (b_lo + b <= b_hi) pre_k[b] = uload(g.adapter_of_out + b_lo + b);
#pragma unroll
            for (int u = 0; u < 16 / (2 * V); ++u) pre_s[u] = load_s(0, min(tw + lm, Tlim - 1), 2 * V * u);
#pragma unroll
            for (int b = 0; b < PB; ++b)
                if (pre_k[b] >= 0)
#pragma unroll
                    for (int u = 0; u < 16 / (2 * V); ++u) pre_w[b][u] = load_w(pre_k[b], 2 * V * u);
        }
        if (g.mode == EPI_RESID && g.res)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                int row = min(tw + 8 * q + rrow, Tlim - 1);
                if (g.res_block_of_out) { const int b = row / Tblk; row += (g.res_block_of_out[b] - b) * Tblk; }
                pre_r[q] = *(const f32x4 *)(g.res + (long)row * g.N + min(col, g.N - 4));
            }
    } else if (!SHRINK && fin) {
        const int o0 = g.out_off ? uload(g.out_off + b_lo) : b_lo, o1 = g.out_off ? uload(g.out_off + b_lo + 1) : b_lo + 1;
        if (o0 < o1) {
            ob_pre = o0;
            const int trow0 = flat ? tw - b_lo * Tblk : tw;
            if (has_lora) {
                const int s0 = g.set_off ? uload(g.set_off + o0) : o0, s1 = g.set_off ? uload(g.set_off + o0 + 1) : o0 + 1;
                const int k_ad = s0 < s1 ? uload(g.adapter_of_out + s0) : -1;
                if (k_ad >= 0) {
#pragma unroll
                    for (int u = 0; u < 16 / (2 * V); ++u) {
                        pre_s[u] = load_s(s0, min(max(trow0 + lm, 0), Tblk - 1), 2 * V * u);
                        pre_w[0][u] = load_w(k_ad, 2 * V * u);
                    }
                }
            }
            if (g.mode == EPI_RESID && g.res && vec) load_res(pre_r, o0, trow0, Tblk);
        }
    }

    // ---- main loop: no barrier.  k-tile i has landed once at most the loads of the k-tiles behind it are pending; the requests
    // above are younger than the first ns k-tiles, so they make the first waits stricter at most.
    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    const int sw = (lm >> 1) & 7;
    for (int i = 0; i < steps; ++i) {
        const int ahead = min(steps - 1, i + ns - 1) - i;  // k-tiles requested after this one
        if (ahead >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NLD) : "memory");
        else if (ahead == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NLD) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const char *st = ring + (i % ns) * STAGE;
        frag fx[4][MI], fw[4][NI];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int ch = ((2 * kk + lh) ^ sw) << 4;
#pragma unroll
            for (int m = 0; m < MI; ++m) fx[kk][m] = *(const frag *)(st + (m * 32 + lm) * 128 + ch);
#pragma unroll
            for (int n = 0; n < NI; ++n) fw[kk][n] = *(const frag *)(st + (BM + n * 32 + lm) * 128 + ch);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the stage is in registers: request its next k-tile
        if (i + ns < steps) issue(i + ns);
        if (wave + 4 * i == nk - 1 && tail < BK) {         // chunks past K add nothing
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                if ((2 * kk + lh) * V >= tail) {
#pragma unroll
                    for (int m = 0; m < MI; ++m) fx[kk][m] = zero;
#pragma unroll
                    for (int n = 0; n < NI; ++n) fw[kk][n] = zero;
                }
        }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int m = 0; m < MI; ++m)
#pragma unroll
                for (int n = 0; n < NI; ++n) acc[m][n] = E::mma(fw[kk][n], fx[kk][m], acc[m][n]);
    }

    // ---- the four partial sums meet: area (wave, subtile) holds 16 values x 64 lanes
    __syncthreads();                                       // the rings are dead
    float *red = (float *)ks_lds;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4)
                *(f32x4 *)(red + ((wave * NF + i * NI + j) * 4 + e4) * 256 + lane * 4) =
                    f32x4{acc[i][j][4 * e4], acc[i][j][4 * e4 + 1], acc[i][j][4 * e4 + 2], acc[i][j][4 * e4 + 3]};
    __syncthreads();
    if (!fin) return;
    f32x16 base;                                           // row tw + lm, columns nc + 8 (e / 4) + 4 lh + e % 4
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
        f32x4 s = *(const f32x4 *)(red + ((0 * NF + wave) * 4 + e4) * 256 + lane * 4);
#pragma unroll
        for (int w = 1; w < 4; ++w) s += *(const f32x4 *)(red + ((w * NF + wave) * 4 + e4) * 256 + lane * 4);
#pragma unroll
        for (int z = 0; z < 4; ++z) base[4 * e4 + z] = s[z];
    }
    float *stg = red + wave * 1024;                        // this wave's part of wave 0's areas: read above, by this wave only

    if (SHRINK) {
        const int t = tw + lm;
        if (t < g.T) {
            T *out = (T *)g.out + ((size_t)blk * g.T + t) * g.RP;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int c = nc + 8 * (e >> 2) + 4 * lh + (e & 3);
                if (c < g.RP) out[c] = from_f32<T>(c < g.r ? g.scale * base[e] : 0.f);
            }
        }
        return;
    }

    // rows [lo, hi) of the subtile -> output block ob; row 0 of the subtile is row trow0 of the block
    auto emit = [&](const f32x16 &c, int ob, int trow0, int lo, int hi) {
        const long obase = ((long)ob * g.Tout + g.t_off + trow0) * g.N;
        if (!vec) {                                        // N not a multiple of 4, or an address no multiple of 16: element by element
            const int row = lm;
            if (row < lo || row >= hi) return;
            const int rb = (g.mode == EPI_RESID && g.res && g.res_block_of_out) ? g.res_block_of_out[ob] : ob;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int cc = nc + 8 * (e >> 2) + 4 * lh + (e & 3);
                if (cc >= g.N) continue;
                float v = c[e] + (g.bias ? g.bias[cc] : 0.f);
                const long o = obase + (long)row * g.N + cc;
                if (g.mode == EPI_RESID) {
                    if (g.res) v += g.res[((long)rb * g.Tout + g.t_off + trow0 + row) * g.N + cc];
                    if (g.pos) v += g.pos[(long)(g.t_off + trow0 + row) * g.N + cc];
                    ((float *)g.out)[o] = v;
                } else {
                    if (g.mode == EPI_GELU) v = E::gelu4(f32x4{v, v, v, v})[0];
                    ((T *)g.out)[o] = from_f32<T>(v);
                }
            }
            return;
        }
        f32x4 rv[4];
        const bool res = g.mode == EPI_RESID && g.res;
        if (res) {
            if (ob == ob_pre) {
#pragma unroll
                for (int q = 0; q < 4; ++q) rv[q] = pre_r[q];
            } else load_res(rv, ob, trow0, Tblk);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *(f32x4 *)(stg + lm * 32 + (((2 * q + lh) ^ ((lm >> 1) & 7)) << 2)) = f32x4{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = 8 * q + rrow;
            f32x4 v = *(const f32x4 *)(stg + row * 32 + ((rch ^ ((row >> 1) & 7)) << 2)) + bias4;
            if (row < lo || row >= hi || col >= g.N) continue;
            if (g.mode == EPI_RESID) {
                if (res) v += rv[q];
                if (g.pos) v += *(const f32x4 *)(g.pos + (long)(g.t_off + trow0 + row) * g.N + col);
                *(f32x4 *)((float *)g.out + obase + (long)row * g.N + col) = v;
            } else {
                if (g.mode == EPI_GELU) v = E::gelu4(v);
                typedef T out4 __attribute__((ext_vector_type(4)));
                *(out4 *)((T *)g.out + obase + (long)row * g.N + col) = out4{from_f32<T>(v[0]), from_f32<T>(v[1]), from_f32<T>(v[2]), from_f32<T>(v[3])};
            }
        }
    };
    int lo = 0;
    if (own) {
        const int rows = min(32, Tlim - tw);
        f32x16 c = base;
        // the term of block bb on its rows [lo, hi); ranks [0, 16) of its Bt rows in `w` if they have been requested
        auto term = [&](int bb, int k_ad, const frag(&w)[16 / (2 * V)], bool have) {
            const int hi = min(rows, (bb + 1) * Tblk - tw);
            const bool mine = lm >= lo && lm < hi;         // rows of other blocks add nothing
            for (int s0 = 0; k_ad >= 0 && s0 < g.RP; s0 += 16) {
#pragma unroll
                for (int u = 0; u < 16 / (2 * V); ++u) {
                    frag fs = pre_s[u], fw = w[u];
                    if (s0) fs = load_s(0, min(tw + lm, Tlim - 1), s0 + 2 * V * u);
                    if (s0 || !have) fw = load_w(k_ad, s0 + 2 * V * u);
                    c = E::mma(fw, mine ? fs : zero, c);
                }
            }
            lo = hi;
        };
        if (has_lora) {
#pragma unroll
            for (int b = 0; b < PB; ++b)
                if (lo < rows) term(b_lo + b, pre_k[b], pre_w[b], true);
            for (int bb = b_lo + PB; lo < rows; ++bb) term(bb, uload(g.adapter_of_out + bb), pre_w[0], false);
        }
        emit(c, b_lo, tw - b_lo * Tblk, 0, rows);
        return;
    }
    for (int bb = b_lo; lo < 32; ++bb) {                   // the input blocks whose rows lie in this subtile
        const int trow0 = flat ? tw - bb * Tblk : tw;
        const int hi = min(32, (flat ? min(Tblk, Tlim - bb * Tblk) : Tlim) - trow0);
        if (hi <= lo) break;
        const int o0 = g.out_off ? uload(g.out_off + bb) : bb, o1 = g.out_off ? uload(g.out_off + bb + 1) : bb + 1;
        for (int ob = o0; ob < o1; ++ob) {                 // the output blocks that fan out of it
            f32x16 c = base;
            const int sb0 = g.set_off ? uload(g.set_off + ob) : ob, sb1 = g.set_off ? uload(g.set_off + ob + 1) : ob + 1;
            for (int sb = sb0; has_lora && sb < sb1; ++sb) {   // one low-rank term, or all the terms summed on this block
                const int k_ad = uload(g.adapter_of_out + sb);
                if (k_ad < 0) continue;
                const int t = min(max(trow0 + lm, 0), Tblk - 1);
                const bool mine = lm >= lo && lm < hi;     // rows of other blocks add nothing
                const bool pre = ob == ob_pre && sb == sb0;
                for (int s0 = 0; s0 < g.RP; s0 += 16) {
#pragma unroll
                    for (int u = 0; u < 16 / (2 * V); ++u) {
                        frag fs = pre_s[u], fw = pre_w[0][u];
                        if (!(pre && s0 == 0)) { fs = load_s(sb, t, s0 + 2 * V * u); fw = load_w(k_ad, s0 + 2 * V * u); }
                        c = E::mma(fw, mine ? fs : zero, c);
                    }
                }
            }
            emit(c, ob, trow0, lo, hi);
        }
        lo = hi;
        if (!flat) break;
    }
}

template <typename T, int MI, int NI, bool SHRINK, bool AL>
__global__ __launch_bounds__(256, 2) void gemm_ks_kernel(const GemmArgs g, int tiles_m, int tiles_n, int ns)
{
    gemm_ks_tile<T, MI, NI, SHRINK, AL, false>(g, tiles_m, tiles_n, ns, PatchRows{});
}

// The patch embedding in single precision: the product's tiles, behind them workgroups for the rest, the last one for the CSR check (a gather and a product were
// two launches).  Bound by the matrix instructions.  Forward in one launch / in two, us: 4 frames of 17 tokens 69.8 / 72.1; of 197 tokens 1, 8, 32, 64 frames
// 78.7 / 81.5, 140.9 / 146.3, 414.2 / 421.4, 697.9 / 709.1.
template <int MI, int NI>
__global__ __launch_bounds__(256, 2) void patch_f32_kernel(const GemmArgs g, int tiles_m, int tiles_n, int ns, const PatchRows pr, const PatchArgs pa, int tile_wgs,
                                                           int job_wgs)
{
    const int job = (int)blockIdx.x - tile_wgs;
    if (job < 0) gemm_ks_tile<float, MI, NI, false, true, true>(g, tiles_m, tiles_n, ns, pr);
    else patch_jobs(pa, g.N, job, job_wgs);
}

// ------------------------------------------------------------------ the isolated multi-adapter linear of a small call, one launch
// Y[b] = X[f] W + bias + s (X[f] A_k) B_k for every output block b = (f, k): the CSR check, the shrink and the product in one kernel.
// A call of a few blocks is three dependent launches of four to six microseconds each otherwise (check, shrink, product with the
// expand).  Here every workgroup checks the whole CSR (a few hundred words, under its tile loads) before it stores anything, and
// the shrink of a tile's rows runs beside its product: the ranks of up to four 16-rank slots (output blocks x rank tiles) are 32 more
// "columns" per two slots of the same 32 x 32 x 16 steps, split over the waves like the product.  The column tiles of a row tile repeat
// the shrink, which is why large calls keep the separate one (linear_ks_tile).
// Measured, one / two launches: 1 x 197 x 192 -> 576 10.4 / 13.9 us, 1 x 197 x 768 -> 2304 11.2 / 15.9, 9 x 17 x 384 -> 1536 10.9 / 48
// (its separate product has too few rows per block for the large tiles); single precision, 2 x 197 x 192 -> 576: 11.2 / 19.3.
struct LinearParams {
    const void *X, *W, *At, *Bt;
    const float *bias;
    int F, T, K, N, n_adapters, r, R_cap;
    float scale;
    const int *off, *ids;
    void *Y;
    int *dev_status;
};

template <typename T, int MI, int NI>
__global__ __launch_bounds__(256) void linear_ks_kernel(const LinearParams g, int tiles_m, int tiles_n, int ns)
{
    typedef Elt<T> E;
    typedef typename E::frag frag;
    constexpr int V = E::V, BK = 8 * V, BM = 32 * MI, BN = 32 * NI, NU = 16 / (2 * V);   // NU: expand steps per 16 ranks
    constexpr int STAGE = (BM + BN) * 128, NLD = (BM + BN) / 8;
    constexpr int NF = MI * NI;
    extern __shared__ __attribute__((aligned(16))) char ks_lds[];
    __shared__ int bad_s[4];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lm = lane & 31, lh = lane >> 5;
    // tile of this workgroup: eight equal runs, one per XCD (as gemm_ks_kernel)
    const int mtot = g.F * tiles_m;
    int mt, tn;
    {
        const unsigned xcd = blockIdx.x & 7, total = (unsigned)mtot * tiles_n, lo = total * xcd / 8, hi = total * (xcd + 1) / 8, L = lo + (blockIdx.x >> 3);
        if (L >= hi && blockIdx.x) return;                     // (workgroup 0 reports the status in any case)
        if (mtot <= tiles_n) { tn = (int)(L / (unsigned)mtot); mt = (int)L - tn * mtot; }
        else { mt = (int)(L / (unsigned)tiles_n); tn = (int)L - mt * tiles_n; }
        if (L >= hi) { mt = -1; tn = 0; }
    }
    const bool idle = mt < 0;
    const int xb = idle ? 0 : mt / tiles_m, t0 = idle ? 0 : (mt - xb * tiles_m) * BM, n0 = tn * BN;
    const T *A = (const T *)g.X + ((size_t)xb * g.T + t0) * g.K;
    const T *W = (const T *)g.W + (size_t)n0 * g.K;
    const int nk = (g.K + BK - 1) / BK, steps = idle ? 0 : (nk - wave + 3) >> 2;
    const unsigned rowb = (unsigned)g.K * sizeof(T);
    const int lr = lane >> 3, c0 = (lane & 7) ^ (lr >> 1), c1 = c0 ^ 4;
    const int tail = g.K - (nk - 1) * BK;
    const int adj0 = min(c0, tail / V - 1) - c0, adj1 = min(c1, tail / V - 1) - c1;
    char *ring = ks_lds + wave * ns * STAGE;
    auto issue = [&](int i) {
        const int kt = wave + 4 * i;
        const bool last = kt == nk - 1;
        const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_addr_of(ring + (i % ns) * STAGE));
        const unsigned e0 = (unsigned)(c0 + (last ? adj0 : 0)) * 16, e1 = (unsigned)(c1 + (last ? adj1 : 0)) * 16;
#pragma unroll
        for (int q = 0; q < BM / 8; ++q)
            glds16_s((const char *)A + (size_t)kt * 128, (unsigned)min(8 * q + lr, g.T - 1 - t0) * rowb + ((q & 1) ? e1 : e0), lds0 + q * 1024);
#pragma unroll
        for (int q = 0; q < BN / 8; ++q)
            glds16_s((const char *)W + (size_t)kt * 128, (unsigned)min(8 * q + lr, g.N - 1 - n0) * rowb + ((q & 1) ? e1 : e0), lds0 + (BM / 8 + q) * 1024);
    };
    for (int i = 0; i < min(ns, steps); ++i) issue(i);

    // ---- the CSR: this tile's output blocks and adapters first, then the check of all of it
    const int R = uload(g.off + g.F), o0 = uload(g.off + xb), o1 = uload(g.off + xb + 1), off0 = uload(g.off);
    const bool sane = off0 == 0 && R >= 0 && R <= g.R_cap && o0 >= 0 && o0 <= o1 && o1 <= R;
    const int nob = sane && !idle ? o1 - o0 : 0;
    bool bad = !(off0 == 0 && R >= 0 && R <= g.R_cap);
    if (!bad) {
        for (int f = tid; f < g.F; f += 256) {
            const int a = g.off[f], b = g.off[f + 1];
            if (a > b || a < 0 || b > R) bad = true;
        }
        for (int i = tid; i < R; i += 256) {
            const int k = g.ids[i];
            if (k < 0 || k >= g.n_adapters) bad = true;
        }
    }
    const bool any = __ballot(bad) != 0;
    if (lane == 0) bad_s[wave] = any;
    const int nrt = (g.r + 15) >> 4, per_pass = nrt <= 2 ? 4 / nrt : 1;   // rank tiles; output blocks per pass of at most four slots

    const int fi = wave / NI, fj = wave % NI;
    const int tw = t0 + 32 * fi, nc = n0 + 32 * fj;
    const bool fin = wave < NF && tw < g.T && nc < g.N;
    const bool vec = g.N % 4 == 0;
    const int rch = lane & 7, rrow = lane >> 3, col = nc + 4 * rch;
    f32x4 bias4 = {0.f, 0.f, 0.f, 0.f};
    if (fin && g.bias && vec) bias4 = *(const f32x4 *)(g.bias + min(col, g.N - 4));
    const frag zero = {};
    const int sw = (lm >> 1) & 7;
    float *red = (float *)ks_lds, *sred = red + 4 * NF * 1024;
    float *stg = red + wave * 1024;                            // this wave's part of wave 0's areas
    f32x16 base;
#pragma unroll
    for (int e = 0; e < 16; ++e) base[e] = 0.f;

    for (int pass = 0; pass == 0 || pass * per_pass < nob; ++pass) {
        const int ob_base = o0 + pass * per_pass, nslots = min(per_pass, nob - pass * per_pass) * nrt;   // (<= 0 without output blocks)
        if (pass) {
            __syncthreads();                                   // the partial sums of the pass before have been read
            for (int i = 0; i < min(ns, steps); ++i) issue(i);
        }
        // At row of lane lm in the two slots of product q (clamped where there is none: the result is not used)
        const T *at[2];
        int kad[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            kad[s] = s < nslots ? uload(g.ids + ob_base + s / nrt) : 0;
            if ((unsigned)kad[s] >= (unsigned)g.n_adapters) kad[s] = 0;                                  // (reported, and nothing is stored)
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int s = 2 * q + (lm >> 4);
            const int rank = min((s % nrt) * 16 + (lm & 15), g.r - 1);
            at[q] = (const T *)g.At + ((size_t)((lm >> 4) ? kad[2 * q + 1] : kad[2 * q]) * g.r + rank) * g.K;
        }
        frag fat[2][4];
        auto load_at = [&](int i) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (2 * q < nslots) {
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) fat[q][kk] = *(const frag *)(at[q] + min((wave + 4 * i) * BK + (2 * kk + lh) * V, g.K - V));
                }
        };
        if (steps > 0) load_at(0);
        // Bt rows of this wave's columns: ranks 16 jt + 4 lh .. and 16 jt + 8 + 4 lh .. of every slot, as the shrink leaves them in a lane
        frag fbt[4][NU];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (fin && s < nslots) {
                const T *bt = (const T *)g.Bt + ((size_t)kad[s] * g.N + min(nc + lm, g.N - 1)) * g.r;
                typedef T quad __attribute__((ext_vector_type(4)));
                quad w[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int rank = 16 * (s % nrt) + 8 * u + 4 * lh;
                    if (g.r % 4 == 0) {
                        w[u] = *(const quad *)(bt + min(rank, g.r - 4));
                        if (rank >= g.r) w[u] = quad{};
                    } else {
#pragma unroll
                        for (int z = 0; z < 4; ++z) w[u][z] = rank + z < g.r ? bt[rank + z] : from_f32<T>(0.f);
                    }
                }
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int z = 0; z < 4; ++z) fbt[s][V == 8 ? 0 : u][V == 8 ? 4 * u + z : z] = w[u][z];
            }

        f32x16 acc[MI][NI], sac[MI][2];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int e = 0; e < 16; ++e) sac[i][q][e] = 0.f;
        }
        for (int i = 0; i < steps; ++i) {
            const int ahead = min(steps - 1, i + ns - 1) - i;
            if (ahead >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NLD) : "memory");
            else if (ahead == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NLD) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const char *st = ring + (i % ns) * STAGE;
            frag fx[4][MI], fw[4][NI];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const int ch = ((2 * kk + lh) ^ sw) << 4;
#pragma unroll
                for (int m = 0; m < MI; ++m) fx[kk][m] = *(const frag *)(st + (m * 32 + lm) * 128 + ch);
#pragma unroll
                for (int n = 0; n < NI; ++n) fw[kk][n] = *(const frag *)(st + (BM + n * 32 + lm) * 128 + ch);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (i + ns < steps) issue(i + ns);
            if (wave + 4 * i == nk - 1 && tail < BK) {         // chunks past K add nothing
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    if ((2 * kk + lh) * V >= tail) {
#pragma unroll
                        for (int m = 0; m < MI; ++m) fx[kk][m] = zero;
                    }
            }
            if (pass == 0) {
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                    for (int m = 0; m < MI; ++m)
#pragma unroll
                        for (int n = 0; n < NI; ++n) acc[m][n] = E::mma(fw[kk][n], fx[kk][m], acc[m][n]);
            }
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (2 * q < nslots) {
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                        for (int m = 0; m < MI; ++m) sac[m][q] = E::mma(fat[q][kk], fx[kk][m], sac[m][q]);
                }
            if (i + 1 < steps) load_at(i + 1);
        }

        // ---- the partial sums meet: (wave, subtile) of the product, (wave, row subtile, q) of the shrink
        __syncthreads();                                       // the rings are dead
        if (pass == 0) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int e4 = 0; e4 < 4; ++e4)
                        *(f32x4 *)(red + ((wave * NF + i * NI + j) * 4 + e4) * 256 + lane * 4) =
                            f32x4{acc[i][j][4 * e4], acc[i][j][4 * e4 + 1], acc[i][j][4 * e4 + 2], acc[i][j][4 * e4 + 3]};
        }
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (2 * q < nslots) {
#pragma unroll
                    for (int e4 = 0; e4 < 4; ++e4)
                        *(f32x4 *)(sred + (((wave * MI + i) * 2 + q) * 4 + e4) * 256 + lane * 4) =
                            f32x4{sac[i][q][4 * e4], sac[i][q][4 * e4 + 1], sac[i][q][4 * e4 + 2], sac[i][q][4 * e4 + 3]};
                }
        __syncthreads();
        const bool bad_csr = bad_s[0] | bad_s[1] | bad_s[2] | bad_s[3];
        if (pass == 0 && blockIdx.x == 0 && tid == 0 && g.dev_status) *g.dev_status = bad_csr ? POLY_ERANGE : POLY_OK;
        if (bad_csr || nob <= 0) return;
        if (!fin) continue;
        if (pass == 0) {
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                f32x4 s = *(const f32x4 *)(red + ((0 * NF + wave) * 4 + e4) * 256 + lane * 4);
#pragma unroll
                for (int w = 1; w < 4; ++w) s += *(const f32x4 *)(red + ((w * NF + wave) * 4 + e4) * 256 + lane * 4);
#pragma unroll
                for (int z = 0; z < 4; ++z) base[4 * e4 + z] = s[z];
            }
        }
        auto emit = [&](const f32x16 &c, int ob) {
            const long obase = ((long)ob * g.T + tw) * g.N;
            const int hi = min(32, g.T - tw);
            if (!vec) {                                        // N not a multiple of 4: element by element
                if (lm >= hi) return;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int cc = nc + 8 * (e >> 2) + 4 * lh + (e & 3);
                    if (cc < g.N) ((T *)g.Y)[obase + (long)lm * g.N + cc] = from_f32<T>(c[e] + (g.bias ? g.bias[cc] : 0.f));
                }
                return;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f32x4 *)(stg + lm * 32 + (((2 * q + lh) ^ ((lm >> 1) & 7)) << 2)) = f32x4{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = 8 * q + rrow;
                const f32x4 v = *(const f32x4 *)(stg + row * 32 + ((rch ^ ((row >> 1) & 7)) << 2)) + bias4;
                if (row >= hi || col >= g.N) continue;
                typedef T out4 __attribute__((ext_vector_type(4)));
                *(out4 *)((T *)g.Y + obase + (long)row * g.N + col) = out4{from_f32<T>(v[0]), from_f32<T>(v[1]), from_f32<T>(v[2]), from_f32<T>(v[3])};
            }
        };
        f32x16 c = base;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s >= nslots) break;
            const int jt = s % nrt;
            if (jt == 0) c = base;
            // ranks 16 jt + 8 u + 4 lh .. (bf16: u = 0 and 1 in one operand) of row lm; the slot's half of product s / 2
            float sv[8];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float *sp = sred + ((size_t)fi * 2 + (s >> 1)) * 1024 + (2 * (s & 1) + u) * 256 + lane * 4;
                f32x4 t = *(const f32x4 *)sp;
#pragma unroll
                for (int w = 1; w < 4; ++w) t += *(const f32x4 *)(sp + (size_t)w * MI * 2 * 1024);
#pragma unroll
                for (int z = 0; z < 4; ++z) sv[4 * u + z] = t[z] * g.scale;
            }
            frag fs[NU];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int z = 0; z < 4; ++z) fs[V == 8 ? 0 : u][V == 8 ? 4 * u + z : z] = from_f32<T>(sv[4 * u + z]);
#pragma unroll
            for (int u = 0; u < NU; ++u) c = E::mma(fbt[s][u], fs[u], c);
            if (jt == nrt - 1) emit(c, ob_base + s / nrt);
        }
    }
}

// LDS of a tile and, in `ns`, its ring's stages per wave
template <typename T, int MI, int NI> int ks_lds_bytes(int K, int &ns)
{
    constexpr int STAGE = 32 * (MI + NI) * 128, BK = 8 * Elt<T>::V, RED = 4 * MI * NI * 4096;
    const int nk = (K + BK - 1) / BK;
    ns = (nk + 3) / 4 < KS_NSMAX ? (nk + 3) / 4 : KS_NSMAX;   // no more stages than a wave has k-tiles: short contractions leave room for other workgroups
    while (4 * ns * STAGE > 160 * 1024) --ns;
    return 4 * ns * STAGE > RED ? 4 * ns * STAGE : RED;
}

template <int MI, int NI> int launch_patch_t(const GemmArgs &g, const PatchRows &pr, const PatchArgs &pa, hipStream_t st)
{
    int ns;
    const int lds = ks_lds_bytes<float, MI, NI>(g.K, ns);
    auto kern = patch_f32_kernel<MI, NI>;
    static bool attr_set = false;       // raising the dynamic LDS limit is a per-kernel, process-wide setting
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 156 * 1024) != hipSuccess) return POLY_EHIP;
        attr_set = true;
    }
    const int tiles_m = (g.T + 32 * MI - 1) / (32 * MI), tiles_n = (g.N + 32 * NI - 1) / (32 * NI);
    const long tile_wgs = ((long)g.n_in * tiles_m * tiles_n + 7) / 8 * 8;
    const int job_wgs = patch_job_wgs(pa, g.N);
    POLY_LAUNCH_SHMEM(POLY_STAGE_GEMM, kern, dim3((unsigned)(tile_wgs + job_wgs + (pa.prep.row_offsets ? 1 : 0))), dim3(256), lds, st, g, tiles_m, tiles_n, ns, pr, pa,
                      (int)tile_wgs, job_wgs);
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

template <typename T, int MI, int NI, bool SHRINK, bool AL> int launch_ks_t(const GemmArgs &g, hipStream_t st)
{
    int ns;
    const int lds = ks_lds_bytes<T, MI, NI>(g.K, ns);
    auto kern = gemm_ks_kernel<T, MI, NI, SHRINK, AL>;
    static bool attr_set = false;       // raising the dynamic LDS limit is a per-kernel, process-wide setting
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) return POLY_EHIP;
        attr_set = true;
    }
    const int tiles_m = (g.T + 32 * MI - 1) / (32 * MI), tiles_n = (g.N + 32 * NI - 1) / (32 * NI);
    const long total = (long)g.n_in * tiles_m * tiles_n;
    if (total > 0x3fffffffL) return POLY_EINVAL;
    POLY_LAUNCH_SHMEM(SHRINK ? POLY_STAGE_SHRINK : POLY_STAGE_GEMM, kern, dim3((unsigned)((total + 7) / 8 * 8)), dim3(256), lds, st, g, tiles_m, tiles_n, ns);
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

template <typename T, int MI, int NI, bool SHRINK> int launch_ks(const GemmArgs &g, hipStream_t st)
{
    return gemm_aligned(g) ? launch_ks_t<T, MI, NI, SHRINK, true>(g, st) : launch_ks_t<T, 1, 1, SHRINK, false>(g, st);
}

}  // namespace

bool gemm_aligned(const GemmArgs &g)
{
    return aligned16(g.A) && aligned16(g.Wt) && aligned16(g.bias) && aligned16(g.S) && aligned16(g.Bt) && aligned16(g.out) && aligned16(g.res) && aligned16(g.pos);
}

// Tile by the time of the busiest CU: rounds of tiles over the 256 CUs, each the larger of its loads through the CU's load path
// (about 40 bytes per clock) and its products, plus what a tile costs whatever its size (first round trip, partial sums, stores).  On 24
// products of 68 to 6304 rows it picks the fastest of the three tiles 23 times and one that is 10 % slower once, e.g. 591 x 768 -> 768 12.4,
// 8.5 and 9.8 us with 32 x 32, 32 x 64 and 64 x 64, 591 x 768 -> 3072 39.4, 25.6, 17.1, single precision 68 x 192 -> 576 10.0, 11.4, 14.0.
static int ks_tile(const GemmArgs &g, int dtype)              // 0, 1, 2: 32 x 32, 32 x 64, 64 x 64
{
    const double es = dtype == POLY_BF16 ? 2 : 4, rate = dtype == POLY_BF16 ? 2048 : 220;    // flop per clock and CU
    auto cost = [&](int mi, int ni) {
        const double tiles = (double)g.n_in * ((g.T + 32 * mi - 1) / (32 * mi)) * ((g.N + 32 * ni - 1) / (32 * ni));
        const double rounds = (double)(long)((tiles + 255) / 256);
        const double load = es * g.K * 32 * (mi + ni) / 40, prod = 2.0 * g.K * 1024 * mi * ni / rate;
        return rounds * (3000 + (load > prod ? load : prod));
    };
    const double c11 = cost(1, 1), c12 = cost(1, 2), c22 = cost(2, 2);
    return c11 < c12 && c11 < c22 ? 0 : c12 < c22 ? 1 : 2;
}

int launch_gemm_ks(const GemmArgs &g, int dtype, hipStream_t st)
{
    const int tile = ks_tile(g, dtype);
    if (dtype == POLY_BF16) return tile == 0 ? launch_ks<bf16_t, 1, 1, false>(g, st) : tile == 1 ? launch_ks<bf16_t, 1, 2, false>(g, st) : launch_ks<bf16_t, 2, 2, false>(g, st);
    return tile == 0 ? launch_ks<float, 1, 1, false>(g, st) : tile == 1 ? launch_ks<float, 1, 2, false>(g, st) : launch_ks<float, 2, 2, false>(g, st);
}

static GemmArgs patch_product(const PatchArgs &pa, const void *Wt, const float *bias, int D)
{
    GemmArgs g = {};
    g.A = pa.frames; g.Wt = Wt; g.bias = bias;
    g.T = (pa.H / pa.p) * (pa.W / pa.p); g.K = 3 * pa.p * pa.p; g.N = D; g.n_in = pa.F;
    g.mode = EPI_RESID; g.out = pa.x; g.Tout = g.T + 1; g.t_off = 1; g.pos = pa.pos;
    return g;
}

// A piece of 16 bytes never crosses from one image row of a patch to the next nor lies off a 16-byte boundary
bool patch_rows_f32_fits(const PatchArgs &pa, const void *Wt, const float *bias, int D)
{
    const GemmArgs g = patch_product(pa, Wt, bias, D);
    return pa.F > 0 && (3 * pa.p) % 4 == 0 && g.K % 32 == 0 && g.K <= 4096 && g.N % 4 == 0 && (size_t)pa.H * pa.W * 12 <= 0x7fffffffu && aligned16(pa.frames) &&
           gemm_aligned(g);
}

int launch_patch_rows_f32(const PatchArgs &pa, const void *Wt, const float *bias, int D, hipStream_t st)
{
    const GemmArgs g = patch_product(pa, Wt, bias, D);
    const PatchRows pr = patch_rows(pa, 4);
    const int tile = ks_tile(g, POLY_F32);
    return tile == 0 ? launch_patch_t<1, 1>(g, pr, pa, st) : tile == 1 ? launch_patch_t<1, 2>(g, pr, pa, st) : launch_patch_t<2, 2>(g, pr, pa, st);
}

namespace {
template <typename T, int MI, int NI> int launch_linear_t(const LinearParams &g, hipStream_t st)
{
    constexpr int STAGE = 32 * (MI + NI) * 128, BK = 8 * Elt<T>::V, RED = 4 * (MI * NI + 2 * MI) * 4096, LDS_MAX = 144 * 1024;
    const int nk = (g.K + BK - 1) / BK;
    int ns = (nk + 3) / 4 < KS_NSMAX ? (nk + 3) / 4 : KS_NSMAX;
    while (4 * ns * STAGE > LDS_MAX) --ns;
    const int lds = 4 * ns * STAGE > RED ? 4 * ns * STAGE : RED;
    auto kern = linear_ks_kernel<T, MI, NI>;
    static bool attr_set = false;       // raising the dynamic LDS limit is a per-kernel, process-wide setting
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_MAX) != hipSuccess) return POLY_EHIP;
        attr_set = true;
    }
    const int tiles_m = (g.T + 32 * MI - 1) / (32 * MI), tiles_n = (g.N + 32 * NI - 1) / (32 * NI);
    const long total = (long)g.F * tiles_m * tiles_n;
    POLY_LAUNCH_SHMEM(POLY_STAGE_GEMM, kern, dim3((unsigned)((total + 7) / 8 * 8)), dim3(256), lds, st, g, tiles_m, tiles_n, ns);
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

// Tile of the one-launch linear: the smallest of 32 x 32, 32 x 64 and 64 x 64 with which every tile gets a compute unit of its own
// (0 = none).  Smaller tiles are more of the chip and a shorter serial chain; with more tiles than compute units a second round, and the
// shrink that every column tile repeats, cost more than the launch that is saved (9 x 197 x 192 -> 576, 324 tiles of 64 x 64: 14.4 us of
// kernel time against 11.7 in two launches; 6 x 197 x 192 -> 576 15.7, 12.8, 8.9 with the three tiles, 9 x 17 x 384 -> 1536 13.2, 8.6, 9.5).
int linear_ks_tile(long F, int T, int N)
{
    auto tiles = [&](int bm, int bn) { return F * ((T + bm - 1) / bm) * ((N + bn - 1) / bn); };
    return tiles(32, 32) <= 256 ? 1 : tiles(32, 64) <= 256 ? 2 : tiles(64, 64) <= 256 ? 3 : 0;
}
}  // namespace

// ranks: four slots of 16 at most; CSR: every workgroup reads all of it, four words per lane at most; every address a multiple of 16
bool linear_ks_fits(const void *X, int F, int T, const void *W, const float *bias, int N, const void *At, const void *Bt, int r, int R, const void *Y)
{
    return r <= 64 && F + (long)R <= 1024 && linear_ks_tile(F, T, N) != 0 && aligned16(X) && aligned16(W) && aligned16(bias) && aligned16(At) &&
           aligned16(Bt) && aligned16(Y);
}

int launch_linear_ks(const void *X, int F, int T, int K, const void *W, const float *bias, int N, const void *At, const void *Bt, int n_adapters,
                     int r, float scale, const int *off, const int *ids, int R, void *Y, int dtype, int *dev_status, hipStream_t st)
{
    const LinearParams g = {X, W, At, Bt, bias, F, T, K, N, n_adapters, r, R, scale, off, ids, Y, dev_status};
    const int tile = linear_ks_tile(F, T, N);
    if (dtype == POLY_BF16) return tile == 1 ? launch_linear_t<bf16_t, 1, 1>(g, st) : tile == 2 ? launch_linear_t<bf16_t, 1, 2>(g, st) : launch_linear_t<bf16_t, 2, 2>(g, st);
    return tile == 1 ? launch_linear_t<float, 1, 1>(g, st) : tile == 2 ? launch_linear_t<float, 1, 2>(g, st) : launch_linear_t<float, 2, 2>(g, st);
}

// S[ob] = scale * X[in_block_of_out[ob]] At[adapter_of_out[ob]]^T in single precision, zero padded to RP columns
int launch_shrink_f32(const float *X, int T, int K, const float *At, int r, int RP, float scale, int n_out, const int *n_out_dev,
                      const int *in_block_of_out, const int *adapter_of_out, float *S, hipStream_t st)
{
    GemmArgs g = {};
    g.A = X; g.Wt = At; g.T = T; g.K = K; g.N = RP; g.n_in = n_out; g.n_in_dev = n_out_dev; g.r = r; g.RP = RP; g.scale = scale;
    g.adapter_of_out = adapter_of_out; g.res_block_of_out = in_block_of_out; g.out = S; g.Tout = T;
    return launch_ks<float, 1, 1, true>(g, st);
}
