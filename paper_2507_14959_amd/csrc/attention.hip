// Fused softmax attention of one (token block, head) per workgroup; head width 64.
//
// bf16: K and V^T of the head are staged once in LDS.  Each wave owns 32 queries (or two such tiles, one after the other) and computes
// S^T = K Q^T on the MFMA (keys down the rows, so every lane holds all scores of ONE query), takes the
// softmax over its registers in fp32, and feeds the unnormalised probabilities straight back as the B
// operand of O^T = V^T P^T -- the accumulator layout of S^T is already a valid B layout once the keys of
// each 16-key step are read from V^T in the matching order.  1/sum is applied per lane at the end.
// fp32: the same on fp32 matrix instructions, key tiles streamed through LDS with an online softmax.
#include "poly_dev.h"

#include <type_traits>

namespace {

constexpr float LOG2E = 1.4426950408889634f;
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));

// A wave per query tile and, from 161 keys on, room for others on the CU: at most 168 registers, and where there are more workgroups than CUs half of the waves leave once K
// and V are in LDS, so that the next workgroup's fit beside the others.
constexpr bool att_shares(int nkt, int w) { return nkt == w && nkt >= 6; }
__host__ __device__ constexpr int att_keys(int T) { return (T + 15) & ~15; }      // that have a place in LDS

// Bound by loading in one phase and computing in the next; what helps is another workgroup on the CU in the other phase.  K and V^T alone are in LDS, without padding and for
// 16 keys at a time (53 KB for 197), so that three fit where 80 KB with padded rows and staged outputs let two.  us per launch, before / now, 197 tokens: 72 workgroups 7.8 / 7.9, 144 8.5 /
// 8.1, 264 15.1 / 13.8, 516 22.1 / 18.6, 720 23.9 / 20.8, 999 30.0 / 25.3 (its bytes 20); 113 tokens (four instead of two) 360 8.6 / 7.6, 720 13.6 / 11.4, 999 16.2 / 13.8.
template <int NKT, int W, bool FRAGMENTS, bool SPLIT>  // 32-key tiles: T <= 32 * NKT; waves, each takes the query tiles w, w + live, ..; SPLIT: two workgroups, of the first four and of the other query tiles
__global__ __launch_bounds__(64 * W, att_shares(NKT, W) ? 3 : NKT > W ? 3 : NKT <= 4 ? 4 : 1) void attn_bf16_kernel(const bf16_t *qkv, bf16_t *out, int T, int D, int heads, int n_blocks,
                                                        const int *n_blocks_dev)
{
    extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
    const int TK = att_keys(T), VS = TK + 4; // Vt's rows are an odd number of 8-byte pieces apart: 8-byte reads of 32 rows meet no bank twice
    bf16_t *Ks = smem;                       // [TK][64], 16-byte piece c of row r at c ^ (r >> 1 & 7)
    bf16_t *Vt = Ks + TK * 64;               // [64][VS]

    const int nb = n_blocks_dev ? min(*n_blocks_dev, n_blocks) : n_blocks;
    const int b = blockIdx.x / heads, hd = blockIdx.x % heads;
    if (b >= nb) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lm = lane & 31, lh = lane >> 5;
    const size_t ld = (size_t)3 * D;
    const bf16_t *base = qkv + (size_t)b * T * ld + hd * 64;
    constexpr int nthreads = 64 * W;

    // everything this thread will read from global memory is requested up front: its queries (of its first 32-query
    // tile), then its share of K (16-byte pieces) and of V (an 8 keys x 8 columns block, transposed in registers below).
    // Rows past T repeat row T - 1 (a load under a per-lane condition would be waited for on the spot): such keys are
    // masked in the softmax and get probability 0, such queries are never stored
    bf16x8 qf[4];
    auto load_q = [&](int qs) {
#pragma unroll
        for (int ds = 0; ds < 4; ++ds) qf[ds] = *(const bf16x8 *)(base + (size_t)min(qs * 32 + lm, T - 1) * ld + ds * 16 + lh * 8);
    };
    const int first = SPLIT ? (int)blockIdx.y * 4 : 0;         // query tile of wave 0
    load_q(SPLIT ? min(first + wave, NKT - 1) : wave);
    constexpr int NKP = (256 * NKT + nthreads - 1) / nthreads;     // K pieces (8 TK of up to 256 NKT) per thread
    bf16x8 kp[NKP];
#pragma unroll
    for (int i = 0; i < NKP; ++i) {
        const int v = tid + i * nthreads, key = v >> 3;
        kp[i] = *(const bf16x8 *)(base + (size_t)min(key, T - 1) * ld + D + (v & 7) * 8);
    }
    for (int blk = tid; blk < TK; blk += nthreads) {
        const int cb = blk & 7, kb = blk >> 3;       // consecutive lanes: consecutive 16-byte pieces of a row of V
        bf16x8 vv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int key = kb * 8 + k;
            vv[k] = *(const bf16x8 *)(base + (size_t)min(key, T - 1) * ld + 2 * D + cb * 8);
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            bf16_t *row = Vt + (cb * 8 + c) * VS + kb * 8;
            *(bf16x4 *)row = bf16x4{vv[0][c], vv[1][c], vv[2][c], vv[3][c]};
            *(bf16x4 *)(row + 4) = bf16x4{vv[4][c], vv[5][c], vv[6][c], vv[7][c]};
        }
    }
#pragma unroll
    for (int i = 0; i < NKP; ++i) {
        const int v = tid + i * nthreads;
        if (v < TK * 8) *(bf16x8 *)(Ks + (v >> 3) * 64 + ((v & 7) ^ (v >> 4 & 7)) * 8) = kp[i];
    }
    __syncthreads();

    // the second 16 keys of the last tile may not be there: their scores are read from V^T's place and masked, their step of the second product is left out
    const bool half = TK < 32 * NKT;
    const int sw = lm >> 1 & 7;
    auto k_piece = [&](int kt, int ds) { return *(const bf16x8 *)(Ks + (kt * 32 + lm) * 64 + ((2 * ds + lh) ^ sw) * 8); };
    const int live = att_shares(NKT, W) && nb * heads > 256 ? (NKT + 1) / 2 : W;
    if (wave >= (SPLIT ? 4 : live)) return;
    for (int qs = first + wave; qs * 32 < T; qs += SPLIT ? NKT : live) {
        // S^T tile kt: rows = keys kt*32 + 8*(e/4) + 4*lh + e%4, column = this lane's query.  The K fragments of tile
        // kt + 1 are read while the MFMAs of tile kt run (the scheduling barriers pin that order)
        f32x16 s[NKT];
        bf16x8 kf[2][4];
#pragma unroll
        for (int ds = 0; ds < 4; ++ds) kf[0][ds] = k_piece(0, ds);
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt) {
            if (kt + 1 < NKT) {
#pragma unroll
                for (int ds = 0; ds < 4; ++ds) kf[(kt + 1) & 1][ds] = k_piece(kt + 1, ds);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 16; ++e) s[kt][e] = 0.f;
#pragma unroll
            for (int ds = 0; ds < 4; ++ds) s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kt & 1][ds], qf[ds], s[kt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }

        if (!SPLIT && (att_shares(NKT, W) ? qs + live < NKT : NKT > W)) load_q(min(qs + live, NKT - 1));   // for the next round: arrives under this one's softmax

        // only the last key tile can hold keys past T (T > 32 * (NKT - 1) by construction)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int key = (NKT - 1) * 32 + 8 * (e >> 2) + 4 * lh + (e & 3);
            s[NKT - 1][e] = key < T ? s[NKT - 1][e] : -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
            for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[kt][e]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float sc = 0.125f * LOG2E;  // 1/sqrt(64), folded into the base-2 exponent
        const float off = -mx * sc;
        // probabilities are packed to bf16 as they are produced (they are the B operand of the second product), which
        // frees the fp32 score registers tile by tile
        float sum = 0.f;
        bf16x8 pf[NKT][2];
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
            for (int hs = 0; hs < 2; ++hs)
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(s[kt][hs * 8 + q], sc, off));   // exponent <= 0: no range handling needed
                    sum += p;
                    pf[kt][hs][q] = (bf16_t)p;
                }
        sum += __shfl_xor(sum, 32, 64);

        // O^T = V^T P^T: rows = head columns, column = this lane's query; V^T fragments one step ahead as above
        f32x16 o[2];
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
        bf16x4 vlo[2][2], vhi[2][2];
        auto loadv = [&](int st, int sl) {
            // slots 0..3 = keys kbase + 4*lh + 0..3, slots 4..7 = keys kbase + 8 + 4*lh + 0..3
            const int kbase = st * 16 + 4 * lh;
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) {
                const bf16_t *vr = Vt + (dt * 32 + lm) * VS + kbase;
                vlo[sl][dt] = *(const bf16x4 *)vr;
                vhi[sl][dt] = *(const bf16x4 *)(vr + 8);
            }
        };
        loadv(0, 0);
#pragma unroll
        for (int st = 0; st < 2 * NKT; ++st) {
            if (st + 1 == 2 * NKT && half) break;
            if (st + 2 < 2 * NKT || (st + 2 == 2 * NKT && !half)) loadv(st + 1, (st + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) {
                const bf16x4 lo = vlo[st & 1][dt], hi = vhi[st & 1][dt];
                const bf16x8 vf = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[st >> 1][st & 1], o[dt], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }

        // a lane owns four columns of every eight of one query: the two lanes of a query trade, so that each has 16 bytes in a row and the wave stores 32 of each query
        // (for rowreg.hip 1 KB in a run: 16 columns of 32 rows)
        const float inv = 1.0f / sum;
        const int row = qs * 32 + lm;
        const size_t flat = (size_t)b * T + row;
        bf16_t *dst = FRAGMENTS ? out + (flat >> 5) * (32 * D) + hd * 2048 + (lh * 32 + (flat & 31)) * 8 : out + flat * D + hd * 64 + lh * 8;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unsigned w[2][2];                              // columns 16 i + 8 q + 4 lh + {0, 1}, {2, 3}
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int e = (2 * (i & 1) + q) * 4 + 2 * h;
                    const bf16x2 two = {(bf16_t)(o[i >> 1][e] * inv), (bf16_t)(o[i >> 1][e + 1] * inv)};
                    w[q][h] = __builtin_bit_cast(unsigned, two);
                }
            const u32x2 a = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false), c = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
            if (row < T) *(u32x4 *)(dst + i * (FRAGMENTS ? 512 : 16)) = u32x4{a[0], c[0], a[1], c[1]};
        }
    }
}

// fp32: v_mfma_f32_32x32x2_f32, one wave per 32-query tile and four query tiles per workgroup, keys and values in tiles of 32
// through LDS with an online softmax (any T).  As above, S^T = K Q^T leaves a lane all scores of one query, and the probabilities
// are the B operand of O^T = V^T P^T as they are: step e of the second product takes key 8 (e / 4) + 4 lh + e % 4 from lane half
// lh, so V is read from LDS at that key.  (One thread per query with the dot products on the vector ALU took 44 us for 17 tokens,
// 6 us this way: a 32 x 32 tile is 64 + 64 matrix instructions of 64 cycles.)
__global__ __launch_bounds__(256) void attn_f32_kernel(const float *qkv, float *out, int T, int D, int heads, int n_blocks,
                                                       const int *n_blocks_dev)
{
    constexpr int VS = 72;                                     // row stride of V: the two lane halves (rows 4 apart) hit different banks
    __shared__ __attribute__((aligned(16))) float Ks[32 * 64]; // 16-byte chunk c of row r at c ^ (r & 15)
    __shared__ __attribute__((aligned(16))) float Vs[32 * VS];
    const int nb = n_blocks_dev ? min(*n_blocks_dev, n_blocks) : n_blocks;
    const int groups = (T + 127) / 128;
    const int b = blockIdx.x / (heads * groups), hd = (blockIdx.x / groups) % heads, gq = blockIdx.x % groups;
    if (b >= nb) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lm = lane & 31, lh = lane >> 5;
    const size_t ld = (size_t)3 * D;
    const float *base = qkv + (size_t)b * T * ld + hd * 64;
    const int query = gq * 128 + wave * 32 + lm;
    const bool live = gq * 128 + wave * 32 < T;                // (wave-uniform)
    f32x4 qf[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) qf[kk] = *(const f32x4 *)(base + (size_t)min(query, T - 1) * ld + 8 * kk + 4 * lh) * 0.125f;
    f32x4 kv[4];                                               // this thread's pieces of the next tile: two of K, two of V
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int v = tid + 256 * i;
            const float *row = base + (size_t)min(k0 + (v >> 4), T - 1) * ld + (v & 15) * 4;
            kv[i] = *(const f32x4 *)(row + D);
            kv[2 + i] = *(const f32x4 *)(row + 2 * D);
        }
    };
    load(0);
    f32x16 o[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) o[0][e] = o[1][e] = 0.f;
    float mx = -INFINITY, sum = 0.f;
    for (int k0 = 0; k0 < T; k0 += 32) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int v = tid + 256 * i, r = v >> 4, c = v & 15;
            *(f32x4 *)(Ks + r * 64 + ((c ^ (r & 15)) << 2)) = kv[i];
            *(f32x4 *)(Vs + r * VS + c * 4) = kv[2 + i];
        }
        __syncthreads();
        if (k0 + 32 < T) load(k0 + 32);
        if (!live) continue;
        f32x16 s;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const f32x4 kf = *(const f32x4 *)(Ks + lm * 64 + (((2 * kk + lh) ^ (lm & 15)) << 2));
#pragma unroll
            for (int z = 0; z < 4; ++z) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[z], qf[kk][z], s, 0, 0, 0);
        }
        float m = -INFINITY;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if (k0 + 8 * (e >> 2) + 4 * lh + (e & 3) >= T) s[e] = -INFINITY;
            m = fmaxf(m, s[e]);
        }
        m = fmaxf(mx, fmaxf(m, __shfl_xor(m, 32, 64)));        // (a tile always has a key inside T)
        const float corr = expf(mx - m);
        mx = m;
        float t = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) { s[e] = expf(s[e] - m); t += s[e]; }
        sum = fmaf(sum, corr, t);
#pragma unroll
        for (int e = 0; e < 16; ++e) { o[0][e] *= corr; o[1][e] *= corr; }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float *vr = Vs + (8 * (e >> 2) + 4 * lh + (e & 3)) * VS + lm;
            o[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[0], s[e], o[0], 0, 0, 0);
            o[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[32], s[e], o[1], 0, 0, 0);
        }
    }
    if (query < T) {
        const float inv = 1.0f / (sum + __shfl_xor(sum, 32, 64));
        float *orow = out + ((size_t)b * T + query) * D + hd * 64 + 4 * lh;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f32x4 *)(orow + dt * 32 + 8 * q) = f32x4{o[dt][4 * q], o[dt][4 * q + 1], o[dt][4 * q + 2], o[dt][4 * q + 3]} * inv;
    }
}

// sum over the LPK neighbouring lanes (8 or 16) that hold a row's pieces, in every one of them
template <int LPK> __device__ __forceinline__ float piece_sum(float v)
{
    auto add = [&](auto ctrl) { v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, true)); };
    add(std::integral_constant<int, 0xB1>{});              // quad_perm: lanes l ^ 1, l ^ 2
    add(std::integral_constant<int, 0x4E>{});
    add(std::integral_constant<int, 0x141>{});             // row_half_mirror, row_mirror
    if (LPK == 16) add(std::integral_constant<int, 0x140>{});
    return v;
}

// Attention of a block's first query (the class token), all that the heads read of the last layer: one (block, head) per workgroup, and the block's class row
// of the residual stream beside it, so that what follows works on blocks of one row.  A row of 64 elements is LPK lanes x 16 bytes, for the scores and for the
// second product alike, so nothing changes lanes but the sums: a lane group keeps a maximum, a sum and its part of the output of its own keys, and the 4 KPI
// groups meet in LDS once.  Probabilities stay in fp32.
// Bound by the bytes of K and V (50 KB per workgroup of 197 keys in bf16, all requested up front).
template <typename E, int NI>       // NI: keys per lane group at a time (bf16: T <= 32 NI; fp32 goes on from there with what it has so far)
__global__ __launch_bounds__(256) void attn_class_kernel(const E *qkv, E *out, int T, int D, int heads, int n_blocks, const int *n_blocks_dev, const float *x,
                                                         const int *x_block, int x_fragments, float *x_out)
{
    constexpr int EPL = 16 / (int)sizeof(E), LPK = 64 / EPL, KPI = 64 / LPK, GROUPS = 4 * KPI;      // elements per lane, lanes per key, keys per instruction
    typedef E piece_t __attribute__((ext_vector_type(EPL)));
    constexpr bool BF16 = sizeof(E) == 2;
    __shared__ __attribute__((aligned(16))) float part[GROUPS][64], ml[2][GROUPS];
    const int nb = n_blocks_dev ? min(*n_blocks_dev, n_blocks) : n_blocks;
    const int b = blockIdx.x / heads, hd = blockIdx.x % heads;
    if (b >= nb) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane / LPK, c = lane % LPK;
    const size_t ld = (size_t)3 * D;
    const E *base = qkv + (size_t)b * T * ld + hd * 64 + c * EPL;
    const piece_t qp = *(const piece_t *)base;
    piece_t kp[NI], vp[NI];
    auto key = [&](int t0, int i) { return t0 + (i * 4 + wave) * KPI + g; };
    auto load = [&](int t0) {                              // rows past T repeat row T - 1
#pragma unroll
        for (int i = 0; i < NI; ++i) kp[i] = *(const piece_t *)(base + (size_t)min(key(t0, i), T - 1) * ld + D);
#pragma unroll
        for (int i = 0; i < NI; ++i) vp[i] = *(const piece_t *)(base + (size_t)min(key(t0, i), T - 1) * ld + 2 * D);
    };
    load(0);
    if (wave == 3) {
        const size_t row = (size_t)(x_block ? x_block[b] : b) * T;
        const int col = hd * 64 + lane;
        const float v = x_fragments ? x[(row >> 5) * 32 * D + (col >> 3) * 256 + (col >> 2 & 1) * 128 + (row & 31) * 4 + (col & 3)] : x[row * D + col];
        x_out[(size_t)b * D + col] = v;
    }
    const float scale = BF16 ? 0.125f * LOG2E : 0.125f;
    auto pexp = [&](float v) { return BF16 ? __builtin_amdgcn_exp2f(v) : expf(v); };
    float q[EPL], o[EPL], mx = -INFINITY, sum = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) { q[e] = (float)qp[e] * scale; o[e] = 0.f; }
    for (int t0 = 0;;) {
        float s[NI], m = mx;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            float a = 0.f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) a = fmaf(q[e], (float)kp[i][e], a);
            a = piece_sum<LPK>(a);
            s[i] = key(t0, i) < T ? a : -INFINITY;
            m = fmaxf(m, s[i]);
        }
        const float safe = fmaxf(m, -3.4e38f);             // (a group without keys, or with -infinity in all of them, counts nothing)
        const float corr = pexp(mx - safe);
        mx = m;
        sum *= corr;
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[e] *= corr;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const float p = pexp(s[i] - safe);
            sum += p;
            const bool in = key(t0, i) < T;
#pragma unroll
            for (int e = 0; e < EPL; ++e) o[e] = fmaf(p, in ? (float)vp[i][e] : 0.f, o[e]);
        }
        t0 += NI * GROUPS;
        if (BF16 || t0 >= T) break;
        load(t0);
    }
    const int gr = wave * KPI + g;
#pragma unroll
    for (int e = 0; e < EPL; e += 4) *(f32x4 *)&part[gr][c * EPL + e] = f32x4{o[e], o[e + 1], o[e + 2], o[e + 3]};
    if (c == 0) { ml[0][gr] = mx; ml[1][gr] = sum; }
    __syncthreads();
    if (wave) return;
    float M = -INFINITY, all = 0.f, y = 0.f;
#pragma unroll
    for (int j = 0; j < GROUPS; ++j) M = fmaxf(M, ml[0][j]);
    M = fmaxf(M, -3.4e38f);
#pragma unroll
    for (int j = 0; j < GROUPS; ++j) {
        const float w = pexp(ml[0][j] - M);
        all = fmaf(ml[1][j], w, all);
        y = fmaf(part[j][lane], w, y);
    }
    out[(size_t)b * D + hd * 64 + lane] = (E)(y / all);
}

template <int NKT, int W, bool FRAGMENTS, bool SPLIT>
int launch_bf16(const void *qkv, void *out, int T, int D, int heads, int n_blocks, const int *n_blocks_dev, hipStream_t st)
{
    const int LDS = (att_keys(T) * 128 + 64 * 4) * 2;
    auto kern = attn_bf16_kernel<NKT, W, FRAGMENTS, SPLIT>;
    POLY_LAUNCH_SHMEM(POLY_STAGE_ATTN, kern, dim3((unsigned)(n_blocks * heads), SPLIT ? 2 : 1), dim3(64 * W), LDS, st, (const bf16_t *)qkv, (bf16_t *)out, T, D,
                      heads, n_blocks, n_blocks_dev);
    return POLY_OK;
}
template <int NKT, int W = NKT>
int launch_bf16(const void *qkv, void *out, int T, int D, int heads, int n_blocks, const int *n_blocks_dev, bool fragments, hipStream_t st, bool split = false)
{
    if constexpr (W == NKT && NKT > 4)
        if (split && !fragments) return launch_bf16<NKT, W, false, true>(qkv, out, T, D, heads, n_blocks, n_blocks_dev, st);
    return (fragments ? launch_bf16<NKT, W, true, false> : launch_bf16<NKT, W, false, false>)(qkv, out, T, D, heads, n_blocks, n_blocks_dev, st);
}

}  // namespace

int launch_attention(const void *qkv, void *out, int T, int D, int heads, int n_blocks, const int *n_blocks_dev, int n_usual, int dtype,
                     bool fragments, hipStream_t st)
{
    if (n_blocks == 0) return POLY_OK;
    if (D != heads * 64 || (fragments && dtype != POLY_BF16)) return POLY_EINVAL;
    if (dtype == POLY_BF16) {
        // From 161 keys on, two query tiles per wave and up to three workgroups per CU, one loading while another computes, are faster where there are more
        // workgroups than CUs, and slower below.  Half the waves from the start where the usual count says so, else the form that looks at the true
        // count (whose second workgroup cannot load beside the first).  us, by the count / half the waves, 197 tokens: 96 workgroups 7.7 / 8.8, 192 9.3 / 10.3,
        // 252 10.4 / 11.6, 264 15.2 / 14.3, 360 16.2 / 15.4, 516 21.0 / 19.3, 720 22.8 / 21.2.
        // From 129 keys on, where there are two CUs for every workgroup, it is two: all waves load and four (three, two, one) compute, one per SIMD.  197 tokens: 48 workgroups
        // 7.3 / 6.1, 96 7.6 / 6.5, 120 7.8 / 6.9, 132 8.0 / 9.4; 155 tokens 60 5.7 / 5.2, 120 6.4 / 5.8, 132 6.5 / 7.4.  (Of a bound half of what it has over the usual.)
        const bool many = (long)n_usual * heads > 256, split = ((long)n_usual + n_blocks) * heads <= 256;
        switch ((T + 31) / 32) {
        case 1: if (launch_bf16<1>(qkv, out, T, D, heads, n_blocks, n_blocks_dev, fragments, st) != POLY_OK) return POLY_EHIP; break;
        case 2: if (launch_bf16<2>(qkv, out, T, D, heads, n_blocks, n_blocks_dev, fragments, st) != POLY_OK) return POLY_EHIP; break;
        case 3: if (launch_bf16<3>(qkv, out, T, D, heads, n_blocks, n_blocks_dev, fragments, st) != POLY_OK) return POLY_EHIP; break;
        case 4: if (launch_bf16<4>(qkv, out, T, D, heads, n_blocks, n_blocks_dev, fragments, st) != POLY_OK) return POLY_EHIP; break;
        case 5: if (launch_bf16<5>(qkv, out, T, D, heads, n_blocks, n_blocks_dev, fragments, st, split) != POLY_OK) return POLY_EHIP; break;
        case 6: if ((many ? launch_bf16<6, 3> : launch_bf16<6>)(qkv, out, T, D, heads, n_blocks, n_blocks_dev, fragments, st, split) != POLY_OK) return POLY_EHIP; break;
        case 7: if ((many ? launch_bf16<7, 4> : launch_bf16<7>)(qkv, out, T, D, heads, n_blocks, n_blocks_dev, fragments, st, split) != POLY_OK) return POLY_EHIP; break;
        default: return POLY_EINVAL;  // bf16 attention holds all keys of a block in LDS: T <= 224
        }
    } else {
        POLY_LAUNCH(POLY_STAGE_ATTN, attn_f32_kernel, dim3((unsigned)(n_blocks * heads * ((T + 127) / 128))), dim3(256), st, (const float *)qkv, (float *)out, T, D, heads,
                           n_blocks, n_blocks_dev);
    }
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

int launch_attention_class(const void *qkv, void *out, int T, int D, int heads, int n_blocks, const int *n_blocks_dev, const float *x, const int *x_block,
                           bool x_fragments, float *x_out, int dtype, hipStream_t st)
{
    if (n_blocks == 0) return POLY_OK;
    if (D != heads * 64 || (dtype == POLY_BF16 && T > 224)) return POLY_EINVAL;
    const dim3 grid((unsigned)(n_blocks * heads));
#define ATTN_CLASS(E, NI)                                                                                                                                      \
    POLY_LAUNCH(POLY_STAGE_ATTN, (attn_class_kernel<E, NI>), grid, dim3(256), st, (const E *)qkv, (E *)out, T, D, heads, n_blocks, n_blocks_dev, x, x_block, \
                (int)x_fragments, x_out)
    if (dtype != POLY_BF16) ATTN_CLASS(float, 7);
    else if (T <= 64) ATTN_CLASS(bf16_t, 2);
    else if (T <= 128) ATTN_CLASS(bf16_t, 4);
    else ATTN_CLASS(bf16_t, 7);
#undef ATTN_CLASS
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}
