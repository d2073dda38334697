// A stack of transformer layers on few token blocks in ONE launch: the workgroups take small tasks from a queue and a task starts as
// soon as the tasks that it reads from are done.
//
// With a few blocks a layer is no work for this chip, only a chain of dependent steps: a launch per step costs three to five
// microseconds (issue, dispatch, caches emptied at the boundary), and a kernel that keeps 64 rows to itself through a whole layer
// (rowlayer.hip) leaves most CUs idle while the busy ones pull 885 KB of weights each through one CU's load path.  Here a
// layer is five steps
//     Q  qkv = LayerNorm1(x) Wq + bq (+ low rank)      V is stored transposed, as the second product of attention reads it
//     A  o = softmax(q k^T / 8) v                       one head, 32 queries
//     P  x += o Wp + bp (+ low rank)
//     1  h = GELU(LayerNorm2(x) W1 + b1 (+ low rank))
//     2  x += h W2 + b2 (+ low rank)
// each cut into tasks of 32 rows x 64 columns (A: 32 queries), so that one block of 197 tokens already gives 21 to 84 tasks a step.
// The weights of a task are requested before its inputs are waited for.
//
// Passing data between XCDs, whose L2s do not see each other's writes, without fences: results are stored at device scope (sc1: through to
// memory), the stores are waited for, then the task is counted with an atomic; and every layer of a launch has buffers of its own, so that
// no address is read by this launch before it has been written for good, and no L1 or L2 can hold an old copy of it.  Every 128-byte line
// is written by the tasks of one counter only, so a line is complete when anything in it is read.  Loads are therefore ordinary ones, and
// the many tasks that read the same rows hit the L2.  4 KB change hands in 1.2 us this way between two workgroups of an idle chip, in 2.2 us
// with release and acquire fences, which moreover empty the L2 that holds the weights.
//
// Order and progress: a queue's tickets are numbered layer by layer and step by step, a task waits only for tasks with lower
// numbers of the same queue, and a workgroup works through the tickets it has drawn in ascending order.  The lowest unfinished ticket
// is therefore always being worked on by a running workgroup and waits for nothing, whatever other workgroups are not (yet) running:
// every wait ends, as long as nobody else writes the counters.  Two calls on one workspace at a time would: their results are undefined, but
// the kernel has to come to its end all the same, so a workgroup looks at counters a limited number of times per launch (a million, about
// a second; a whole launch takes under a millisecond), then works on without waiting and the call reports POLY_ESTALL.
//
// What bounds it: the chain of a block, five steps per layer with a hand-over each, four where P is part of the F1 tasks (few tiles: launch_flow_d).  DeiT-tiny,
// one live frame: 14.9 us per layer (15.7 in five steps; two launches of ten and two layers), the matrix unit busy 0.7 % of the time; the lagged loop takes
// 195 us instead of the 473 of row kernels and attention launches.  With many blocks the weights that every 32-row task pulls through its CU's load path bound it, and kernels with
// larger tiles take over (api.hip).
//
// Single precision: the same tasks on v_mfma_f32_16x16x4_f32, elements and buffers of twice the size, one workgroup per CU (190 registers).  The same
// chain bounds it: two layers on 4 frames of 17 tokens, 22 launches of 3 to 13 us each before, 128 us per forward / 74 now (70 with the patches gathered by the product); one frame of
// 197 tokens 168 / 82 (78).  Its products are an eighth of the bf16 rate, so the tasks give way to larger tiles with fewer blocks than in bf16 (api.hip).
#include "flow_dev.h"

namespace {

__device__ __forceinline__ f32x4 gelu(f32x4 v, bf16_t) { return gelu_fine4(v); }
__device__ __forceinline__ f32x4 gelu(f32x4 v, float) { return f32x4{gelu_erf(v[0]), gelu_erf(v[1]), gelu_erf(v[2]), gelu_erf(v[3])}; }

// LDS of a norm task: rows, partial sums that the halves of K hand over (NT x 8 KB; with proj in it KD / 2 x 8 KB), shrink [quarter of K][row half][rank
// tile][lane], with proj in it the rows of the stream
template <typename E> constexpr int norm_red(int kd, int nt, bool pre) { return (pre && kd / 2 > nt ? kd / 2 : nt) * 8192; }
template <typename E> constexpr int norm_lds(int kd, int nt, bool pre)
{
    return 32 * 32 * kd * (int)sizeof(E) + norm_red<E>(kd, nt, pre) + 16384 + (pre ? 32 * (32 * kd + 4) * 4 : 0);
}

// ---- LayerNorm + linear on 32 rows x NT tiles of 64 columns; STAGE: 0 Q, 3 F1.  The normalised rows go through LDS; wave (kh, wc)
// takes half kh of the contraction for the 16 columns 16 wc .. of a tile, both row halves; returns the counter to raise.
// PRE: the rows are not read but made here, x1 = x + o Wp + bp (+ low rank), by every task of these rows, and the first of them stores them for F2
template <typename E, int KD, int STAGE, int NT, bool SUM, bool PRE>
__device__ __forceinline__ unsigned *norm_task(const Task &k, char *lds)
{
    typedef El<E> L;
    typedef typename L::op op_t;
    typedef typename L::quad quad_t;
    constexpr int ES = sizeof(E) / 2;
    constexpr int D = 32 * KD, KT = KD / 2, HK = KD / 2;       // HK: K steps of a wave
    constexpr int NA = (KD + 3) / 4;                           // K steps of a wave's share of the shrink
    E *As = (E *)lds;                                          // rows: 32 x D, chunks of eight swizzled by row
    char *red = lds + 32 * D * sizeof(E), *shr = red + norm_red<E>(KD, NT, PRE);
    const ParamPtr p = params();
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lm = lane & 15, g = lane >> 4;
    const int kh = wave >> 2, wc = wave & 3, T = p->a.T, t0 = k.rt * 32, b = k.b;
    const size_t ld = k.layer;
    const unsigned *dep = counter(k, (STAGE == 0 ? C_F2 : PRE ? C_A : C_P) + k.rt);
    const unsigned want = (k.layer + (STAGE == 0 ? 0 : 1)) * (PRE ? p->a.heads : p->a_p2);
    unsigned seen = 0;
    if (wave == 0) seen = peek(dep);
    const int N = STAGE == 0 ? 3 * D : p->a.Dm, dt = p->ct_d;
    // tile i of the task: q, k and v of one head, or neighbours
    auto tile = [&](int i) { return STAGE == 0 ? k.ct + i * dt : k.ct * NT + i; };
    auto is_v = [&](int i) { return STAGE == 0 && tile(i) >= 2 * dt; };            // V: product untransposed
    constexpr int PT = KT;                                     // PRE: 16-column tiles of proj a wave takes
    op_t wp[PT][HK];
    f32x4 biasp[PT];
    if constexpr (PRE) {
        const E *Wp = (const E *)p->a.Wp + (ld * D + wc * PT * 16 + lm) * D + kh * HK * 32 + 8 * g;
#pragma unroll
        for (int t = 0; t < PT; ++t) {
#pragma unroll
            for (int j = 0; j < HK; ++j) wp[t][j] = *(const op_t *)(Wp + (size_t)t * 16 * D + 32 * j);
            biasp[t] = *(const f32x4_u *)(p->a.bp + ld * D + (wc * PT + t) * 16 + 4 * g);
        }
    }
    const E *W = (const E *)(STAGE == 0 ? p->a.Wq : p->a.W1) + ld * N * D + (size_t)(wc * 16 + lm) * D + kh * HK * 32 + 8 * g;
    const float *bias = (STAGE == 0 ? p->a.bq : p->a.b1) + ld * N + wc * 16;
    op_t wf[NT][HK];
    f32x4 bias4[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
#pragma unroll
        for (int j = 0; j < HK; ++j) wf[i][j] = *(const op_t *)(W + (size_t)tile(i) * 64 * D + 32 * j);
    }
    constexpr bool LEAN = NT > 2;                              // gains and biases are requested later: registers
    auto load_bias = [&]() {
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const float *bp = bias + tile(i) * 64;
            if (is_v(i)) { const float bv = bp[lm]; bias4[i] = f32x4{bv, bv, bv, bv}; }
            else bias4[i] = *(const f32x4_u *)(bp + 4 * g);
        }
    };
    if (!LEAN) load_bias();
    const int row = tid >> 4, part = tid & 15, rrow = min(t0 + row, T - 1);
    const float *gain = (STAGE == 0 ? p->a.ln1_g : p->a.ln2_g) + ld * D + 4 * part, *shift = (STAGE == 0 ? p->a.ln1_b : p->a.ln2_b) + ld * D + 4 * part;
    f32x4 gn[KT], sh[KT];
    auto load_gain = [&]() {
#pragma unroll
        for (int i = 0; i < KT; ++i) { gn[i] = *(const f32x4_u *)(gain + 64 * i); sh[i] = *(const f32x4_u *)(shift + 64 * i); }
    };
    if (!LEAN) load_gain();
    // operands of the low-rank terms of this block's adapter(s); those of the first one are requested here
    constexpr int TGT = STAGE == 0 ? 0 : 2;
    const E *At = (const E *)p->a.At[TGT], *Bt = (const E *)p->a.Bt[TGT];
    const int *set_off = p->a.set_off, *adapter = p->a.adapter_of_row, *in_map = p->a.in_map;
    const int s0 = At ? (SUM ? uload(set_off + b) : b) : 0, s1 = At ? (SUM ? uload(set_off + b + 1) : b + 1) : 0;
    const int r = p->a.r, nrk = (r + 15) >> 4;
    const quad_t z4 = {0, 0, 0, 0};
    op_t fat[NA][2];
    auto load_at = [&](int s) {
        const E *Ak = At + (p->a.n_adapters * ld + uload(adapter + s)) * r * D + 8 * g;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int kk = min(wc + 4 * i, KD - 1);
            fat[i][0] = *(const op_t *)(Ak + (size_t)min(lm, r - 1) * D + 32 * kk);
            if (nrk > 1) fat[i][1] = *(const op_t *)(Ak + (size_t)min(16 + lm, r - 1) * D + 32 * kk);
        }
    };
    op_t fb[NT];
    auto load_bt = [&](int s) {                                // ranks 4 g .. and 16 + 4 g .. of a column
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const E *bt = Bt + ((p->a.n_adapters * ld + uload(adapter + s)) * N + tile(i) * 64 + wc * 16 + lm) * r + 4 * g;
            quad_t lo = *(const quad_t *)(bt + min(0, r - 4 - 4 * g)), hi = z4;
            if (4 * g >= r) lo = z4;
            if (nrk > 1) {
                hi = *(const quad_t *)(bt + min(16, r - 4 - 4 * g));
                if (16 + 4 * g >= r) hi = z4;
            }
            fb[i] = L::join(lo, hi);
        }
    };
    if (s0 < s1) { load_at(s0); load_bt(s0); }
    const bool first = (STAGE == 0 || PRE) && k.layer == 0;    // the stream still lies where the caller put it
    const int xblk = first && in_map ? uload(in_map + b) : b;
    const size_t step = (size_t)p->a.nb * T * D, slot = ld * p->a.nb + b;
    const int TP = p->nrt * 32;
    const float *xs = STAGE == 3 && !PRE ? p->a.x1 + ld * step : first ? p->a.x_in : p->a.x2 + (ld - 1) * step;
    const Buf xb(xs + (size_t)xblk * T * D, (unsigned)T * D * 4);
    // the shrink of a term is shared by the waves (row half kh, K steps wc, wc + 4), the partial sums meet in LDS, and ranks 4 g .. and 16 + 4 g ..
    // of row lm are what a lane feeds to the expand
    auto shrink_store = [&](const f32x4(&sp)[2]) {
        *(f32x4 *)(shr + (((wc * 2 + kh) * 2 + 0) * 64 + lane) * 16) = sp[0];
        if (nrk > 1) *(f32x4 *)(shr + (((wc * 2 + kh) * 2 + 1) * 64 + lane) * 16) = sp[1];
    };
    auto shrink_sum = [&]() {
        quad_t fs[2] = {z4, z4};
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (q < nrk) {
                f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int w = 0; w < 4; ++w) t += *(const f32x4 *)(shr + (((w * 2 + kh) * 2 + q) * 64 + lane) * 16);
                fs[q] = L::round4(t * p->a.scale);
            }
        return L::join(fs[0], fs[1]);
    };
    float *x1s = (float *)(shr + 16384);                       // PRE: rows of D + 4 floats
    // PRE: operands of proj's low-rank terms
    const E *Atp = PRE ? (const E *)p->a.At[1] : nullptr, *Btp = PRE ? (const E *)p->a.Bt[1] : nullptr;
    const int p0 = Atp ? (SUM ? uload(set_off + b) : b) : 0, p1 = Atp ? (SUM ? uload(set_off + b + 1) : b + 1) : 0;
    op_t fap[PRE ? NA : 1][2], fbp[PRE ? PT : 1];
    auto load_p = [&](int s) {
        if constexpr (PRE) {
            const size_t ad = p->a.n_adapters * ld + uload(adapter + s);
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const E *Ak = Atp + ad * r * D + 8 * g + 32 * min(wc + 4 * i, KD - 1);
                fap[i][0] = *(const op_t *)(Ak + (size_t)min(lm, r - 1) * D);
                if (nrk > 1) fap[i][1] = *(const op_t *)(Ak + (size_t)min(16 + lm, r - 1) * D);
            }
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                const E *bt = Btp + (ad * D + (wc * PT + t) * 16 + lm) * r + 4 * g;
                quad_t lo = *(const quad_t *)(bt + min(0, r - 4 - 4 * g)), hi = z4;
                if (4 * g >= r) lo = z4;
                if (nrk > 1) {
                    hi = *(const quad_t *)(bt + min(16, r - 4 - 4 * g));
                    if (16 + 4 * g >= r) hi = z4;
                }
                fbp[t] = L::join(lo, hi);
            }
        }
    };
    if (p0 < p1) load_p(p0);
    // ---- inputs
    if (wave == 0) await(k, dep, seen, want);
    __syncthreads();
    if constexpr (PRE) {
        const Buf src((const E *)p->a.o + slot * TP * D, (unsigned)TP * D * 2 * ES);
        auto load_o = [&](int m, int j) { return L::load(src, (((k.rt * 2 + m) * KD + j) * 1024 + lane * 16) * ES); };
        op_t fo[2][HK], fos[NA];
        f32x4 res[PT];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int j = 0; j < HK; ++j) fo[m][j] = load_o(m, kh * HK + j);
        if (p0 < p1) {
#pragma unroll
            for (int i = 0; i < NA; ++i) fos[i] = load_o(kh, min(wc + 4 * i, KD - 1));
        }
        const int xrow = t0 + 16 * kh + lm;
        const unsigned xoff = ((unsigned)min(xrow, T - 1) * D + wc * PT * 16 + 4 * g) * 4;
#pragma unroll
        for (int t = 0; t < PT; ++t) res[t] = __builtin_bit_cast(f32x4, xb.ld16(xoff + 64 * t));
        auto shrink_o = [&]() {
            f32x4 sp[2] = {};
#pragma unroll
            for (int i = 0; i < NA; ++i)
                if (wc + 4 * i < KD) {
                    sp[0] = L::mma(fap[i][0], fos[i], sp[0]);
                    if (nrk > 1) sp[1] = L::mma(fap[i][1], fos[i], sp[1]);
                }
            shrink_store(sp);
        };
        f32x4 y[PT];
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            f32x4 acc[2] = {};
#pragma unroll
            for (int j = 0; j < HK; ++j)
#pragma unroll
                for (int m = 0; m < 2; ++m) acc[m] = L::mma(wp[t][j], fo[m][j], acc[m]);
            *(f32x4 *)(red + ((t * 8 + wave) * 64 + lane) * 16) = kh ? acc[0] : acc[1];
            y[t] = kh ? acc[1] : acc[0];
        }
        if (p0 < p1) shrink_o();
        __syncthreads();
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            const f32x4 other = *(const f32x4 *)(red + ((t * 8 + (wave ^ 4)) * 64 + lane) * 16);
            y[t] = kh ? other + y[t] : y[t] + other;
        }
        for (int s = p0; s < p1; ++s) {
            if (SUM && s > p0) {                               // further terms summed on this block
                load_p(s);
                __syncthreads();
                shrink_o();
                __syncthreads();
            }
            const op_t fs = shrink_sum();
#pragma unroll
            for (int t = 0; t < PT; ++t) y[t] = L::mma(fbp[t], fs, y[t]);
            if (!SUM) break;
        }
        const Buf xo(p->a.x1 + ld * step + (size_t)b * T * D, (unsigned)T * D * 4);
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            const f32x4 v = y[t] + biasp[t] + res[t];
            *(f32x4 *)(x1s + (16 * kh + lm) * (D + 4) + (wc * PT + t) * 16 + 4 * g) = v;
            if (k.ct == 0 && xrow < T) xo.st16(__builtin_bit_cast(u32x4_, v), xoff + 64 * t);
        }
        __syncthreads();
    }
    {
        f32x4 v[KT];
#pragma unroll
        for (int i = 0; i < KT; ++i) {
            if constexpr (PRE) v[i] = *(const f32x4 *)(x1s + row * (D + 4) + 4 * (part + 16 * i));
            else v[i] = __builtin_bit_cast(f32x4, xb.ld16(((unsigned)rrow * D + 4 * (part + 16 * i)) * 4));
        }
        if (LEAN) load_gain();
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < KT; ++i) t += v[i][0] + v[i][1] + v[i][2] + v[i][3];
        const float mean = L::over(row16_sum(t), D);
        float q = 0.f;
#pragma unroll
        for (int i = 0; i < KT; ++i)
#pragma unroll
            for (int z = 0; z < 4; ++z) { const float d = v[i][z] - mean; q = fmaf(d, d, q); }
        const float inv = rsqrtf(row16_sum(q) * (1.0f / D) + p->a.eps), nmi = -mean * inv;
#pragma unroll
        for (int i = 0; i < KT; ++i) {
            f32x4 o;
#pragma unroll
            for (int z = 0; z < 4; ++z) o[z] = fmaf(L::centred(v[i][z], mean, inv, nmi), gn[i][z], sh[i][z]);
            const int c = 4 * (part + 16 * i);
            *(quad_t *)(As + row * D + (((c >> 3) ^ (row & 7)) << 3) + (c & 4)) = L::round4(o);
        }
    }
    __syncthreads();
    if (tid == 0) draw(k);
    // fragment of rows 16 m + lm, K step i: chunk 4 i + g
    auto frag_a = [&](int m, int i) { return *(const op_t *)(As + (16 * m + lm) * D + (((4 * i + g) ^ (lm & 7)) << 3)); };
    auto shrink_part = [&]() {
        f32x4 sp[2] = {};
#pragma unroll
        for (int i = 0; i < NA; ++i)
            if (wc + 4 * i < KD) {
                const op_t fa = frag_a(kh, wc + 4 * i);
                sp[0] = L::mma(fat[i][0], fa, sp[0]);
                if (nrk > 1) sp[1] = L::mma(fat[i][1], fa, sp[1]);
            }
        shrink_store(sp);
    };
    if (s0 < s1) shrink_part();
    f32x4 y[NT];                                               // the row half that this wave finishes: 16 kh ..
    {
        op_t fa[2][HK];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int j = 0; j < HK; ++j) fa[m][j] = frag_a(m, kh * HK + j);
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int j = 0; j < HK; ++j)
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const op_t u = is_v(i) ? fa[m][j] : wf[i][j], v = is_v(i) ? wf[i][j] : fa[m][j];
                    acc[m] = L::mma(u, v, acc[m]);
                }
            *(f32x4 *)(red + ((i * 8 + wave) * 64 + lane) * 16) = kh ? acc[0] : acc[1];
            y[i] = kh ? acc[1] : acc[0];
        }
    }
    if (LEAN) load_bias();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const f32x4 other = *(const f32x4 *)(red + ((i * 8 + (wave ^ 4)) * 64 + lane) * 16);
        y[i] = kh ? other + y[i] : y[i] + other;
    }
    for (int s = s0; s < s1; ++s) {
        if (SUM && s > s0) {                                   // further terms summed on this block
            load_at(s); load_bt(s);
            __syncthreads();
            shrink_part();
            __syncthreads();
        }
        const op_t fs = shrink_sum();
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const op_t u = is_v(i) ? fs : fb[i], v = is_v(i) ? fb[i] : fs;
            y[i] = L::mma(u, v, y[i]);
        }
        if (!SUM) break;
    }
    // q and k as [head][16 rows][32 columns][lane][8], v as [head][32 rows][16 columns][lane][rows 4 g .., 16 + 4 g ..]: attention
    // reads 1 KB per instruction (rows past T repeat row T - 1: finite, and masked there)
    const Buf vt((const E *)p->a.vt + slot * D * TP, (unsigned)D * TP * 2 * ES), qk((const E *)p->a.qk + slot * TP * 2 * D, (unsigned)TP * 4 * D * ES),
        hb((const E *)p->a.h + slot * TP * N, (unsigned)TP * N * 2 * ES);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const int ct = tile(i);
        const f32x4 v = y[i] + bias4[i];
        if (STAGE == 3) L::store4(hb, gelu(v, E()), frag_off(k.rt, kh, N / 32, ct * 4 + wc, lm, g) * ES);
        else if (is_v(i)) L::store4(vt, v, ((unsigned)(ct - 2 * dt) * TP * 128 + (4 * k.rt + wc) * 1024 + lane * 16 + kh * 8) * ES);
        else L::store4(qk, v, ((unsigned)ct * TP * 128 + frag_off(k.rt, kh, 2, wc, lm, g)) * ES);
    }
    return counter(k, STAGE == 0 ? C_Q + (k.ct < dt ? k.ct : k.ct < 2 * dt ? k.ct - dt : k.ct - 2 * dt) : C_F1 + k.rt);
}

// ---- linear + residual on 32 rows x NT tiles of 16 NC columns; STAGE: 2 P, 4 F2.  Wave w takes the K steps w, w + 8, .. of the whole tile,
// both operands straight from memory in fragment order, and the partial sums meet in LDS; returns the counter to raise
template <typename E, int KD, int CH, int STAGE, int NT, int NC, bool SUM>
__device__ __forceinline__ unsigned *resid_task(const Task &k, char *lds)
{
    typedef El<E> L;
    typedef typename L::op op_t;
    typedef typename L::quad quad_t;
    constexpr int ES = sizeof(E) / 2;
    constexpr int D = 32 * KD, KS = STAGE == 4 ? CH : KD, NS = (KS + 7) / 8;      // K steps of a wave
    static_assert(NT <= 2, "waves 0 - 3 and 4 - 7 finish a tile each");
    char *red = lds, *shr = lds + 32768;                       // [tile][wave][row half][column half][lane]; [wave][row half][rank tile][lane]
    const ParamPtr p = params();
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lm = lane & 15, g = lane >> 4;
    const int T = p->a.T, TP = p->nrt * 32, b = k.b;
    const size_t ld = k.layer;
    const unsigned *dep = counter(k, (STAGE == 2 ? C_A : C_F1) + k.rt);
    const unsigned want = (k.layer + 1) * (STAGE == 2 ? p->a.heads : p->a_1);
    unsigned seen = 0;
    if (wave == 0) seen = peek(dep);
    const int K = STAGE == 4 ? p->a.Dm : D, ks = K / 32, np = min(ks, 8);
    const E *W = (const E *)(STAGE == 2 ? p->a.Wp : p->a.W2) + (ld * D + k.ct * NT * 16 * NC + lm) * K + 8 * g;
    op_t wf[NT][NS][NC];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int n = 0; n < NC; ++n) wf[j][i][n] = *(const op_t *)(W + (size_t)(j * 16 * NC + 16 * n) * K + 32 * min(wave + 8 * i, ks - 1));
    // waves 2 NC j .. finish the subtiles of tile j: rows 16 fm .., columns 16 fn ..
    const int fj = wave / (2 * NC), fm = (wave / NC) & 1, fn = wave & (NC - 1), trow = k.rt * 32 + 16 * fm + lm, fcol = ((k.ct * NT + fj) * NC + fn) * 16;
    const bool fin = wave < 2 * NC * NT;
    const f32x4 bias4 = *(const f32x4_u *)((STAGE == 2 ? p->a.bp : p->a.b2) + ld * D + (fin ? fcol : 0) + 4 * g);
    constexpr int TGT = STAGE == 2 ? 1 : 3;
    const E *At = (const E *)p->a.At[TGT], *Bt = (const E *)p->a.Bt[TGT];
    const int *set_off = p->a.set_off, *adapter = p->a.adapter_of_row, *in_map = p->a.in_map;
    const int s0 = At ? (SUM ? uload(set_off + b) : b) : 0, s1 = At ? (SUM ? uload(set_off + b + 1) : b + 1) : 0;
    const int r = p->a.r, nrk = (r + 15) >> 4;
    const quad_t z4 = {0, 0, 0, 0};
    op_t fat[2];                                               // of one K step
    auto load_at = [&](int s, int i) {
        const E *Ak = At + (p->a.n_adapters * ld + uload(adapter + s)) * r * K + 32 * min(wave + 8 * i, ks - 1) + 8 * g;
        fat[0] = *(const op_t *)(Ak + (size_t)min(lm, r - 1) * K);
        if (nrk > 1) fat[1] = *(const op_t *)(Ak + (size_t)min(16 + lm, r - 1) * K);
    };
    op_t fb;
    auto load_bt = [&](int s) {
        const E *bt = Bt + ((p->a.n_adapters * ld + uload(adapter + s)) * D + (fin ? fcol : 0) + lm) * r + 4 * g;
        quad_t lo = *(const quad_t *)(bt + min(0, r - 4 - 4 * g)), hi = z4;
        if (4 * g >= r) lo = z4;
        if (nrk > 1) {
            hi = *(const quad_t *)(bt + min(16, r - 4 - 4 * g));
            if (16 + 4 * g >= r) hi = z4;
        }
        fb = L::join(lo, hi);
    };
    if (s0 < s1) { load_at(s0, 0); load_bt(s0); }
    const bool first = STAGE == 2 && k.layer == 0;
    const int xblk = first && in_map ? uload(in_map + b) : b;
    const size_t step = (size_t)p->a.nb * T * D, slot = ld * p->a.nb + b;
    const float *xs = STAGE == 4 ? p->a.x1 + ld * step : first ? p->a.x_in : p->a.x2 + (ld - 1) * step;
    float *xd = STAGE == 2 ? p->a.x1 + ld * step : (int)k.layer + 1 == p->a.layers ? p->a.x : p->a.x2 + ld * step;
    const Buf xi(xs + (size_t)xblk * T * D, (unsigned)T * D * 4), xo(xd + (size_t)b * T * D, (unsigned)T * D * 4);
    const Buf src((const E *)(STAGE == 2 ? p->a.o : p->a.h) + slot * TP * K, (unsigned)TP * K * 2 * ES);
    // ---- inputs
    if (wave == 0) await(k, dep, seen, want);
    __syncthreads();
    op_t fa[NS][2];
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int m = 0; m < 2; ++m)
            fa[i][m] = L::load(src, (((k.rt * 2 + m) * ks + min(wave + 8 * i, ks - 1)) * 1024 + lane * 16) * ES);
    const unsigned xoff = ((unsigned)min(trow, T - 1) * D + (fin ? fcol : 0) + 4 * g) * 4;
    const f32x4 res = __builtin_bit_cast(f32x4, xi.ld16(xoff));
    auto shrink_part = [&](int s) {                            // (K step 0 of the term is in registers)
        f32x4 sp[2][2] = {};
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (wave + 8 * i < ks) {
                if (i) load_at(s, i);
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    sp[m][0] = L::mma(fat[0], fa[i][m], sp[m][0]);
                    if (nrk > 1) sp[m][1] = L::mma(fat[1], fa[i][m], sp[m][1]);
                }
            }
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            *(f32x4 *)(shr + (((wave * 2 + m) * 2 + 0) * 64 + lane) * 16) = sp[m][0];
            if (nrk > 1) *(f32x4 *)(shr + (((wave * 2 + m) * 2 + 1) * 64 + lane) * 16) = sp[m][1];
        }
    };
    auto shrink_sum = [&]() {
        quad_t fs[2] = {z4, z4};
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (q < nrk) {
                f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int w = 0; w < 8; ++w) {
                    const f32x4 u = *(const f32x4 *)(shr + (((min(w, np - 1) * 2 + fm) * 2 + q) * 64 + lane) * 16);
                    if (w < np) t += u;
                }
                fs[q] = L::round4(t * p->a.scale);
            }
        return L::join(fs[0], fs[1]);
    };
    op_t fs1 = {};                                             // the first term's
    if (s0 < s1) shrink_part(s0);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        if (j == 1 && s0 < s1) {                               // (the second tile takes the place of the shrink's partial sums)
            __syncthreads();
            fs1 = shrink_sum();
            __syncthreads();
        }
        f32x4 acc[2][NC] = {};
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (wave + 8 * i < ks) {
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int n = 0; n < NC; ++n) acc[m][n] = L::mma(wf[j][i][n], fa[i][m], acc[m][n]);
            }
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < NC; ++n) *(f32x4 *)(red + j * 32768 + (((wave * 2 + m) * 2 + n) * 64 + lane) * 16) = acc[m][n];
    }
    __syncthreads();
    if (tid == 0) draw(k);
    f32x4 y = {0.f, 0.f, 0.f, 0.f};
    if (fin) {
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const f32x4 t = *(const f32x4 *)(red + fj * 32768 + (((min(w, np - 1) * 2 + fm) * 2 + fn) * 64 + lane) * 16);
            if (w < np) y += t;
        }
    }
    for (int s = s0; s < s1; ++s) {
        if (SUM && s > s0) {                                   // further terms summed on this block
            load_at(s, 0); load_bt(s);
            __syncthreads();
            shrink_part(s);
            __syncthreads();
            fs1 = shrink_sum();
        } else if (NT == 1) {
            fs1 = shrink_sum();
        }
        y = L::mma(fb, fs1, y);
        if (!SUM) break;
    }
    if (fin && trow < T) xo.st16(__builtin_bit_cast(u32x4_, y + bias4 + res), xoff);
    return counter(k, (STAGE == 2 ? C_P : C_F2) + k.rt);
}

// KD: K steps of 32 in the model width.  CH: K steps at most in the hidden width
// PRE: proj is in the F1 tasks
template <typename E, int KD, int CH, int NQ, int N1, int NP, int NC, bool SUM, bool PRE>
__global__ __launch_bounds__(FL_THREADS, sizeof(E) == 2 && !PRE ? 4 : 2) void flow_kernel(const FlowParams)
{
    extern __shared__ __attribute__((aligned(16))) char fl_lds[];
    __shared__ unsigned s_ticket;
    __shared__ int s_patience;
    const int tid = threadIdx.x;
    int nb, nq;
    {
        const ParamPtr p = params();
        const int *nb_dev = p->a.nb_dev;
        nb = p->a.nb; nq = p->a.n_queues;
        if (nb_dev) nb = min(uload(nb_dev), nb);
        if (tid == 0) s_patience = p->a.patience;
    }
    if (nb <= 0) return;
    for (int qi = 0; qi < nq; ++qi) {
        const int qn = ((int)blockIdx.x + qi) % nq;
        const int nbq = nb > qn ? (nb - qn + nq - 1) / nq : 0; // blocks of this queue: qn, qn + nq, ..
        if (nbq == 0) continue;
        unsigned *qc = params()->queue + qn * 16;
        if (tid == 0) s_ticket = __hip_atomic_fetch_add(qc, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        unsigned ticket = __builtin_amdgcn_readfirstlane(s_ticket), layer = 0, lbase = 0;
        for (;;) {
            const ParamPtr p = params();
            const unsigned tpl = nbq * p->tpb;
            while (ticket >= lbase + tpl) { lbase += tpl; ++layer; }
            if (layer >= (unsigned)p->a.layers) break;
            // The model's last layer, of which the class token alone is read: behind Q the first row tile of every block
            const bool end = p->a.class_rows && layer + 1 == (unsigned)p->a.layers;
            if (end && ticket - lbase >= nbq * p->tpb_end) break;
            // ---- which task
            unsigned rem = ticket - lbase, bi;
            int stage = 0;
            const Div dQ = {p->dQ.d, p->dQ.m}, dA = {end ? p->eA.d : p->dA.d, end ? p->eA.m : p->dA.m},
                      dP = {end ? p->eP.d : p->dP.d, end ? p->eP.m : p->dP.m}, d1 = {end ? p->e1.d : p->d1.d, end ? p->e1.m : p->d1.m};
            if (rem < nbq * dQ.d) bi = div(rem, dQ), rem -= bi * dQ.d;
            else if ((rem -= nbq * dQ.d) < nbq * dA.d) stage = 1, bi = div(rem, dA), rem -= bi * dA.d;
            else if ((rem -= nbq * dA.d) < (PRE ? 0 : nbq * dP.d)) stage = 2, bi = div(rem, dP), rem -= bi * dP.d;
            else if ((rem -= (PRE ? 0 : nbq * dP.d)) < nbq * d1.d) stage = 3, bi = div(rem, d1), rem -= bi * d1.d;
            else rem -= nbq * d1.d, stage = 4, bi = div(rem, dP), rem -= bi * dP.d;
            Task k;
            unsigned next = 0;
            k.queue = qc; k.next = &next; k.patience = &s_patience;
            k.layer = layer;
            if (end && stage) k.ct = rem, k.rt = 0;
            else k.ct = div(rem, Div{p->drt.d, p->drt.m}), k.rt = rem - k.ct * p->nrt;
            k.b = qn + bi * nq;
            k.cnt = p->cnt + (size_t)k.b * p->ncnt * 16;
            unsigned *done;
            if (stage == 0) done = norm_task<E, KD, 0, NQ, SUM, false>(k, fl_lds);
            else if (stage == 1) done = attention_task<E, KD, false>(k, fl_lds);
            else if (!PRE && stage == 2) done = resid_task<E, KD, CH, 2, NP, NC, SUM>(k, fl_lds);
            else if (stage == 3) done = norm_task<E, KD, 3, N1, SUM, PRE>(k, fl_lds);
            else done = resid_task<E, KD, CH, 4, NP, NC, SUM>(k, fl_lds);
            // ---- done: every wave's stores have reached device scope, then the task is counted
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (tid == 0) s_ticket = next;
            __syncthreads();
            if (tid == 0) __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ticket = __builtin_amdgcn_readfirstlane(s_ticket);
        }
        __syncthreads();                                       // (s_ticket is written again for the next queue)
    }
    if (tid == 0 && s_patience < 0) {                          // no later launch of the call finds a block to work on, and the caller is told
        const ParamPtr p = params();
        PolyMeta *meta = p->a.meta;
        int *status = p->a.dev_status;
        meta->stalled = 1; meta->R = 0; meta->F_ok = 0; meta->status = POLY_ESTALL;
        if (status) *status = POLY_ESTALL;
    }
}

Div make_div(unsigned d) { return Div{d, d == 1 ? 0u : (unsigned)((0x100000000ull + d - 1) / d)}; }

template <typename E, int KD, int NQ, int N1, int NP, int NC, bool SUM, bool PRE> int launch_flow_t(FlowParams &p, hipStream_t st)
{
    constexpr int PER_CU = sizeof(E) == 2 && !PRE ? 2 : 1;     // (single precision: fragments of twice the registers; proj in F1: more of them)
    constexpr int ATT = 8 * 8192 + 2048, Q = norm_lds<E>(KD, NQ, false), F1 = norm_lds<E>(KD, N1, PRE);
    constexpr int LDS = ATT > Q ? (ATT > F1 ? ATT : F1) : Q > F1 ? Q : F1;                // ATT: attention's partial outputs
    static_assert(PER_CU * LDS <= 160 * 1024 - 128, "LDS budget");
    const FlowArgs &a = p.a;
    const int nrt = p.nrt;
    p.nQ = NQ;
    p.dQ = make_div(nrt * 3 * p.ct_d / NQ); p.dA = make_div(nrt * a.heads); p.dP = make_div(nrt * 4 / NC * p.ct_d / NP); p.d1 = make_div(nrt * p.ct_m / N1);
    p.drt = make_div(nrt);
    p.tpb = p.dQ.d + p.dA.d + (PRE ? 1 : 2) * p.dP.d + p.d1.d;
    p.eA = make_div(a.heads); p.eP = make_div(4 / NC * p.ct_d / NP); p.e1 = make_div(p.ct_m / N1);
    p.tpb_end = p.dQ.d + p.eA.d + (PRE ? 1 : 2) * p.eP.d + p.e1.d;
    p.a_p2 = 4 / NC * p.ct_d / NP; p.a_1 = p.ct_m / N1;
    // one workgroup per CU while that gives every block of a queue 32 of them or more, else two (DeiT-tiny, twelve layers, 256 / 512 of them:
    // 4 blocks 249 / 271 us, 8 blocks 314 / 334, 9 blocks 372 / 368, 12 blocks 426 / 408, 20 blocks 599 / 488)
    const long all = (long)p.tpb * a.nb, most = a.nb <= FL_MAXQ || PER_CU == 1 ? 256 : 512;
    auto kern = flow_kernel<E, KD, 24, NQ, N1, NP, NC, SUM, PRE>;
    static bool attr_set = false;   // raising the dynamic LDS limit is a per-kernel, process-wide setting
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS) != hipSuccess) return POLY_EHIP;
        attr_set = true;
    }
    POLY_LAUNCH_SHMEM(POLY_STAGE_GEMM, kern, dim3((unsigned)(all < most ? all : most)), dim3(FL_THREADS), LDS, st, p);
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

template <typename E, int KD, int NQ, int N1, int NP, int NC, bool PRE> int launch_flow_n(FlowParams &p, hipStream_t st)
{
    return p.a.set_off ? launch_flow_t<E, KD, NQ, N1, NP, NC, true, PRE>(p, st) : launch_flow_t<E, KD, NQ, N1, NP, NC, false, PRE>(p, st);
}

template <int KD> int launch_flow_d(FlowParams &p, int dtype, hipStream_t st)
{
    // Single precision: up to 16 tiles the products of a task are what its step waits for, and half as many columns of them a task takes (us, tasks of
    // 128 and 32 / 64 and 16 columns: 1 block of 17 tokens 72.7 / 65.3, 8 82.5 / 77.5, 16 84.1 / 81.8, 24 85.8 / 88.7; 1 of 197 (7 tiles) 81.3 / 79.3, 4 (28) 95 / 108).
    if constexpr (KD == 6) {
        if (dtype == POLY_F32) return p.a.nb * p.nrt <= 16 ? launch_flow_n<float, KD, 1, 1, 1, 1, false>(p, st) : launch_flow_n<float, KD, 1, 2, 1, 2, false>(p, st);
    }
    if (dtype == POLY_F32) return POLY_EINVAL;
    // With few row tiles the chain of a block is what counts: proj goes into the F1 tasks, a hand-over less per layer for 74 KB more of weights in each, with
    // one workgroup per CU.  From 25 tiles on coarse tasks (all three tiles of a head, four of the hidden width, two of the output) load the rows and hand over
    // once for several tiles; beyond 64 tiles proj is a step of its own again and two workgroups share a CU.
    // Twelve layers of DeiT-tiny, us, fine with proj in F1 / coarse with it / coarse: 1 block of 197 tokens 191 / 206 / 232, 3 (21 tiles) 215 / 215 / 237,
    // 4 (28) 231 / 225 / 254, 5 (35) 276 / 230 / 252, 8 (56) . / 296 / 312, 10 (70) . / 385 / 374; 6 of 113 (24) 219 / 219 / 247, 16 (64) . / 300 / 320,
    // 24 (96) . / 388 / 386; 8 of 17 182 / 203 / 228, 24 210 / 208 / 254, 36 250 / 229 / 269, 64 . / 277 / 291, 100 . / 399 / 355.
    // Where the device alone knows how many blocks fan out, five eighths of the bound are taken for there (a call has room for three adapters a frame, the
    // lagged loop for four, and uses fewer).
    const int tiles = (p.a.nb_dev && !p.a.set_off ? (5 * p.a.nb + 7) / 8 : p.a.nb) * p.nrt;
    if (p.ct_m % 4 != 0) return tiles <= 30 ? launch_flow_n<bf16_t, KD, 1, 2, 1, 2, true>(p, st) : launch_flow_n<bf16_t, KD, 1, 2, 1, 2, false>(p, st);
    if (tiles <= 24) return launch_flow_n<bf16_t, KD, 1, 2, 1, 2, true>(p, st);
    return tiles <= 64 ? launch_flow_n<bf16_t, KD, 3, 4, 2, 2, true>(p, st) : launch_flow_n<bf16_t, KD, 3, 4, 2, 2, false>(p, st);
}

}  // namespace

bool flow_supported(int T, int D, int Dm, int heads, int r, bool lora)
{
    if (!(D == 64 || D == 128 || D == 192) || Dm % 128 || Dm > 768 || D != heads * 64 || T > 224 || T <= 0) return false;
    return !lora || (r % 4 == 0 && r <= 32);
}

size_t flow_counter_bytes(int nb, int heads) { return 64 * (size_t)(FL_MAXQ + (size_t)nb * (C_Q + heads)); }
size_t flow_elements(int T, int D) { return (size_t)D * ((T + 31) / 32 * 32); }

int launch_flow(const FlowArgs &args, int dtype, hipStream_t st)
{
    if (args.nb <= 0 || args.layers <= 0) return POLY_OK;
    if (args.D > 192) return launch_flow_wide(args, FL_PATIENCE, st);
    FlowParams p;
    p.a = args;
    const int nrt = (args.T + 31) / 32;
    p.nrt = nrt; p.ct_d = args.D / 64; p.ct_m = args.Dm / 64;
    if (p.a.patience < 0) p.a.patience = FL_PATIENCE;
    p.a.n_queues = args.nb < FL_MAXQ ? args.nb : FL_MAXQ;
    p.ncnt = C_Q + args.heads;
    p.queue = args.counters;
    p.cnt = args.counters + FL_MAXQ * 16;
    switch (args.D) {
    case 64: return launch_flow_d<2>(p, dtype, st);
    case 128: return launch_flow_d<4>(p, dtype, st);
    case 192: return launch_flow_d<6>(p, dtype, st);
    default: return POLY_EINVAL;
    }
}
