// A stack of layers of a wide model on few token blocks in one launch: the tasks of flow.hip at 768 columns.
//
// A frame (197 rows) through the 768-wide backbone is 84 and more dependent launches of 4 to 14 us layer by layer: LayerNorm, four products on a part of the chip
// each, attention, with adapters four shrinks.  Here a layer is the five steps of flow.hip in tasks of 32 rows: Q one head's q, k and v (LayerNorm1 in it), A one head on 32 queries,
// P and F2 64 columns, F1 256 columns (LayerNorm2 in it).  Rows, weights in operand order, hand-over through device-scope stores and counters: as there.
//
// What bounds it: one frame, the chain of a block, 36 us a layer (layer by layer 52, with adapters 75) of which 5 x 1.2 are hand-overs and the rest a task's rows, partial
// sums and what of its weights is not there yet.  With more blocks the weights on their way into the registers: a load of 16 rows x 64 bytes takes
// the address unit 40 clocks (25 bytes per clock and CU, 3.4 us for 196 KB), and every 32 rows pull all 14 MB: 47 us a layer for two blocks, 57 for three,
// where larger tiles take no longer (api.hip).  The way of the operands into the XCDs would be a bound too.  A layer's weights are 14 MB, more than an L2, and come out of the Infinity Cache at
// 0.9 TB/s per XCD: with tasks drawn in any order every XCD pulls nearly all of them.  So a step's tasks, ordered by column tile and then row tile,
// are cut into eight equal runs, a queue for each XCD: an XCD pulls an eighth of the weights and all of the rows.  Six adapted layers of one frame, one of the three
// blocks that there is room for in use, 270 us: 134 MiB come from outside the L2s, of which the weights are 81 once (every XCD pulling them all: 648); the matrix unit is busy 3 %.
//
// Order and progress.  A queue's tickets are numbered layer by layer and step by step, and a task may wait for tasks of earlier steps of ANY queue.  Were all
// running workgroups those of one queue, the others' tasks would be nobody's.  A task whose inputs are not there for long is therefore put off, and its
// workgroup draws a ticket of the earliest step that any queue has left, if that is before its own, works on it, and so on until there is none; then it looks
// at its own inputs again.  At the time such a ticket is drawn no
// ticket of an earlier step is left, so all of those are in the hands of running workgroups; a workgroup works on the earliest ticket it holds; so the
// earliest unfinished ticket is always being worked on, or will be once somebody's patience with a later one has run out, and waits for nothing.
// A put-off costs FW_LOOKS of the workgroup's patience, so it must not be one per ticket of the other queues (three blocks of 197 tokens in six layers are 7500
// tickets, which a lone workgroup would give up on): what was left before its step is done when it comes back, and only tasks in others' hands put it off again.
// Two calls on one workspace at a time: as in flow.hip, the waits are bounded and the call reports POLY_ESTALL.
#include "flow_dev.h"

namespace {

constexpr int FW_LOOKS = 256;          // looks of a task at its inputs before it is put off: far more than any step takes
constexpr int FW_Q = 8;                // queues: XCDs

// The thread's number, as if new in every task: what follows from it is worked out where it is needed, not once ahead of all tasks and kept (in scratch
// memory, whose loads wait for all weights in flight)
__device__ __forceinline__ int task_tid()
{
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid;
}

// ---- LayerNorm + linear on 32 rows x NT tiles of 64 columns; STAGE: 0 Q, 3 F1.  Wave (kh, wc): half kh of the contraction for columns 16 wc .. of a
// tile.  Two tiles of weights in registers: requested before the inputs are waited for, then each K step's are replaced by those of the next two tiles
template <int KD, int STAGE, int NT>
__device__ __forceinline__ unsigned *wide_norm_task(const Task &k, char *lds)
{
    typedef El<bf16_t> L;
    constexpr int D = 32 * KD, KT = KD / 2, HK = KD / 2, NA = (KD + 3) / 4, GC = 4;       // GC: gains in flight
    static_assert(NT >= 2 && KT % GC == 0, "tiles");
    bf16_t *As = (bf16_t *)lds;                                // rows: 32 x D, chunks of eight swizzled by row
    char *red = lds + 32 * D * 2;                              // partial sums that the halves of K hand over: NT x 8 KB
    char *shr = red + NT * 8192;                               // shrink [quarter of K][row half][lane]: 8 KB
    const ParamPtr p = params();
    const int tid = task_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lm = lane & 15, g = lane >> 4;
    const int kh = wave >> 2, wc = wave & 3, T = p->a.T, t0 = k.rt * 32, b = k.b;
    const size_t ld = k.layer;
    const unsigned *dep = counter(k, (STAGE == 0 ? C_F2 : C_P) + k.rt);
    const unsigned want = (k.layer + (STAGE == 0 ? 0 : 1)) * p->a_p2;
    unsigned seen = 0;
    if (wave == 0) seen = peek(dep);
    const int N = STAGE == 0 ? 3 * D : p->a.Dm, dt = p->ct_d;
    auto tile = [&](int i) { return STAGE == 0 ? k.ct + i * dt : k.ct * NT + i; };        // q, k, v of one head, or neighbours
    const bf16_t *W = (const bf16_t *)(STAGE == 0 ? p->a.Wq : p->a.W1) + ld * N * D + (size_t)(wc * 16 + lm) * D + kh * HK * 32 + 8 * g;
    const float *bias = (STAGE == 0 ? p->a.bq : p->a.b1) + ld * N + wc * 16;
    bf16x8 wf[2][HK];
    auto load_w = [&](int i, int j) { return *(const bf16x8 *)(W + (size_t)tile(i) * 64 * D + 32 * j); };
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < HK; ++j) wf[i][j] = load_w(i, j);
    constexpr int TGT = STAGE == 0 ? 0 : 2;
    const bf16_t *At = (const bf16_t *)p->a.At[TGT], *Bt = (const bf16_t *)p->a.Bt[TGT];
    const int r = p->a.r;
    const bool lora = At != nullptr;
    const bf16x4 z4 = {0, 0, 0, 0};
    bf16x8 fat[NA];
    bf16x4 fb[NT];
    if (lora) {
        const size_t ad = p->a.n_adapters * ld + uload(p->a.adapter_of_row + b);
        const bf16_t *Ak = At + ad * r * D + 8 * g + (size_t)min(lm, r - 1) * D;
#pragma unroll
        for (int i = 0; i < NA; ++i) fat[i] = *(const bf16x8 *)(Ak + 32 * min(wc + 4 * i, KD - 1));
#pragma unroll
        for (int i = 0; i < NT; ++i) {                         // ranks 4 g .. of a column
            fb[i] = *(const bf16x4 *)(Bt + (ad * N + tile(i) * 64 + wc * 16 + lm) * r + min(4 * g, r - 4));
        }
    }
    const int row = tid >> 4, part = tid & 15, rrow = min(t0 + row, T - 1);
    const float *gain = (STAGE == 0 ? p->a.ln1_g : p->a.ln2_g) + ld * D + 4 * part, *shift = (STAGE == 0 ? p->a.ln1_b : p->a.ln2_b) + ld * D + 4 * part;
    const bool first = STAGE == 0 && k.layer == 0;             // the stream still lies where the caller put it
    const int xblk = first && p->a.in_map ? uload(p->a.in_map + b) : b;
    const size_t step = (size_t)p->a.nb * T * D;
    const float *xs = STAGE == 3 ? p->a.x1 + ld * step : first ? p->a.x_in : p->a.x2 + (ld - 1) * step;
    const Buf xb(xs + (size_t)xblk * T * D, (unsigned)T * D * 4);
    // ---- inputs
    if (!inputs_there<true>(k, wave, dep, seen, want)) return nullptr;
    {
        f32x4 v[KT], gn[GC], sh[GC];
#pragma unroll
        for (int i = 0; i < KT; ++i) v[i] = __builtin_bit_cast(f32x4, xb.ld16(((unsigned)rrow * D + 4 * (part + 16 * i)) * 4));
        auto load_gain = [&](int i) { gn[i % GC] = *(const f32x4_u *)(gain + 64 * i); sh[i % GC] = *(const f32x4_u *)(shift + 64 * i); };
#pragma unroll
        for (int i = 0; i < GC; ++i) load_gain(i);
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < KT; ++i) t += v[i][0] + v[i][1] + v[i][2] + v[i][3];
        const float mean = row16_sum(t) / D;
        float q = 0.f;
#pragma unroll
        for (int i = 0; i < KT; ++i)
#pragma unroll
            for (int z = 0; z < 4; ++z) { const float d = v[i][z] - mean; q = fmaf(d, d, q); }
        const float inv = rsqrtf(row16_sum(q) * (1.0f / D) + p->a.eps);
#pragma unroll
        for (int i = 0; i < KT; ++i) {
            f32x4 o;
#pragma unroll
            for (int z = 0; z < 4; ++z) o[z] = fmaf((v[i][z] - mean) * inv, gn[i % GC][z], sh[i % GC][z]);     // (x inv - mean inv: an instruction less, see flow_dev.h)
            if (i + GC < KT) load_gain(i + GC);
            const int c = 4 * (part + 16 * i);
            *(bf16x4 *)(As + row * D + (((c >> 3) ^ (row & 7)) << 3) + (c & 4)) = pack4(o);
        }
    }
    f32x4 bias4[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const float *bp = bias + tile(i) * 64;
        if (STAGE == 0 && i == 2) { const float bv = bp[lm]; bias4[i] = f32x4{bv, bv, bv, bv}; }
        else bias4[i] = *(const f32x4_u *)(bp + 4 * g);
    }
    __syncthreads();
    if (tid == 0 && k.queue) draw(k);
    // fragment of rows 16 m + lm, K step i: chunk 4 i + g
    auto frag_a = [&](int m, int i) { return *(const bf16x8 *)(As + (16 * m + lm) * D + (((4 * i + g) ^ (lm & 7)) << 3)); };
    if (lora) {                                                // the shrink is shared by the waves: row half kh, K steps wc, wc + 4, ..
        f32x4 sp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NA; ++i)
            if (wc + 4 * i < KD) sp = L::mma(fat[i], frag_a(kh, wc + 4 * i), sp);
        *(f32x4 *)(shr + ((wc * 2 + kh) * 64 + lane) * 16) = sp;
    }
    f32x4 y[NT];                                               // the row half that this wave finishes: 16 kh ..
#pragma unroll
    for (int i0 = 0; i0 < NT; i0 += 2) {
        f32x4 acc[2][2] = {};
        bf16x8 fr[2][2] = {{frag_a(0, kh * HK), frag_a(1, kh * HK)}};
#pragma unroll
        for (int j = 0; j < HK; ++j) {
            const bf16x8 *fa = fr[j & 1];
            if (j + 1 < HK) { fr[(j + 1) & 1][0] = frag_a(0, kh * HK + j + 1); fr[(j + 1) & 1][1] = frag_a(1, kh * HK + j + 1); }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if (i0 + i >= NT) continue;
                const bool v = STAGE == 0 && i0 + i == 2;      // V: product untransposed
#pragma unroll
                for (int m = 0; m < 2; ++m) acc[i][m] = v ? L::mma(fa[m], wf[i][j], acc[i][m]) : L::mma(wf[i][j], fa[m], acc[i][m]);
                if (i0 + 2 + i < NT) wf[i][j] = load_w(i0 + 2 + i, j);
            }
            __builtin_amdgcn_sched_barrier(0);                 // (or the requests sink to where they are needed)
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (i0 + i < NT) {
                *(f32x4 *)(red + (((i0 + i) * 8 + wave) * 64 + lane) * 16) = kh ? acc[i][0] : acc[i][1];
                y[i0 + i] = kh ? acc[i][1] : acc[i][0];
            }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const f32x4 other = *(const f32x4 *)(red + ((i * 8 + (wave ^ 4)) * 64 + lane) * 16);
        y[i] = kh ? other + y[i] : y[i] + other;
    }
    if (lora) {
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) t += *(const f32x4 *)(shr + ((w * 2 + kh) * 64 + lane) * 16);
        const bf16x8 fs = L::join(pack4(t * p->a.scale), z4);
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const bf16x8 f = L::join(4 * g < r ? fb[i] : z4, z4);
            y[i] = STAGE == 0 && i == 2 ? L::mma(fs, f, y[i]) : L::mma(f, fs, y[i]);
        }
    }
    const size_t slot = ld * p->a.nb + b;
    const int TP = p->nrt * 32;
    const Buf vt((const bf16_t *)p->a.vt + slot * D * TP, (unsigned)D * TP * 2), qk((const bf16_t *)p->a.qk + slot * TP * 2 * D, (unsigned)TP * 4 * D),
        hb((const bf16_t *)p->a.h + slot * TP * N, (unsigned)TP * N * 2);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const int ct = tile(i);
        const f32x4 v = y[i] + bias4[i];
        if (STAGE == 3) L::store4(hb, gelu_fine4(v), frag_off(k.rt, kh, N / 32, ct * 4 + wc, lm, g));
        else if (i == 2) L::store4(vt, v, (unsigned)(ct - 2 * dt) * TP * 128 + (4 * k.rt + wc) * 1024 + lane * 16 + kh * 8);
        else L::store4(qk, v, (unsigned)ct * TP * 128 + frag_off(k.rt, kh, 2, wc, lm, g));
    }
    return counter(k, STAGE == 0 ? C_Q + k.ct : C_F1 + k.rt);
}

// ---- linear + residual on 32 rows x NT tiles of 32 columns; STAGE: 2 P, 4 F2.  Wave w takes the K steps w, w + 8, .. of all of it, six (two
// tiles) or twelve steps of weights in flight, the weights' from before the inputs are waited for; the partial sums meet in LDS and waves 4 j .. finish tile j, 16 rows x 16 columns each
template <int KD, int CH, int STAGE, int NT>
__device__ __forceinline__ unsigned *wide_resid_task(const Task &k, char *lds)
{
    typedef El<bf16_t> L;
    constexpr int D = 32 * KD, KS = STAGE == 4 ? CH : KD, NS = (KS + 7) / 8, CK = NS < 6 ? NS : 6, CW = NT == 1 ? NS : CK;   // steps in flight: rows, weights
    char *red = lds, *shr = lds + 65536;                       // [tile][wave][row half][column half][lane]; [wave][row half][lane]
    const ParamPtr p = params();
    const int tid = task_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lm = lane & 15, g = lane >> 4;
    const int T = p->a.T, TP = p->nrt * 32, b = k.b;
    const size_t ld = k.layer;
    const unsigned *dep = counter(k, (STAGE == 2 ? C_A : C_F1) + k.rt);
    const unsigned want = (k.layer + 1) * (STAGE == 2 ? p->a.heads : p->a_1);
    unsigned seen = 0;
    if (wave == 0) seen = peek(dep);
    const int K = STAGE == 4 ? p->a.Dm : D, ks = K / 32, np = min(ks, 8);
    const bf16_t *W = (const bf16_t *)(STAGE == 2 ? p->a.Wp : p->a.W2) + (ld * D + k.ct * NT * 32 + lm) * K + 8 * g;
    bf16x8 wf[CW][NT][2], fa[CK][2], fat[CK];
    auto load_w = [&](int i) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int n = 0; n < 2; ++n) wf[i % CW][j][n] = *(const bf16x8 *)(W + (size_t)(j * 32 + 16 * n) * K + 32 * min(wave + 8 * i, ks - 1));
    };
#pragma unroll
    for (int i = 0; i < CW; ++i) load_w(i);
    const bool fin = wave < 4 * NT;
    const int fj = fin ? wave >> 2 : 0, fm = (wave >> 1) & 1, fn = wave & 1;   // this wave finishes rows 16 fm .., columns 16 fn .. of tile fj
    const int trow = k.rt * 32 + 16 * fm + lm, fcol = (k.ct * NT + fj) * 32 + 16 * fn;
    const f32x4 bias4 = *(const f32x4_u *)((STAGE == 2 ? p->a.bp : p->a.b2) + ld * D + fcol + 4 * g);
    constexpr int TGT = STAGE == 2 ? 1 : 3;
    const bf16_t *At = (const bf16_t *)p->a.At[TGT], *Bt = (const bf16_t *)p->a.Bt[TGT];
    const int r = p->a.r;
    const bool lora = At != nullptr;
    const bf16x4 z4 = {0, 0, 0, 0};
    const bf16_t *Ak = At;
    bf16x4 fb = z4;
    auto load_at = [&](int i) { fat[i % CK] = *(const bf16x8 *)(Ak + 32 * min(wave + 8 * i, ks - 1)); };
    if (lora) {
        const size_t ad = p->a.n_adapters * ld + uload(p->a.adapter_of_row + b);
        Ak = At + ad * r * K + (size_t)min(lm, r - 1) * K + 8 * g;
#pragma unroll
        for (int i = 0; i < CK; ++i) load_at(i);
        fb = *(const bf16x4 *)(Bt + (ad * D + fcol + lm) * r + min(4 * g, r - 4));        // ranks 4 g .. of a column
    }
    const bool first = STAGE == 2 && k.layer == 0;
    const int xblk = first && p->a.in_map ? uload(p->a.in_map + b) : b;
    const size_t step = (size_t)p->a.nb * T * D, slot = ld * p->a.nb + b;
    const float *xs = STAGE == 4 ? p->a.x1 + ld * step : first ? p->a.x_in : p->a.x2 + (ld - 1) * step;
    float *xd = STAGE == 2 ? p->a.x1 + ld * step : (int)k.layer + 1 == p->a.layers ? p->a.x : p->a.x2 + ld * step;
    const Buf xi(xs + (size_t)xblk * T * D, (unsigned)T * D * 4), xo(xd + (size_t)b * T * D, (unsigned)T * D * 4);
    const Buf src((const bf16_t *)(STAGE == 2 ? p->a.o : p->a.h) + slot * TP * K, (unsigned)TP * K * 2);
    // ---- inputs
    if (!inputs_there<true>(k, wave, dep, seen, want)) return nullptr;
    auto load_a = [&](int i) {
#pragma unroll
        for (int m = 0; m < 2; ++m) fa[i % CK][m] = L::load(src, ((k.rt * 2 + m) * ks + min(wave + 8 * i, ks - 1)) * 1024 + lane * 16);
    };
#pragma unroll
    for (int i = 0; i < CK; ++i) load_a(i);
    const unsigned xoff = ((unsigned)min(trow, T - 1) * D + fcol + 4 * g) * 4;
    const f32x4 res = __builtin_bit_cast(f32x4, xi.ld16(xoff));
    f32x4 acc[NT][2][2] = {}, sp[2] = {};
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int s = i % CK;
        if (wave + 8 * i < ks) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int n = 0; n < 2; ++n) acc[j][m][n] = L::mma(wf[i % CW][j][n], fa[s][m], acc[j][m][n]);
                if (lora) sp[m] = L::mma(fat[s], fa[s][m], sp[m]);
            }
        }
        if (i + CW < NS) load_w(i + CW);
        if (i + CK < NS) {
            load_a(i + CK);
            if (lora) load_at(i + CK);
        }
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int n = 0; n < 2; ++n) *(f32x4 *)(red + j * 32768 + (((wave * 2 + m) * 2 + n) * 64 + lane) * 16) = acc[j][m][n];
        if (lora) *(f32x4 *)(shr + ((wave * 2 + m) * 64 + lane) * 16) = sp[m];
    }
    __syncthreads();
    if (tid == 0 && k.queue) draw(k);
    f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const f32x4 t = *(const f32x4 *)(red + fj * 32768 + (((min(w, np - 1) * 2 + fm) * 2 + fn) * 64 + lane) * 16);
        if (w < np) y += t;
    }
    if (lora) {
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const f32x4 u = *(const f32x4 *)(shr + ((min(w, np - 1) * 2 + fm) * 64 + lane) * 16);
            if (w < np) t += u;
        }
        y = L::mma(L::join(4 * g < r ? fb : z4, z4), L::join(pack4(t * p->a.scale), z4), y);
    }
    if (fin && trow < T) xo.st16(__builtin_bit_cast(u32x4_, y + bias4 + res), xoff);
    return counter(k, (STAGE == 2 ? C_P : C_F2) + k.rt);
}

// n / d, the same for all lanes (the compiler divides on the vector unit, and a task that it takes for different from lane to lane has its buffers accessed
// lane by lane)
__device__ __forceinline__ unsigned udiv(unsigned n, unsigned d) { return __builtin_amdgcn_readfirstlane(n / d); }

struct Steps {
    unsigned n[5];                     // tasks of a step: row tiles times column tiles
    __device__ __forceinline__ unsigned lo(int s, unsigned q) const { return n[s] * q / FW_Q; }
    __device__ __forceinline__ unsigned len(int s, unsigned q) const { return lo(s, q + 1) - lo(s, q); }
    __device__ __forceinline__ unsigned layer(unsigned q) const { return len(0, q) + len(1, q) + len(2, q) + len(3, q) + len(4, q); }
    // layer and step of a ticket of queue q; what is left of the ticket is its place in the step's run
    __device__ __forceinline__ unsigned find(unsigned q, unsigned &ticket, int &s) const
    {
        const unsigned all = layer(q), l = udiv(ticket, all);
        ticket -= l * all;
        for (s = 0; s < 4 && ticket >= len(s, q); ++s) ticket -= len(s, q);
        return l;
    }
};

// N1: 64-column tiles of an F1 task; NP: 32-column tiles of a P or F2 task
template <int KD, int CH, int N1, int NP>
__global__ __launch_bounds__(FL_THREADS, 2) void flow_wide_kernel(const FlowParams)
{
    extern __shared__ __attribute__((aligned(16))) char fl_lds[];
    __shared__ unsigned s_ticket, s_help[2];
    __shared__ int s_patience, s_go;
    const int tid = threadIdx.x;
    unsigned tiles;                                            // row tiles of all blocks
    Steps st;
    {
        const ParamPtr p = params();
        int nb = p->a.nb;
        if (p->a.nb_dev) nb = min(uload(p->a.nb_dev), nb);
        if (tid == 0) s_patience = p->a.patience;
        if (nb <= 0) return;
        tiles = nb * p->nrt;
        // more than work on three steps only wait, and get in the others' way (12 shared layers, one tile: 444 us with 40 workgroups, 503 with 256, 537 with 24)
        if (blockIdx.x >= (3 * tiles * p->a.heads + 7) / 8 * 8) return;
        st.n[0] = st.n[1] = tiles * p->a.heads;
        st.n[2] = st.n[4] = tiles * p->a_p2;
        st.n[3] = tiles * p->a_1;
    }
    for (unsigned qi = 0; qi < FW_Q; ++qi) {
        const unsigned own = (blockIdx.x + qi) % FW_Q;
        if (tid == 0) s_ticket = __hip_atomic_fetch_add(params()->queue + own * 16, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        unsigned ticket = __builtin_amdgcn_readfirstlane(s_ticket);
        unsigned hq = FW_Q, hticket = 0, own_step = 0;         // a ticket of another queue that goes first; the step of the ticket that was put off
        auto help = [&]() {                                    // is there a ticket of a step before that one that nobody has?
            if (tid == 0) {
                const ParamPtr p = params();
                unsigned best = own_step, bt = 0, bq = FW_Q;
                for (unsigned c = 0; c < FW_Q; ++c) {
                    const unsigned t = peek(p->queue + c * 16);
                    unsigned left = t;
                    int s;
                    const unsigned l = st.find(c, left, s);
                    if (l < (unsigned)p->a.layers && l * 5 + s < best) { best = l * 5 + s; bt = t; bq = c; }
                }
                unsigned expect = bt;
                if (bq < FW_Q && !__hip_atomic_compare_exchange_strong(p->queue + bq * 16, &expect, bt + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) bq = FW_Q;
                s_help[0] = bq; s_help[1] = bt;
            }
            __syncthreads();
            hq = __builtin_amdgcn_readfirstlane(s_help[0]); hticket = __builtin_amdgcn_readfirstlane(s_help[1]);
            __syncthreads();
        };
        for (;;) {
            const ParamPtr p = params();
            const bool helping = hq < FW_Q;
            const unsigned q = helping ? hq : own;
            unsigned rem = helping ? hticket : ticket, next = 0;
            int stage;
            const unsigned layer = __builtin_amdgcn_readfirstlane(st.find(q, rem, stage));
            if (layer >= (unsigned)p->a.layers) break;         // (own queue: done)
            stage = __builtin_amdgcn_readfirstlane(stage);
            rem = __builtin_amdgcn_readfirstlane(rem + st.lo(stage, q));
            Task k;
            k.queue = helping ? nullptr : p->queue + own * 16; k.next = &next; k.patience = &s_patience; k.go = &s_go;
            k.looks = helping ? 0x7fffffff : FW_LOOKS;
            k.layer = layer;
            unsigned tile;                                     // row tile of all blocks
            if (stage == 1) {                                  // block by block and head by head: its keys and values come to one or two XCDs
                const unsigned bh = udiv(rem, p->nrt);
                k.rt = rem - bh * p->nrt; k.b = udiv(bh, p->a.heads); k.ct = bh - k.b * p->a.heads;
            } else {
                k.ct = udiv(rem, tiles); tile = rem - k.ct * tiles;
                k.b = udiv(tile, p->nrt); k.rt = tile - k.b * p->nrt;
            }
            k.cnt = p->cnt + (size_t)k.b * p->ncnt * 16;
            unsigned *done;
            if (stage == 0) done = wide_norm_task<KD, 0, 3>(k, fl_lds);
            else if (stage == 1) done = attention_task<bf16_t, KD, true>(k, fl_lds);
            else if (stage == 2) done = wide_resid_task<KD, CH, 2, NP>(k, fl_lds);
            else if (stage == 3) done = wide_norm_task<KD, 3, N1>(k, fl_lds);
            else done = wide_resid_task<KD, CH, 4, NP>(k, fl_lds);
            if (!done) {                                       // its inputs are not there for long
                own_step = layer * 5 + stage;
                help();
                continue;
            }
            // ---- done: every wave's stores have reached device scope, then the task is counted
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (tid == 0) s_ticket = next;
            __syncthreads();
            if (tid == 0) __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (helping) help();
            else ticket = __builtin_amdgcn_readfirstlane(s_ticket);
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

}  // namespace

// (queues need at least a task each in every layer: heads = 12)
bool flow_wide_supported(int T, int D, int Dm, int heads, int r, bool lora)
{
    if (D != 768 || Dm % 256 || Dm > 3072 || Dm <= 0 || D != heads * 64 || T > 224 || T <= 0) return false;
    return !lora || (r % 4 == 0 && r <= 16);
}

template <int N1, int NP> static int launch_wide_t(const FlowArgs &args, int patience, hipStream_t st)
{
    constexpr int KD = 24, CH = 96, LDS = 32 * 32 * KD * 2 + 4 * 8192 + 8192;
    static_assert(LDS >= 65536 + 16384 && LDS >= 8 * 8192 + 2048, "partial sums and shrink of a residual task; attention's partial outputs");
    FlowParams p = {};
    p.a = args;
    p.nrt = (args.T + 31) / 32; p.ct_d = args.D / 64; p.ct_m = args.Dm / 64;
    p.nQ = 3; p.a_p2 = 2 * p.ct_d / NP; p.a_1 = p.ct_m / N1;
    if (p.a.patience < 0) p.a.patience = patience;
    p.ncnt = C_Q + args.heads;
    p.queue = args.counters;
    p.cnt = args.counters + FL_MAXQ * 16;
    auto kern = flow_wide_kernel<KD, CH, N1, NP>;
    static bool attr_set = false;   // raising the dynamic LDS limit is a per-kernel, process-wide setting
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS) != hipSuccess) return POLY_EHIP;
        attr_set = true;
    }
    POLY_LAUNCH_SHMEM(POLY_STAGE_GEMM, kern, dim3(args.workgroups > 0 && args.workgroups < 256 ? args.workgroups : 256), dim3(FL_THREADS), LDS, st, p);
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

// Up to 10 row tiles P and F2 tasks of 32 columns leave no CU idle that 64 would keep busy, and hold all their weights before their inputs are there (12 layers
// of 7 tiles 433 / 493 us with tasks of 32 / 64 columns, 14 tiles 594 / 565).
int launch_flow_wide(const FlowArgs &args, int patience, hipStream_t st)
{
    return args.nb * ((args.T + 31) / 32) <= 10 ? launch_wide_t<4, 1>(args, patience, st) : launch_wide_t<4, 2>(args, patience, st);
}
