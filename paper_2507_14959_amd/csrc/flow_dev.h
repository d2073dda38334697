// What the kernels that run layers as tasks share (flow.hip, flow_wide.hip): the counters, device-scope stores, the order in which activations lie between
// the steps, attention.
#pragma once
#include "poly_dev.h"
#include "rowtile.h"

namespace {

constexpr int FL_THREADS = 512;
constexpr int FL_MAXQ = 8;             // queues
constexpr int FL_SC1 = 16;             // cache policy bit of a buffer access: device scope
constexpr int FL_PATIENCE = 1 << 20;   // counter reads of a workgroup that find its inputs not there yet, per launch
constexpr float FL_LOG2E = 1.4426950408889634f;

// counters of a block, 64 bytes apart: per row tile (8 of each) F2 done, A done, P done, F1 done, then per head Q done
enum { C_F2 = 0, C_A = 8, C_P = 16, C_F1 = 24, C_Q = 32 };

struct Div { unsigned d, m; };         // n / d, exact for n * d < 2^32
__device__ __forceinline__ unsigned div(unsigned n, Div v) { return v.d == 1 ? n : __umulhi(n, v.m); }

struct FlowParams {
    FlowArgs a;
    int nrt, ct_d, ct_m;               // row tiles per block; 64-column tiles of D and Dm
    Div dQ, dA, dP, d1, drt;           // tasks per block of every step (F2: as P); row tiles
    unsigned tpb;                      // tasks per block and layer
    Div eA, eP, e1;                    // the same on one row tile, and all of a block's in the layer whose class token alone is read
    unsigned tpb_end;
    int nQ;                            // column tiles of a Q task
    unsigned a_p2, a_1;                // tasks per row tile: P and F2; F1
    unsigned ncnt;                     // counters per block
    unsigned *queue, *cnt;
};

typedef unsigned u32x4_ __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_ __attribute__((ext_vector_type(2)));

// accesses to one block of a buffer (bounds-checked: reads past the end give 0, writes past it are dropped); stores at device scope
struct Buf {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Buf(const void *p, unsigned bytes) { r = __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, bytes, 0x00027000); }
    __device__ __forceinline__ u32x4_ ld16(unsigned off) const { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0); }
    __device__ __forceinline__ void st16(u32x4_ v, unsigned off) const { __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, FL_SC1); }
    __device__ __forceinline__ void st8(u32x2_ v, unsigned off) const { __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, FL_SC1); }
};

__device__ __forceinline__ bf16x4 pack4(f32x4 v) { return bf16x4{(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]}; }

// What the tasks do with elements of either type.  `op`: eight consecutive contraction elements of a row, a lane's share of a K step of 32: one
// 16 x 16 x 32 product in bf16, eight of 16 x 16 x 4 in single precision (both operands in the same order).  `quad`: four elements.
// over, centred, scaled: t / n, (x - mean) inv (nmi = -mean inv), (s - m) sc (off = -m sc).  In bf16 by an instruction less each, with one rounding more of what
// the row's elements share.  In single precision that rounding shows where a mean is far above its row's spread (it is 2^-24 of the mean in every element): logits of
// rows of 1027 and eighths up to 9e-3 off the short way, 4e-5 this way, which is the stream's own rounding.
struct f32x8_ { f32x4 a, b; };
template <typename E> struct El;
template <> struct El<bf16_t> {
    typedef bf16x8 op;
    typedef bf16x4 quad;
    static __device__ __forceinline__ op load(const Buf &b, unsigned off) { return __builtin_bit_cast(op, b.ld16(off)); }
    static __device__ __forceinline__ void store4(const Buf &b, f32x4 v, unsigned off) { b.st8(__builtin_bit_cast(u32x2_, pack4(v)), off); }
    static __device__ __forceinline__ quad round4(f32x4 v) { return pack4(v); }
    static __device__ __forceinline__ op join(quad lo, quad hi) { return op{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]}; }
    static __device__ __forceinline__ f32x4 mma(op u, op v, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(u, v, c, 0, 0, 0); }
    static __device__ __forceinline__ float over(float t, int n) { return t * (1.0f / n); }
    static __device__ __forceinline__ float centred(float x, float, float inv, float nmi) { return fmaf(x, inv, nmi); }
    static __device__ __forceinline__ float scaled(float s, float, float sc, float off) { return fmaf(s, sc, off); }
};
template <> struct El<float> {
    typedef f32x8_ op;
    typedef f32x4 quad;
    static __device__ __forceinline__ op load(const Buf &b, unsigned off) { return op{__builtin_bit_cast(f32x4, b.ld16(off)), __builtin_bit_cast(f32x4, b.ld16(off + 16))}; }
    static __device__ __forceinline__ void store4(const Buf &b, f32x4 v, unsigned off) { b.st16(__builtin_bit_cast(u32x4_, v), off); }
    static __device__ __forceinline__ quad round4(f32x4 v) { return v; }
    static __device__ __forceinline__ float over(float t, int n) { return t / n; }
    static __device__ __forceinline__ float centred(float x, float mean, float inv, float) { return (x - mean) * inv; }
    static __device__ __forceinline__ float scaled(float s, float m, float sc, float) { return (s - m) * sc; }
    static __device__ __forceinline__ op join(quad lo, quad hi) { return op{lo, hi}; }
    static __device__ __forceinline__ f32x4 mma(op u, op v, f32x4 c)
    {
#pragma unroll
        for (int z = 0; z < 4; ++z) c = __builtin_amdgcn_mfma_f32_16x16x4f32(u.a[z], v.a[z], c, 0, 0, 0);
#pragma unroll
        for (int z = 0; z < 4; ++z) c = __builtin_amdgcn_mfma_f32_16x16x4f32(u.b[z], v.b[z], c, 0, 0, 0);
        return c;
    }
};

// The kernel's arguments are read where they are used (a scalar load that hits the scalar cache): held in registers across the loop over
// the tasks they would be five times what fits.
typedef const __attribute__((address_space(4))) FlowParams *ParamPtr;
__device__ __forceinline__ ParamPtr params()
{
    ParamPtr p = (ParamPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// The next ticket is drawn when this task's inputs are there: the answer arrives under the work, and no workgroup sits on a second
// ticket while it waits for the inputs of its first.
struct Task {
    unsigned *queue, *next;            // ticket counter; thread 0's next ticket
    unsigned layer;
    int b, ct, rt;                     // block, 64-column tile (A: head), row tile
    unsigned *cnt;                     // the block's counters
    int *patience;                     // in LDS, wave 0's: how often the workgroup may still find a counter too low; < 0: given up
    int looks;                         // HELP: how often this task may before it is put off
    int *go;                           // HELP: in LDS, whether its inputs are there
};

__device__ __forceinline__ void draw(const Task &t) 
{
    // (an increment: an addition of a uniform value would be rewritten for a whole wave, which waits for the answer on the spot)
    *t.next = __builtin_amdgcn_atomic_inc32(t.queue, 0xffffffffu, __ATOMIC_RELAXED, "agent");
}
// a value that an earlier launch has written, at a wave-uniform address: through the scalar cache
__device__ __forceinline__ int uload(const int *q) { return *(const int __attribute__((address_space(4))) *)(uintptr_t)q; }

__device__ __forceinline__ unsigned *counter(const Task &t, int id) { return t.cnt + id * 16; }

// Inputs ready?  The counter is read once before the weights are requested (answers come in order: behind them it would take a
// microsecond longer), and again and again afterwards if it was too early.  By wave 0, for all: a barrier follows.
__device__ __forceinline__ unsigned peek(const unsigned *c) { return __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <bool HELP = false> __device__ __forceinline__ bool await(const Task &t, const unsigned *c, unsigned seen, unsigned want)
{
    int looks = HELP ? t.looks : 0;
    while (seen < want) {
        if (HELP && --looks < 0) return false;
        __builtin_amdgcn_s_sleep(1);
        const unsigned now = peek(c);                          // in flight while the look is counted
        const int left = *t.patience - 1;
        *t.patience = left;
        if (left < 0) break;
        seen = now;
    }
    return true;
}
// The same for all waves.  HELP: false if the task has to be put off
template <bool HELP> __device__ __forceinline__ bool inputs_there(const Task &t, int wave, const unsigned *c, unsigned seen, unsigned want)
{
    if (wave == 0) {
        const bool ok = await<HELP>(t, c, seen, want);
        if (HELP) *t.go = ok;
    }
    __syncthreads();
    return !HELP || __builtin_amdgcn_readfirstlane(*t.go) != 0;
}

// Fragment order of an activation matrix of ks K steps of 32 columns: [32 rows][16 rows][K step][lane][8], what a wave reads as the rows'
// operand of a 16 x 16 x 32 product with one load of 1 KB (single precision: two).  Byte offset, in bf16, of the four columns 16 c16 + 4 g .. of row 16 m + lm of row tile rt
__device__ __forceinline__ unsigned frag_off(int rt, int m, int ks, int c16, int lm, int g)
{
    return ((rt * 2 + m) * ks + (c16 >> 1)) * 1024u + (((c16 & 1) * 2 + (g >> 1)) * 16 + lm) * 16 + (g & 1) * 8;
}

// ---- attention of one head on 32 queries: wave w takes the keys 32 w ..; returns the counter to raise
// (HELP: or null if its inputs are not there for long)
template <typename E, int KD, bool HELP>
__device__ __forceinline__ unsigned *attention_task(const Task &k, char *lds)
{
    typedef El<E> L;
    typedef typename L::op op_t;
    constexpr int D = 32 * KD, ES = sizeof(E) / 2;             // ES: of offsets in bf16
    const ParamPtr p = params();
    float *op = (float *)lds;                                  // partial outputs [wave][2][4][64 lanes] x 4
    float *ml = op + 8 * 2048;                                 // [wave][32] maxima, [wave][32] sums
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lm = lane & 15, g = lane >> 4;
    const int T = p->a.T, nrt = p->nrt, TP = nrt * 32;
    if (!inputs_there<HELP>(k, wave, counter(k, C_Q + k.ct), 0, (k.layer + 1) * (3 / p->nQ) * nrt)) return nullptr;
    const size_t slot = k.layer * (size_t)p->a.nb + k.b;
    const Buf qk((const E *)p->a.qk + slot * TP * 2 * D, (unsigned)TP * 4 * D * ES), vt((const E *)p->a.vt + slot * D * TP, (unsigned)D * TP * 2 * ES);
    const unsigned hq = (unsigned)k.ct * TP * 128 * ES, hk = hq + (unsigned)D * TP * 2 * ES;   // bytes: this head's queries, keys (and values)
    if (wave < nrt) {
        op_t qf[2][2], kf[2][2], vf[4];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                qf[i][ks] = L::load(qk, hq + (((2 * k.rt + i) * 2 + ks) * 1024 + lane * 16) * ES);
                kf[i][ks] = L::load(qk, hk + (((2 * wave + i) * 2 + ks) * 1024 + lane * 16) * ES);
            }
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) vf[dt] = L::load(vt, hq + ((4 * wave + dt) * 1024 + lane * 16) * ES);
        f32x4 s[2][2];                                         // [key subtile][query subtile]: keys 16 i + 4 g + e of query lm
        const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                s[i][j] = L::mma(kf[i][0], qf[j][0], z4);
                s[i][j] = L::mma(kf[i][1], qf[j][1], s[i][j]);
            }
        const float sc = 0.125f * FL_LOG2E;
        op_t pf[2];
        float mx[2], sum[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float m = -INFINITY;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (32 * wave + 16 * i + 4 * g + e >= T) s[i][j][e] = -INFINITY;
                    m = fmaxf(m, s[i][j][e]);
                }
            m = fmaxf(m, __shfl_xor(m, 16, 64));
            m = fmaxf(fmaxf(m, __shfl_xor(m, 32, 64)), -3.4e38f);    // (the tile has a key inside T; where all its scores are -infinity its keys count nothing)
            const float off = -m * sc;
            float t = 0.f;
            f32x4 pr[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    pr[i][e] = __builtin_amdgcn_exp2f(L::scaled(s[i][j][e], m, sc, off));
                    t += pr[i][e];
                }
            pf[j] = L::join(L::round4(pr[0]), L::round4(pr[1]));
            t += __shfl_xor(t, 16, 64);
            t += __shfl_xor(t, 32, 64);
            mx[j] = m; sum[j] = t;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) {
                const f32x4 o = L::mma(vf[dt], pf[j], z4);
                *(f32x4 *)(op + ((wave * 2 + j) * 4 + dt) * 256 + lane * 4) = o;
            }
        if (g == 0) {
#pragma unroll
            for (int j = 0; j < 2; ++j) { ml[wave * 32 + 16 * j + lm] = mx[j]; ml[256 + wave * 32 + 16 * j + lm] = sum[j]; }
        }
    }
    __syncthreads();
    if (tid == 0 && (!HELP || k.queue)) draw(k);
    // wave (j, dt) brings its piece of the key tiles' partial outputs together
    const int j = wave >> 2, dt = wave & 3;
    float mw[8], M = -INFINITY, sum = 0.f;
    f32x4 ow[8], o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const int v = min(w, nrt - 1);
        mw[w] = ml[v * 32 + 16 * j + lm];
        ow[w] = *(const f32x4 *)(op + ((v * 2 + j) * 4 + dt) * 256 + lane * 4);
        M = fmaxf(M, mw[w]);
    }
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const float c = w < nrt ? __builtin_amdgcn_exp2f((mw[w] - M) * (0.125f * FL_LOG2E)) : 0.f;
        sum = fmaf(ml[256 + min(w, nrt - 1) * 32 + 16 * j + lm], c, sum);
        o += ow[w] * c;
    }
    const Buf ob((const E *)p->a.o + slot * TP * D, (unsigned)TP * D * 2 * ES);
    L::store4(ob, o * (1.0f / sum), frag_off(k.rt, j, KD, k.ct * 4 + dt, lm, g) * ES);
    return counter(k, C_A + k.rt);
}

}  // namespace
