// Device-side helpers shared by the libpoly kernels (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include "../../include/poly.h"
#include "../../include/poly_profile.h"
#include "gemm_tiles.h"

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));   // the caller's vectors of floats: no more than a float's alignment

#define POLY_WAVE 64

// Device-visible bookkeeping at the head of the workspace.
struct PolyMeta {
    int32_t R;       // row_offsets[F] as read on the device (0 when the inputs are rejected)
    int32_t status;  // POLY_OK, POLY_ERANGE or POLY_ESTALL
    int32_t F_ok;    // number of frames, or 0 when the inputs are rejected
    int32_t stalled; // 1 when the task queue has given up waiting in this call (flow.hip): cleared by the first launch of a forward
    int32_t pad[60];
};

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

template <typename T> __device__ __forceinline__ float to_f32(T v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v) { return (T)v; }

__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752440f)); }

// erf-GELU without transcendental instructions, for results that are rounded to bf16 afterwards:
//     GELU(x) = x * Phi(x),   Phi(x) - 1/2 = erf(x / sqrt 2) / 2 ~= xc * Q(xc^2),   xc = clamp(x, -4.4, 4.4),
// Q a degree-8 polynomial (weighted least-squares fit on Chebyshev nodes of [0, 4.4^2]).  The constant is a hair
// under 1/2 so that Phi reaches exactly 0 on the negative tail (max with 0) instead of a tiny positive slope.
// Against the double-precision definition: absolute error at most 6.3e-5 on |x| <= 8 (5e-5 on |x| <= 4, root mean square 1.9e-5 for
// normal x), relative error below 3.2e-4 wherever |GELU| > 0.05 -- a sixth of half a bf16 ulp.  14 plain fp32 instructions.
__device__ __forceinline__ float gelu_poly(float x)
{
    const float xc = __builtin_amdgcn_fmed3f(x, -4.4f, 4.4f);
    const float s = xc * xc;
    float q = fmaf(3.446953140e-11f, s, -3.649543778e-09f);
    q = fmaf(q, s, 1.703905070e-07f);
    q = fmaf(q, s, -4.655028533e-06f);
    q = fmaf(q, s, 8.353321027e-05f);
    q = fmaf(q, s, -1.050237101e-03f);
    q = fmaf(q, s, 9.626936167e-03f);
    q = fmaf(q, s, -6.605132669e-02f);
    q = fmaf(q, s, 3.987498879e-01f);
    return x * fmaxf(fmaf(xc, q, 0.499994f), 0.f);
}
// four at a time, written so that the four dependency chains advance together: one chain alone leaves the vector
// pipeline idle between dependent instructions
__device__ __forceinline__ f32x4 gelu_poly4(f32x4 x)
{
    f32x4 xc, s, q;
#pragma unroll
    for (int i = 0; i < 4; ++i) xc[i] = __builtin_amdgcn_fmed3f(x[i], -4.4f, 4.4f);
    s = xc * xc;
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = fmaf(3.446953140e-11f, s[i], -3.649543778e-09f);
    const float c[7] = {1.703905070e-07f, -4.655028533e-06f, 8.353321027e-05f, -1.050237101e-03f, 9.626936167e-03f, -6.605132669e-02f, 3.987498879e-01f};
#pragma unroll
    for (int j = 0; j < 7; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = fmaf(q[i], s[i], c[j]);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = x[i] * fmaxf(fmaf(xc[i], q[i], 0.499994f), 0.f);
    return q;
}

// The same with a polynomial of degree 9 in t = min(2 x^2 / 4.4^2 - 1, 1), whose terms do not cancel (least maximum of |x dPhi| on [0, 4.4], half
// as much weight past 3.4), and Phi cut off at 0 and 1 by the clamp of its last instruction: exact tails, no clamped copy of x.
// Absolute error at most 2.4e-5 (8.6e-6 on |x| <= 4), root mean square 2.8e-6 for normal x, relative error below 6e-5 wherever |GELU| > 0.05.  The
// table below has 1.6e-5, 1.8e-6 and 7e-5 (an interpolated one of the same size 2.7e-5, 3.9e-6, 1.4e-4): next to the bf16 rounding of the result,
// 2e-3 of it, it does not matter whether a call runs in a kernel with the table or in one with this.  14 plain fp32 instructions and no LDS.
__device__ __forceinline__ f32x4 gelu_fine4(f32x4 x)
{
    f32x4 t, q;
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = fminf(fmaf(x[i], x[i] * 1.033057868e-01f, -1.0f), 1.0f);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = fmaf(-1.346726320e-03f, t[i], 3.855216317e-03f);
    const float c[8] = {-5.589226261e-03f, 9.236665443e-03f, -1.722279564e-02f, 2.764520608e-02f,
                        -3.985336795e-02f, 5.512621254e-02f, -7.862353325e-02f, 1.604070514e-01f};
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = fmaf(q[i], t[i], c[j]);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = x[i] * __builtin_amdgcn_fmed3f(fmaf(x[i], q[i], 0.5f), 0.f, 1.f);
    return q;
}

// erf-GELU through a table of Phi in LDS, for kernels whose inner loop is bound by the number of instructions it
// issues: GELU(x) = x * Phi(x), Phi on the 1/64-wide interval around x_i = (i - 288) / 64, i = 0 .. 576, by the line whose error changes sign
// twice on it, 0 and 1 on and past the outermost ones (Phi(-4.49) = 3.6e-6).  Error <= h^2 / 16 * max|Phi''| = 3.7e-6.  Entry i holds the line as (value at 0, slope):
// 4616 bytes.  Rounding 64 x + 288 by adding 1.5 * 2^23 leaves i in the low bits of the sum, so the address is one shift-and-add of its bit
// pattern: six vector instructions per value and one 8-byte LDS read.
constexpr int GELU_TAB_ENTRIES = 577;
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f32x2 gelu_tab_entry(int i)
{
    const float x = (i - 288) * (1.0f / 64), h = 1.0f / 128;
    const float lo = 0.5f * erfcf((h - x) * 0.70710678118654752440f), hi = 0.5f * erfcf((-h - x) * 0.70710678118654752440f);
    const float slope = (hi - lo) * 64.0f, mid = 0.5f * (0.5f * erfcf(-x * 0.70710678118654752440f) + 0.5f * (lo + hi));
    if (i == 0 || i == GELU_TAB_ENTRIES - 1) return f32x2{i == 0 ? 0.f : 1.f, 0.f};
    return f32x2{fmaf(-slope, x, mid), slope};
}
// the entry of a value (tab: LDS address of the table), and the GELU of four from theirs: apart, so that other work can stand between a read and
// its use
__device__ __forceinline__ void gelu_look(float x, unsigned tab, float &xc, f32x2 &e)
{
    xc = __builtin_amdgcn_fmed3f(x, -4.5f, 4.5f);
    const unsigned u = __builtin_bit_cast(unsigned, fmaf(xc, 64.0f, 12582912.0f + 288.0f));
    e = *(const __attribute__((address_space(3))) f32x2 *)(size_t)((u << 3) + (tab - (0x4b400000u << 3)));
}
__device__ __forceinline__ f32x4 gelu_tab4(f32x4 x, const float (&xc)[4], const f32x2 (&e)[4])
{
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = x[i] * fmaf(xc[i], e[i][1], e[i][0]);
    return v;
}

// ---- launch with optional per-stage timing (profile.hip) ----
bool poly_prof_next(int stage, hipEvent_t *a, hipEvent_t *b);
int poly_patience();     // FlowArgs::patience of this thread's calls
int poly_workgroups();   // and FlowArgs::workgroups

#define POLY_LAUNCH(stage, kernel, grid, block, st, ...)                                         \
    do {                                                                                         \
        hipEvent_t ea_, eb_;                                                                     \
        if (poly_prof_next(stage, &ea_, &eb_))                                                   \
            hipExtLaunchKernelGGL(kernel, grid, block, 0, st, ea_, eb_, 0, __VA_ARGS__);         \
        else                                                                                     \
            hipLaunchKernelGGL(kernel, grid, block, 0, st, __VA_ARGS__);                         \
    } while (0)

#define POLY_LAUNCH_SHMEM(stage, kernel, grid, block, shmem, st, ...)                            \
    do {                                                                                         \
        hipEvent_t ea_, eb_;                                                                     \
        if (poly_prof_next(stage, &ea_, &eb_))                                                   \
            hipExtLaunchKernelGGL(kernel, grid, block, shmem, st, ea_, eb_, 0, __VA_ARGS__);     \
        else                                                                                     \
            hipLaunchKernelGGL(kernel, grid, block, shmem, st, __VA_ARGS__);                     \
    } while (0)

// ---- stage launchers (defined in the .hip files, used by the entry points in api.hip) ----


// C = A Wt^T with per-block structure.  Rows come in blocks of T; input block xb feeds the output
// blocks [out_off[xb], out_off[xb+1]) (or block xb itself when out_off is null).  Each output block ob
// may add its own low-rank term S[ob] Bt[adapter_of_out[ob]]^T before the epilogue.
struct GemmArgs {
    const void *A;    // elt [n_in*T][K]
    const void *Wt;   // elt [N][K]
    const float *bias;  // [N] or null
    int T, K, N;
    int n_in;             // upper bound of the number of input blocks (grid size)
    const int *n_in_dev;  // true count on the device, or null (= n_in)
    const int *out_off;   // [n_in+1] or null
    const void *S;        // elt [n_out*T][RP], zero padded to RP columns, or null
    int RP;
    const void *Bt;       // elt [n_adapters][N][r]
    int r;
    const int *adapter_of_out;  // [n_out], < 0 = no adapter
    const int *set_off;   // null: output block ob has the one low-rank term (S[ob], adapter_of_out[ob]).  Else [n_out+1]: output block
                          // ob sums the terms (S[sb], adapter_of_out[sb]) for sb in [set_off[ob], set_off[ob+1]) -- several adapters
                          // on one hidden state; S and adapter_of_out are then indexed by sb
    int mode;             // EPI_*
    void *out;            // EPI_STORE / EPI_GELU: elt [n_out*Tout][N]; EPI_RESID: float, same shape
    int Tout, t_off;      // output row of (ob, t) is ob*Tout + t_off + t
    const float *res;     // EPI_RESID: float [..*Tout][N] added (row res_block*Tout + t_off + t), or null
    const int *res_block_of_out;  // null = ob
    const float *pos;     // EPI_RESID: float [Tout][N] added (row t_off + t), or null
    float scale;          // launch_shrink_f32 only
    // set by launch_gemm only.  Tb > 0: the nb input blocks of Tb rows are tiled as ONE run of nb * Tb rows (T = nb * Tb,
    // n_in = 1; n_in_dev still counts blocks and Tout = Tb still places the output blocks), so that row tiles ignore block
    // boundaries; row t of the run belongs to input block t / Tb
    int Tb, nb;
};

// What the choice of a tile goes by beside the arguments (kept out of them: the kernels' arguments are a round trip per 64 bytes).
struct GemmCount {
    bool known;           // *n_in_dev is n_in or, where the CSR was rejected, 0
    int terms;            // (input block, adapter) pairs where rows fan out or terms are summed, about
};
int launch_gemm(const GemmArgs &g, GemmCount count, int dtype, hipStream_t st);
int launch_gemm_ks(const GemmArgs &g, int dtype, hipStream_t st);    // small calls, fp32 and any alignment (gemm_ks.hip); called by launch_gemm
bool gemm_aligned(const GemmArgs &g);                                // every address a multiple of 16
inline bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }
// the isolated linear of a small call in one launch (gemm_ks.hip): CSR check, shrink, product and expand
bool linear_ks_fits(const void *X, int F, int T, const void *W, const float *bias, int N, const void *At, const void *Bt, int r, int R, const void *Y);
int launch_linear_ks(const void *X, int F, int T, int K, const void *W, const float *bias, int N, const void *At, const void *Bt, int n_adapters,
                     int r, float scale, const int *off, const int *ids, int R, void *Y, int dtype, int *dev_status, hipStream_t st);
int launch_shrink_f32(const float *X, int T, int K, const float *At, int r, int RP, float scale, int n_out, const int *n_out_dev,
                      const int *in_block_of_out, const int *adapter_of_out, float *S, hipStream_t st);

// Row-tile linear for K <= 192 (rowlin.hip): y = [LN](x) Wt^T + b + scale ([LN](x) At_k^T) Bt_k^T with the
// LayerNorm and the low-rank shrink computed inside the kernel.
struct RowLinArgs {
    const float *x_ln;            // LayerNorm mode: fp32 rows [n_in*T][K] (null = plain mode)
    const float *ln_g, *ln_b;     // [K]
    float eps;
    const bf16_t *a_in;           // plain mode: bf16 rows [n_in*T][K]
    const int *in_block_of_out;   // null = identity
    int T, K, N;
    int n_out;                    // upper bound of the number of output blocks (grid size)
    const int *n_out_dev;         // true count on the device, or null
    const bf16_t *Wt;             // [N][K]
    const float *bias;            // [N] or null
    const bf16_t *At, *Bt;        // [n_adapters][r][K], [n_adapters][N][r]; null = no adapters
    int r;
    float scale;
    const int *adapter_of_out;
    int mode;                     // EPI_STORE / EPI_GELU: bf16 out [n_out*T][N]; EPI_RESID: fp32 out = res + y
    void *out;
    const float *res;             // EPI_RESID: fp32 [..*T][N]
    const int *res_block_of_out;  // null = ob
};
bool rowlin_supported(int K, int N, int r, bool lora, bool f32out);

// x <- x + GELU(LayerNorm(x) W1 + b1) W2 + b2 on blocks of T rows (mlp.hip); bf16 weights stored contraction-fastest
struct MlpArgs {
    float *x;                    // [n_out][T][D] fp32, updated in place
    const float *ln_g, *ln_b;    // [D]
    float eps;
    int T, D, Dm, n_out;
    const int *n_out_dev;        // optional device-side block count (the smaller of the two is used)
    const bf16_t *W1t;           // [Dm][D]
    const float *b1;             // [Dm]
    const bf16_t *W2t;           // [D][Dm]
    const float *b2;             // [D]
};
bool mlp_supported(int D, int Dm);
int launch_mlp(const MlpArgs &a, hipStream_t st);

// The row-wise part of a layer in one launch (rowlayer.hip):
//   A                       x' = res + o Wp + bp + scale (o Ap_k) Bp_k
//   B                       x_out = x' + GELU(LayerNorm2(x') W1 + b1) W2 + b2
//   C (if qkv_out != null)  qkv_out = LayerNorm1'(x_out) Wq + bq + scale (.. Aq_k) Bq_k     (the next layer's qkv)
// o == null: C alone, on res instead of x_out
// bf16 weights stored contraction-fastest, adapter stacks indexed by adapter_of_out[block]
struct RowLayerArgs {
    int T, D, Dm, n_out;
    const int *n_out_dev;            // optional device-side block count (the smaller of the two is used)
    const int *adapter_of_out;       // [n_out] or null: no adapters in this launch
    int r;
    float scale, eps;
    // A
    const bf16_t *o;                 // [n_out][T][D]
    const bf16_t *Wpt;               // [D][D]
    const float *bp;                 // [D]
    const bf16_t *Apt, *Bpt;         // [n_adapters][r][D], [n_adapters][D][r]; null = no adapters on proj
    const float *res;                // [..][T][D] fp32 residual stream going in
    const int *res_block_of_out;     // null = same block
    // B
    const float *ln2_g, *ln2_b;      // [D]
    const bf16_t *W1t;               // [Dm][D]
    const float *b1;                 // [Dm]
    const bf16_t *W2t;               // [D][Dm]
    const float *b2;                 // [D]
    float *x_out;                    // [n_out][T][D] fp32 residual stream going out (may be the same buffer as res)
    // C
    const float *lnq_g, *lnq_b;      // [D]
    const bf16_t *Wqt;               // [3 D][D]
    const float *bq;                 // [3 D]
    const bf16_t *Aqt, *Bqt;         // [n_adapters][r][D], [n_adapters][3 D][r]; null = no adapters on qkv
    bf16_t *qkv_out;                 // [n_out][T][3 D]
    int row_first;                   // set by launch_rowreg
    bool res_fragments, out_fragments;   // launch_rowreg only: res / x_out lie in its order (below); o always does there
};
bool rowlayer_supported(int D, int Dm, int r);
int launch_rowlayer(const RowLayerArgs &a, hipStream_t st);
// The same with 32 rows per wave, all of a wave's rows in its registers (rowreg.hip; row_waves.h says where).
// waves: 4, 8 or ROWREG_BOTH.  Its order, of o and where the flags say so of the residual stream, on the rows of all blocks as one run: groups of 32 rows; in a group, of a 16-bit
// value, [column / 16][column / 8 % 2][row][column % 8], of a float [column / 8][column / 4 % 2][row][column % 4].  The last group of a buffer may reach
// 31 rows past the last row.
int launch_rowreg(const RowLayerArgs &a, int waves, hipStream_t st);
int launch_rowlin(const RowLinArgs &a, hipStream_t st);

// A run of whole layers on few blocks in one launch: bf16 at 64, 128 and 192 columns and single precision at 192 (flow.hip), bf16 at 768 (flow_wide.hip).  Weight pointers are those of the first layer of the
// run, one layer of a stack behind the other.
struct FlowArgs {
    int T, D, Dm, heads, layers;
    int nb;                          // upper bound of the number of blocks
    const int *nb_dev;               // true count on the device, or null
    float eps;
    const float *x_in;               // residual stream into the first layer: block in_map[b] (null: b) of [..][T][D]
    const int *in_map;
    float *x;                        // [nb][T][D]: the residual stream after the last layer (may be x_in)
    float *x1, *x2;                  // [layers][nb][T][D]: after proj, and [layers - 1][nb][T][D]: after the layer
    const float *ln1_g, *ln1_b, *ln2_g, *ln2_b;
    const void *Wq, *Wp, *W1, *W2;   // these, the adapters and q .. h: elements of the model's type
    const float *bq, *bp, *b1, *b2;
    const void *At[4], *Bt[4];       // adapter stacks of qkv, proj, fc1, fc2; null = none
    int n_adapters, r;
    float scale;
    const int *adapter_of_row;
    const int *set_off;              // null: block b has the one term adapter_of_row[b]; else the sum of the terms [set_off[b], set_off[b + 1])
    void *qk, *vt, *o, *h;           // [layers][nb][flow_elements(T, ..)] of 2 D, D, D and Dm
    unsigned *counters;              // flow_counter_bytes, cleared by an earlier launch
    int patience;                    // looks at a counter that is not there yet, per workgroup; < 0: as many as flow.hip finds enough
    int workgroups;                  // at most so many of them in a launch of flow_wide.hip; 0: as many as there are CUs
    PolyMeta *meta;                  // a workgroup that has run out of them sets stalled, no blocks, and the status here ..
    int *dev_status;                 // .. and here (or null)
    int class_rows;                  // of the last layer's x only the first row of every block is read: the others need not be there
    int n_queues;                    // set by launch_flow
};
bool flow_supported(int T, int D, int Dm, int heads, int r, bool lora);
bool flow_wide_supported(int T, int D, int Dm, int heads, int r, bool lora);   // the same for a wide model (flow_wide.hip): bf16, one term per block
size_t flow_counter_bytes(int nb, int heads);
size_t flow_elements(int T, int D);
int launch_flow(const FlowArgs &a, int dtype, hipStream_t st);
int launch_flow_wide(const FlowArgs &a, int patience, hipStream_t st);   // called by launch_flow

// A run of whole layers of a model 192 wide on tiles of 64 or 32 rows in one launch (rowrun.hip).  Weight pointers are those of the first layer of the run, one layer of a
// stack behind the other.
struct RowRunArgs {
    int T, Dm, layers;
    int nb;                          // upper bound of the number of blocks
    const int *nb_dev;               // true count on the device, or null
    int capacity, launch;            // blocks x layers that there are buffers for (nb or more); this launch takes the launch-th so many layers, if there are any left
    int rows;                        // of a tile: 64 or 32
    int tiles;                       // set by launch_rowrun: tiles of a block
    float eps;
    const float *x_in;               // residual stream into the first layer: block in_map[b] (null: b) of [..][T][192]
    const int *in_map;
    float *x_out;                    // [nb][T][192] after the last layer (may be x_in where there is no map)
    int class_rows;                  // of x_out only the first row of every block is read: the others need not be there
    const float *ln1_g, *ln1_b, *ln2_g, *ln2_b;
    const bf16_t *Wq, *Wp, *W1, *W2;
    const float *bq, *bp, *b1, *b2;
    const bf16_t *Aq, *Bq, *Ap, *Bp; // adapter stacks of qkv and proj; null = none
    int n_adapters, r;
    float scale;
    const int *adapter_of_row;       // null: no adapters
    const int *set_off;              // null: block b has the one term adapter_of_row[b]; else (32-row tiles) the sum of the terms [set_off[b], set_off[b + 1])
    bf16_t *k, *v;                   // [capacity][rowrun_elements(T)]
    unsigned *counters;              // rowrun_counter_bytes, cleared by an earlier launch
    int patience;                    // as in FlowArgs, as are these
    int workgroups;
    PolyMeta *meta;
    int *dev_status;
};
bool rowrun_supported(int T, int D, int Dm, int heads, int r);
size_t rowrun_counter_bytes(int nb);
size_t rowrun_elements(int T);
int launch_rowrun(const RowRunArgs &a, hipStream_t st);

// y = LayerNorm(x) row-wise; x float [n*T][D] -> elt [n*T][D]
int launch_layernorm(const float *x, void *y, const float *gain, const float *shift, int D, float eps, int T,
                     int n_blocks, const int *n_blocks_dev, int dtype, hipStream_t st);

// One block.  Validates row_offsets / adapter_ids against (F, R_cap, n_adapters) and builds
// frame_of_row / adapter_of_row.  On any violation nothing downstream runs (meta->R = 0).
__device__ __forceinline__ void prep_block(const int32_t *row_offsets, const int32_t *adapter_ids, int F, int R_cap, int n_adapters,
                                           PolyMeta *meta, int32_t *frame_of_row, int32_t *adapter_of_row, int32_t *dev_status)
{
    __shared__ int bad;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    const int R = row_offsets[F];
    if (row_offsets[0] != 0 || R < 0 || R > R_cap) {
        if (threadIdx.x == 0) bad = 1;
    } else {
        for (int f = threadIdx.x; f < F; f += blockDim.x) {
            const int a = row_offsets[f], b = row_offsets[f + 1];
            if (a > b || a < 0 || b > R) { bad = 1; continue; }
            for (int i = a; i < b; ++i) {
                const int k = adapter_ids[i];
                if (k < 0 || k >= n_adapters) bad = 1;
                frame_of_row[i] = f;
                adapter_of_row[i] = k;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        meta->R = bad ? 0 : R;
        meta->F_ok = bad ? 0 : F;
        meta->status = bad ? POLY_ERANGE : POLY_OK;
        if (dev_status) *dev_status = meta->status;
    }
}
struct PrepArgs {       // the CSR check as the last block of another launch (row_offsets == nullptr: none)
    const int32_t *row_offsets, *adapter_ids;
    int F, R_cap, n_adapters;
    PolyMeta *meta;
    int32_t *frame_of_row, *adapter_of_row, *dev_status;
};

// The patch embedding in one launch with what else comes first: x[f][1 + t] = patch_t Wt^T + bias + pos[1 + t] with the patches gathered from the frames by
// the product itself, the class-token rows x[f][0] = cls + pos[0], `merged` and `zero` cleared, the CSR check and the row maps
struct PatchArgs {
    const void *frames;              // [F][H][W][3]
    int F, H, W, p;
    const float *cls, *pos;
    float *x;                        // [F][T][D]
    float *merged;
    size_t n_merged;
    unsigned *zero;
    size_t n_zero;
    PrepArgs prep;                   // row_offsets == nullptr: none
};
// Where a row of patches lies: a run of 3 p elements (a patch's part of an image row) is a whole number of 16-byte pieces
struct PatchRows {
    int p, gw, gh, run;                                    // patch, patches per row and column; pieces of a run
    unsigned magic, pitch;                                 // n / run = umulhi(n, magic) for the pieces of a patch; bytes of an image row
};
inline PatchRows patch_rows(const PatchArgs &pa, int es)
{
    const unsigned run = (unsigned)(3 * pa.p * es / 16);   // a multiple of three
    return {pa.p, pa.W / pa.p, pa.H / pa.p, (int)run, (unsigned)((0x100000000ull + run - 1) / run), (unsigned)(3 * pa.W * es)};
}
__device__ __forceinline__ unsigned patch_start(const PatchRows &pr, int row, int es)      // first byte of patch `row` of all frames
{
    const int ty = row / pr.gw;                            // (frames are whole rows of patches)
    return (unsigned)(ty * pr.p) * pr.pitch + (unsigned)(row - ty * pr.gw) * (unsigned)(3 * pr.p * es);
}
__device__ __forceinline__ unsigned patch_piece(const PatchRows &pr, unsigned n)           // byte of a patch's 16-byte piece n, from its first
{
    const unsigned dy = __umulhi(n, pr.magic);
    return dy * pr.pitch + (n - dy * pr.run) * 16u;
}
inline int patch_job_wgs(const PatchArgs &pa, int D)       // workgroups behind the product's tiles, one more where pa.prep asks for it
{
    size_t most = (size_t)pa.F * D;
    if (pa.n_merged > most) most = pa.n_merged;
    if (pa.n_zero > most) most = pa.n_zero;
    return most / 1024 + 1 < 64 ? (int)(most / 1024 + 1) : 64;
}
__device__ __forceinline__ void patch_jobs(const PatchArgs &pa, int D, int job, int job_wgs)
{
    if (job == job_wgs) {
        prep_block(pa.prep.row_offsets, pa.prep.adapter_ids, pa.prep.F, pa.prep.R_cap, pa.prep.n_adapters, pa.prep.meta, pa.prep.frame_of_row,
                   pa.prep.adapter_of_row, pa.prep.dev_status);
        return;
    }
    const size_t T = (size_t)(pa.H / pa.p) * (pa.W / pa.p) + 1, first = (size_t)job * blockDim.x + threadIdx.x, step = (size_t)job_wgs * blockDim.x;
    for (size_t i = first; i < (size_t)pa.F * D; i += step) {
        const size_t f = i / D, c = i - f * D;
        pa.x[f * T * D + c] = pa.cls[c] + pa.pos[c];
    }
    for (size_t i = first; i < pa.n_merged; i += step) pa.merged[i] = 0.f;
    for (size_t i = first; i < pa.n_zero; i += step) pa.zero[i] = 0u;
    if (first == 0 && pa.prep.meta) pa.prep.meta->stalled = 0;
}
// bf16 (patch.hip) and single precision (gemm_ks.hip); false where a kernel gathers the patches and another multiplies them
bool patch_rows_fits(const PatchArgs &pa, const void *Wt, const float *bias, int D);
int launch_patch_rows(const PatchArgs &pa, const void *Wt, const float *bias, int D, hipStream_t st);
bool patch_rows_f32_fits(const PatchArgs &pa, const void *Wt, const float *bias, int D);
int launch_patch_rows_f32(const PatchArgs &pa, const void *Wt, const float *bias, int D, hipStream_t st);

// LayerNorm + linear of few rows in one launch (norm_gemm.hip): out[row] = [GELU](LayerNorm(x[row]) Wt^T + bias), no low-rank terms
struct NormGemmArgs {
    const float *x;                  // [nb * T][D], D = 768
    const float *gain, *shift;
    float eps;
    const bf16_t *W;                 // [N][D]
    const float *bias;
    bf16_t *out;                     // [nb * T][N]
    int N, T, nb;
    const int *nb_dev;               // true count on the device, or null
    bool gelu;
};
bool norm_gemm_fits(const NormGemmArgs &a, int D);
int launch_norm_gemm(const NormGemmArgs &a, hipStream_t st);

// LayerNorm of n_blocks blocks and S = scale * y At[adapter_of_out[ob]]^T of their outputs ob (out_off: CSR offsets of every block's, null: block b itself)
// in one launch; two launches do it where that does not fit
bool layernorm_shrink_fits(const float *x, const void *y, const float *gain, const float *shift, int D, int n_blocks, const void *At, int RP, int n_out,
                           const void *S, int dtype);
int launch_layernorm_shrink(const float *x, void *y, const float *gain, const float *shift, int D, float eps, int T, int n_blocks, const int *n_blocks_dev,
                            const void *At, int r, float scale, int n_out, const int *n_out_dev, const int *out_off, const int *adapter_of_out, void *S,
                            hipStream_t st);

// S[ob] = scale * X[in_block_of_out[ob]] At[adapter_of_out[ob]]^T, zero padded to RP columns.  pair_off (nullable): CSR offsets
// [n_in + 1] of the output blocks of every input block, when the output blocks of one input block are consecutive (fan-out):
// lets one workgroup serve two of them from one read of the input rows
int launch_shrink(const void *X, int T, int K, const void *At, int r, int RP, float scale, int n_in, int n_out,
                  const int *n_out_dev, const int *in_block_of_out, const int *adapter_of_out, const int *out_off, void *S,
                  int dtype, hipStream_t st);

// the CSR check, the row maps and the shrink of an isolated bf16 linear in one launch
bool shrink_csr_fits(int F, int T, int K, int dtype);
int launch_shrink_csr(const void *X, int T, int K, const void *At, int r, int RP, float scale, const int32_t *row_offsets, const int32_t *adapter_ids,
                      int F, int R_cap, int n_adapters, PolyMeta *meta, int32_t *frame_of_row, int32_t *adapter_of_row, int32_t *dev_status, void *S,
                      hipStream_t st);

// softmax attention of every (block, head); qkv elt [n*T][3D] -> out elt [n*T][D].  n_usual: blocks that a call of n_blocks at most has as a rule (<= n_blocks);
// fragments (bf16): out in the order that launch_rowreg takes
int launch_attention(const void *qkv, void *out, int T, int D, int heads, int n_blocks, const int *n_blocks_dev, int n_usual,
                     int dtype, bool fragments, hipStream_t st);
// the same for the first query of every block alone: out elt [n][D], and x_out float [n][D], row 0 of block x_block[b] (null: b) of x [..][T][D] (fragments: in
// the order of launch_rowreg)
int launch_attention_class(const void *qkv, void *out, int T, int D, int heads, int n_blocks, const int *n_blocks_dev, const float *x, const int *x_block,
                           bool x_fragments, float *x_out, int dtype, hipStream_t st);

// poly_select with what the lagged loop needs right behind it done in the same launch (select.hip): meta != null: the row maps and
// the bookkeeping words of the CSR arrays just written (nothing is selected and state and carry stay where meta->stalled is set); carry != null: K floats carry_src -> carry
struct SelectFollow {
    PolyMeta *meta;
    int32_t *frame_of_row, *adapter_of_row, *dev_status;
    float *carry;
    const float *carry_src;
};
int launch_select(const float *label_scores, int F, int K, const uint8_t *group_membership, int M, const poly_select_opts *opts, void *state,
                  int32_t *row_offsets, int32_t *adapter_ids, int cap, int32_t *counters, const SelectFollow &fo, hipStream_t st);

// ---- bookkeeping and row-wise stages (rowops.hip) ----
int launch_prep(const int32_t *row_offsets, const int32_t *adapter_ids, int F, int R_cap, int n_adapters, PolyMeta *meta,
                int32_t *frame_of_row, int32_t *adapter_of_row, int32_t *dev_status, hipStream_t st);
// patches <- frames (im2col), x[f][0][:] <- cls + pos[0], merged[0 .. n_merged) <- 0, zero[0 .. n_zero) <- 0; and, when row_offsets is given, the work of
// launch_prep as one more block of the same launch
int launch_im2col(const void *frames, void *patches, int F, int H, int W, int p, int dtype, float *x, const float *cls, const float *pos,
                  int T_tok, int D, float *merged, size_t n_merged, unsigned *zero, size_t n_zero, const int32_t *row_offsets, const int32_t *adapter_ids, int R_cap,
                  int n_adapters, PolyMeta *meta, int32_t *frame_of_row, int32_t *adapter_of_row, int32_t *dev_status, hipStream_t st);
// base head of the lagged loop: scores of frame f -> lag[f + 1][K] and out[f][K] (nullable); lag[0] = carry (or zeros)
int launch_base_head(const float *x, int T, int D, const float *gain, const float *shift, float eps, const void *Wb, const float *bb,
                     int K, int F, float *lag, float *out, const float *carry, int dtype, hipStream_t st);
int launch_head(const float *x, const int *src_block_of_row, int T, int D, const float *gain, const float *shift, float eps,
                const void *head_w, const float *head_b, int C, const int *adapter_of_row, const int *frame_of_row,
                const int32_t *class_map, int K, const PolyMeta *meta, int R_cap, float *logits, float *scores, float *merged, int dtype,
                hipStream_t st);
