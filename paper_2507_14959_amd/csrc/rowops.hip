// Row-wise and bookkeeping kernels of the forward: CSR validation, patch gathering, LayerNorm,
// LoRA shrink (x A_k), per-adapter heads with sigmoid, and the optional merge to label space.
#include "rowtile.h"

#include <type_traits>

namespace {

// ------------------------------------------------------------------ CSR check + row maps
__global__ void prep_kernel(const int32_t *row_offsets, const int32_t *adapter_ids, int F, int R_cap, int n_adapters,
                            PolyMeta *meta, int32_t *frame_of_row, int32_t *adapter_of_row, int32_t *dev_status)
{
    prep_block(row_offsets, adapter_ids, F, R_cap, n_adapters, meta, frame_of_row, adapter_of_row, dev_status);
}

// ------------------------------------------------------------------ patch gathering
// patches[(f*P + ty*gw + tx)][(i*p + j)*3 + c] = frame[f][ty*p + i][tx*p + j][c]; a run of 3p values
// (fixed i) is contiguous in the NHWC frame.
// VEC elements (16 bytes) per thread when the run length allows it.  The same launch also writes the class-token
// rows x[f][0][:] = cls + pos[0] and clears the merged-score buffer (both are needed much later: two launches less).
template <typename T, int VEC>
__global__ void im2col_kernel(const T *frames, T *patches, int F, int H, int W, int p, float *x, const float *cls, const float *pos,
                              int T_tok, int D, float *merged, size_t n_merged, unsigned *zero, size_t n_zero, const PrepArgs pa)
{
    const int nblk = pa.row_offsets ? gridDim.x - 1 : gridDim.x;   // the last block checks the CSR arrays (one launch less)
    if ((int)blockIdx.x == nblk) {
        prep_block(pa.row_offsets, pa.adapter_ids, pa.F, pa.R_cap, pa.n_adapters, pa.meta, pa.frame_of_row, pa.adapter_of_row, pa.dev_status);
        return;
    }
    const int gw = W / p, gh = H / p, run = 3 * p / VEC;         // vectors per contiguous run
    const size_t total = (size_t)F * gh * gw * p * run;
    const size_t gtid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, gsz = (size_t)nblk * blockDim.x;
    typedef T vec_t __attribute__((ext_vector_type(VEC)));
    for (size_t idx = gtid; idx < total; idx += gsz) {
        size_t q = idx;
        const int e = q % run; q /= run;
        const int i = q % p; q /= p;
        const int tx = q % gw; q /= gw;
        const int ty = q % gh; const size_t f = q / gh;
        const T *src = frames + ((f * H + (size_t)ty * p + i) * W + (size_t)tx * p) * 3 + (size_t)e * VEC;
        if (VEC == 1) patches[idx] = *src;
        else *(vec_t *)(patches + idx * VEC) = *(const vec_t *)src;
    }
    for (size_t idx = gtid; idx < (size_t)F * D; idx += gsz) {
        const size_t f = idx / D; const int c = idx % D;
        x[f * T_tok * D + c] = cls[c] + pos[c];
    }
    for (size_t idx = gtid; idx < n_merged; idx += gsz) merged[idx] = 0.f;
    for (size_t idx = gtid; idx < n_zero; idx += gsz) zero[idx] = 0u;
    if (gtid == 0 && pa.meta) pa.meta->stalled = 0;
}

// ------------------------------------------------------------------ LayerNorm
// One wave per row; fp32 statistics (mean, then centred second moment), output in the activation type.
template <typename T>
__global__ __launch_bounds__(256) void layernorm_kernel(const float *x, T *y, const float *gain, const float *shift, int D,
                                                        float eps, int rows_per_block, int n_blocks, const int *n_blocks_dev)
{
    const int nb = n_blocks_dev ? min(*n_blocks_dev, n_blocks) : n_blocks;
    const size_t rows = (size_t)nb * rows_per_block;
    const size_t row = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int lane = threadIdx.x & 63;
    const float *xr = x + row * D;
    float s = 0.f;
    for (int k = lane; k < D; k += 64) s += xr[k];
    const float mean = wave_sum(s) / D;
    float v = 0.f;
    for (int k = lane; k < D; k += 64) { const float d = xr[k] - mean; v += d * d; }
    const float inv = rsqrtf(wave_sum(v) / D + eps);
    T *yr = y + row * D;
    for (int k = lane; k < D; k += 64) yr[k] = from_f32<T>((xr[k] - mean) * inv * gain[k] + shift[k]);
}

// D = 256 NV: the row stays in registers (NV 16-byte pieces per lane), read once and written in 8- or 16-byte pieces
template <typename T, int NV>
__global__ __launch_bounds__(256) void layernorm_vec_kernel(const float *x, T *y, const float *gain, const float *shift, float eps,
                                                            int rows_per_block, int n_blocks, const int *n_blocks_dev)
{
    constexpr int D = 256 * NV;
    const int lane = threadIdx.x & 63;
    const size_t row = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const size_t rows_cap = (size_t)n_blocks * rows_per_block;
    const float *xr = x + (row < rows_cap ? row : rows_cap - 1) * D + 4 * lane;     // requested before the row count is known
    f32x4 v[NV], g[NV], b[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = *(const f32x4 *)(xr + 256 * i);
#pragma unroll
    for (int i = 0; i < NV; ++i) { g[i] = *(const f32x4 *)(gain + 4 * lane + 256 * i); b[i] = *(const f32x4 *)(shift + 4 * lane + 256 * i); }
    const int nb = n_blocks_dev ? min(*n_blocks_dev, n_blocks) : n_blocks;
    if (row >= (size_t)nb * rows_per_block) return;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) s += v[i][0] + v[i][1] + v[i][2] + v[i][3];
    const float mean = wave_sum(s) / D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int z = 0; z < 4; ++z) { const float d = v[i][z] - mean; q += d * d; }
    const float inv = rsqrtf(wave_sum(q) / D + eps);
    T *yr = y + row * D + 4 * lane;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        typedef T out4 __attribute__((ext_vector_type(4)));
        out4 o;
#pragma unroll
        for (int z = 0; z < 4; ++z) o[z] = from_f32<T>((v[i][z] - mean) * inv * g[i][z] + b[i][z]);
        *(out4 *)(yr + 256 * i) = o;
    }
}

// LayerNorm of 16 rows and their shrink with the adapters of the block's outputs (ranks up to 16) in one launch: the normalised rows, rounded to bf16, are
// stored for the product and shrunk out of LDS.  Launches of their own read them back, 10 us of 35 MB for 115 blocks of ViT-base, or pay for a launch, 5 us.
// Bound by the bytes, 120 MB in and 60 out at 768 columns and 40000 rows: many workgroups per CU (32 KB of LDS, five), a wave's four rows requested at once.
// Wave w shrinks with quarter w of the columns, the partial sums meet in LDS.
template <int NV>
__global__ __launch_bounds__(256) void layernorm_shrink_kernel(const float *x, bf16_t *y, const float *gain, const float *shift, float eps, int T, int subs,
                                                               int n_blocks, const int *n_blocks_dev, const bf16_t *At, int r, float scale, const int *out_off,
                                                               const int *n_out_dev, int n_out, const int *adapter_of_out, bf16_t *S)
{
    constexpr int D = 256 * NV, NS = 2 * NV;                   // K steps of a wave
    __shared__ __attribute__((aligned(16))) bf16_t rows_s[16 * D];
    __shared__ __attribute__((aligned(16))) float red[2][4][256];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lm = lane & 15, g4 = lane >> 4;
    const int blk = blockIdx.x / subs, t0 = (blockIdx.x - blk * subs) * 16;
    f32x4 v[4][NV], g[NV], b[NV];
#pragma unroll
    for (int q = 0; q < 4; ++q)                                // (requested before the counts are known)
#pragma unroll
        for (int i = 0; i < NV; ++i) v[q][i] = *(const f32x4 *)(x + ((size_t)blk * T + min(t0 + 4 * wave + q, T - 1)) * D + 4 * lane + 256 * i);
#pragma unroll
    for (int i = 0; i < NV; ++i) { g[i] = *(const f32x4 *)(gain + 4 * lane + 256 * i); b[i] = *(const f32x4 *)(shift + 4 * lane + 256 * i); }
    const int nb = n_blocks_dev ? min(*n_blocks_dev, n_blocks) : n_blocks, R = min(*n_out_dev, n_out);     // (0 outputs if the CSR arrays are rejected)
    if (blk >= nb) return;
    const int o0 = out_off ? max(out_off[blk], 0) : blk, o1 = min(out_off ? out_off[blk + 1] : blk + 1, R);
    bf16x8 at[NS];
    auto load_at = [&](int ob) {
        const int k = adapter_of_out[ob];
        const bf16_t *p = At + ((size_t)max(k, 0) * r + min(lm, r - 1)) * D + wave * (D / 4) + 8 * g4;
#pragma unroll
        for (int j = 0; j < NS; ++j) at[j] = *(const bf16x8 *)(p + 32 * j);
        return k;
    };
    int k = o0 < o1 ? load_at(o0) : -1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) s += v[q][i][0] + v[q][i][1] + v[q][i][2] + v[q][i][3];
        const float mean = wave_sum(s) / D;
        float p = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int z = 0; z < 4; ++z) { const float d = v[q][i][z] - mean; p += d * d; }
        const float inv = rsqrtf(wave_sum(p) / D + eps);
        const int row = 4 * wave + q;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            bf16x4 o;
#pragma unroll
            for (int z = 0; z < 4; ++z) o[z] = (bf16_t)((v[q][i][z] - mean) * inv * g[i][z] + b[i][z]);
            if (t0 + row < T) *(bf16x4 *)(y + ((size_t)blk * T + t0 + row) * D + 4 * lane + 256 * i) = o;
            *(bf16x4 *)(rows_s + row * D + ((((lane >> 1) + 32 * i) ^ (row & 7)) << 3) + 4 * (lane & 1)) = o;
        }
    }
    __syncthreads();
    for (int ob = o0; ob < o1; ++ob) {
        f32x4 sp = {0.f, 0.f, 0.f, 0.f};                       // ranks 4 g4 .. of row lm
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const int chunk = wave * (D / 32) + 4 * j + g4;
            sp = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at[j], *(const bf16x8 *)(rows_s + lm * D + ((chunk ^ (lm & 7)) << 3)), sp, 0, 0, 0);
        }
        float (*part)[256] = red[(ob - o0) & 1];
        *(f32x4 *)(part[wave] + 4 * lane) = sp;
        const int k_now = k;
        if (ob + 1 < o1) k = load_at(ob + 1);
        __syncthreads();
        if (wave == ((ob - o0) & 3) && k_now >= 0 && t0 + lm < T) {
            f32x4 s = *(const f32x4 *)(part[0] + 4 * lane);
#pragma unroll
            for (int w = 1; w < 4; ++w) s += *(const f32x4 *)(part[w] + 4 * lane);
            bf16x4 o;
#pragma unroll
            for (int z = 0; z < 4; ++z) o[z] = (bf16_t)(4 * g4 + z < r ? scale * s[z] : 0.f);
            *(bf16x4 *)(S + ((size_t)ob * T + t0 + lm) * 16 + 4 * g4) = o;
        }
    }
}

// ------------------------------------------------------------------ LoRA shrink
// bf16: S = scale * X At_k^T (zero padded to RP columns) with v_mfma_f32_16x16x32_bf16, operands read straight from
// global memory: a lane's 16 bytes are 8 consecutive K elements of one row, four lanes cover 64 contiguous bytes.
//
// The kernel moves few bytes per workgroup, so its time is the length of a workgroup's chain of dependent memory
// round trips and the number of workgroups in flight, not arithmetic.  Hence:
//  - a workgroup covers only 16 * MS = 32 rows of one output block (many workgroups per CU; more rows per workgroup
//    would re-read At_k less often but measured slower) and its four waves split K; the partial sums meet in LDS,
//    where every wave finishes a quarter of the values;
//  - everything that needs only the block index is requested in one go (true count, input block, adapter ids), then
//    -- when output blocks are paired -- the fan-out offsets, then At_k and the rows of a whole batch of K steps at
//    once; the rows of subtile m + 1 are requested before the MFMAs of subtile m.  Rows past T and ranks past r are
//    clamped, not predicated: they feed results that are dropped or zeroed at the store.
// A 16-column MFMA tile is one "group": NG = 2 groups are the two rank halves of an adapter of rank 17-32 or, with
// ranks of at most 16, two adapters: where consecutive output blocks read the same input block (the fan-out of a
// frame into its row-blocks; pair_off = the CSR offsets of the input blocks) the workgroup of the even one does
// both and the input rows are read once instead of twice.
constexpr int SH_NS = 6;    // 32-element K steps whose operands are in flight together
constexpr int SH_CSR_MAX = 1024;   // input blocks at most where the kernel reads the CSR arrays itself

// What a workgroup of output block ob works on: input block xb, adapter k_ad, and the output block ob2 (adapter k_ad2, -1: none) that it does
// along with its own.  False: nothing to do (past the true count, no adapter, done by the workgroup of ob - 1, arrays that the check rejects).
template <bool CSR>
__device__ __forceinline__ bool shrink_blocks(int ob, bool paired, int n_out, const int *n_out_dev, const int *in_block_of_out,
                                              const int *adapter_of_out, const int *pair_off, const PrepArgs &pa, int &xb, int &k_ad,
                                              int &k_ad2, int &ob2)
{
    ob2 = -1;
    if constexpr (CSR) {
        __shared__ int offs[SH_CSR_MAX + 1];
        for (int f = threadIdx.x; f <= pa.F; f += 256) offs[f] = pa.row_offsets[f];
        __syncthreads();
        const int R = offs[pa.F];
        if (offs[0] != 0 || R < 0 || R > pa.R_cap || ob >= R) return false;    // (rejected, or past the true count)
        k_ad = pa.adapter_ids[ob];
        k_ad2 = pa.adapter_ids[min(ob + 1, R - 1)];
        int before = 0;                                          // input blocks whose rows all lie before output block ob
        for (int f = threadIdx.x & 63; f < ((pa.F + 63) & ~63); f += 64) before += __popcll(__ballot(f < pa.F && offs[f + 1] <= ob));
        xb = min(before, pa.F - 1);
        if (paired) {
            const int p0 = offs[xb], p1 = offs[xb + 1];
            if ((ob - p0) & 1) return false;                     // done by the workgroup of ob - 1
            if (ob + 1 < min(p1, R)) ob2 = ob + 1;
        }
        if ((unsigned)k_ad >= (unsigned)pa.n_adapters || (ob2 >= 0 && (unsigned)k_ad2 >= (unsigned)pa.n_adapters)) return false;   // (rejected)
        if (ob2 < 0) k_ad2 = -1;
    } else {
        // first round trip: four loads with unconditional addresses, so that they are requested together.  The arrays have
        // n_out entries; those past the true count are read here but never used.
        // (volatile: the compiler would otherwise sink each load below the early exit that precedes its first use)
        const int *pn = n_out_dev ? n_out_dev : adapter_of_out, *pi = in_block_of_out ? in_block_of_out + ob : adapter_of_out + ob;
        const int n_ld = *(const volatile int *)pn, xb_ld = *(const volatile int *)pi;
        const int k1_raw = *(const volatile int *)(adapter_of_out + ob), k2_raw = *(const volatile int *)(adapter_of_out + min(ob + 1, n_out - 1));
        const int n = n_out_dev ? min(n_ld, n_out) : n_out;
        xb = in_block_of_out ? xb_ld : ob;
        if (ob >= n) return false;
        if (paired) {                                                // second round trip
            const int p0 = *(const volatile int *)(pair_off + xb), p1 = *(const volatile int *)(pair_off + xb + 1);
            if ((ob - p0) & 1) return false;                         // done by the workgroup of ob - 1
            if (ob + 1 < min(p1, n)) ob2 = ob + 1;
        }
        k_ad = k1_raw;
        k_ad2 = ob2 >= 0 ? k2_raw : -1;
        if (k_ad < 0 && k_ad2 < 0) return false;
    }
    return true;
}

template <int MS, int NG, bool CSR>
__global__ __launch_bounds__(256) void shrink_bf16_kernel(const bf16_t *X, int T, int K, const bf16_t *At, int r, int RP,
                                                          float scale, int n_out, const int *n_out_dev,
                                                          const int *in_block_of_out, const int *adapter_of_out, const int *pair_off,
                                                          bf16_t *S, const PrepArgs pa)
{
    constexpr int NV = MS * NG * 4;                              // values per lane and wave
    constexpr int RV = NV < 32 ? NV : 32;                        // values per reduction round
    static_assert(RV % 4 == 0, "reduction rounds");
    __shared__ float red[4][RV][64];
    const int subs = (T + 16 * MS - 1) / (16 * MS);
    // CSR: no launch before this one has built the row maps.  The last workgroup checks the arrays and builds them for the product;
    // the others look their output block up in the offsets themselves (one launch less: 3.5 of the 15.6 us of a call on 9 blocks)
    if (CSR && blockIdx.x == gridDim.x - 1) {
        prep_block(pa.row_offsets, pa.adapter_ids, pa.F, pa.R_cap, pa.n_adapters, pa.meta, pa.frame_of_row, pa.adapter_of_row, pa.dev_status);
        return;
    }
    const int ob = blockIdx.x / subs, row0 = (blockIdx.x % subs) * (16 * MS);
    const bool paired = NG == 2 && RP == 16 && (CSR || (pair_off && in_block_of_out));
    int xb, k_ad, k_ad2, ob2;
    if (!shrink_blocks<CSR>(ob, paired, n_out, n_out_dev, in_block_of_out, adapter_of_out, pair_off, pa, xb, k_ad, k_ad2, ob2)) return;
    const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 15, lc = lane >> 4;
    const bf16_t *xblk = X + (size_t)xb * T * K + lc * 8;
    int xoff[MS];                                                // row li of subtile m (the host has checked T * K < 2^31)
#pragma unroll
    for (int m = 0; m < MS; ++m) xoff[m] = min(row0 + 16 * m + li, T - 1) * K;
    const bf16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
    const int steps = K >> 5, per = (steps + 3) / 4;             // full steps; what is left of K (8, 16 or 24) goes to wave 3
    const int s0 = min(q * per, steps), s1 = min(steps, s0 + per);
    for (int j0 = 0; j0 < (paired ? 16 : RP); j0 += 16 * NG) {
        // group g, lane column li: rank `rank` of adapter `ksel`, stored to column `rank` of output block `osel`
        int ksel[NG], osel[NG], rank[NG];
        const bf16_t *ar[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const bool other = paired && g == 1;
            ksel[g] = other ? k_ad2 : k_ad;
            osel[g] = other ? ob2 : ob;
            rank[g] = paired ? li : j0 + 16 * g + li;
            ar[g] = At + ((size_t)max(ksel[g], 0) * r + min(rank[g], r - 1)) * K + lc * 8;
        }
        f32x4 acc[MS][NG];
#pragma unroll
        for (int m = 0; m < MS; ++m)
#pragma unroll
            for (int g = 0; g < NG; ++g) acc[m][g] = f32x4{0.f, 0.f, 0.f, 0.f};
        // NB steps from step st on
        auto batch = [&](auto nb, int st) {
            constexpr int NB = decltype(nb)::value;
            bf16x8 fb[NG][NB], fa[2][NB];
#pragma unroll
            for (int u = 0; u < NB; ++u)
#pragma unroll
                for (int g = 0; g < NG; ++g) fb[g][u] = *(const bf16x8 *)(ar[g] + (st + u) * 32);
#pragma unroll
            for (int u = 0; u < NB; ++u) fa[0][u] = *(const bf16x8 *)(xblk + xoff[0] + (st + u) * 32);
#pragma unroll
            for (int m = 0; m < MS; ++m) {
                if (m + 1 < MS) {
#pragma unroll
                    for (int u = 0; u < NB; ++u) fa[(m + 1) & 1][u] = *(const bf16x8 *)(xblk + xoff[m + 1] + (st + u) * 32);
                }
                __builtin_amdgcn_sched_barrier(0);               // the next rows are requested before these MFMAs wait
#pragma unroll
                for (int u = 0; u < NB; ++u)
#pragma unroll
                    for (int g = 0; g < NG; ++g)
                        acc[m][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[m & 1][u], fb[g][u], acc[m][g], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int st = s0;                                             // (the counts are the same for the whole wave: scalar branches)
        for (; st + SH_NS <= s1; st += SH_NS) batch(std::integral_constant<int, SH_NS>(), st);
        for (; st + 2 <= s1; st += 2) batch(std::integral_constant<int, 2>(), st);
        for (; st < s1; ++st) batch(std::integral_constant<int, 1>(), st);
        if ((K & 31) && q == 3) {                                // the rest of K: chunks past the end of the row are zero
            const bool in = steps * 32 + lc * 8 + 8 <= K;
            bf16x8 fb[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) fb[g] = in ? *(const bf16x8 *)(ar[g] + steps * 32) : zero8;
#pragma unroll
            for (int m = 0; m < MS; ++m) {
                const bf16x8 fa = in ? *(const bf16x8 *)(xblk + xoff[m] + steps * 32) : zero8;
#pragma unroll
                for (int g = 0; g < NG; ++g) acc[m][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb[g], acc[m][g], 0, 0, 0);
            }
        }
        // value v = (m * NG + g) * 4 + e of a lane: row row0 + 16 m + 4 lc + e, column li of group g.  RV values per round;
        // wave q finishes values [q RV / 4, (q + 1) RV / 4) of the round.
#pragma unroll
        for (int v0 = 0; v0 < NV; v0 += RV) {
            if (v0 || j0) __syncthreads();
#pragma unroll
            for (int v = 0; v < RV; ++v)
                if (v0 + v < NV) red[q][v][lane] = acc[(v0 + v) / (NG * 4)][((v0 + v) / 4) % NG][(v0 + v) & 3];
            __syncthreads();
#pragma unroll
            for (int w = 0; w < RV / 4; ++w) {
                const int vr = q * (RV / 4) + w, v = v0 + vr;    // (q is scalar: the three selections below are uniform)
                const int m = v / (NG * 4), g = (v / 4) % NG, e = v & 3;
                const float sum = red[0][vr][lane] + red[1][vr][lane] + red[2][vr][lane] + red[3][vr][lane];
                const int tt = row0 + 16 * m + 4 * lc + e;
                int ks = ksel[0], os = osel[0], rk = rank[0];
#pragma unroll
                for (int gg = 1; gg < NG; ++gg)
                    if (g == gg) { ks = ksel[gg]; os = osel[gg]; rk = rank[gg]; }
                if (v < NV && tt < T && ks >= 0 && os >= 0 && rk < RP)
                    S[((size_t)os * T + tt) * RP + rk] = rk < r ? (bf16_t)(scale * sum) : (bf16_t)0.f;
            }
        }
    }
}

// The same product with the rows streamed through LDS and a workgroup that stays with them (K a multiple of 128 or 192).
// A wave owns a ring of items of 16 rows x 32 CS columns (global_load_lds_dwordx4, contiguous runs of 64 CS bytes; the other slots are on
// their way while one is read) and needs no barrier for it.  Per chunk of 32 CS columns it holds the At rows of its one or two groups
// as fragments and passes over up to SH_MS subtiles of X, so an adapter's At is read once per 16 SH_MS rows.  The four waves are WK
// parts of K times 4 / WK runs of subtiles (WK = 4, 2 or 1, the largest that divides the chunks of K); partial sums meet in LDS once, at the end.
// The product is transposed (At is the A operand): a lane ends up with four consecutive ranks of one row and stores them in one piece.
// Where output blocks fan out of input blocks (MODE 1: row maps made before; 2: the CSR arrays themselves, checked by the last workgroup) the
// grid runs over the input blocks and `units` shares of their branches: the rows are requested before anything else is known.
template <int CS> constexpr int sh_ring() { return CS == 6 ? 3 : 4; }
constexpr int SH_MS = 7;

template <int CS, int MODE>
__global__ __launch_bounds__(256, 2) void shrink_stream_kernel(const bf16_t *X, int T, int K, const bf16_t *At, int r, int RP, float scale, int n_out,
                                                               const int *n_out_dev, const int *in_block_of_out, const int *adapter_of_out,
                                                               const int *out_off, bf16_t *S, int wk_log, int parts, int wgs, int units, const PrepArgs pa)
{
    constexpr int ROW = 64 * CS, ITEM = 16 * ROW, RING = sh_ring<CS>();      // bytes, bytes, items
    __shared__ __attribute__((aligned(16))) char ring[4][RING * ITEM];
    static_assert(SH_MS * 2 * 1024 <= RING * ITEM, "a wave's partial sums fit its ring");
    if (MODE == 2 && blockIdx.x == gridDim.x - 1) {
        prep_block(pa.row_offsets, pa.adapter_ids, pa.F, pa.R_cap, pa.n_adapters, pa.meta, pa.frame_of_row, pa.adapter_of_row, pa.dev_status);
        return;
    }
    const int b = MODE == 0 ? blockIdx.x / wgs : blockIdx.x / (wgs * units);          // output block (MODE 0) or input block
    const int unit = MODE == 0 ? 0 : blockIdx.x / wgs % units;                      // of the branches, pair by pair (RP = 16) or one by one
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 15, lc = lane >> 4;
    const int wk = wave & ((1 << wk_log) - 1), wr = wave >> wk_log;
    // subtiles of 16 rows, cut into `parts` runs that differ by one at most (wgs workgroups of 4 / WK runs each)
    const int nt = (T + 15) >> 4, part = (blockIdx.x % wgs) * (4 >> wk_log) + wr;
    const int m0 = part < parts ? (int)((long)nt * part / parts) : nt, ms = part < parts ? (int)((long)nt * (part + 1) / parts) - m0 : 0;
    const int chunks = (K / (32 * CS)) >> wk_log;                // of this wave
    // item layout: 16-byte piece c of row i at position c ^ f(i) of the row, where the 16 lanes of a fragment read (one piece of 16 rows) then
    // lie in 16 different groups of four banks; the lane that fills a position fetches the piece that belongs there
    auto swz = [](int i) { return CS == 6 ? (i >> 1) & 7 : i & 15; };
    int d_row[CS], d_col[CS];
#pragma unroll
    for (int i = 0; i < CS; ++i) {
        const int p = 64 * i + lane;
        d_row[i] = p / (4 * CS);
        d_col[i] = ((p % (4 * CS)) ^ swz(d_row[i])) * 16;
    }
    const char *const mine = ring[wave];
    const unsigned ring0 = __builtin_amdgcn_readfirstlane(lds_addr_of(mine));
    int xb = b, ob = b, ob_end = b + 1;
    if constexpr (MODE == 0) {
        const int *pn = n_out_dev ? n_out_dev : adapter_of_out;
        const int n_ld = *(const volatile int *)pn, xb_ld = *(const volatile int *)(in_block_of_out ? in_block_of_out + b : adapter_of_out + b);
        if (b >= (n_out_dev ? min(n_ld, n_out) : n_out)) return;
        if (in_block_of_out) xb = __builtin_amdgcn_readfirstlane(xb_ld);
    }
    const char *const xbase = (const char *)(X + (size_t)xb * T * K + (size_t)wk * chunks * (32 * CS));
    const char *const abase = (const char *)(At + (size_t)wk * chunks * (32 * CS));
    // Items of one pass, in order: subtiles 0 .. ms - 1 of chunk 0, then for every further chunk the At rows of its groups (item < 0) and the
    // subtiles.  Chunk 0's At comes straight into registers.
    int q_item = 0, q_chunk = 0, ng = 1;
    unsigned q_slot = 0, slot = 0;
    const char *a_row[2];
    int a_last[2];
    auto request = [&]() {
        const bool is_a = q_item < 0;
        const int g = q_item == -1 ? ng - 1 : 0, row = 16 * (m0 + q_item);
        // rows past the last one repeat it: they feed results that are dropped (X) or zeroed (At) at the store
        const char *base = (is_a ? (g ? a_row[1] : a_row[0]) : xbase + (size_t)row * K * 2) + (size_t)q_chunk * ROW;
        const int last = is_a ? (g ? a_last[1] : a_last[0]) : T - 1 - row;
#pragma unroll
        for (int i = 0; i < CS; ++i) glds16_s(base, (unsigned)(min(d_row[i], last) * (2 * K) + d_col[i]), ring0 + q_slot + i * 1024);
        if (++q_item == ms) { q_item = -ng; ++q_chunk; }
        q_slot = q_slot == (RING - 1) * ITEM ? 0 : q_slot + ITEM;
    };
    const int first = max(0, min(RING - 1, ms - 1));                     // requested before the groups are known (the last subtile's successor depends on them)
    bool asked = unit == 0;                                      // (of the later ones it is not known whether there is work)
    for (int i = 0; asked && i < first; ++i) request();
    if constexpr (MODE > 0) {
        const int *off = MODE == 2 ? pa.row_offsets : out_off;
        const int p0 = off[b], p1 = off[b + 1], n = MODE == 2 ? off[pa.F] : n_out_dev ? min(*n_out_dev, n_out) : n_out;
        ob = __builtin_amdgcn_readfirstlane(p0);
        ob_end = __builtin_amdgcn_readfirstlane(p1);
        if (ob < 0 || ob_end > n || n > n_out || (MODE == 2 && off[0] != 0)) ob_end = ob;      // (rejected)
    }
    const bool paired = MODE > 0 && RP == 16;
    const int *ids = MODE == 2 ? pa.adapter_ids : adapter_of_out;
    const int step = paired ? 2 : 1;
    bool again = false;
    for (ob += step * unit; ob < ob_end; ob += step * units) {
        int ksel[2], osel[2] = {ob, ob};
        ksel[0] = ksel[1] = __builtin_amdgcn_readfirstlane(ids[ob]);
        if (paired) {
            osel[1] = ob + 1 < ob_end ? ob + 1 : -1;
            ksel[1] = __builtin_amdgcn_readfirstlane(ids[min(ob + 1, ob_end - 1)]);
        }
        if (MODE == 2 && ((unsigned)ksel[0] >= (unsigned)pa.n_adapters || (unsigned)ksel[1] >= (unsigned)pa.n_adapters)) break;     // (rejected)
        if (ksel[0] < 0 && (ksel[1] < 0 || osel[1] < 0)) continue;
        for (int j0 = 0; j0 < (paired ? 16 : RP); j0 += 32) {
            ng = paired ? (osel[1] >= 0 ? 2 : 1) : RP - j0 > 16 ? 2 : 1;
            const int rank0[2] = {j0, paired ? 0 : j0 + 16};
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int r0 = min(rank0[g], r - 1);
                a_row[g] = abase + ((size_t)max(ksel[g], 0) * r + r0) * K * 2;
                a_last[g] = r - 1 - r0;
            }
            if (again) {                                         // another pass over the rows: the ring is free once all have read the sums
                __syncthreads();
                q_item = q_chunk = 0; q_slot = slot = 0;
            }
            if (again || !asked)
                for (int i = 0; i < first; ++i) request();
            again = asked = true;
            bf16x8 fa[2][CS], fx[CS];
#pragma unroll
            for (int g = 0; g < 2; ++g)
                if (g < ng)
#pragma unroll
                    for (int u = 0; u < CS; ++u) fa[g][u] = *(const bf16x8 *)(a_row[g] + (size_t)min(li, a_last[g]) * (2 * K) + (4 * u + lc) * 16);
            f32x4 acc[SH_MS][2];
#pragma unroll
            for (int m = 0; m < SH_MS; ++m) acc[m][0] = acc[m][1] = f32x4{0.f, 0.f, 0.f, 0.f};
            int left = ms > 0 ? ms * chunks + ng * (chunks - 1) : 0;   // items not yet requested
            const int ahead = min(RING - 1, left);
            for (int i = first; i < ahead; ++i) request();
            left -= ahead;
            // the next item: request one more (its slot was read before the last MFMAs), wait for this one's loads, read it
            auto next = [&](bf16x8 (&f)[CS]) {
                if (left > 0) {
                    request();
                    --left;
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((RING - 1) * CS) : "memory");
                } else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                const char *it = mine + slot + li * ROW;
#pragma unroll
                for (int u = 0; u < CS; ++u) f[u] = *(const bf16x8 *)(it + ((4 * u + lc) ^ swz(li)) * 16);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // before the slot is requested again
                slot = slot == (RING - 1) * ITEM ? 0 : slot + ITEM;
            };
            if (ms > 0)
                for (int c = 0; c < chunks; ++c) {
                    if (c > 0) {
                        next(fa[0]);
                        if (ng == 2) next(fa[1]);
                    }
#pragma unroll
                    for (int m = 0; m < SH_MS; ++m)
                        if (m < ms) {
                            next(fx);
#pragma unroll
                            for (int u = 0; u < CS; ++u) acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[0][u], fx[u], acc[m][0], 0, 0, 0);
                            if (ng == 2) {
#pragma unroll
                                for (int u = 0; u < CS; ++u) acc[m][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[1][u], fx[u], acc[m][1], 0, 0, 0);
                            }
                        }
                }
            // partial sums of the WK waves of a run: wave wk finishes the values v = 2 m + g with v % WK == wk
            if (wk_log > 0) {
                f32x4 *red = (f32x4 *)ring[wave];
#pragma unroll
                for (int v = 0; v < 2 * SH_MS; ++v)
                    if (v / 2 < ms && v % 2 < ng) red[v * 64 + lane] = acc[v / 2][v % 2];
                __syncthreads();
            }
            const int share = wk_log == 0 ? 0 : ng == 2 ? wk : 2 * wk, stride = wk_log == 0 ? 1 : (ng == 2 ? 1 : 2) << wk_log;
#pragma unroll
            for (int v = 0; v < 2 * SH_MS; ++v) {
                const int m = v / 2, g = v % 2;
                if (m >= ms || g >= ng || (v & (stride - 1)) != share) continue;
                f32x4 sum = acc[m][g];
                if (wk_log > 0) {
                    sum = ((const f32x4 *)ring[wr << wk_log])[v * 64 + lane];
                    for (int w = 1; w < 1 << wk_log; ++w) sum += ((const f32x4 *)ring[(wr << wk_log) + w])[v * 64 + lane];
                }
                const int tt = 16 * (m0 + m) + li, rk = rank0[g] + 4 * lc;
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = rk + e < r ? (bf16_t)(scale * sum[e]) : (bf16_t)0.f;
                if (tt < T && ksel[g] >= 0 && osel[g] >= 0 && rk < RP) *(bf16x4 *)(S + ((size_t)osel[g] * T + tt) * RP + rk) = o;
            }
        }
    }
    if (!again) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // nothing lands in this LDS once another workgroup owns it
}

// ------------------------------------------------------------------ heads and merge to label space
// One wave per row-block: z = LN(x[src][0][:]); logits = z H_k + hb_k; scores = sigmoid(logits); lane c
// then folds class c into the frame's label vector.  Scores are in (0, 1): the order of positive floats
// is the order of their bit patterns, so an integer atomic max merges overlapping adapters without
// depending on arrival order.
// NX = D/64 values of the row per lane (0: any D, strided loops).  With NX fixed the row, gain, shift and
// the first head row are requested together and each later head row one class ahead of its use.
template <typename T, int NX>
__global__ __launch_bounds__(64) void head_kernel(const float *x, const int *src_block_of_row, int Tn, int D, const float *gain,
                                                  const float *shift, float eps, const T *head_w, const float *head_b, int C,
                                                  const int *adapter_of_row, const int *frame_of_row, const int32_t *class_map,
                                                  int K, const PolyMeta *meta, float *logits, float *scores, float *merged)
{
    const int b = blockIdx.x;
    if (b >= meta->R) return;
    const int lane = threadIdx.x;
    const int src = src_block_of_row ? src_block_of_row[b] : b;
    const int k_ad = adapter_of_row[b];
    const int fr = merged ? frame_of_row[b] : 0;
    const float *xr = x + (size_t)src * Tn * D;
    const int cl = lane < C ? lane : C - 1;
    const float hb = head_b[k_ad * C + cl];
    const int cls = merged ? class_map[k_ad * C + cl] : -1;
    float mine = 0.f;
    if constexpr (NX > 0) {
        float xv[NX], g[NX], sh[NX], hw[NX], hn[NX];
        const T *hk = head_w + (size_t)k_ad * C * D + lane;
#pragma unroll
        for (int i = 0; i < NX; ++i) xv[i] = xr[lane + 64 * i];
#pragma unroll
        for (int i = 0; i < NX; ++i) { g[i] = gain[lane + 64 * i]; sh[i] = shift[lane + 64 * i]; hw[i] = to_f32(hk[64 * i]); }
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < NX; ++i) s += xv[i];
        const float mean = wave_sum(s) / D;
        float v = 0.f;
#pragma unroll
        for (int i = 0; i < NX; ++i) { const float d = xv[i] - mean; v += d * d; }
        const float inv = rsqrtf(wave_sum(v) / D + eps);
#pragma unroll
        for (int i = 0; i < NX; ++i) xv[i] = (xv[i] - mean) * inv * g[i] + sh[i];
        for (int c = 0; c < C; ++c) {
            const T *hnext = hk + (size_t)(c + 1 < C ? c + 1 : c) * D;
#pragma unroll
            for (int i = 0; i < NX; ++i) hn[i] = to_f32(hnext[64 * i]);
            float a = 0.f;
#pragma unroll
            for (int i = 0; i < NX; ++i) a = fmaf(xv[i], hw[i], a);
            a = wave_sum(a);
            if (lane == c) mine = a;
#pragma unroll
            for (int i = 0; i < NX; ++i) hw[i] = hn[i];
        }
    } else {
        float s = 0.f;
        for (int k = lane; k < D; k += 64) s += xr[k];
        const float mean = wave_sum(s) / D;
        float v = 0.f;
        for (int k = lane; k < D; k += 64) { const float d = xr[k] - mean; v += d * d; }
        const float inv = rsqrtf(wave_sum(v) / D + eps);
        for (int c = 0; c < C; ++c) {
            const T *hw = head_w + ((size_t)k_ad * C + c) * D;
            float a = 0.f;
            for (int k = lane; k < D; k += 64) a = fmaf((xr[k] - mean) * inv * gain[k] + shift[k], to_f32(hw[k]), a);
            a = wave_sum(a);
            if (lane == c) mine = a;
        }
    }
    if (lane < C) {
        const float lg = mine + hb;
        const float sc = 1.0f / (1.0f + expf(-lg));
        if (logits) logits[(size_t)b * C + lane] = lg;
        scores[(size_t)b * C + lane] = sc;
        if (cls >= 0 && cls < K) atomicMax((int *)(merged + (size_t)fr * K + cls), __float_as_int(sc));
    }
}

}  // namespace

// ------------------------------------------------------------------ launchers

static inline int hip_ok() { return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP; }

int launch_prep(const int32_t *row_offsets, const int32_t *adapter_ids, int F, int R_cap, int n_adapters, PolyMeta *meta,
                int32_t *frame_of_row, int32_t *adapter_of_row, int32_t *dev_status, hipStream_t st)
{
    POLY_LAUNCH(POLY_STAGE_OTHER, prep_kernel, dim3(1), dim3(256), st, row_offsets, adapter_ids, F, R_cap, n_adapters, meta, frame_of_row,
                       adapter_of_row, dev_status);
    return hip_ok();
}

int launch_im2col(const void *frames, void *patches, int F, int H, int W, int p, int dtype, float *x, const float *cls, const float *pos,
                  int T_tok, int D, float *merged, size_t n_merged, unsigned *zero, size_t n_zero, const int32_t *row_offsets, const int32_t *adapter_ids, int R_cap,
                  int n_adapters, PolyMeta *meta, int32_t *frame_of_row, int32_t *adapter_of_row, int32_t *dev_status, hipStream_t st)
{
    const PrepArgs pa = {row_offsets, adapter_ids, F, R_cap, n_adapters, meta, frame_of_row, adapter_of_row, dev_status};
    const size_t total = (size_t)F * H * W * 3;
    if (total == 0 && n_merged == 0 && n_zero == 0) {
        if (row_offsets) return launch_prep(row_offsets, adapter_ids, F, R_cap, n_adapters, meta, frame_of_row, adapter_of_row, dev_status, st);
        return POLY_OK;
    }
    // 16-byte vectors when a run of 3p elements is a whole number of them and rows of the frame keep them aligned
    const int vec = dtype == POLY_BF16 ? 8 : 4;
    const bool wide = (3 * p) % vec == 0 && (3 * W) % vec == 0 && ((uintptr_t)frames & 15) == 0 && ((uintptr_t)patches & 15) == 0;
    const size_t work = (wide ? total / vec : total) > n_merged ? (wide ? total / vec : total) : n_merged;
    const unsigned blocks = (unsigned)((work + 255) / 256 > 65536 ? 65536 : (work + 255) / 256 < 1 ? 1 : (work + 255) / 256) + (row_offsets ? 1 : 0);
    if (dtype == POLY_BF16) {
        if (wide) POLY_LAUNCH(POLY_STAGE_OTHER, (im2col_kernel<bf16_t, 8>), dim3(blocks), dim3(256), st, (const bf16_t *)frames, (bf16_t *)patches, F, H, W, p, x, cls, pos, T_tok, D, merged, n_merged, zero, n_zero, pa);
        else POLY_LAUNCH(POLY_STAGE_OTHER, (im2col_kernel<bf16_t, 1>), dim3(blocks), dim3(256), st, (const bf16_t *)frames, (bf16_t *)patches, F, H, W, p, x, cls, pos, T_tok, D, merged, n_merged, zero, n_zero, pa);
    } else {
        if (wide) POLY_LAUNCH(POLY_STAGE_OTHER, (im2col_kernel<float, 4>), dim3(blocks), dim3(256), st, (const float *)frames, (float *)patches, F, H, W, p, x, cls, pos, T_tok, D, merged, n_merged, zero, n_zero, pa);
        else POLY_LAUNCH(POLY_STAGE_OTHER, (im2col_kernel<float, 1>), dim3(blocks), dim3(256), st, (const float *)frames, (float *)patches, F, H, W, p, x, cls, pos, T_tok, D, merged, n_merged, zero, n_zero, pa);
    }
    return hip_ok();
}

int launch_layernorm(const float *x, void *y, const float *gain, const float *shift, int D, float eps, int T, int n_blocks,
                     const int *n_blocks_dev, int dtype, hipStream_t st)
{
    const size_t rows = (size_t)n_blocks * T;
    if (rows == 0) return POLY_OK;
    const unsigned blocks = (unsigned)((rows + 3) / 4);
    const bool aligned = ((uintptr_t)x & 15) == 0 && ((uintptr_t)y & 15) == 0 && ((uintptr_t)gain & 15) == 0 && ((uintptr_t)shift & 15) == 0;
    if (dtype == POLY_BF16 && aligned && D == 768) {
        POLY_LAUNCH(POLY_STAGE_NORM, (layernorm_vec_kernel<bf16_t, 3>), dim3(blocks), dim3(256), st, x, (bf16_t *)y, gain, shift, eps, T, n_blocks, n_blocks_dev);
    } else if (dtype == POLY_BF16 && aligned && D == 1024) {
        POLY_LAUNCH(POLY_STAGE_NORM, (layernorm_vec_kernel<bf16_t, 4>), dim3(blocks), dim3(256), st, x, (bf16_t *)y, gain, shift, eps, T, n_blocks, n_blocks_dev);
    } else if (dtype == POLY_BF16 && aligned && D == 512) {
        POLY_LAUNCH(POLY_STAGE_NORM, (layernorm_vec_kernel<bf16_t, 2>), dim3(blocks), dim3(256), st, x, (bf16_t *)y, gain, shift, eps, T, n_blocks, n_blocks_dev);
    } else if (dtype == POLY_BF16 && aligned && D == 256) {
        POLY_LAUNCH(POLY_STAGE_NORM, (layernorm_vec_kernel<bf16_t, 1>), dim3(blocks), dim3(256), st, x, (bf16_t *)y, gain, shift, eps, T, n_blocks, n_blocks_dev);
    } else if (dtype == POLY_BF16)
        POLY_LAUNCH(POLY_STAGE_NORM, layernorm_kernel<bf16_t>, dim3(blocks), dim3(256), st, x, (bf16_t *)y, gain, shift, D, eps, T, n_blocks, n_blocks_dev);
    else
        POLY_LAUNCH(POLY_STAGE_NORM, layernorm_kernel<float>, dim3(blocks), dim3(256), st, x, (float *)y, gain, shift, D, eps, T, n_blocks, n_blocks_dev);
    return hip_ok();
}

bool layernorm_shrink_fits(const float *x, const void *y, const float *gain, const float *shift, int D, int n_blocks, const void *At, int RP, int n_out,
                           const void *S, int dtype)
{
    return dtype == POLY_BF16 && RP == 16 && D % 256 == 0 && D > 0 && D <= 1024 && n_blocks > 0 && n_out > 0 && aligned16(x) && aligned16(y) && aligned16(gain) &&
           aligned16(shift) && aligned16(At) && aligned16(S);
}

int launch_layernorm_shrink(const float *x, void *y, const float *gain, const float *shift, int D, float eps, int T, int n_blocks, const int *n_blocks_dev,
                            const void *At, int r, float scale, int n_out, const int *n_out_dev, const int *out_off, const int *adapter_of_out, void *S,
                            hipStream_t st)
{
    const int subs = (T + 15) / 16;
    const dim3 grid((unsigned)((size_t)n_blocks * subs));
#define LN_SHRINK_CASE(N)                                                                                                                                       \
    case 256 * N:                                                                                                                                               \
        POLY_LAUNCH(POLY_STAGE_NORM, layernorm_shrink_kernel<N>, grid, dim3(256), st, x, (bf16_t *)y, gain, shift, eps, T, subs, n_blocks, n_blocks_dev,         \
                    (const bf16_t *)At, r, scale, out_off, n_out_dev, n_out, adapter_of_out, (bf16_t *)S);                                                       \
        return hip_ok();
    switch (D) {
        LN_SHRINK_CASE(1) LN_SHRINK_CASE(2) LN_SHRINK_CASE(3) LN_SHRINK_CASE(4)
        default: return POLY_EINVAL;
    }
#undef LN_SHRINK_CASE
}

template <int MS, int NG, bool CSR>
static void launch_shrink_bf16(hipStream_t st, const bf16_t *X, int T, int K, const bf16_t *At, int r, int RP, float scale, int n_out,
                               const int *n_out_dev, const int *in_block_of_out, const int *adapter_of_out, const int *pair_off, bf16_t *S,
                               const PrepArgs &pa)
{
    const int subs = (T + 16 * MS - 1) / (16 * MS);
    POLY_LAUNCH(POLY_STAGE_SHRINK, (shrink_bf16_kernel<MS, NG, CSR>), dim3((unsigned)((size_t)n_out * subs + (CSR ? 1 : 0))), dim3(256), st, X, T, K, At, r,
                RP, scale, n_out, n_out_dev, in_block_of_out, adapter_of_out, pair_off, S, pa);
}

// False where the other kernel is to run: columns that the items do not divide, addresses that their 16-byte loads do not allow, and little work.
// The other one's chain is shorter where a wave has one batch of columns (K <= 768) and few workgroups; per call on 197-token blocks of rank 16, us,
// other / this: 16 blocks x 2 branches x 768 6.3 / 6.8, 32 x 2 8.7 / 7.9, 256 x 2 42.4 / 18.2 (77 MB of rows, in a call of poly_lora_linear on
// 2304 columns; 77 MB at the rate of a large copy take 16); 64 x 2 x 384 8.3 / 8.6, 128 x 2 12.2 / 9.8; 128 x 2 x 192 8.5 / 8.0;
// 4 x 1 x 1024 5.5 / 5.1, 4 x 1 x 3072 11.9 / 7.0, 64 x 2 x 3072 34.6 / 19.4.  Of rank 32, 113 tokens: 64 x 2 x 768 8.6 / 9.9, 128 x 2 15.4 / 12.6.
// Runs of 16 to 112 rows, the shortest with which all workgroups are on the chip at once (two per CU).
// blocks: output blocks (MODE 0) or input blocks
template <int MODE>
static bool launch_shrink_stream(hipStream_t st, const bf16_t *X, int T, int K, const bf16_t *At, int r, int RP, float scale, int blocks, int n_out,
                                 const int *n_out_dev, const int *in_block_of_out, const int *adapter_of_out, const int *out_off, bf16_t *S,
                                 const PrepArgs &pa)
{
    const int cs = K % 192 == 0 ? 6 : K % 128 == 0 ? 4 : 0;
    if (!cs || (((uintptr_t)X | (uintptr_t)At) & 15) || ((uintptr_t)S & 7) || RP % 4) return false;
    if ((RP > 16 || K <= 768) && (long)n_out * T * K < (RP > 16 ? 12L : 8L) * 1000000) return false;
    const int units = MODE == 0 ? 1 : RP == 16 ? (n_out + 2 * blocks - 1) / (2 * blocks) : (n_out + blocks - 1) / blocks;
    const int chunks = K / (32 * cs), wk_log = chunks % 4 == 0 ? 2 : chunks % 2 == 0 ? 1 : 0, runs = 4 >> wk_log, nt = (T + 15) / 16;
    int parts = 0, wgs = 0;
    for (int per = 1; per <= SH_MS; ++per) {
        parts = (nt + per - 1) / per;
        wgs = (parts + runs - 1) / runs;
        if ((long)blocks * units * wgs <= 512) break;
    }
    const dim3 grid((unsigned)((size_t)blocks * units * wgs + (MODE == 2 ? 1 : 0)));
    if (cs == 6)
        POLY_LAUNCH(POLY_STAGE_SHRINK, (shrink_stream_kernel<6, MODE>), grid, dim3(256), st, X, T, K, At, r, RP, scale, n_out, n_out_dev,
                    in_block_of_out, adapter_of_out, out_off, S, wk_log, parts, wgs, units, pa);
    else
        POLY_LAUNCH(POLY_STAGE_SHRINK, (shrink_stream_kernel<4, MODE>), grid, dim3(256), st, X, T, K, At, r, RP, scale, n_out, n_out_dev,
                    in_block_of_out, adapter_of_out, out_off, S, wk_log, parts, wgs, units, pa);
    return true;
}

// launch_prep and launch_shrink of an isolated linear (bf16, output blocks of one input block consecutive) in one launch
bool shrink_csr_fits(int F, int T, int K, int dtype) { return dtype == POLY_BF16 && F <= SH_CSR_MAX && K % 8 == 0 && (long)T * K <= 0x7fffffffL; }
int launch_shrink_csr(const void *X, int T, int K, const void *At, int r, int RP, float scale, const int32_t *row_offsets, const int32_t *adapter_ids,
                      int F, int R_cap, int n_adapters, PolyMeta *meta, int32_t *frame_of_row, int32_t *adapter_of_row, int32_t *dev_status, void *S,
                      hipStream_t st)
{
    const PrepArgs pa = {row_offsets, adapter_ids, F, R_cap, n_adapters, meta, frame_of_row, adapter_of_row, dev_status};
    if (!launch_shrink_stream<2>(st, (const bf16_t *)X, T, K, (const bf16_t *)At, r, RP, scale, F, R_cap, nullptr, nullptr, nullptr, nullptr, (bf16_t *)S, pa))
        launch_shrink_bf16<2, 2, true>(st, (const bf16_t *)X, T, K, (const bf16_t *)At, r, RP, scale, R_cap, nullptr, nullptr, nullptr, nullptr, (bf16_t *)S, pa);
    return hip_ok();
}

// out_off: offsets of the output blocks of the n_in input blocks where they fan out (then in_block_of_out is their map), else nullptr
int launch_shrink(const void *X, int T, int K, const void *At, int r, int RP, float scale, int n_in, int n_out, const int *n_out_dev,
                  const int *in_block_of_out, const int *adapter_of_out, const int *out_off, void *S, int dtype, hipStream_t st)
{
    if (n_out == 0) return POLY_OK;
    if (dtype != POLY_BF16)
        return launch_shrink_f32((const float *)X, T, K, (const float *)At, r, RP, scale, n_out, n_out_dev, in_block_of_out, adapter_of_out, (float *)S, st);
    if (K % 8 != 0 || (long)T * K > 0x7fffffffL) return POLY_EINVAL;
    const bf16_t *x = (const bf16_t *)X, *at = (const bf16_t *)At;
    const bool fan = out_off && in_block_of_out;
    if (fan ? launch_shrink_stream<1>(st, x, T, K, at, r, RP, scale, n_in, n_out, n_out_dev, nullptr, adapter_of_out, out_off, (bf16_t *)S, PrepArgs{})
            : launch_shrink_stream<0>(st, x, T, K, at, r, RP, scale, n_out, n_out, n_out_dev, in_block_of_out, adapter_of_out, nullptr, (bf16_t *)S, PrepArgs{}))
        return hip_ok();
    if (RP > 16 || fan)
        launch_shrink_bf16<2, 2, false>(st, x, T, K, at, r, RP, scale, n_out, n_out_dev, in_block_of_out, adapter_of_out, out_off, (bf16_t *)S, PrepArgs{});
    else
        launch_shrink_bf16<2, 1, false>(st, x, T, K, at, r, RP, scale, n_out, n_out_dev, in_block_of_out, adapter_of_out, out_off, (bf16_t *)S, PrepArgs{});
    return hip_ok();
}

template <typename T>
static void launch_head_t(int nx, dim3 grid, hipStream_t st, const float *x, const int *src_block_of_row, int Tn, int D, const float *gain,
                          const float *shift, float eps, const T *head_w, const float *head_b, int C, const int *adapter_of_row,
                          const int *frame_of_row, const int32_t *class_map, int K, const PolyMeta *meta, float *logits, float *scores,
                          float *merged)
{
#define HEAD_CASE(N)                                                                                                             \
    case N:                                                                                                                      \
        POLY_LAUNCH(POLY_STAGE_OTHER, (head_kernel<T, N>), grid, dim3(64), st, x, src_block_of_row, Tn, D, gain, shift, eps, head_w, head_b, \
                    C, adapter_of_row, frame_of_row, class_map, K, meta, logits, scores, merged);                               \
        break;
    switch (nx) {
        HEAD_CASE(1) HEAD_CASE(2) HEAD_CASE(3) HEAD_CASE(4) HEAD_CASE(6) HEAD_CASE(8) HEAD_CASE(12)
        default: HEAD_CASE(0)
    }
#undef HEAD_CASE
}

// ------------------------------------------------------------------ base head of the lagged loop
// Block f: LayerNorm of frame f's class token (row 0 of its block of x) and the K label scores
// sigmoid(z Wb[c] + bb[c]).  The scores go to lag[f + 1] (the selection of frame
// f + 1 reads them there) and to out[f]; block 0 also copies the carried scores of the previous call to lag[0].
template <typename T>
__global__ __launch_bounds__(256) void base_head_kernel(const float *x, int T_tok, int D, const float *gain, const float *shift, float eps,
                                                        const T *Wb, const float *bb, int K, float *lag, float *out, const float *carry)
{
    extern __shared__ float bh_s[];      // z [D], then 8 partial sums
    float *z = bh_s, *part = bh_s + D;
    const int f = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float *xr = x + (size_t)f * T_tok * D;
    if (f == 0)
        for (int c = tid; c < K; c += 256) lag[c] = carry ? carry[c] : 0.f;
    float s = 0.f;
    for (int i = tid; i < D; i += 256) s += xr[i];
    s = wave_sum(s);
    if (lane == 0) part[wave] = s;
    __syncthreads();
    const float mean = (part[0] + part[1] + part[2] + part[3]) / D;
    float q = 0.f;
    for (int i = tid; i < D; i += 256) { const float d = xr[i] - mean; q += d * d; }
    q = wave_sum(q);
    if (lane == 0) part[4 + wave] = q;
    __syncthreads();
    const float inv = rsqrtf((part[4] + part[5] + part[6] + part[7]) / D + eps);
    for (int i = tid; i < D; i += 256) z[i] = (xr[i] - mean) * inv * gain[i] + shift[i];
    __syncthreads();
    // eight classes per wave and round: their weight loads are in flight together (one class at a time pays a memory
    // round trip per class), and lane u finishes class c0 + u
    for (int c0 = wave * 8; c0 < K; c0 += 32) {
        float d[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) d[u] = 0.f;
        for (int i = lane; i < D; i += 64) {
            const float zi = z[i];
#pragma unroll
            for (int u = 0; u < 8; ++u) d[u] = fmaf(zi, (float)Wb[(size_t)min(c0 + u, K - 1) * D + i], d[u]);
        }
        float mine = 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float t = wave_sum(d[u]);
            if (lane == u) mine = t;
        }
        const int c = c0 + lane;
        if (lane < 8 && c < K) {
            const float sc = 1.0f / (1.0f + expf(-(mine + bb[c])));
            lag[(size_t)(f + 1) * K + c] = sc;
            if (out) out[(size_t)f * K + c] = sc;
        }
    }
}

// D = 64 ND: no LDS and no workgroup barrier -- every wave normalises the row for itself (lane l holds elements l + 64 j,
// the layout its dot products need), and the weights of the next eight classes are requested before the sums of the
// current eight are reduced, so that a round costs one memory round trip instead of one per K step
template <typename T, int ND>
__global__ __launch_bounds__(256) void base_head_nd_kernel(const float *x, int T_tok, const float *gain, const float *shift, float eps,
                                                           const T *Wb, const float *bb, int K, float *lag, float *out, const float *carry)
{
    constexpr int D = 64 * ND, CW = 8;
    const int f = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float *xr = x + (size_t)f * T_tok * D;
    float xv[ND], g[ND], sh[ND];
#pragma unroll
    for (int j = 0; j < ND; ++j) { xv[j] = xr[lane + 64 * j]; g[j] = gain[lane + 64 * j]; sh[j] = shift[lane + 64 * j]; }
    auto loadw = [&](T(&w)[CW][ND], int c0) {
#pragma unroll
        for (int u = 0; u < CW; ++u)
#pragma unroll
            for (int j = 0; j < ND; ++j) w[u][j] = Wb[(size_t)min(c0 + u, K - 1) * D + lane + 64 * j];
    };
    T w0[CW][ND];
    loadw(w0, wave * CW);
    if (f == 0)
        for (int c = tid; c < K; c += 256) lag[c] = carry ? carry[c] : 0.f;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < ND; ++j) s += xv[j];
    const float mean = wave_sum(s) / D;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < ND; ++j) { const float d = xv[j] - mean; q += d * d; }
    const float inv = rsqrtf(wave_sum(q) / D + eps);
    float z[ND];
#pragma unroll
    for (int j = 0; j < ND; ++j) z[j] = (xv[j] - mean) * inv * g[j] + sh[j];
    for (int c0 = wave * CW; c0 < K; c0 += 4 * CW) {
        T w1[CW][ND];
        const bool more = c0 + 4 * CW < K;          // uniform
        if (more) loadw(w1, c0 + 4 * CW);
        float mine = 0.f;
#pragma unroll
        for (int u = 0; u < CW; ++u) {
            float d = 0.f;
#pragma unroll
            for (int j = 0; j < ND; ++j) d = fmaf(z[j], (float)w0[u][j], d);
            d = wave_sum(d);
            if (lane == u) mine = d;
        }
        const int c = c0 + lane;
        if (lane < CW && c < K) {
            const float sc = 1.0f / (1.0f + expf(-(mine + bb[c])));
            lag[(size_t)(f + 1) * K + c] = sc;
            if (out) out[(size_t)f * K + c] = sc;
        }
        if (more) {
#pragma unroll
            for (int u = 0; u < CW; ++u)
#pragma unroll
                for (int j = 0; j < ND; ++j) w0[u][j] = w1[u][j];
        }
    }
}

template <typename T>
static bool launch_base_head_nd(int D, int F, hipStream_t st, const float *x, int T_tok, const float *gain, const float *shift, float eps,
                                const T *Wb, const float *bb, int K, float *lag, float *out, const float *carry)
{
    switch (D) {
#define POLY_BH_CASE(ND)                                                                                                            \
    case 64 * ND:                                                                                                                   \
        POLY_LAUNCH(POLY_STAGE_OTHER, (base_head_nd_kernel<T, ND>), dim3(F), dim3(256), st, x, T_tok, gain, shift, eps, Wb, bb, K, lag, out, carry); \
        return true;
        POLY_BH_CASE(1) POLY_BH_CASE(2) POLY_BH_CASE(3) POLY_BH_CASE(4) POLY_BH_CASE(6) POLY_BH_CASE(8) POLY_BH_CASE(12)
#undef POLY_BH_CASE
    default: return false;
    }
}

int launch_base_head(const float *x, int T, int D, const float *gain, const float *shift, float eps, const void *Wb, const float *bb,
                     int K, int F, float *lag, float *out, const float *carry, int dtype, hipStream_t st)
{
    if (F == 0) return POLY_OK;
    if (dtype == POLY_BF16 ? launch_base_head_nd<bf16_t>(D, F, st, x, T, gain, shift, eps, (const bf16_t *)Wb, bb, K, lag, out, carry)
                           : launch_base_head_nd<float>(D, F, st, x, T, gain, shift, eps, (const float *)Wb, bb, K, lag, out, carry))
        return hip_ok();
    const size_t lds = sizeof(float) * (size_t)(D + 8);
    if (dtype == POLY_BF16)
        POLY_LAUNCH_SHMEM(POLY_STAGE_OTHER, base_head_kernel<bf16_t>, dim3(F), dim3(256), lds, st, x, T, D, gain, shift, eps, (const bf16_t *)Wb, bb,
                          K, lag, out, carry);
    else
        POLY_LAUNCH_SHMEM(POLY_STAGE_OTHER, base_head_kernel<float>, dim3(F), dim3(256), lds, st, x, T, D, gain, shift, eps, (const float *)Wb, bb,
                          K, lag, out, carry);
    return hip_ok();
}

// heads, and the merge to the label space when merged is given (zeroed by the caller, F x K)
int launch_head(const float *x, const int *src_block_of_row, int T, int D, const float *gain, const float *shift, float eps,
                const void *head_w, const float *head_b, int C, const int *adapter_of_row, const int *frame_of_row,
                const int32_t *class_map, int K, const PolyMeta *meta, int R_cap, float *logits, float *scores, float *merged, int dtype,
                hipStream_t st)
{
    if (R_cap == 0) return POLY_OK;
    const int nx = D % 64 == 0 ? D / 64 : 0;
    if (dtype == POLY_BF16)
        launch_head_t<bf16_t>(nx, dim3(R_cap), st, x, src_block_of_row, T, D, gain, shift, eps, (const bf16_t *)head_w, head_b, C,
                              adapter_of_row, frame_of_row, class_map, K, meta, logits, scores, merged);
    else
        launch_head_t<float>(nx, dim3(R_cap), st, x, src_block_of_row, T, D, gain, shift, eps, (const float *)head_w, head_b, C,
                             adapter_of_row, frame_of_row, class_map, K, meta, logits, scores, merged);
    return hip_ok();
}
