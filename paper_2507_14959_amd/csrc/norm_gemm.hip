// LayerNorm + linear of few rows of a wide model in one launch: y = [GELU](LayerNorm(x) W + b), bf16, shared weights only.
//
// On a few hundred rows both are launches of 5 to 10 us that are mostly their first round trips: 591 rows of 768 columns 4.8 us of LayerNorm and 9 to 10 us
// of product on tiles of 64 x 64.  Here a workgroup normalises its 64 rows itself while the first weights are on their way, and keeps them in LDS for the
// whole contraction (96 KB at 768 columns; the rows are read once per 128 columns, out of the L2 that the product before left them behind).
// 591 rows -> 2304 11.1 us.  Bound by the loads of a CU: 196 KB of rows and 196 KB of weights, the latter through a ring of three 16 KB stages in what LDS is left.
#include "rowtile.h"

namespace {

constexpr int NG_BN = 128, NG_NS = 3, NG_STAGE = NG_BN * 64;   // columns of a tile, stages, elements of a stage

// 64 rows x 128 columns, eight waves of 32 x 32: wave (wr, wc)
template <int KT>
__global__ __launch_bounds__(512, 2) void norm_gemm_kernel(const NormGemmArgs a, int tiles_n)
{
    constexpr int K = 64 * KT, NV = K / 32;                    // NV: 16-byte pieces of a thread, eight threads per row
    extern __shared__ __attribute__((aligned(16))) bf16_t ng_lds[];
    bf16_t *As = ng_lds, *ring = ng_lds + KT * 4096;
    float *gb_s = (float *)(ring + NG_NS * NG_STAGE);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lm = lane & 31, lh = lane >> 5;
    const int wr = wave >> 2, wc = wave & 3;
    const int rows = a.T * (a.nb_dev ? __builtin_amdgcn_readfirstlane(min(*a.nb_dev, a.nb)) : a.nb), mtot = (rows + 63) / 64;
    int mt, tn;
    {   // eight equal runs, one per XCD, of columns with all their rows: a column's weights come to one L2
        const long total = (long)mtot * tiles_n, lo = total * (blockIdx.x & 7) / 8, hi = total * ((blockIdx.x & 7) + 1) / 8, L = lo + (blockIdx.x >> 3);
        if (L >= hi) return;
        tn = __builtin_amdgcn_readfirstlane((int)(L / mtot));
        mt = (int)(L - (long)tn * mtot);
    }
    const int t0 = mt * 64, n0 = tn * NG_BN;
    // weights: each wave 16 of a stage's 128 rows, two loads of 8 rows x 128 bytes
    const int lr = lane >> 3;
    unsigned off[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (wave * 2 + i) * 8 + lr;
        off[i] = 2u * (unsigned)(min(n0 + row, a.N - 1) * K + (((lane & 7) ^ ((row >> 1) & 7)) << 3));
    }
    const unsigned ring_at = __builtin_amdgcn_readfirstlane(lds_addr_of(ring));
    auto issue = [&](int kt, int s) {
#pragma unroll
        for (int i = 0; i < 2; ++i) glds16_if(a.W + (size_t)kt * 64, off[i], ring_at + s * (NG_STAGE * 2) + (wave * 2 + i) * 1024, KT - kt);
    };
    f32x4 v[NV];
    const int row = tid >> 3, part = tid & 7;
    const float *xr = a.x + (size_t)min(t0 + row, rows - 1) * K + 4 * part;
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = *(const f32x4 *)(xr + 32 * i);
    const f32x4 gbv = ln_gb_load<KT>(a.gain, a.shift, tid);
    f32x4 bias4[4];                                            // columns 8 q + 4 lh .. of this wave's 32
#pragma unroll
    for (int q = 0; q < 4; ++q) bias4[q] = *(const f32x4 *)(a.bias + min(n0 + 32 * wc + 8 * q + 4 * lh, a.N - 4));
#pragma unroll
    for (int s = 0; s < NG_NS; ++s) issue(s, s);
    ln_gb_store<KT>(gbv, gb_s, tid);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) s += v[i][0] + v[i][1] + v[i][2] + v[i][3];
        const float mean = row_group_sum<8>(s) / K;
        float p = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int z = 0; z < 4; ++z) { const float d = v[i][z] - mean; p += d * d; }
        const float inv = rsqrtf(row_group_sum<8>(p) / K + a.eps);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int k = 32 * i + 4 * part;
            const f32x4 g = *(const f32x4 *)(gb_s + k), b = *(const f32x4 *)(gb_s + K + k);
            bf16x4 o;
#pragma unroll
            for (int z = 0; z < 4; ++z) o[z] = (bf16_t)((v[i][z] - mean) * inv * g[z] + b[z]);
            *(bf16x4 *)(As + (k >> 6) * 4096 + tile_off(row, (k & 63) >> 3) + (k & 4)) = o;
        }
    }
    f32x16 acc;                                                // row 32 wr + lm, columns 32 wc + 8 q + 4 lh + z
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int z = 0; z < 4; ++z) acc[4 * q + z] = bias4[q][z];
    const int sw = (lm >> 1) & 7;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
        // k-tile kt has landed once this wave's loads of the one behind it alone are pending; past the barrier everybody is done with the stage before
        if (kt == 0) rl_wait_barrier<2 * (NG_NS - 1)>();
        else rl_wait_barrier<2 * (NG_NS - 2)>();
        if (kt > 0) issue(kt - 1 + NG_NS, (kt - 1) % NG_NS);
        const bf16_t *at = As + kt * 4096 + (32 * wr + lm) * 64, *wt = ring + (kt % NG_NS) * NG_STAGE + (32 * wc + lm) * 64;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int ko = ((2 * kk + lh) ^ sw) << 3;
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8 *)(wt + ko), *(const bf16x8 *)(at + ko), acc, 0, 0, 0);
        }
    }
    // the wave's 32 x 32 results through LDS of its own (the ring is dead once every wave is here), 64 bytes of a row from four lanes
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    bf16_t *stg = ring + wave * 1024;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        f32x4 r = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        if (a.gelu) r = gelu_poly4(r);
        *(bf16x4 *)(stg + lm * 32 + ((q ^ ((lm >> 1) & 3)) << 3) + 4 * lh) = bf16x4{(bf16_t)r[0], (bf16_t)r[1], (bf16_t)r[2], (bf16_t)r[3]};
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int srow = 16 * q + (lane >> 2), ch = lane & 3, t = t0 + 32 * wr + srow, col = n0 + 32 * wc + 8 * ch;
        const bf16x8 r = *(const bf16x8 *)(stg + srow * 32 + ((ch ^ ((srow >> 1) & 3)) << 3));
        if (t < rows && col < a.N) *(bf16x8 *)(a.out + (size_t)t * a.N + col) = r;
    }
}

}  // namespace

// From six row tiles on, with fewer the two launches read less and are as fast, and as long as every tile has a CU of its own.  Forward of ViT-base, ten layers
// shared, us, as one / two launches: 3 frames of 197 tokens (10 row tiles) 643 / 668, 2 (7) 609 / 618, 6 of 101 (10) 649 / 676, 30 of 17 (8) 626 / 680; 16 of 17 (5)
// 546 / 548, 8 of 17 (3) 509 / 492; 5 of 197 (16, up to 384 tiles) 940 / 844.
bool norm_gemm_fits(const NormGemmArgs &a, int D)
{
    const long tiles_m = ((long)a.nb * a.T + 63) / 64, tiles_n = (a.N + NG_BN - 1) / NG_BN;
    return D == 768 && a.N % 8 == 0 && tiles_m >= 6 && tiles_m * tiles_n <= 256 && aligned16(a.x) && aligned16(a.gain) && aligned16(a.shift) && aligned16(a.W) &&
           aligned16(a.bias) && aligned16(a.out);
}

int launch_norm_gemm(const NormGemmArgs &a, hipStream_t st)
{
    constexpr int KT = 12, LDS = KT * 8192 + NG_NS * NG_STAGE * 2 + 64 * KT * 8;
    static_assert(LDS <= 160 * 1024, "LDS budget");
    auto kern = norm_gemm_kernel<KT>;
    static bool attr_set = false;   // raising the dynamic LDS limit is a per-kernel, process-wide setting
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS) != hipSuccess) return POLY_EHIP;
        attr_set = true;
    }
    const int tiles_n = (a.N + NG_BN - 1) / NG_BN;
    const long total = ((long)a.nb * a.T + 63) / 64 * tiles_n;
    POLY_LAUNCH_SHMEM(POLY_STAGE_GEMM, kern, dim3((unsigned)((total + 7) / 8 * 8)), dim3(512), LDS, st, a, tiles_n);
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}
