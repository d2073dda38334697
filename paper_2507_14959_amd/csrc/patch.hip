// The patch embedding in bf16: x[f][1 + t] = patch_t W + b + pos[1 + t], the patches gathered from the frames by the loads of the product, in one launch with
// what else comes first in a forward (PatchArgs).
//
// Bound by the bytes (frames in, fp32 rows out; 150 MB for 333 frames of 224 x 224 at 192 columns) and, on few frames, by the round trips of the ring.  A gather
// of its own writes every patch once more and has it read back, a launch and two passes over the frames that the product does not need: it is told
// where a row's next 16 bytes lie instead.  Gather and product 40 + 69 us there, 6.7 + 10.2 for 32 frames; us per forward before / now, 192 columns: 1 frame
// 190.3 / 188.9, 32 452 / 445, 333 1927 / 1852, 900 of 112 x 112 1046 / 948; 768 columns: 4 frames 822 / 805, 24 1879 / 1825, 64 3466 / 3454.
// Rows run across frames.  As in gemm.hip: 128-byte k-tiles of rows and weights go straight to LDS, swizzled, two of them ahead of the one in work.  (Four
// stages of 64 x 64 tiles, two of the others, 64 x 192, 64 x 96 and 128 x 96 are slower by up to 2 % of a forward where these are used.)
#include "rowtile.h"

namespace {

// WM x WN waves of 32 rows x 32 WC columns
template <int WM, int WN, int WC, int NS>
__global__ __launch_bounds__(64 * WM * WN, 2) void patch_rows_kernel(const PatchArgs pa, const PatchRows pr, const bf16_t *W, const float *bias, int D, int K, int tiles_m,
                                                                     int tiles_n, int tile_wgs, int job_wgs)
{
    constexpr int BM = 32 * WM, BN = 32 * WN * WC, NW = WM * WN, LA = BM / 8 / NW, LW = BN / 8 / NW, STAGE = (BM + BN) * 128, PITCH = 36;
    static_assert(BM / 8 % NW == 0 && BN / 8 % NW == 0 && NW * 32 * PITCH * 4 <= NS * STAGE, "loads of a wave, staging area");
    extern __shared__ __attribute__((aligned(16))) char pt_lds[];
    if ((int)blockIdx.x >= tile_wgs) {
        patch_jobs(pa, D, (int)blockIdx.x - tile_wgs, job_wgs);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lm = lane & 31, lh = lane >> 5;
    const int wr = wave / WN, wc = wave % WN, P = pr.gw * pr.gh, rows = pa.F * P, nk = K / 64;
    int mt, tn;
    {   // eight equal runs, one per XCD, of rows with all their columns: a frame comes to one L2
        const long total = (long)tiles_m * tiles_n, lo = total * (blockIdx.x & 7) / 8, hi = total * ((blockIdx.x & 7) + 1) / 8, L = lo + (blockIdx.x >> 3);
        if (L >= hi) return;
        mt = (int)(L / tiles_n);
        tn = (int)(L - (long)mt * tiles_n);
    }
    const int t0 = mt * BM, n0 = tn * BN;
    // a wave's loads: 8 rows x 128 bytes each; row 8 q + lane / 8, position lane % 8 takes chunk c0 (q even) or c0 ^ 4
    const int lr = lane >> 3, c0 = (lane & 7) ^ (lr >> 1);
    unsigned oa[LA], ow[LW];
#pragma unroll
    for (int i = 0; i < LA; ++i) oa[i] = patch_start(pr, min(t0 + 8 * (wave + NW * i) + lr, rows - 1), 2);
#pragma unroll
    for (int i = 0; i < LW; ++i) {
        const int q = wave + NW * i;
        ow[i] = 2u * (unsigned)(min(n0 + 8 * q + lr, D - 1) * K) + ((q & 1) ? c0 ^ 4 : c0) * 16u;
    }
    const unsigned ring_at = __builtin_amdgcn_readfirstlane(lds_addr_of(pt_lds));
    auto issue = [&](int kt, int s) {
        const unsigned at = ring_at + s * STAGE, p0 = patch_piece(pr, 8 * kt + c0), p1 = patch_piece(pr, 8 * kt + (c0 ^ 4));
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int q = wave + NW * i;
            glds16_if(pa.frames, oa[i] + ((q & 1) ? p1 : p0), at + q * 1024, nk - kt);
        }
#pragma unroll
        for (int i = 0; i < LW; ++i) glds16_if(W + (size_t)kt * 64, ow[i], at + (BM / 8 + wave + NW * i) * 1024, nk - kt);
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue(s, s);
    f32x16 acc[WC] = {};                                       // row 32 wr + lm, columns 32 (WC wc + j) + 8 q + 4 lh + z
    const int sw = (lm >> 1) & 7;
    int s = 0;
    for (int kt = 0; kt < nk; ++kt) {
        // k-tile kt has landed once the loads of the NS - 2 behind it alone are pending; past the barrier everybody is done with the stage before
        rl_wait_barrier<(NS - 2) * (LA + LW)>();
        issue(kt + NS - 1, s == 0 ? NS - 1 : s - 1);
        const bf16_t *at = (const bf16_t *)(pt_lds + s * STAGE) + (32 * wr + lm) * 64, *wt = (const bf16_t *)(pt_lds + s * STAGE) + (BM + 32 * WC * wc + lm) * 64;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int ko = ((2 * kk + lh) ^ sw) << 3;
            const bf16x8 x = *(const bf16x8 *)(at + ko);
#pragma unroll
            for (int j = 0; j < WC; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8 *)(wt + j * 2048 + ko), x, acc[j], 0, 0, 0);
        }
        s = s + 1 == NS ? 0 : s + 1;
    }
    // 32 x 32 results at a time through LDS of the wave's own (the ring is dead once every wave is here), 128 bytes of a row from eight lanes
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    float *stg = (float *)pt_lds + wave * (32 * PITCH);
    const int ch = lane & 7;
    size_t to[4];
    int from[4];
    bool there[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = t0 + 32 * wr + 8 * q + lr, f = r / P, t = r - f * P;
        there[q] = r < rows;
        to[q] = ((size_t)f * (P + 1) + 1 + t) * D;
        from[q] = (1 + t) * D;
    }
#pragma unroll
    for (int j = 0; j < WC; ++j) {
        const int col = n0 + 32 * (WC * wc + j) + 4 * ch, cc = min(col, D - 4);
        const f32x4 b = *(const f32x4 *)(bias + cc);
        f32x4 pos[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) pos[q] = *(const f32x4 *)(pa.pos + from[q] + cc);
#pragma unroll
        for (int q = 0; q < 4; ++q) *(f32x4 *)(stg + lm * PITCH + 8 * q + 4 * lh) = f32x4{acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 v = *(const f32x4 *)(stg + (8 * q + lr) * PITCH + 4 * ch) + b + pos[q];
            if (there[q] && col < D) *(f32x4 *)(pa.x + to[q] + col) = v;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

template <int WM, int WN, int WC, int NS> int launch_rows_t(const PatchArgs &pa, const PatchRows &pr, const bf16_t *W, const float *bias, int D, hipStream_t st)
{
    constexpr int BM = 32 * WM, BN = 32 * WN * WC, LDS = NS * (BM + BN) * 128;
    auto kern = patch_rows_kernel<WM, WN, WC, NS>;
    static bool attr_set = false;       // raising the dynamic LDS limit is a per-kernel, process-wide setting
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS) != hipSuccess) return POLY_EHIP;
        attr_set = true;
    }
    const int tiles_m = (pa.F * pr.gw * pr.gh + BM - 1) / BM, tiles_n = (D + BN - 1) / BN, job_wgs = patch_job_wgs(pa, D);
    const long tile_wgs = ((long)tiles_m * tiles_n + 7) / 8 * 8;
    POLY_LAUNCH_SHMEM(POLY_STAGE_GEMM, kern, dim3((unsigned)(tile_wgs + job_wgs + (pa.prep.row_offsets ? 1 : 0))), dim3(64 * WM * WN), LDS, st, pa, pr, W, bias, D,
                      3 * pa.p * pa.p, tiles_m, tiles_n, (int)tile_wgs, job_wgs);
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

}  // namespace

// A piece of 16 bytes never crosses from one image row of a patch to the next nor lies off a 16-byte boundary
bool patch_rows_fits(const PatchArgs &pa, const void *Wt, const float *bias, int D)
{
    const size_t row_bytes = (size_t)pa.W * 6, K = 3 * (size_t)pa.p * pa.p;
    return pa.F > 0 && K % 64 == 0 && K <= 4096 && (3 * pa.p) % 8 == 0 && D % 64 == 0 && row_bytes * pa.H * pa.F <= 0x7fffffffu && row_bytes % 16 == 0 &&
           aligned16(pa.frames) && aligned16(Wt) && aligned16(bias) && aligned16(pa.pos) && aligned16(pa.x);
}

// Small tiles as long as a few rounds of them are all, then tiles that read the frames once per 192 columns.  us per forward, 64 x 64 / 128 x 192: 192 columns, 200
// frames of 224 x 224 (1839 tiles of 64 x 64) 989 / 992, 250 (2298) 1084 / 1067, 333 (3063) 1871 / 1852, 64 469 / 471, 32 445 / 451; 768 columns, 48 frames
// (1764) 2663 / 2667, 64 (2352) 3460 / 3454.
int launch_patch_rows(const PatchArgs &pa, const void *Wt, const float *bias, int D, hipStream_t st)
{
    const PatchRows pr = patch_rows(pa, 2);
    const long small = ((long)pa.F * pr.gw * pr.gh + 63) / 64 * (D / 64);
    return small > 2048 && D % 192 == 0 ? launch_rows_t<4, 2, 3, 3>(pa, pr, (const bf16_t *)Wt, bias, D, st)
                                        : launch_rows_t<2, 2, 1, 3>(pa, pr, (const bf16_t *)Wt, bias, D, st);
}
