// A run of whole layers of a model 192 wide in ONE launch, on tiles of 64 token rows: a workgroup keeps its rows from the first layer of the run to the last.
//
// rowlayer.hip and attention.hip are two launches a layer: every one starts cold (4 us to issue and dispatch, 2 to 3 us until the first tile written by the launch
// before is usable), the residual stream goes out and comes back, and attention stages keys and values in LDS once more.  Here the up to four workgroups that
// hold a block's rows run side by side, one per CU, and meet once a layer:
//     C   [q k v] = LayerNorm1(x) Wq + bq (+ low rank)      q stays in LDS; k and v, in the order attention reads them, go out at device scope
//     ..  the tiles of the block have all done so
//     att o = softmax(q k^T / 8) v                          a wave per (head, 32 queries), k and v straight into registers, o over q in LDS
//     A, B of rowlayer.hip                                  x, 24 fp32 registers of a lane, never leaves them
// The products, LayerNorms and the GELU are rowlayer.hip's, on the same slots of weights, in the same order of sums.
//
// Handing k and v over without fences: as in flow.hip.  They are stored at device scope, the stores are waited for, then the tile is counted; every layer of a
// launch has buffers of its own, so no address is read by this launch before it has been written for good and no cache holds an old copy of it.  A 1 KB
// piece is written by one workgroup.
//
// Order and progress: tickets of eight queues, block b in queue b % 8, the tiles of a block consecutive.  (Workgroups are dealt to the XCDs in turn, so a block's
// tiles mostly share an L2; nothing rests on that.)  A workgroup finishes the tile it has drawn before it draws another, from its own queue first, then from
// the others, and leaves when all are empty.  A tile waits only for tiles of its own block.  At any time at most one block per queue has tickets not
// yet drawn, so at most 8 x 3 workgroups wait for tiles that nobody has; all others come to their end, and with 25 CUs for the launch one of them draws the next
// ticket.  Nobody else writes the counters; should two calls use one workspace at a time, the looks at a counter are limited as in flow.hip.
#include "flow_dev.h"

#include <type_traits>

namespace {

constexpr int RN_THREADS = 512;
constexpr int RN_TILE = 8192;       // bytes of a [64][64] bf16 tile in LDS: 128 bytes a row, its 16-byte pieces permuted
constexpr int RN_TILES = 4;         // of activations
constexpr int RN_MAX_DM = 768;
constexpr int RN_GELU = (GELU_TAB_ENTRIES + 1) & ~1;    // (what lies behind is read in 16-byte pieces)
constexpr int RN_AT_STRIDE = 200;   // elements per rank row of At_k in LDS (192 + 8: rows start 4 banks apart)
constexpr int RN_QUEUES = 8;
constexpr int KT = 3, D = 64 * KT, HEADS = KT, Nq = 3 * D, NQ = (Nq + 127) / 128;
constexpr int CT = KT;                                     // column tiles of 16 per wave of a product with D columns
constexpr int SLOT = KT * 2048;                            // bytes of a slot: 16 rows of D columns, or 16 CT rows of 64 columns
constexpr int RN_END = 16384;                              // the region from stat_s on
constexpr int RN_LDS = RN_TILES * RN_TILE + 16 * SLOT + (RN_MAX_DM + Nq + 2 * D + 4 * D) * 4 + RN_GELU * 8 + RN_END + 64;
static_assert(RN_LDS <= 160 * 1024, "LDS budget");

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) char *lds_ptr;
typedef const __attribute__((address_space(4))) RowRunArgs *RunPtr;

// The arguments are read where they are used (scalar loads that hit the scalar cache): held in registers across the layers they would push others out
__device__ __forceinline__ RunPtr run_args()
{
    RunPtr p = (RunPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48 that share a token row, in every one of them
__device__ __forceinline__ float quad16_sum(float v)
{
    unsigned p = __builtin_bit_cast(unsigned, v);
    const u32x2 a = __builtin_amdgcn_permlane32_swap(p, p, false, false);
    const unsigned a0 = a[0], a1 = a[1];
    p = __builtin_bit_cast(unsigned, __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1));
    const u32x2 b = __builtin_amdgcn_permlane16_swap(p, p, false, false);
    const unsigned b0 = b[0], b1 = b[1];
    return __builtin_bit_cast(float, b0) + __builtin_bit_cast(float, b1);
}

// NKT: key tiles of 32 at most
template <int NKT> __global__ __launch_bounds__(RN_THREADS, 2) void rowrun_kernel(const RowRunArgs)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char *As = lds;                                        // activations: KT tiles [64][64] bf16; two pairs of tiles for the hidden columns
    char *Ws = lds + RN_TILES * RN_TILE;                   // two slots per wave
    float *b1_s = (float *)(Ws + 16 * SLOT);               // [Dm]
    float *bq_s = b1_s + RN_MAX_DM;                        // [3 D]
    float *bp_s = bq_s + Nq;                               // [D]
    float *b2_s = bp_s + D;                                // [D]
    float *gb2_s = b2_s + D;                               // LayerNorm2 gain [D], shift [D]
    float *gbq_s = gb2_s + 2 * D;                          // LayerNorm1 gain, shift
    float *gelu_s = gbq_s + 2 * D;
    f32x2 *stat_s = (f32x2 *)(gelu_s + 2 * RN_GELU);       // [64][4]: mean and squared deviations of a wave's columns of a row
    s16x4 *sh_s = (s16x4 *)stat_s;                         // in C: shrink output, [4][64 lanes]; from its second round on two tiles of keys
    bf16_t *at_s = (bf16_t *)(stat_s + 64 * 4);            // At_k of the phase, [16][RN_AT_STRIDE]
    bf16_t *bt_s = at_s + 16 * RN_AT_STRIDE;               // Bt_k of A, [D][r]
    int *word_s = (int *)((char *)stat_s + RN_END);        // [0] ticket, [1] looks left

    const int tid0 = threadIdx.x;
    const int nb = [&]() { const RunPtr p = run_args(); const int *dev = p->nb_dev; return dev ? min(uload(dev), p->nb) : p->nb; }();
    if (tid0 == 0) word_s[1] = run_args()->patience;
#pragma unroll
    for (int j = 0; j < 2; ++j) {                          // Phi table of the GELU
        const int i = tid0 + RN_THREADS * j;
        if (i < GELU_TAB_ENTRIES) *(f32x2 *)(gelu_s + 2 * i) = gelu_tab_entry(i);
    }
    if (nb <= 0) return;
    // this launch's layers: as many as there are buffers for, of the blocks that exist
    int l0, l1;
    {
        const RunPtr p = run_args();
        const int n = min(p->layers, p->capacity / nb);
        l0 = p->launch * n;
        l1 = min(l0 + n, p->layers);
    }
    int queue = blockIdx.x & (RN_QUEUES - 1), left = l0 < l1 ? RN_QUEUES : 0;
    while (left > 0) {
    // ---- the next tile
    unsigned ticket;
    {
        const RunPtr p = run_args();
        __syncthreads();
        if (tid0 == 0) word_s[0] = (int)__hip_atomic_fetch_add(p->counters + queue * 16, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        ticket = __builtin_amdgcn_readfirstlane(word_s[0]);
    }
    const int tiles = run_args()->tiles;
    const int nbq = nb > queue ? (nb - queue + RN_QUEUES - 1) / RN_QUEUES : 0;
    if (ticket >= (unsigned)(nbq * tiles)) {
        --left;
        queue = (queue + 1) & (RN_QUEUES - 1);
        continue;
    }
    const int ob = queue + RN_QUEUES * (int)(ticket / (unsigned)tiles), tile = (int)(ticket % (unsigned)tiles);
    // Everything made of the thread's number is made anew for every phase from a copy that the compiler cannot see through: kept from phase to phase, or hoisted
    // out of the loop over the layers, it would be spilled.
    int tid, lane, wave, kh, wc, lm, lg, lr, wrow, wcol;
    unsigned slot0, off_d, off_m;
    lds_ptr act[2], wn[2];                                 // [k & 1]: rows of activations, rows of a slot
    auto renew = [&]() {
        tid = tid0;
        asm volatile("" : "+v"(tid));
        lane = tid & 63; wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        kh = wave >> 2; wc = wave & 3; lm = lane & 15; lg = lane >> 4; lr = lane >> 3;
        // slots of weights: 8 rows x 128 bytes per instruction, the swizzle of the LDS rows applied on the global side
        slot0 = __builtin_amdgcn_readfirstlane(lds_addr_of(Ws)) + wave * (2 * SLOT);                // N slot, then K slot
        const unsigned piece = (unsigned)(((lane & 7) ^ (lr >> 1)) << 4);                           // of rows lr; of rows 8 + lr: ^ 64
        off_d = (unsigned)lr * (D * 2) + piece;
        off_m = (unsigned)lr * (run_args()->Dm * 2) + piece;
        // the residual stream of the row half kh: row lm of tile rt, columns 16 CT wc + 16 ct + 4 lg + {0..3}
        wrow = 32 * kh; wcol = 16 * CT * wc + 4 * lg;
        // operands: a fragment is 16 rows x 32 contraction columns, lane (lm, lg) holds columns 8 lg .. + 7 of row lm, the 16-byte piece
        // (4 kk + lg) ^ (row >> 1 & 7) of a 128-byte row
        const int fo0 = lm * 128 + ((lg ^ ((lm >> 1) & 7)) << 4);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            act[k] = (lds_ptr)(As + (fo0 ^ (64 * k)));
            wn[k] = (lds_ptr)(Ws + wave * (2 * SLOT) + (fo0 ^ (64 * k)));
            asm("" : "+v"(act[k]));
            asm("" : "+v"(wn[k]));
        }
    };
    renew();
    const int T = run_args()->T, Dm = run_args()->Dm, nc = (Dm + 127) >> 7, r = run_args()->r;
    const int t0 = tile * 64, rows = min(64, T - t0), nkt = (T + 31) >> 5;        // key tiles of 32
    const float scale = run_args()->scale, eps = run_args()->eps;
    int k_ad = -1;
    { const RunPtr p = run_args(); if (p->adapter_of_row) k_ad = uload(p->adapter_of_row + ob); }
    const bool lora_p = k_ad >= 0 && run_args()->Ap, lora_q = k_ad >= 0 && run_args()->Aq;

    auto issue_n = [&](const bf16_t *W, int row, unsigned slot) {      // 16 rows of a matrix with D columns from row `row`
#pragma unroll
        for (int j = 0; j < 2 * KT; ++j) glds16_s(W + (size_t)(row + 8 * (j & 1)) * D + 64 * (j >> 1), off_d ^ (64 * (j & 1)), slot + j * 1024);
    };
    // first row of W1 / first column of W2 that this wave multiplies of chunk c (the last chunk may be half a one: what lies past it is not used)
    auto row_n = [&](int c) { return min(128 * c + 16 * wave, Dm - 16); };
    auto col_k = [&](int c) { return min(128 * c + 64 * kh, Dm - 64); };
    // rounds of C: 128 columns of Wq at a time, keys first, then values, queries last (they stay here, so keys and values are on their way under them)
    auto round_of = [](int s) { return s == 0 ? 2 : s == 1 ? 1 : s == 2 ? 3 : s == 3 ? 4 : 0; };
    auto row_q = [&](int s) { const int q = round_of(s); return 128 * q + 16 * (q < 4 ? wave : wc); };
    auto slot_q = [&](int s) { return slot0 + (s & 1 ? 0 : SLOT); };
    // vectors -> LDS, 64 floats per instruction (any alignment of a float), shared out by wave
    auto vec = [&](const float *src, int from, int to, const float *dst) {
        for (int i = from; i < to; i += 64) glds4(src + i + lane, __builtin_amdgcn_readfirstlane(lds_addr_of(dst)) + i * 4);
    };
    auto vectors_q = [&](int l) {                          // of C
        const RunPtr p = run_args();
        if (wave == 4) { vec(p->ln1_g + (size_t)l * D, 0, D, gbq_s); vec(p->ln1_b + (size_t)l * D, 0, D, gbq_s + D); }
        if (wave == 5 || wave == 6) vec(p->bq + (size_t)l * Nq, (wave - 5) * 320, wave == 5 ? 320 : Nq, bq_s);
    };
    auto vectors = [&](int l) {                            // of A and B
        const RunPtr p = run_args();
        if (wave == 0) vec(p->b1 + (size_t)l * Dm, 0, Dm >> 1 & ~63, b1_s);
        if (wave == 1) vec(p->b1 + (size_t)l * Dm, Dm >> 1 & ~63, Dm, b1_s);
        if (wave == 2) { vec(p->bp + (size_t)l * D, 0, D, bp_s); vec(p->b2 + (size_t)l * D, 0, D, b2_s); }
        if (wave == 3) { vec(p->ln2_g + (size_t)l * D, 0, D, gb2_s); vec(p->ln2_b + (size_t)l * D, 0, D, gb2_s + D); }
    };
    // At_k [r][D] -> at_s, a rank row per instruction
    auto issue_at = [&](const bf16_t *At_k) {
        for (int rk = wave; rk < r; rk += 8)
            if (lane < D / 8) glds16(At_k + rk * D + lane * 8, __builtin_amdgcn_readfirstlane(lds_addr_of(at_s + rk * RN_AT_STRIDE)));
    };
    // the adapter's slab of layer l in a stack with `width` elements per rank
    auto slab = [&](const bf16_t *stack, int l, int width) { return stack + ((size_t)l * run_args()->n_adapters + k_ad) * r * width; };
    // rank lm (repeated past r: such ranks meet zeros of Bt_k), columns 32 k + 8 lg + {0..7}
    auto at_frag = [&](int k) { return *(const bf16x8 *)(at_s + min(lm, r - 1) * RN_AT_STRIDE + 32 * k + 8 * lg); };
    // column n of Bt_k [.][r], ranks 4 lg + {0..3} (r is a multiple of 4; zero where the rank does not exist)
    auto bt_frag = [&](const bf16_t *Bt_k, int n) { return *(const s16x4 *)(Bt_k + n * r + min(4 * lg, r - 4)); };
    // four ranks of a lane as a step of 32, the other four zeros on both sides: v_mfma_f32_16x16x16_bf16 takes several times as long (the five rounds of C 10.0 k cycles with
    // it, 7.8 k like this)
    auto wide = [](s16x4 v) { return __builtin_bit_cast(bf16x8, __builtin_shufflevector(v, s16x4{0, 0, 0, 0}, 0, 1, 2, 3, 4, 5, 6, 7)); };
    auto bt_operand = [&](s16x4 v) { return 4 * lg < r ? v : s16x4{0, 0, 0, 0}; };
    auto rd = [&](lds_ptr p, int off) { return *(const __attribute__((address_space(3))) bf16x8 *)(p + off); };
    auto act_frag = [&](int tile, int rt, int kk) { return rd(act[kk], tile * RN_TILE + rt * 2048); };
    f32x4 x[CT][2];
    bf16x8 fa[2 * KT][4];                                  // the resident rows as the B operand of the transposed product
    auto load_fa = [&]() {
#pragma unroll
        for (int k = 0; k < 2 * KT; ++k)
#pragma unroll
            for (int rt = 0; rt < 4; ++rt) fa[k][rt] = act_frag(k >> 1, rt, k & 1);
    };
    // s (x At_k): ranks 4 lg + {0..3} of row lm, the operand of the expand as it is
    auto shrink_out = [&](f32x4 c) {
        const bf16x4 o = {(bf16_t)(scale * c[0]), (bf16_t)(scale * c[1]), (bf16_t)(scale * c[2]), (bf16_t)(scale * c[3])};
        return __builtin_bit_cast(s16x4, o);
    };
    // 4 columns 16 cg + 4 lg + {0..3} (cg < 4) of row 16 rt + lm -> a [64][64] tile
    auto put = [&](char *tile, int cg, int rt, f32x4 v) {
        const bf16x4 o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
        *(bf16x4 *)(tile + (16 * rt + lm) * 128 + (((2 * cg + (lg >> 1)) ^ ((lm >> 1) & 7)) << 4) + 8 * (lg & 1)) = o;
    };
    // The sums over the two halves of the contraction meet: a wave hands the row half that is not its own to the wave with the same columns, through
    // a slot of its own, and adds what it is handed.
    auto exchange = [&](f32x4 (&acc)[CT][4], f32x4 (&own)[CT][2], int slot) {
        f32x4 *mine = (f32x4 *)(Ws + wave * (2 * SLOT) + slot) + lane;
        const f32x4 *theirs = (const f32x4 *)(Ws + (wave ^ 4) * (2 * SLOT) + slot) + lane;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                mine[(ct * 2 + rt) * 64] = kh ? acc[ct][rt] : acc[ct][2 + rt];
                own[ct][rt] = kh ? acc[ct][2 + rt] : acc[ct][rt];
            }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) own[ct][rt] += theirs[(ct * 2 + rt) * 64];
    };
    // LayerNorm (fp32 statistics, centred second moments of 16 CT columns each, put together by Chan's rule) of x -> bf16 tiles at As -> fragments.
    // Behind the first barrier every wave is done with what it read before: `between` runs there.
    auto layernorm = [&](const float *gb_s, auto between) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            float t = 0.f;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) t += (x[ct][rt][0] + x[ct][rt][1]) + (x[ct][rt][2] + x[ct][rt][3]);
            const float m = quad16_sum(t) * (1.0f / (16 * CT));
            float q = 0.f;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int z = 0; z < 4; ++z) { const float d = x[ct][rt][z] - m; q = fmaf(d, d, q); }
            q = quad16_sum(q);
            if (lg == 0) stat_s[(wrow + 16 * rt + lm) * 4 + wc] = f32x2{m, q};
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        between();
        f32x4 g[CT], b[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) { g[ct] = *(const f32x4 *)(gb_s + wcol + 16 * ct); b[ct] = *(const f32x4 *)(gb_s + D + wcol + 16 * ct); }
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            const int row = wrow + 16 * rt + lm;
            const f32x4 s0 = *(const f32x4 *)(stat_s + row * 4), s1 = *(const f32x4 *)(stat_s + row * 4 + 2);
            const float mean = 0.25f * ((s0[0] + s0[2]) + (s1[0] + s1[2]));
            const float d0 = s0[0] - mean, d1 = s0[2] - mean, d2 = s1[0] - mean, d3 = s1[2] - mean;
            const float q = (s0[1] + s0[3]) + (s1[1] + s1[3]) + (16 * CT) * ((d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3));
            const float inv = rsqrtf(q * (1.0f / D) + eps), nmi = -mean * inv;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                bf16x4 o;
#pragma unroll
                for (int z = 0; z < 4; ++z) o[z] = (bf16_t)fmaf(fmaf(x[ct][rt][z], inv, nmi), g[ct][z], b[ct][z]);   // ((x - mean) inv) g + b
                const int col = wcol + 16 * ct;
                *(bf16x4 *)(As + (col >> 6) * RN_TILE + row * 128 + ((((col & 63) >> 3) ^ ((lm >> 1) & 7)) << 4) + 2 * (col & 4)) = o;
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        load_fa();
    };
    constexpr int NS = 4 * KT;                             // MFMAs of a segment
    // a segment: every MFMA is followed by a share of the other work
    auto segment = [&](auto mfma, auto side) {
#pragma unroll
        for (int n = 0; n < NS; ++n) {
            mfma(n);
            side(n);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // pieces 0 .. count - 1 over the slots [first, last) of a segment
    auto share = [&](int n, int first, int last, int count, auto piece) {
#pragma unroll
        for (int j = 0; j < count; ++j)
            if (n == first + j * (last - first) / count) piece(j);
    };


    // ---- prologue: the rows, and what the first C needs
    {
        const RunPtr p = run_args();
        issue_n(p->Wq + (size_t)l0 * Nq * D, row_q(0), slot_q(0));
        vectors_q(l0);
        if (lora_q) issue_at(slab(p->Aq, l0, D));
        const float *src = (l0 ? p->x_out : p->x_in) + ((size_t)(p->in_map && l0 == 0 ? uload(p->in_map + ob) : ob) * T + t0) * D;
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) x[ct][rt] = *(const f32x4 *)(src + (unsigned)(min(wrow + 16 * rt + lm, rows - 1) * D + wcol + 16 * ct));
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
#pragma unroll 1
    for (int l = l0; l < l1; ++l) {
        renew();
        const size_t slot = (size_t)(l - l0) * nb + ob;                // of keys and values
        const bool end = l + 1 == run_args()->layers && run_args()->class_rows;        // nothing but the first row of a block is read of what comes out
        // ============================================================ C: q, k, v = LayerNorm1(x) Wq + bq + lora
        {
            const bf16_t *Wq = run_args()->Wq + (size_t)l * Nq * D;
            s16x4 b2[NQ] = {};                                         // Bt_k of the rounds
            if (lora_q) {
                const bf16_t *Bq_k = slab(run_args()->Bq, l, Nq);
#pragma unroll
                for (int s = 0; s < NQ; ++s) b2[s] = bt_frag(Bq_k, row_q(s) + lm);
            }
            layernorm(gbq_s, [&]() {
#pragma unroll
                for (int s = 0; s < NQ; ++s) asm volatile("" : "+v"(b2[s]));   // (waited for here: behind loads that the compiler does not know it would wait for those too)
                issue_n(Wq, row_q(1), slot_q(1));
            });
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * KT) : "memory");     // round 0 and At_k; round 1 is on its way
            s16x4 fs[4];
            if (lora_q) {                                              // one row tile per wave, to every wave
                asm volatile("s_barrier" ::: "memory");
                f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 2 * KT; ++k) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at_frag(k), rd(act[k & 1], (k >> 1) * RN_TILE + wc * 2048), c, 0, 0, 0);
                if (!kh) sh_s[wc * 64 + lane] = shrink_out(c);
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
                for (int rt = 0; rt < 4; ++rt) fs[rt] = sh_s[rt * 64 + lane];
            }
            char *const keys = (char *)stat_s;                         // of heads 1 and 2; of head 0 in tile 3
            const RunPtr p = run_args();
            // of a block, per 32 keys and head: 4 KB in the order of the fragments (what a tile has past the last 32 is past the end, where stores are dropped)
            const size_t piece = HEADS * 2048;
            const Buf kb(p->k + slot * nkt * piece, (unsigned)(nkt * piece) * 2u), vb(p->v + slot * nkt * piece, (unsigned)(nkt * piece) * 2u);
            bf16x8 W[2][2 * KT];
            auto fetch = [&](int s, int j) { W[s & 1][j] = rd(wn[j & 1], (s & 1 ? 0 : SLOT) + (j >> 1) * 2048); };
#pragma unroll
            for (int j = 0; j < 2 * KT; ++j) fetch(0, j);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int s = 0; s < NQ; ++s) {
                const bool full = s != 3, values = s == 2 || s == 3;   // values: rows down the accumulator, so that a lane has four keys of a column
                const int col = row_q(s);
                if (s + 2 < NQ) issue_n(Wq, row_q(s + 2), slot_q(s + 2));      // W[s & 1] is in registers
                f32x4 b;
                if (values) { const float t = bq_s[col + lm]; b = f32x4{t, t, t, t}; }
                else b = *(const f32x4 *)(bq_s + col + 4 * lg);
                f32x4 acc[4] = {b, b, b, b};
                if (lora_q) {
                    const bf16x8 w = wide(bt_operand(b2[s]));
#pragma unroll
                    for (int rt = 0; rt < 4; ++rt)
                        acc[rt] = values ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(wide(fs[rt]), w, b, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, wide(fs[rt]), b, 0, 0, 0);
                }
                auto mfma = [&](int n, int rt0) {
                    const int k = n / 2, rt = rt0 + n % 2;
                    const f32x4 c = acc[rt];
                    acc[rt] = values ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[k][rt], W[s & 1][k], c, 0, 0, 0)
                                     : __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[s & 1][k], fa[k][rt], c, 0, 0, 0);
                };
                auto next = [&](int n) {                               // the operands of the next round
                    if (s + 1 == NQ) return;
                    // behind the next round's weights: those of the round after it; the three stores of the keys; the four of a full round of values
                    if (n == 0 && s == 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * KT) : "memory");
                    if (n == 0 && s == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * KT) : "memory");
                    if (n == 0 && s == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * KT + 3) : "memory");
                    if (n == 0 && s == 3) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
                    share(n, 0, NS - 2, 2 * KT, [&](int j) { fetch(s + 1, j); });
                };
                if (full) {
                    segment([&](int n) { mfma(n, 0); }, next);
                    segment([&](int n) { mfma(n, 2); }, [&](int n) {});
                } else {                                               // half a round: 64 columns, every wave 16 of them for its row half
                    if (kh) {
                        segment([&](int n) { mfma(n, 2); }, next);
                        acc[0] = acc[2];
                        acc[1] = acc[3];
                    } else {
                        segment([&](int n) { mfma(n, 0); }, next);
                    }
                }
                if (values) {
                    // keys 16 kt + 4 lg + {0..3} of column 16 cg + lm of a head: half lg / 2 of lane 32 (lg % 2) + column % 32 of a fragment of 16 keys x 32 columns
                    const int head = full ? kh : 2, cg = wc;
                    const unsigned off = (unsigned)((tile * 2 * HEADS + head) * 4 + (cg >> 1)) * 1024u + (unsigned)((lg & 1) * 32 + (cg & 1) * 16 + lm) * 16u + (unsigned)(lg >> 1) * 8u;
#pragma unroll
                    for (int rt = 0; rt < (full ? 4 : 2); ++rt) {
                        const unsigned k16 = (unsigned)(full ? rt : 2 * kh + rt);
                        vb.st8(__builtin_bit_cast(u32x2_, pack4(acc[rt])), off + (k16 >> 1) * (HEADS * 4096u) + (k16 & 1) * 2048u);
                    }
                } else {
                    if (s == 0) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // every wave has its operands and the shrink output
                    char *const to = s == 0 ? keys + kh * RN_TILE : As + (s == 1 ? 2 + kh : kh) * RN_TILE;
#pragma unroll
                    for (int rt = 0; rt < 4; ++rt) put(to, wc, rt, acc[rt]);
                    if (s == 1) {                                      // all keys are staged: 16 columns x 32 rows of every head per wave
                        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                        const int row = 32 * kh + (lane & 31), at = row * 128 + (((2 * wc + (lane >> 5)) ^ ((row >> 1) & 7)) << 4);
                        u32x4_ v[HEADS];
#pragma unroll
                        for (int h = 0; h < HEADS; ++h) v[h] = *(const u32x4_ *)((h == 0 ? As + 3 * RN_TILE : keys + (h - 1) * RN_TILE) + at);
#pragma unroll
                        for (int h = 0; h < HEADS; ++h) kb.st16(v[h], (unsigned)(((tile * 2 + kh) * HEADS + h) * 4 + wc) * 1024u + lane * 16u);
                    }
                }
            }
        }
        // ---- keys and values have reached device scope: the tile is counted, and its block's others are waited for
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        renew();
        unsigned *const count = run_args()->counters + (RN_QUEUES + ob) * 16;
        if (tid == 0) __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (end && tile) break;
        auto proj_loads = [&]() {
            // Wp: rows 16 CT wc .., columns 64 t + 32 kh .. + 31 as [16 CT][32], 16 rows x 64 bytes per instruction
            const RunPtr p = run_args();
            const bf16_t *Wp = p->Wp + (size_t)l * D * D;
            const unsigned vo = (unsigned)(lane >> 2) * (D * 2) + (((lane & 3) ^ ((lane >> 4) & 3)) << 4);
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) glds16_s(Wp + (size_t)(16 * CT * wc + 16 * ct) * D + 64 * t + 32 * kh, vo, slot0 + (t * CT + ct) * 1024);
            vectors(l);
            if (l + 1 < l1) vectors_q(l + 1);
            if (lora_p) {
                issue_at(slab(p->Ap, l, D));
                const char *Bt_k = (const char *)slab(p->Bp, l, D);
                const int n16 = D * r / 8;                             // 16-byte pieces
                for (int i = wave * 64; i < n16; i += 512)
                    if (i + lane < n16) glds16(Bt_k + (i + lane) * 16, __builtin_amdgcn_readfirstlane(lds_addr_of(bt_s)) + i * 16);
            }
        };
        // (the wave that waits requests its own behind the barrier: it has nothing to do in attention)
        if (wave == 7) {
            const unsigned want = tiles > 1 ? (unsigned)(l - l0 + 1) * tiles : 0;
            while (want && peek(count) < want) {
                const int looks = word_s[1] - 1;
                word_s[1] = looks;
                if (looks < 0) break;
                __builtin_amdgcn_s_sleep(1);
            }
        } else {
            proj_loads();
        }
        asm volatile("s_barrier" ::: "memory");
        if (wave == 7) proj_loads();
        // ============================================================ attention: waves 0 .. 2 rows 0 .. 31 of a head each, 3 .. 5 the others
        if (wave < HEADS || (wave < 2 * HEADS && rows > 32 && !end)) {
            const int h = wave < HEADS ? wave : wave - HEADS, j = wave < HEADS ? 0 : 1, am = lane & 31, ah = lane >> 5;
            const RunPtr p = run_args();
            const size_t at = (slot * nkt * HEADS + h) * 2048 + lane * 8;
            const bf16_t *const kp = p->k + at, *const vp = p->v + at;
            char *const q = As + h * RN_TILE + (32 * j + am) * 128;    // this lane's query
            const int sw = (am >> 1) & 7;
            bf16x8 qf[4], kf[4][4], vf[2 * NKT][2];
#pragma unroll
            for (int ds = 0; ds < 4; ++ds) qf[ds] = *(const bf16x8 *)(q + (((2 * ds + ah) ^ sw) << 4));
            // (tiles past the last repeat it: their probabilities are 0)
            auto load_k = [&](int kt) {
#pragma unroll
                for (int ds = 0; ds < 4; ++ds) kf[kt & 3][ds] = *(const bf16x8 *)(kp + min(kt, nkt - 1) * (HEADS * 2048) + ds * 512);
            };
            auto load_v = [&](int kt) {
#pragma unroll
                for (int st = 0; st < 2; ++st)
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt) vf[2 * kt + st][dt] = *(const bf16x8 *)(vp + min(kt, nkt - 1) * (HEADS * 2048) + (st * 2 + dt) * 512);
            };
#pragma unroll
            for (int kt = 0; kt < (NKT < 4 ? NKT : 4); ++kt) load_k(kt);
            f32x16 s[NKT];
#pragma unroll
            for (int kt = 0; kt < NKT; ++kt) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 16; ++e) s[kt][e] = 0.f;
#pragma unroll
                for (int ds = 0; ds < 4; ++ds) s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kt & 3][ds], qf[ds], s[kt], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (kt + 4 < NKT) load_k(kt + 4);
                else load_v(kt + 4 - NKT < 0 ? 0 : NKT < 4 ? kt : kt + 4 - NKT);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kt = 0; kt < NKT; ++kt)
                if (32 * kt + 32 > T) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) s[kt][e] = 32 * kt + 8 * (e >> 2) + 4 * ah + (e & 3) < T ? s[kt][e] : -INFINITY;
                }
            float mx = -INFINITY;
#pragma unroll
            for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
                for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[kt][e]);
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float sc = 0.125f * FL_LOG2E, off = -mx * sc;        // 1/sqrt(64), folded into the base-2 exponent
            float sum = 0.f;
            bf16x8 pf[NKT][2];
#pragma unroll
            for (int kt = 0; kt < NKT; ++kt) {
#pragma unroll
                for (int hs = 0; hs < 2; ++hs)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float pr = __builtin_amdgcn_exp2f(fmaf(s[kt][hs * 8 + e], sc, off));
                        sum += pr;
                        pf[kt][hs][e] = (bf16_t)pr;
                    }
                __builtin_amdgcn_sched_barrier(0);
                if (kt >= 4) load_v(kt);
            }
            sum += __shfl_xor(sum, 32, 64);
            f32x16 o[2];
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
#pragma unroll
            for (int st = 0; st < 2 * NKT; ++st)
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[st][dt], pf[st >> 1][st & 1], o[dt], 0, 0, 0);
            const float inv = 1.0f / sum;
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *(bf16x4 *)(q + (((dt * 4 + g) ^ sw) << 4) + 8 * ah) = pack4(f32x4{o[dt][4 * g] * inv, o[dt][4 * g + 1] * inv, o[dt][4 * g + 2] * inv, o[dt][4 * g + 3] * inv});
        }
        renew();
        const bf16_t *W1 = run_args()->W1 + (size_t)l * Dm * D, *W2 = run_args()->W2 + (size_t)l * Dm * D;
        // W2: rows 16 CT wc .., 64 columns from column `col`
        auto issue_k1 = [&](int col, int j) { glds16_s(W2 + (size_t)(16 * CT * wc + 8 * j) * Dm + col, off_m ^ (64 * (j & 1)), slot0 + SLOT + j * 1024); };
        // ============================================================ A: x' = x + o Wp + bp + lora
        f32x4 y[CT][4];
        rl_wait_barrier<0>();                              // o is there, Wp, At_k, Bt_k and the vectors have landed
        {
            const lds_ptr wp = (lds_ptr)(Ws + wave * (2 * SLOT) + lm * 64 + ((lg ^ ((lm >> 2) & 3)) << 4));
            bf16x8 w[KT][CT], h[KT][4];
#pragma unroll
            for (int t = 0; t < KT; ++t) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) w[t][ct] = rd(wp, (t * CT + ct) * 1024);
#pragma unroll
                for (int rt = 0; rt < 4; ++rt) h[t][rt] = rd(kh ? act[1] : act[0], t * RN_TILE + rt * 2048);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue_n(W1, row_n(0), slot0);
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int rt = 0; rt < 4; ++rt)
                        y[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t][ct], h[t][rt], t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : y[ct][rt], 0, 0, 0);
        }
        {
            f32x4 own[CT][2];
            exchange(y, own, SLOT);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const f32x4 b = *(const f32x4 *)(bp_s + wcol + 16 * ct);
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) x[ct][rt] += own[ct][rt] + b;
            }
        }
        if (lora_p) {
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 2 * KT; ++k) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at_frag(k), rd(act[k & 1], (k >> 1) * RN_TILE + wrow * 128 + rt * 2048), c, 0, 0, 0);
                const s16x4 fs = shrink_out(c);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) x[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wide(bt_operand(bt_frag(bt_s, 16 * CT * wc + 16 * ct + lm))), wide(fs), x[ct][rt], 0, 0, 0);
            }
        }
        renew();
        layernorm(gb2_s, [&]() {
#pragma unroll
            for (int j = 0; j < 2 * CT; ++j) issue_k1(col_k(0), j);
        });
        // The second product of B adds to x' + b2 on half 0 of its contraction in every row, so that a row's bits do not depend on its place in the tile: the
        // waves of half 1 hand their rows over, in LDS that is in no use until the second chunk (tile 3, and what LayerNorm and A are done with).  0.3 us of a
        // launch of 248 tiles (twelve of them and the rest of 32 frames of 224 x 224, 62 blocks: 498 / 502 us; through the weight slots, before the first of
        // W1 is requested, 504).
        auto handed = [&](int ct, int rt) {
            const int i = ct * 2 + rt;
            return (f32x4 *)((i < 2 ? As + 3 * RN_TILE + i * 4096 : (char *)stat_s + (i - 2) * 4096) + wc * 1024) + lane;
        };
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const f32x4 b = *(const f32x4 *)(b2_s + wcol + 16 * ct), z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                if (kh) *handed(ct, rt) = x[ct][rt] + b;
                y[ct][rt] = kh ? z : x[ct][rt] + b;
                y[ct][2 + rt] = z;
            }
        }

        // ============================================================ B: x'' = x' + b2 + GELU(LayerNorm2(x') W1 + b1) W2
        bf16x8 wN[2 * KT], wK[2][CT], hk[2][4];
        f32x4 h[4];
        float xc[4];
        f32x2 en[4];
        const unsigned gelu_a = lds_addr_of(gelu_s);
        auto fetch_n1 = [&](int j) { wN[j] = rd(wn[j & 1], (j >> 1) * 2048); };
        auto fetch_w1 = [&](int kk, int j) { wK[kk][j] = rd(wn[kk], SLOT + j * 2048); };
        auto fetch_h1 = [&](int kk, int buf, int rt) { hk[kk][rt] = rd(act[kk], buf * (2 * RN_TILE) + kh * RN_TILE + rt * 2048); };
        auto mfma_n = [&](int n, int rt0, f32x4 b) {       // rows of two tiles
            const int k = n / 2, rt = rt0 + n % 2;
            h[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wN[k], fa[k][rt], k == 0 ? b : h[rt], 0, 0, 0);
        };
        auto mfma_k = [&](int n, int kk) {
            const int ct = n / 4, rt = n % 4;
            y[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wK[kk][ct], hk[kk][rt], y[ct][rt], 0, 0, 0);
        };
        // GELU of one row tile: four lookups, then (fin) the results
        auto look = [&](int rt, int j) { gelu_look(h[rt][j], gelu_a, xc[j], en[j]); };
        auto fin = [&](int rt, int buf) { put(As + buf * (2 * RN_TILE) + kh * RN_TILE, wc, rt, gelu_tab4(h[rt], xc, en)); };
        auto gelu_side = [&](int n, int rt0, int buf) {    // of two row tiles in a segment of NS slots
            share(n, 0, NS / 4, 4, [&](int j) { look(rt0, j); });
            if (n == NS / 2 - 1) fin(rt0, buf);
            share(n, NS / 2, 3 * NS / 4, 4, [&](int j) { look(rt0 + 1, j); });
            if (n == NS - 1) fin(rt0 + 1, buf);
        };
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * CT) : "memory");  // the first of W1; W2 is on its way
#pragma unroll
        for (int j = 0; j < 2 * KT; ++j) fetch_n1(j);
        auto chunk = [&](int c, auto FIRST) {              // first product of chunk c, second of chunk c - 1
            constexpr bool first = decltype(FIRST)::value;
            const int buf = c & 1;
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");     // hidden columns of chunk c - 1 are there; wN is in registers
            const f32x4 b = *(const f32x4 *)(b1_s + min(128 * c + 16 * wave, Dm - 16) + 4 * lg);
            if (c + 1 < nc) issue_n(W1, row_n(c + 1), slot0);
            if (first && !kh) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt) y[ct][2 + rt] = *handed(ct, rt);
            }
            segment([&](int n) { mfma_n(n, 0, b); }, [&](int n) {});
            segment([&](int n) { mfma_n(n, 2, b); },
                    [&](int n) {
                        gelu_side(n, 0, buf);
                        if (!first) {
                            share(n, 0, NS / 2, 4, [&](int j) { fetch_h1(0, buf ^ 1, j); });
                            if (n == NS / 2) {
                                if (c + 1 < nc) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * KT) : "memory");
                                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                            }
                            share(n, NS / 2, NS, CT, [&](int j) { fetch_w1(0, j); });
                        }
                    });
            if (first) {
#pragma unroll
                for (int n = 0; n < NS; ++n) gelu_side(n, 2, buf);
            } else {
                segment([&](int n) { mfma_k(n, 0); },
                        [&](int n) {
                            gelu_side(n, 2, buf);
                            share(n, 0, NS / 2, 4, [&](int j) { fetch_h1(1, buf ^ 1, j); });
                            share(n, NS / 2, NS - 1, CT, [&](int j) { fetch_w1(1, j); });
                        });
            }
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            if (first) {
                if (c + 1 < nc) {
#pragma unroll
                    for (int j = 0; j < 2 * KT; ++j) fetch_n1(j);
                }
            } else {
                segment([&](int n) { mfma_k(n, 1); },
                        [&](int n) {
                            share(n, 0, NS, 2 * CT, [&](int j) { issue_k1(col_k(c), j); });
                            if (c + 1 < nc) share(n, 0, NS - 1, 2 * KT, [&](int j) { fetch_n1(j); });
                        });
            }
        };
        chunk(0, std::true_type{});
#pragma unroll 1
        for (int c = 1; c < nc; ++c) chunk(c, std::false_type{});
        {                                                  // second product of the last chunk; where that is half a chunk, the second half has nothing
            const int buf = (nc - 1) & 1;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int j = 0; j < CT; ++j) fetch_w1(kk, j);
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int j = 0; j < 4; ++j) fetch_h1(kk, buf, j);
            if (l + 1 < l1) {
                const RunPtr p = run_args();
                issue_n(p->Wq + (size_t)(l + 1) * Nq * D, row_q(0), slot_q(0));
                if (lora_q) issue_at(slab(p->Aq, l + 1, D));
            }
            if (!kh || !(Dm & 64)) {
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                    for (int n = 0; n < NS; ++n) mfma_k(n, kk);
            }
        }
        exchange(y, x, 0);
        if (l + 1 == l1) {
            float *dst = run_args()->x_out + ((size_t)ob * T + t0) * D + wcol;
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const int row = wrow + 16 * rt + lm;
                    if (row < rows) *(f32x4 *)(dst + row * D + 16 * ct) = x[ct][rt];
                }
        }
    }
    }
    if (tid0 == 7 * 64 && word_s[1] < 0) {                     // no later launch of the call finds a block to work on, and the caller is told
        const RunPtr p = run_args();
        PolyMeta *meta = p->meta;
        int *status = p->dev_status;
        meta->stalled = 1; meta->R = 0; meta->F_ok = 0; meta->status = POLY_ESTALL;
        if (status) *status = POLY_ESTALL;
    }
}

template <int NKT> int launch_t(const RowRunArgs &a, hipStream_t st)
{
    auto kern = rowrun_kernel<NKT>;
    static bool attr_set = false;   // raising the dynamic LDS limit is a per-kernel, process-wide setting
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, RN_LDS) != hipSuccess) return POLY_EHIP;
        attr_set = true;
    }
    // a multiple of the queues, and all of a small call's at once on CUs of their own
    const int all = (a.nb * a.tiles + RN_QUEUES - 1) / RN_QUEUES * RN_QUEUES, most = 256;
    POLY_LAUNCH_SHMEM(POLY_STAGE_GEMM, kern, dim3((unsigned)(all < most ? all : most)), dim3(RN_THREADS), RN_LDS, st, a);
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

}  // namespace

bool rowrun_supported(int T, int width, int Dm, int heads, int r)
{
    return width == D && heads == HEADS && T > 0 && T <= 224 && Dm >= 128 && Dm % 64 == 0 && Dm <= RN_MAX_DM && (r == 0 || (r >= 4 && r <= 16 && r % 4 == 0));
}
size_t rowrun_counter_bytes(int nb) { return 64 * (size_t)(RN_QUEUES + nb); }
size_t rowrun_elements(int T) { return (size_t)((T + 31) / 32) * 32 * D; }

int launch_rowrun(const RowRunArgs &args, hipStream_t st)
{
    if (args.nb <= 0 || args.layers <= 0) return POLY_OK;
    if (args.capacity < args.nb) return POLY_EINVAL;
    RowRunArgs a = args;
    a.tiles = (a.T + 63) / 64;
    if (a.patience < 0) a.patience = FL_PATIENCE;
    return a.T <= 64 ? launch_t<2>(a, st) : a.T <= 128 ? launch_t<4>(a, st) : launch_t<7>(a, st);
}
