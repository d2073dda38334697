// A run of whole layers of a model 192 wide in ONE launch, on tiles of 64 or 32 token rows: a workgroup keeps its rows from the first layer of the run to the last.
//
// rowlayer.hip and attention.hip are two launches a layer: every one starts cold (4 us to issue and dispatch, 2 to 3 us until the first tile written by the launch
// before is usable), the residual stream goes out and comes back, and attention stages keys and values in LDS once more.  Here the up to four (of 32 rows: seven)
// workgroups that hold a block's rows run side by side, one per CU, and meet once a layer:
//     C   [q k v] = LayerNorm1(x) Wq + bq (+ low rank)      q stays in LDS; k and v, in the order attention reads them, go out at device scope
//     ..  the tiles of the block have all done so
//     att o = softmax(q k^T / 8) v                          a wave per (head, 32 queries), k and v straight into registers, o over q in LDS
//     A, B of rowlayer.hip                                  x, 24 fp32 registers of a lane (12), never leaves them
// The products, LayerNorms and the GELU are rowlayer.hip's, on the same slots of weights.
//
// Tiles of 32 rows are for few blocks, which give every CU one: half the rows for the same weights, and of attention three (head, 32 queries) whose keys are shared out over
// two waves each.  They alone take the sum of several adapters' terms: two of them are a step of 32 in the expand, and A_k (in A B_k too) of up to four lie in LDS.
//
// What bounds it, in cycles of a layer of DeiT-tiny with adapters: 64 rows (62 k, 26 us) feed-forward 22 k -- the LDS: weights in and out, lookups of the GELU, hidden columns --,
// qkv 8.5 k, attention 11.5 k (360 KB of keys and values through the CU's load path, 6 tasks on 4 SIMDs), the two LayerNorms 8.5 k, proj 5 k, handing over 5 k of which about
// 2 k are the round trip of the counter.  32 rows (50 k, 20.5 us) 18 k (15.5 k of it the chunks of 128 hidden columns: 14.7 k with no weights coming in), 7.3 k, 9.3 k, 6.5 k, 3.7 k, 4.5 k.
// Twelve layers and everything else of a forward, us, two launches a layer before / now: 62 blocks of 197 tokens (32 frames) 497 / 349, 24 blocks 448 / 270; 24 of 113
// with summed terms (small tasks) 417 / 298.  Tried and dropped: the next weights pulled into the L2 ahead (64 rows 1.5 % slower, 32 the same); a tile counted halfway through the q
// products, with proj's weights requested there too (0 to 1 % slower, on few blocks 2 %); a feed-forward part of its own for the class row's tile of the last layer, a quarter of the
// products of 64 rows (60 registers spilled, everything half as long again).
//
// Handing k and v over without fences: as in flow.hip.  They are stored at device scope, the stores are waited for, then the tile is counted; every layer of a
// launch has buffers of its own, so no address is read by this launch before it has been written for good and no cache holds an old copy of it.  A 1 KB
// piece is written by one workgroup.
//
// Order and progress: tickets of eight queues, block b in queue b % 8, the tiles of a block consecutive.  (Workgroups are dealt to the XCDs in turn, so a block's
// tiles mostly share an L2: 62 blocks of 197 tokens 349 us, drawn from one queue after the other 355.)  A workgroup finishes the tile it has drawn before it draws another, from the
// queue it starts at first, then from the others, and leaves when all are empty.  A tile waits only for tiles of its own block.  Whoever starts at queue 0 comes to a queue
// once those before it are empty, so at any time at most one block has some of its tickets drawn by these and others not, and `tiles` workgroups, up to seven, always get on.
// To start at its own XCD's queue a workgroup must have seen that 8 (tiles - 1) + 1 workgroups are there: at most one block per queue is partly drawn, so one of those that are there
// does not wait for tickets nobody has.  They are given some 30 us to come; where the GPU has no CUs for them (a partition or a stream with few of them, other kernels), work
// starts at queue 0.  Counted under the GELU's table, on a line for each XCD, that costs what a workgroup saves that looks for a queue with tickets left in all of them at once (in turn: eight
// round trips before it leaves): lagged loop on 64 frames, DeiT-tiny on 32, summed terms on 24, us, without / with both 410.7 / 408.6, 349.0 / 348.0, 299.7 / 298.1;
// counted on one line, queues in turn 414.2, 354.1, 299.4.
// How long the last of a block's tickets takes to be drawn is up to whatever else runs on the GPU, so the first wait of a tile, for that, has
// a limit of its own, of half a minute; behind it all of a block's workgroups are at work.  Nobody else writes the counters; should two calls use one workspace at a time, or
// fewer CUs than a block has tiles be free for that long, these limits end the waits and the call reports POLY_ESTALL, as in flow.hip.
#include "flow_dev.h"

#include <type_traits>

namespace {

constexpr int RN_THREADS = 512;
constexpr int rn_tile(int rt) { return rt * 2048; }        // bytes of a [16 rt][64] bf16 tile in LDS: 128 bytes a row, its 16-byte pieces permuted
constexpr int RN_TILES = 4;         // of activations
constexpr int RN_MAX_DM = 768;
constexpr int RN_GELU = (GELU_TAB_ENTRIES + 1) & ~1;    // (what lies behind is read in 16-byte pieces)
constexpr int RN_AT_STRIDE = 200;   // elements per rank row of At_k in LDS (192 + 8: rows start 4 banks apart)
constexpr int RN_QUEUES = 8;
constexpr int RN_GATHER = 32;        // looks, of 1 us and more, for enough workgroups to start at eight queues
constexpr int RN_FORMING = 1 << 24;  // looks, of 1.5 us and more, for a block's last ticket
constexpr int KT = 3, D = 64 * KT, HEADS = KT, Nq = 3 * D, NQ = (Nq + 127) / 128;
constexpr int CT = KT;                                     // column tiles of 16 per wave of a product with D columns
constexpr int SLOT = KT * 2048;                            // bytes of a slot: 16 rows of D columns, or 16 CT rows of 64 columns
constexpr int rn_end(bool sum) { return sum ? 32768 : 16384; }      // the region from stat_s on
constexpr int rn_lds(int rt, bool sum) { return RN_TILES * rn_tile(rt) + 16 * SLOT + (RN_MAX_DM + Nq + 2 * D + 4 * D) * 4 + RN_GELU * 8 + rn_end(sum) + 64; }
static_assert(rn_lds(4, false) <= 160 * 1024 && rn_lds(2, true) <= 160 * 1024, "LDS budget");

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

// Two loads of 16 bytes per lane straight into LDS, at `lds` + D0 and `lds` + D1, from base + v0 + I0 and base + v1 + I1 (an instruction's offset counts on both sides).
// go <= 0: loads that move nothing, but are counted as loads all the same (rowtile.h: glds16_if).
template <int I0, int I1, int D0, int D1> __device__ __forceinline__ void glds16_two(const void *base, unsigned v0, unsigned v1, unsigned lds, int go)
{
    asm volatile("s_add_u32 m0, %0, %4\n\ts_cmp_gt_i32 %8, 0\n\ts_cselect_b64 exec, -1, 0\n\tglobal_load_lds_dwordx4 %1, %3 offset:%6\n\ts_add_u32 m0, %0, %5\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %2, %3 offset:%7\n\ts_mov_b64 exec, -1" ::"s"(lds),
                 "v"(v0), "v"(v1), "s"(base), "n"(D0 - I0), "n"(D1 - I1), "n"(I0), "n"(I1), "s"(__builtin_amdgcn_readfirstlane(go))
                 : "memory", "m0", "scc");
}

// RT: 16-row tiles of a workgroup.  NKT: key tiles of 32 at most.  SUM: a block has the sum of several adapters' terms
template <int RT, int NKT, bool SUM> __global__ __launch_bounds__(RN_THREADS, 2) void rowrun_kernel(const RowRunArgs)
{
    constexpr int OT = RT / 2, ROWS = 16 * RT, RN_TILE = rn_tile(RT);      // OT: row tiles that a wave owns between the products
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
    int *word_s = (int *)((char *)stat_s + rn_end(SUM));        // [0] ticket, [1] looks left, [2] queue

    const int tid0 = threadIdx.x;
    // this workgroup has come (nobody waits for the answer; a line for each XCD: on one line 256 of these take 2 us)
    if (tid0 == 0) __hip_atomic_fetch_add(run_args()->counters + (blockIdx.x & (RN_QUEUES - 1)) * 16 + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int nb = [&]() { const RunPtr p = run_args(); const int *dev = p->nb_dev; return dev ? min(uload(dev), p->nb) : p->nb; }();
    if (nb <= 0) return;
    // this launch's layers: as many as there are buffers for, of the blocks that exist.  The host counts its launches by a bound, so there may be none left:
    // such a launch leaves before it touches LDS, which holds what others left in it (past here the word of the looks is written in front of a barrier).
    int l0, l1;
    {
        const RunPtr p = run_args();
        const int n = min(p->layers, p->capacity / nb);
        l0 = p->launch * n;
        l1 = min(l0 + n, p->layers);
    }
    if (l0 >= l1) return;
    if (tid0 == 0) word_s[1] = run_args()->patience;
    unsigned there = 0;
    if (tid0 < RN_QUEUES) there = peek(run_args()->counters + tid0 * 16 + 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {                          // Phi table of the GELU
        const int i = tid0 + RN_THREADS * j;
        if (i < GELU_TAB_ENTRIES) *(f32x2 *)(gelu_s + 2 * i) = gelu_tab_entry(i);
    }
    if (tid0 < 64) {
        const RunPtr p = run_args();
        const unsigned enough = (unsigned)(min(nb, RN_QUEUES) * (p->tiles - 1) + 1);
        for (int looks = RN_GATHER;;) {
            unsigned all = there;                          // (of lanes 0 .. 7)
#pragma unroll
            for (int d = 1; d < RN_QUEUES; d *= 2) all += __shfl_xor(all, d, RN_QUEUES);
            const bool own = __builtin_amdgcn_readfirstlane(all) >= enough;
            if (own || --looks < 0) {
                if (tid0 == 0) word_s[2] = own ? blockIdx.x & (RN_QUEUES - 1) : 0;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
            if (tid0 < RN_QUEUES) there = peek(p->counters + tid0 * 16 + 1);
        }
    }
    const int tiles = run_args()->tiles;
    for (;;) {
    // ---- the next tile: a ticket of the queue this workgroup is at, or of the next one that is not empty (which a queue stays)
    __syncthreads();
    if (tid0 < 64) {
        unsigned *const counters = run_args()->counters;
        auto tickets = [&](int q) { return nb > q ? (unsigned)((nb - q + RN_QUEUES - 1) / RN_QUEUES * tiles) : 0u; };
        int q = __builtin_amdgcn_readfirstlane(word_s[2]);
        for (;;) {
            unsigned t = 0;
            if (tid0 == 0) t = __hip_atomic_fetch_add(counters + q * 16, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            t = __builtin_amdgcn_readfirstlane(t);
            const bool got = t < tickets(q);
            unsigned some = 0;
            if (!got) {
                const int at = (q + 1 + tid0) & (RN_QUEUES - 1);
                some = (unsigned)__ballot(tid0 < RN_QUEUES && peek(counters + at * 16) < tickets(at));
            }
            if (got || !some) {
                if (tid0 == 0) { word_s[0] = got ? (int)t : -1; word_s[2] = q; }
                break;
            }
            q = (q + 1 + __builtin_ctz(some)) & (RN_QUEUES - 1);
        }
    }
    __syncthreads();
    const int ticket = __builtin_amdgcn_readfirstlane(word_s[0]), queue = __builtin_amdgcn_readfirstlane(word_s[2]);
    if (ticket < 0) break;
    const int ob = queue + RN_QUEUES * (int)((unsigned)ticket / (unsigned)tiles), tile = (int)((unsigned)ticket % (unsigned)tiles);
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
        wrow = 16 * OT * kh; wcol = 16 * CT * wc + 4 * lg;
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
    const int t0 = tile * ROWS, rows = min(ROWS, T - t0), nkt = (T + 31) >> 5;        // key tiles of 32
    const float scale = run_args()->scale, eps = run_args()->eps;
    // the block's terms: one, or (SUM) those of the pairs [first, first + n_terms)
    int k_ad = -1, first = 0, n_terms = 1;
    {
        const RunPtr p = run_args();
        if (SUM) {
            first = uload(p->set_off + ob);
            n_terms = uload(p->set_off + ob + 1) - first;
        }
        if (p->adapter_of_row && n_terms > 0) k_ad = uload(p->adapter_of_row + (SUM ? first : ob));
    }
    const bool lora_p = k_ad >= 0 && run_args()->Ap, lora_q = k_ad >= 0 && run_args()->Aq;
    // (SUM) At_k, and in A Bt_k, of the first `nt` terms, up to four, have a place in LDS; the rest of them are made from memory where they are needed
    constexpr int NT = SUM ? 4 : 1;
    const int cap = SUM ? min(NT, (rn_end(SUM) - 2048) / (r * (RN_AT_STRIDE + D) * 2)) : 1, nt = min(n_terms, cap);
    bf16_t *const bt_s = at_s + (SUM ? cap * r : 16) * RN_AT_STRIDE;       // Bt_k of A, [term][D][r]
    auto term = [&](int t) { return uload(run_args()->adapter_of_row + first + min(t, n_terms - 1)); };      // (past the last: the last, whose operand is zero then)
    int kt[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) kt[t] = SUM && k_ad >= 0 ? term(t) : k_ad;

    // 16 rows of a matrix with D columns from row `row`
    auto issue_n1 = [&](const bf16_t *W, int row, unsigned slot, int j) { glds16_s(W + (size_t)(row + 8 * (j & 1)) * D + 64 * (j >> 1), off_d ^ (64 * (j & 1)), slot + j * 1024); };
    auto issue_n = [&](const bf16_t *W, int row, unsigned slot) {
#pragma unroll
        for (int j = 0; j < 2 * KT; ++j) issue_n1(W, row, slot, j);
    };
    // first row of W1 / first column of W2 that this wave multiplies of chunk c (the last chunk may be half a one: what lies past it is not used)
    auto row_n = [&](int c) { return min(128 * c + 16 * wave, Dm - 16); };     // (past the last chunk: rows that are there)
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
    // an adapter's slab of layer l in a stack with `width` elements per rank
    auto slab_of = [&](const bf16_t *stack, int l, int width, int k) { return stack + ((size_t)l * run_args()->n_adapters + k) * r * width; };
    auto slab = [&](const bf16_t *stack, int l, int width) { return slab_of(stack, l, width, k_ad); };
    // At_k [r][D] of the terms of layer l -> at_s, a rank row per instruction
    auto issue_at = [&](const bf16_t *stack, int l) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (SUM && t >= nt) break;
            const bf16_t *At_k = slab_of(stack, l, D, kt[t]);
            for (int rk = wave; rk < r; rk += 8)
                if (lane < D / 8) glds16(At_k + rk * D + lane * 8, __builtin_amdgcn_readfirstlane(lds_addr_of(at_s + (t * r + rk) * RN_AT_STRIDE)));
        }
    };
    auto at_global = [&](const bf16_t *At_k, int k) { return *(const bf16x8 *)(At_k + min(lm, r - 1) * D + 32 * k + 8 * lg); };       // the same straight from memory
    // rank lm (repeated past r: such ranks meet zeros of Bt_k), columns 32 k + 8 lg + {0..7}
    auto at_frag = [&](int k, int t) { return *(const bf16x8 *)(at_s + (t * r + min(lm, r - 1)) * RN_AT_STRIDE + 32 * k + 8 * lg); };
    // column n of Bt_k [.][r], ranks 4 lg + {0..3} (r is a multiple of 4; zero where the rank does not exist)
    auto bt_frag = [&](const bf16_t *Bt_k, int n) { return *(const s16x4 *)(Bt_k + n * r + min(4 * lg, r - 4)); };
    // four ranks of a lane as a step of 32, the other four zeros on both sides: v_mfma_f32_16x16x16_bf16 takes several times as long (the five rounds of C 10.0 k cycles with
    // it, 7.8 k like this)
    auto pair = [](s16x4 u, s16x4 v) { return __builtin_bit_cast(bf16x8, __builtin_shufflevector(u, v, 0, 1, 2, 3, 4, 5, 6, 7)); };    // of two terms
    auto wide = [](s16x4 v) { return __builtin_bit_cast(bf16x8, __builtin_shufflevector(v, s16x4{0, 0, 0, 0}, 0, 1, 2, 3, 4, 5, 6, 7)); };
    auto bt_operand = [&](s16x4 v) { return 4 * lg < r ? v : s16x4{0, 0, 0, 0}; };
    auto bt_term = [&](s16x4 v, int t) { return 4 * lg < r && t < nt ? v : s16x4{0, 0, 0, 0}; };
    auto rd = [&](lds_ptr p, int off) { return *(const __attribute__((address_space(3))) bf16x8 *)(p + off); };
    auto act_frag = [&](int tile, int rt, int kk) { return rd(act[kk], tile * RN_TILE + rt * 2048); };
    f32x4 x[CT][OT];
    bf16x8 fa[2 * KT][RT];                                  // the resident rows as the B operand of the transposed product
    auto load_fa = [&]() {
#pragma unroll
        for (int k = 0; k < 2 * KT; ++k)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) fa[k][rt] = act_frag(k >> 1, rt, k & 1);
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
    auto exchange = [&](f32x4 (&acc)[CT][RT], f32x4 (&own)[CT][OT], int slot) {
        f32x4 *mine = (f32x4 *)(Ws + wave * (2 * SLOT) + slot) + lane;
        const f32x4 *theirs = (const f32x4 *)(Ws + (wave ^ 4) * (2 * SLOT) + slot) + lane;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int rt = 0; rt < OT; ++rt) {
                mine[(ct * OT + rt) * 64] = kh ? acc[ct][rt] : acc[ct][OT + rt];
                own[ct][rt] = kh ? acc[ct][OT + rt] : acc[ct][rt];
            }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int rt = 0; rt < OT; ++rt) own[ct][rt] += theirs[(ct * OT + rt) * 64];
    };
    // LayerNorm (fp32 statistics, centred second moments of 16 CT columns each, put together by Chan's rule) of x -> bf16 tiles at As -> fragments.
    // Behind the first barrier every wave is done with what it read before: `between` runs there.
    auto layernorm = [&](const float *gb_s, auto between) {
#pragma unroll
        for (int rt = 0; rt < OT; ++rt) {
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
        for (int rt = 0; rt < OT; ++rt) {
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
        if (lora_q) issue_at(p->Aq, l0);
        const float *src = (l0 ? p->x_out : p->x_in) + ((size_t)(p->in_map && l0 == 0 ? uload(p->in_map + ob) : ob) * T + t0) * D;
#pragma unroll
        for (int rt = 0; rt < OT; ++rt)
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
            s16x4 b2[NT][NQ] = {};                                     // Bt_k of the rounds
            if (lora_q) {
                const bf16_t *Bq = run_args()->Bq;
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (t < 2 || nt > 2) {
                        const bf16_t *Bq_k = slab_of(Bq, l, Nq, kt[t]);
#pragma unroll
                        for (int s = 0; s < NQ; ++s) b2[t][s] = bt_frag(Bq_k, row_q(s) + lm);
                    }
            }
            layernorm(gbq_s, [&]() {
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int s = 0; s < NQ; ++s) asm volatile("" : "+v"(b2[t][s]));    // (waited for here: behind loads that the compiler does not know it would wait for those too)
                issue_n(Wq, row_q(1), slot_q(1));
            });
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * KT) : "memory");     // round 0 and At_k; round 1 is on its way
            constexpr int NF = SUM ? 2 : 1;                            // terms whose shrink output is in registers; the others' stays in tile 3
            s16x4 fs[NF][RT];
            s16x4 *const sh = SUM ? (s16x4 *)(As + 3 * RN_TILE) : sh_s;
            auto shrunk = [&](const bf16x8(&av)[2 * KT], int rt) {
                f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 2 * KT; ++k) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[k], fa[k][rt], c, 0, 0, 0);
                return shrink_out(c);
            };
            if (lora_q) {                                              // a row tile of a term per wave, to every wave
                const int rt0 = RT == 4 ? wc : wave & 1, t0 = SUM ? wave >> 1 : 0;
                asm volatile("s_barrier" ::: "memory");
                if (!SUM || t0 < nt) {
                    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int k = 0; k < 2 * KT; ++k) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at_frag(k, t0), rd(act[k & 1], (k >> 1) * RN_TILE + rt0 * 2048), c, 0, 0, 0);
                    if (SUM || wave < RT) sh[wave * 64 + lane] = shrink_out(c);
                }
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
                for (int t = 0; t < NF; ++t)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) fs[t][rt] = sh[(min(t, nt - 1) * RT + rt) * 64 + lane];
            }
            char *const keys = (char *)stat_s, *const keys0 = SUM ? keys + 2 * RN_TILE : As + 3 * RN_TILE;     // of heads 1 and 2; of head 0
            const RunPtr p = run_args();
            // of a block, per 32 keys and head: 4 KB in the order of the fragments (what a tile has past the last 32 is past the end, where stores are dropped)
            const size_t piece = HEADS * 2048;
            constexpr int KEY_STORES = RT == 4 ? HEADS : 2;            // of a wave
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
                f32x4 acc[RT];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) acc[rt] = b;
                auto mma = [&](bf16x8 w, bf16x8 f, f32x4 c) { return values ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, w, c, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, f, c, 0, 0, 0); };
                if (lora_q) {
                    if constexpr (SUM) {
                        const bf16x8 w = pair(bt_term(b2[0][s], 0), bt_term(b2[1][s], 1));
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) acc[rt] = mma(w, pair(fs[0][rt], fs[1][rt]), acc[rt]);
                        if (nt > 2) {
                            const bf16x8 w2 = pair(bt_term(b2[2][s], 2), bt_term(b2[3][s], 3));
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) acc[rt] = mma(w2, pair(sh[(2 * RT + rt) * 64 + lane], sh[(min(3, nt - 1) * RT + rt) * 64 + lane]), acc[rt]);
                        }
#pragma unroll 1
                        for (int t = cap; t < n_terms; ++t) {          // more of them: made again for every round
                            const RunPtr p = run_args();
                            const bf16_t *Aq_k = slab_of(p->Aq, l, D, term(t));
                            const bf16x8 w = wide(bt_operand(bt_frag(slab_of(p->Bq, l, Nq, term(t)), col + lm)));
                            bf16x8 av[2 * KT];
#pragma unroll
                            for (int k = 0; k < 2 * KT; ++k) av[k] = at_global(Aq_k, k);
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) acc[rt] = mma(w, wide(shrunk(av, rt)), acc[rt]);
                        }
                    } else {
                        const bf16x8 w = wide(bt_operand(b2[0][s]));
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) acc[rt] = mma(w, wide(fs[0][rt]), acc[rt]);
                    }
                }
                auto mfma = [&](int n, int rt0) {
                    const int k = n / 2, rt = rt0 + n % 2;
                    acc[rt] = mma(W[s & 1][k], fa[k][rt], acc[rt]);
                };
                auto next = [&](int n, int slots) {                    // the operands of the next round
                    if (s + 1 == NQ) return;
                    // behind the next round's weights: those of the round after it; the stores of the keys; those of a full round of values
                    if (n == 0 && s == 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * KT) : "memory");
                    if (n == 0 && s == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * KT) : "memory");
                    if (n == 0 && s == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * KT + KEY_STORES) : "memory");
                    if (n == 0 && s == 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(RT) : "memory");
                    share(n, 0, slots, 2 * KT, [&](int j) { fetch(s + 1, j); });
                };
                if (full) {
                    segment([&](int n) { mfma(n, 0); }, [&](int n) { next(n, NS - 2); });
                    if constexpr (RT == 4) segment([&](int n) { mfma(n, 2); }, [&](int n) {});
                } else if constexpr (RT == 4) {                        // half a round: 64 columns, every wave 16 of them for its row half
                    if (kh) {
                        segment([&](int n) { mfma(n, 2); }, [&](int n) { next(n, NS - 2); });
                        acc[0] = acc[2];
                        acc[1] = acc[3];
                    } else {
                        segment([&](int n) { mfma(n, 0); }, [&](int n) { next(n, NS - 2); });
                    }
                } else {
                    if (kh) acc[0] = acc[1];
#pragma unroll
                    for (int k = 0; k < 2 * KT; ++k) {
                        acc[0] = mma(W[s & 1][k], kh ? fa[k][1] : fa[k][0], acc[0]);
                        next(k, 2 * KT);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if (values) {
                    // keys 16 kt + 4 lg + {0..3} of column 16 cg + lm of a head: half lg / 2 of lane 32 (lg % 2) + column % 32 of a fragment of 16 keys x 32 columns
                    const int head = full ? kh : 2;
                    const unsigned off = (unsigned)(head * 4 + (wc >> 1)) * 1024u + (unsigned)((lg & 1) * 32 + (wc & 1) * 16 + lm) * 16u + (unsigned)(lg >> 1) * 8u;
#pragma unroll
                    for (int rt = 0; rt < (full ? RT : OT); ++rt) {
                        const unsigned k16 = (unsigned)(tile * RT + (full ? rt : OT * kh + rt));
                        vb.st8(__builtin_bit_cast(u32x2_, pack4(acc[rt])), off + (k16 >> 1) * (HEADS * 4096u) + (k16 & 1) * 2048u);
                    }
                } else {
                    if (s == 0) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // every wave has its operands and the shrink output
                    char *const to = s == 0 ? keys + kh * RN_TILE : s == 1 && kh ? keys0 : As + (s == 1 ? 2 : kh) * RN_TILE;
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) put(to, wc, rt, acc[rt]);
                    if (s == 1) {                                      // all keys are staged: 16 columns x 32 rows at a time
                        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                        u32x4_ v[KEY_STORES];
                        unsigned to[KEY_STORES];
#pragma unroll
                        for (int j = 0; j < KEY_STORES; ++j) {
                            // four tiles: of every head, rows of half kh, columns 16 wc ..; two: the twelve pieces in order, the last four of sixteen go nowhere
                            const int i = wave + 8 * j, h = RT == 4 ? j : min(i >> 2, HEADS - 1), ds = RT == 4 ? wc : i & 3, half = RT == 4 ? kh : 0;
                            const int row = 32 * half + (lane & 31), at = row * 128 + (((2 * ds + (lane >> 5)) ^ ((row >> 1) & 7)) << 4);
                            v[j] = *(const u32x4_ *)((h == 0 ? keys0 : keys + (h - 1) * RN_TILE) + at);
                            to[j] = (unsigned)(((tile * OT + half) * HEADS + h) * 4 + ds) * 1024u + lane * 16u;
                            if (RT == 2 && i >= 4 * HEADS) to[j] = 0x40000000u;
                        }
#pragma unroll
                        for (int j = 0; j < KEY_STORES; ++j) kb.st16(v[j], to[j]);
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
            // Wp: of the rows 16 CT wc .. + 47, which the waves of both halves of the contraction multiply, 24 each, as KT tiles [24][64]
            const RunPtr p = run_args();
            const bf16_t *Wp = p->Wp + (size_t)l * D * D;
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int g = 0; g < CT; ++g) {
                    const int row = 24 * kh + 8 * g;
                    glds16_s(Wp + (size_t)(16 * CT * wc + row) * D + 64 * t, (unsigned)lr * (D * 2) + (((lane & 7) ^ ((row >> 1) + (lr >> 1) & 7)) << 4), slot0 + (t * CT + g) * 1024);
                }
            vectors(l);
            if (l + 1 < l1) vectors_q(l + 1);
            if (lora_p) issue_at(p->Ap, l);
            if (lora_p) {
                const int n16 = D * r / 8;                             // 16-byte pieces
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    if (SUM && t >= nt) break;
                    const char *Bt_k = (const char *)slab_of(p->Bp, l, D, kt[t]);
                    for (int i = wave * 64; i < n16; i += 512)
                        if (i + lane < n16) glds16(Bt_k + (i + lane) * 16, __builtin_amdgcn_readfirstlane(lds_addr_of(bt_s)) + (t * n16 + i) * 16);
                }
            }
        };
        // (the wave that waits requests its own behind the barrier: it has nothing to do in attention)
        if (wave == 7) {
            const unsigned want = tiles > 1 ? (unsigned)(l - l0 + 1) * tiles : 0;
            if (want && l == l0) {
                const unsigned *const drawn = run_args()->counters + (ob & (RN_QUEUES - 1)) * 16;
                const unsigned all = (unsigned)(ob / RN_QUEUES + 1) * tiles;
                const int most = run_args()->patience;
                for (int looks = word_s[1] < 0 ? 0 : most < FL_PATIENCE ? most : RN_FORMING; peek(drawn) < all;) {
                    if (--looks < 0) { word_s[1] = -1; break; }
                    __builtin_amdgcn_s_sleep(16);
                }
            }
            while (want) {                                             // (every look counts, so that without any patience no wait ends well)
                const int looks = word_s[1] - 1;
                word_s[1] = looks;
                if (looks < 0 || peek(count) >= want) break;
                __builtin_amdgcn_s_sleep(1);
            }
        } else {
            proj_loads();
        }
        asm volatile("s_barrier" ::: "memory");
        if (wave == 7) proj_loads();
        if constexpr (RT == 2) {
            // ======================================================== attention: waves 0 .. 2 a head each on the first half of the keys, 3 .. 5 on the others, whose
            // maxima, sums and outputs go through LDS (what Wp leaves of the slots) and meet those of the first half
            constexpr int H = (NKT + 1) / 2;                           // key tiles of the first half
            const int h = wave % HEADS, kg = wave / HEADS, am = lane & 31, ah = lane >> 5, sw = (am >> 1) & 7;
            char *const q = As + h * RN_TILE + am * 128;               // this lane's query
            float *const ml = (float *)stat_s;                         // [head][maxima, sums][32]
            auto part = [&](int i) { const int j = h * 8 + i; return (f32x4 *)(Ws + j / 3 * (2 * SLOT) + 9 * 1024 + j % 3 * 1024) + lane; };
            const float sc = 0.125f * FL_LOG2E;                        // 1/sqrt(64), folded into the base-2 exponent
            f32x16 o[2];
            float mx = -INFINITY, sum = 0.f;
            auto half = [&](auto N) {
                constexpr int n = decltype(N)::value;
                const RunPtr p = run_args();
                const size_t at = (slot * nkt * HEADS + h) * 2048 + lane * 8;
                const bf16_t *const kp = p->k + at, *const vp = p->v + at;
                bf16x8 qf[4], kf[n][4], vf[2 * n][2];
                // (tiles past the last repeat it: their probabilities are 0)
#pragma unroll
                for (int i = 0; i < n; ++i)
#pragma unroll
                    for (int ds = 0; ds < 4; ++ds) kf[i][ds] = *(const bf16x8 *)(kp + min(kg * H + i, nkt - 1) * (HEADS * 2048) + ds * 512);
#pragma unroll
                for (int i = 0; i < n; ++i)
#pragma unroll
                    for (int st = 0; st < 2; ++st)
#pragma unroll
                        for (int dt = 0; dt < 2; ++dt) vf[2 * i + st][dt] = *(const bf16x8 *)(vp + min(kg * H + i, nkt - 1) * (HEADS * 2048) + (st * 2 + dt) * 512);
#pragma unroll
                for (int ds = 0; ds < 4; ++ds) qf[ds] = *(const bf16x8 *)(q + (((2 * ds + ah) ^ sw) << 4));
                f32x16 s[n];
#pragma unroll
                for (int i = 0; i < n; ++i) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int e = 0; e < 16; ++e) s[i][e] = 0.f;
#pragma unroll
                    for (int ds = 0; ds < 4; ++ds) s[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i][ds], qf[ds], s[i], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < n; ++i) {
                    const int key = 32 * (kg * H + i);
                    if (key + 32 > T) {
#pragma unroll
                        for (int e = 0; e < 16; ++e) s[i][e] = key + 8 * (e >> 2) + 4 * ah + (e & 3) < T ? s[i][e] : -INFINITY;
                    }
                }
#pragma unroll
                for (int i = 0; i < n; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[i][e]);
                mx = fmaxf(fmaxf(mx, __shfl_xor(mx, 32, 64)), -3.4e38f);       // (a half without keys, or with -infinity in all of them, counts nothing)
                const float off = -mx * sc;
                bf16x8 pf[n][2];
#pragma unroll
                for (int i = 0; i < n; ++i)
#pragma unroll
                    for (int hs = 0; hs < 2; ++hs)
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float pr = __builtin_amdgcn_exp2f(fmaf(s[i][hs * 8 + e], sc, off));
                            sum += pr;
                            pf[i][hs][e] = (bf16_t)pr;
                        }
                sum += __shfl_xor(sum, 32, 64);
#pragma unroll
                for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                    for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
#pragma unroll
                for (int st = 0; st < 2 * n; ++st)
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[st][dt], pf[st >> 1][st & 1], o[dt], 0, 0, 0);
                if (kg) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) *part(i) = f32x4{o[i >> 2][4 * (i & 3)], o[i >> 2][4 * (i & 3) + 1], o[i >> 2][4 * (i & 3) + 2], o[i >> 2][4 * (i & 3) + 3]};
                    if (ah == 0) { ml[h * 64 + am] = mx; ml[h * 64 + 32 + am] = sum; }
                }
            };
            if (kg == 0) half(std::integral_constant<int, H>{});
            else if (kg == 1) half(std::integral_constant<int, NKT - H>{});
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (kg == 0) {
                const float m1 = ml[h * 64 + am], M = fmaxf(mx, m1), c0 = __builtin_amdgcn_exp2f((mx - M) * sc), c1 = __builtin_amdgcn_exp2f((m1 - M) * sc);
                const float inv = 1.0f / fmaf(ml[h * 64 + 32 + am], c1, sum * c0), w0 = c0 * inv, w1 = c1 * inv;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const f32x4 u = *part(i);
                    f32x4 y;
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = fmaf(u[e], w1, o[i >> 2][4 * (i & 3) + e] * w0);
                    *(bf16x4 *)(q + ((i ^ sw) << 4) + 8 * ah) = pack4(y);
                }
            }
        } else
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
        f32x4 y[CT][RT];
        rl_wait_barrier<0>();                              // o is there, Wp, At_k, Bt_k and the vectors have landed
        {
            // rows 16 ct + lm, columns 64 t + 32 kh + 8 lg ..
            auto wp = [&](int ct) {
                const int row = 16 * ct + lm, part = row >= 24;
                return (lds_ptr)(Ws + (wc + 4 * part) * (2 * SLOT) + (row - 24 * part) * 128 + (((4 * kh + lg) ^ ((row >> 1) & 7)) << 4));
            };
            bf16x8 w[KT][CT], h[KT][RT];
#pragma unroll
            for (int t = 0; t < KT; ++t) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) w[t][ct] = rd(wp(ct), t * 3072);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) h[t][rt] = rd(kh ? act[1] : act[0], t * RN_TILE + rt * 2048);
            }
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            issue_n(W1, row_n(0), slot0);
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        y[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t][ct], h[t][rt], t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : y[ct][rt], 0, 0, 0);
        }
        {
            f32x4 own[CT][OT];
            exchange(y, own, SLOT);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const f32x4 b = *(const f32x4 *)(bp_s + wcol + 16 * ct);
#pragma unroll
                for (int rt = 0; rt < OT; ++rt) x[ct][rt] += own[ct][rt] + b;
            }
        }
        if (!SUM && lora_p) {
#pragma unroll
            for (int rt = 0; rt < OT; ++rt) {
                f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 2 * KT; ++k) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at_frag(k, 0), rd(act[k & 1], (k >> 1) * RN_TILE + wrow * 128 + rt * 2048), c, 0, 0, 0);
                const s16x4 fs = shrink_out(c);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) x[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wide(bt_operand(bt_frag(bt_s, 16 * CT * wc + 16 * ct + lm))), wide(fs), x[ct][rt], 0, 0, 0);
            }
        }
        if (SUM && lora_p) {
#pragma unroll
            for (int rt = 0; rt < OT; ++rt) {
                bf16x8 ho[2 * KT];
#pragma unroll
                for (int k = 0; k < 2 * KT; ++k) ho[k] = rd(act[k & 1], (k >> 1) * RN_TILE + wrow * 128 + rt * 2048);
                auto shrunk = [&](auto at) {
                    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int k = 0; k < 2 * KT; ++k) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at(k), ho[k], c, 0, 0, 0);
                    return shrink_out(c);
                };
                auto bt = [&](int t, int ct) { return bt_frag(bt_s + t * D * r, 16 * CT * wc + 16 * ct + lm); };
                auto add = [&](int t) {                    // terms t and t + 1
                    const bf16x8 f = pair(shrunk([&](int k) { return at_frag(k, min(t, nt - 1)); }), shrunk([&](int k) { return at_frag(k, min(t + 1, nt - 1)); }));
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) x[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pair(bt_term(bt(t, ct), t), bt_term(bt(min(t + 1, nt - 1), ct), t + 1)), f, x[ct][rt], 0, 0, 0);
                };
                if constexpr (SUM) {
                    add(0);
                    if (nt > 2) add(2);
                }
#pragma unroll 1
                for (int t = cap; t < n_terms; ++t) {
                    const RunPtr p = run_args();
                    const bf16_t *At_k = slab_of(p->Ap, l, D, term(t)), *Bt_k = slab_of(p->Bp, l, D, term(t));
                    const s16x4 fs = shrunk([&](int k) { return at_global(At_k, k); });
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) x[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wide(bt_operand(bt_frag(Bt_k, 16 * CT * wc + 16 * ct + lm))), wide(fs), x[ct][rt], 0, 0, 0);
                }
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
            const int i = ct * OT + rt;
            return (f32x4 *)((i < OT ? As + 3 * RN_TILE + i * 4096 : (char *)stat_s + (i - OT) * 4096) + wc * 1024) + lane;
        };
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const f32x4 b = *(const f32x4 *)(b2_s + wcol + 16 * ct), z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int rt = 0; rt < OT; ++rt) {
                if (kh) *handed(ct, rt) = x[ct][rt] + b;
                y[ct][rt] = kh ? z : x[ct][rt] + b;
                y[ct][OT + rt] = z;
            }
        }

        // ============================================================ B: x'' = x' + b2 + GELU(LayerNorm2(x') W1 + b1) W2
        const unsigned gelu_a = lds_addr_of(gelu_s);
        float xc[4];
        f32x2 en[4];
        // GELU of one row tile: four lookups, then (fin) the results
        auto look = [&](const f32x4 &v, int j) { gelu_look(v[j], gelu_a, xc[j], en[j]); };
        auto fin = [&](const f32x4 &v, int rt, int buf) { put(As + buf * (2 * RN_TILE) + kh * RN_TILE, wc, rt, gelu_tab4(v, xc, en)); };
        auto next_q = [&]() {                              // the first weights of the next layer's C
            if (l + 1 < l1) {
                const RunPtr p = run_args();
                issue_n(p->Wq + (size_t)(l + 1) * Nq * D, row_q(0), slot_q(0));
            }
        };
        auto next_at = [&]() { if (lora_q && l + 1 < l1) issue_at(run_args()->Aq, l + 1); };      // (over what half 1 handed: behind a barrier)
        if constexpr (RT == 2) {
            // Half the rows for the same weights: what counts is that they keep coming.  Both products' operands have two sets of registers, and a wave's slots are a ring
            // of six items of 2 KB (16 rows x 64 columns), each read into them as soon as it has landed and refilled: three of W2(c), three of W1(c + 1), ..
            bf16x8 wN[2][2 * KT], wK[2][2][CT], hk[2][RT];
            f32x4 h[RT];
            auto fetch_n1 = [&](int p, int j) { wN[p][j] = rd(wn[j & 1], (j >> 1) * 2048); };
            auto fetch_h1 = [&](int kk, int buf, int rt) { hk[kk][rt] = rd(act[kk], buf * (2 * RN_TILE) + kh * RN_TILE + rt * 2048); };
            auto mfma_k = [&](int n, int kk, int p) {
                const int ct = n / RT, rt = n % RT;
                y[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wK[p][kk][ct], hk[kk][rt], y[ct][rt], 0, 0, 0);
            };
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * CT) : "memory");      // the first of W1; W2 is on its way
#pragma unroll
            for (int j = 0; j < 2 * KT; ++j) fetch_n1(0, j);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            const unsigned stride8 = 16u * (unsigned)Dm;   // bytes of eight rows of W2
            const bf16_t *const W2w = W2 + (size_t)(16 * CT * wc) * Dm;
            issue_n(W1, row_n(1), slot0);                  // (of a single chunk: the same once more)
            auto chunk = [&](int c, auto FIRST, auto P) {  // first product of chunk c, second of chunk c - 1
                constexpr bool first = decltype(FIRST)::value;
                constexpr int p = decltype(P)::value;      // c & 1
                // item i, of W2(c) and of W1(c + 1): waited for with the five behind it in flight, read, refilled once it is in registers (past the last chunk by loads
                // that move nothing)
                const int go1 = nc - 1 - c, go2 = nc - 2 - c;
                const unsigned ko = 2u * (unsigned)col_k(c + 1), no = (unsigned)row_n(c + 2) * (D * 2), k0 = off_m + ko, k1 = (off_m ^ 64) + ko, n0 = off_d + no, n1 = (off_d ^ 64) + no;
                auto refill = [&](auto I) {
                    constexpr int i = decltype(I)::value;
                    if constexpr (i < CT) glds16_two<0, 0, SLOT + i * 2048, SLOT + i * 2048 + 1024>(W2w, k0 + 2 * i * stride8, k1 + (2 * i + 1) * stride8, slot0, go1);
                    else glds16_two<(i - CT) * 128, 8 * D * 2 + (i - CT) * 128, (i - CT) * 2048, (i - CT) * 2048 + 1024>(W1, n0, n1, slot0, go2);
                };
                auto item = [&](auto I) {
                    constexpr int i = decltype(I)::value;
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    if constexpr (i > 0) refill(std::integral_constant<int, i - 1>{});
                    asm volatile("s_waitcnt vmcnt(10)" ::: "memory");
                    if constexpr (i < CT) {
#pragma unroll
                        for (int kk = 0; kk < 2; ++kk) wK[p][kk][i] = rd(wn[kk], SLOT + i * 2048);
                    } else {
                        fetch_n1(p ^ 1, 2 * (i - CT));
                        fetch_n1(p ^ 1, 2 * (i - CT) + 1);
                    }
                };
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");       // hidden columns of chunk c - 1 are there; wN[p] is in registers
                const f32x4 b = *(const f32x4 *)(b1_s + min(128 * c + 16 * wave, Dm - 16) + 4 * lg);
                if (first && !kh) {
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                        for (int rt = 0; rt < OT; ++rt) y[ct][OT + rt] = *handed(ct, rt);
                }
                if (!first) {
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) fetch_h1(kk, p ^ 1, rt);
                }
                segment(
                    [&](int n) {
                        const int k = n / 2, rt = n % 2;
                        h[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wN[p][k], fa[k][rt], k == 0 ? b : h[rt], 0, 0, 0);
                    },
                    [&](int n) {
                        if (n == 0) item(std::integral_constant<int, 0>{});
                        if (n == 4) item(std::integral_constant<int, 1>{});
                        if (n == 8) item(std::integral_constant<int, 2>{});
                    });
                constexpr int NK = CT * RT;
                auto gelu_side = [&](int n, int rt) {
                    share(n, 0, 4, 4, [&](int j) { look(h[rt], j); });
                    if (n == NK - 1) fin(h[rt], rt, p);
                };
#pragma unroll
                for (int n = 0; n < 2 * NK; ++n) {
                    if (!first) mfma_k(n % NK, n / NK, p ^ 1);
                    gelu_side(n % NK, n / NK);
                    if (n == 0) item(std::integral_constant<int, 3>{});
                    if (n == 4) item(std::integral_constant<int, 4>{});
                    if (n == 8) item(std::integral_constant<int, 5>{});
                    __builtin_amdgcn_sched_barrier(0);
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                refill(std::integral_constant<int, 5>{});
            };
            chunk(0, std::true_type{}, std::integral_constant<int, 0>{});
#pragma unroll 1
            for (int c = 1; c < nc; c += 2) {
                chunk(c, std::false_type{}, std::integral_constant<int, 1>{});
                if (c + 1 < nc) chunk(c + 1, std::false_type{}, std::integral_constant<int, 0>{});
            }
            // second product of the last chunk; where that is half a chunk, the second half has nothing
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            next_q();
            next_at();
            auto last = [&](auto P) {
                constexpr int p = decltype(P)::value;
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                    for (int j = 0; j < RT; ++j) fetch_h1(kk, p, j);
                if (!kh || !(Dm & 64)) {
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                        for (int n = 0; n < CT * RT; ++n) mfma_k(n, kk, p);
                }
            };
            if ((nc - 1) & 1) last(std::integral_constant<int, 1>{});
            else last(std::integral_constant<int, 0>{});
        } else {
            bf16x8 wN[2 * KT], wK[2][CT], hk[2][4];
            f32x4 h[4];
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
            auto gelu_side = [&](int n, int rt0, int buf) {    // of two row tiles in a segment of NS slots
                share(n, 0, NS / 4, 4, [&](int j) { look(h[rt0], j); });
                if (n == NS / 2 - 1) fin(h[rt0], rt0, buf);
                share(n, NS / 2, 3 * NS / 4, 4, [&](int j) { look(h[rt0 + 1], j); });
                if (n == NS - 1) fin(h[rt0 + 1], rt0 + 1, buf);
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
                next_q();
                next_at();
                if (!kh || !(Dm & 64)) {
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                        for (int n = 0; n < NS; ++n) mfma_k(n, kk);
                }
            }
        }
        exchange(y, x, 0);
        if (l + 1 == l1) {
            float *dst = run_args()->x_out + ((size_t)ob * T + t0) * D + wcol;
#pragma unroll
            for (int rt = 0; rt < OT; ++rt)
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

template <int RT, int NKT, bool SUM> int launch_t(const RowRunArgs &a, hipStream_t st)
{
    auto kern = rowrun_kernel<RT, NKT, SUM>;
    constexpr int LDS = rn_lds(RT, SUM);
    static bool attr_set = false;   // raising the dynamic LDS limit is a per-kernel, process-wide setting
    if (!attr_set) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS) != hipSuccess) return POLY_EHIP;
        attr_set = true;
    }
    // a multiple of the queues, and all of a small call's at once on CUs of their own
    const int all = (a.nb * a.tiles + RN_QUEUES - 1) / RN_QUEUES * RN_QUEUES, most = a.workgroups > 0 && a.workgroups < 256 ? a.workgroups : 256;
    POLY_LAUNCH_SHMEM(POLY_STAGE_GEMM, kern, dim3((unsigned)(all < most ? all : most)), dim3(RN_THREADS), LDS, st, a);
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}
template <int RT, bool SUM> int launch_rt(const RowRunArgs &a, hipStream_t st)
{
    return a.T <= 64 ? launch_t<RT, 2, SUM>(a, st) : a.T <= 128 ? launch_t<RT, 4, SUM>(a, st) : launch_t<RT, 7, SUM>(a, st);
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
    if (args.capacity < args.nb || (args.rows != 32 && (args.rows != 64 || args.set_off))) return POLY_EINVAL;
    RowRunArgs a = args;
    a.tiles = (a.T + a.rows - 1) / a.rows;
    if (a.patience < 0) a.patience = FL_PATIENCE;
    if (a.rows == 64) return launch_rt<4, false>(a, st);
    return a.set_off ? launch_rt<2, true>(a, st) : launch_rt<2, false>(a, st);
}
