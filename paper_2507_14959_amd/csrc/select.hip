// Context detection (Alg. 2, Sec. 3.5): label threshold -> greedy cover by contexts in (size, id)
// order -> CSR adapter sets.  Integer work on 64-bit sets, one workgroup per call: a batch is
// F x K = 64 x 80 scores, so the length of the chain of dependent steps, not throughput, is what matters.
//
// Label sets are bitsets built with wave ballots (one 64-label word per ballot, coalesced score
// reads).  Contexts are renumbered by scan position, so a context set is a 64-bit mask whose
// ascending bit order IS the selection order.  One thread per frame, up to 1024 frames per pass:
//
//  - Greedy cover.  A context is taken iff it provides a label that is still uncovered, so the next context taken is the
//    lowest first[l] over the uncovered labels l (first[l] = lowest scan position that provides l): whatever precedes it
//    provides none of them.  The candidates are therefore the first[] of the frame's few labels, not all M positions.
//  - Reuse branches.  S_t = S_{t-1} where the labels repeat or (context copy) where S_{t-1} provides them all, so every S_t is
//    the greedy set of the last frame that was NOT reused.  If frame t took its own set, the next frame to do so is
//    next[t] = the first t' > t whose labels are new and not all provided by the greedy set of t -- a function of t alone, found
//    for all t side by side: every thread whose labels are new walks over the later frames with new labels to the next break.  The frames
//    that really took their own set are the ones on the chain that starts at the first frame of the pass that the carried set does not serve;
//    they are marked by pointer quadrupling (log4 n rounds), and a scan gives every frame the last marked one before it.
//
// 1024 frames x 80 labels, 45 overlapping contexts with an accuracy table and context copy: 1665 us per call with M tests per frame
// and a sequential pass over the frames, 17.0 us this way (kernel 16.4); labels that never change: 102 us while the walk went over all
// frames, 15.7 without.  328 KB of scores through one CU are 12 k of the 38 k cycles, whatever the form of their loop
// (ballots instead of atomics, more loads in flight: the same).
// 64 frames, 16 contexts, in a queue of calls: 17.9 -> 8.8 us; 6.9 us (17.9 -> 13.3 k cycles) with everything the call reads in one round trip,
// barriers that do not wait for it, eight waves, and no search for the set in use by waves without frames.
#include "poly_dev.h"

namespace {

constexpr int MMAX = POLY_MAX_CONTEXTS;
constexpr int FEW_LABELS = 24;       // active labels up to which looking up first[] beats testing every context

struct SelState {       // device image of (Y_{t-1}, S_{t-1})
    int32_t valid, pad;
    uint64_t set_ids;   // S_{t-1} as a mask over context ids
    uint64_t labels[1]; // KW words
};

// all waves' LDS accesses so far, without waiting for loads that are still on their way to registers
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ const uint64_t no_state[2 + POLY_MAX_LABELS / 64] = {};   // read in place of what a caller has not given

// NW: words per label set (64 labels each).  One thread per frame of a pass; wide label sets get fewer frames per pass so that
// the two bitset arrays stay at 16 KB each.  VEC: scores per load (4 when K and the address allow 16-byte loads).
// Every phase runs once per call, so its instructions come from memory once: short code is worth more here than unrolled loops.
template <int NW, int VEC, int SEL_THREADS>
__global__ __launch_bounds__(SEL_THREADS) void select_kernel(const float *scores, int F, int K, const uint8_t *member, int M, float theta,
                                                             int context_copy, const float *acc, float tau, SelState *state,
                                                             int32_t *row_offsets, int32_t *adapter_ids, int cap, int32_t *counters,
                                                             const SelectFollow fo)
{
    constexpr int SEL_WAVES = SEL_THREADS / 64;
    constexpr int CH = NW <= 2 ? SEL_THREADS : NW <= 4 ? 512 : 128;   // frames per pass
    static_assert(SEL_THREADS >= 64 * NW && SEL_THREADS >= CH, "one thread per label and per frame");
    constexpr int LB = 4;                                      // score loads a thread has in flight
    __shared__ uint64_t cmask[MMAX][NW];       // labels that the context at a scan position provides
    __shared__ uint64_t prov_id[MMAX][NW];     // provided labels by context id
    __shared__ uint64_t Y[CH][NW];             // Y_t
    __shared__ uint64_t P[CH][NW];             // labels that the greedy set of frame t provides
    __shared__ uint64_t S[CH];                 // greedy set of frame t as a mask over scan positions
    __shared__ uint64_t prevY[NW], prevP[NW], prevS;      // of the frame before the pass
    __shared__ uint64_t wmask[SEL_WAVES], fresh[SEL_WAVES];
    __shared__ int order[MMAX];                // scan position -> context id
    __shared__ int size_of[MMAX], first[64 * NW];
    __shared__ __attribute__((aligned(16))) int wtot[SEL_WAVES];
    __shared__ int unc_s;
    __shared__ uint16_t nxt[2][CH + 1];
    __shared__ uint8_t reach[CH + 1];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KW = NW <= 2 ? NW : (K + 63) / 64;
    const bool sequential = state != nullptr || context_copy != 0;

    // (all arguments in one round trip instead of one each where they are first used)
    asm volatile("" ::"s"(scores), "s"(F), "s"(K), "s"(member), "s"(M), "s"(acc), "s"(state), "s"(fo.meta));

    // Scores: thread i takes the VEC scores at i, i + SEL_THREADS, .. of a pass, LB loads in flight (addresses clamped, not predicated).
    // Few labels are active, so each piece that has one sets its bits in the frame's words with an LDS atomic.
    typedef float vec_t __attribute__((ext_vector_type(VEC)));
    const int KV = K / VEC, step_t = SEL_THREADS / KV, step_q = SEL_THREADS - step_t * KV;
    vec_t sv[LB];
    auto load_scores = [&](int f0, int tot, int i0) {
#pragma unroll
        for (int u = 0; u < LB; ++u) sv[u] = *(const vec_t *)(scores + (size_t)f0 * K + (size_t)min(i0 + u * SEL_THREADS, tot - 1) * VEC);
    };
    // Everything the call reads is requested here, in one round trip, and no barrier before its use waits for it
    constexpr int MB = 4096 / SEL_THREADS;                     // membership words of a wave in flight
    uint8_t mb[MB];
    float ac[MB];
    auto load_members = [&](int w0) {
        unsigned at[MB];
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            const unsigned w = min(w0 + u * SEL_WAVES, M * KW - 1), c = w / (unsigned)KW;
            at[u] = c * (unsigned)K + min((w - c * (unsigned)KW) * 64u + lane, (unsigned)K - 1u);
            mb[u] = member[at[u]];
        }
        if (acc)
#pragma unroll
            for (int u = 0; u < MB; ++u) ac[u] = acc[at[u]];
    };
    const SelState *from = state ? state : (const SelState *)no_state;
    const int carried = from->valid, stalled = *(fo.meta ? &fo.meta->stalled : (const int *)no_state);
    const uint64_t carried_ids = from->set_ids;
    uint64_t carried_y[NW];
#pragma unroll
    for (int j = 0; j < NW; ++j) carried_y[j] = from->labels[min(j, (K - 1) >> 6)];
    __builtin_amdgcn_sched_barrier(0);
    load_members(wave);
    if (F > 0) load_scores(0, min(CH, F) * KV, tid);

    for (int i = tid; i < min(CH, F) * NW; i += SEL_THREADS) (&Y[0][0])[i] = 0;
    if (tid < 64 * NW) first[tid] = 64;
    if (tid < MMAX) size_of[tid] = 0;
    if (tid == 0) { unc_s = 0; prevS = 0; row_offsets[0] = 0; }
    lds_barrier();
    // membership and provided-label bitsets, one ballot per (context id, 64-label word); a context's size is the sum of its words'
    for (int w0 = wave; w0 < M * KW; w0 += MB * SEL_WAVES) {
        if (w0 != wave) load_members(w0);
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            const int w = w0 + u * SEL_WAVES, c = w / KW, j = w - c * KW;
            const bool mem = j * 64 + lane < K && mb[u] != 0;
            const uint64_t mm = __ballot(mem), pm = __ballot(mem && (acc == nullptr || ac[u] >= tau));
            if (lane == 0 && w < M * KW) { prov_id[c][j] = pm; atomicAdd(&size_of[c], __popcll(mm)); }
        }
    }
    if (tid == 0) {
#pragma unroll
        for (int j = 0; j < NW; ++j) { prevY[j] = carried && j < KW ? carried_y[j] : 0ull; prevP[j] = 0; }
    }
    lds_barrier();
    // contexts in scan order: size ascending, id ascending.  The rank of context c is the number of contexts before it: one ballot
    for (int c = wave; c < M; c += SEL_WAVES) {
        const int sz_l = lane < M ? size_of[lane] : 0x7fffffff, sz_c = size_of[c];
        const int rank = __popcll(__ballot(sz_l < sz_c || (sz_l == sz_c && lane < c)));
        if (lane == 0) order[rank] = c;
#pragma unroll 2
        for (int j = 0; j < KW; ++j) {
            const uint64_t pm = prov_id[c][j];
            if (lane == 0) cmask[rank][j] = pm;
            if ((pm >> lane) & 1ull) atomicMin(&first[j * 64 + lane], rank);
        }
    }

    int running = 0;                                           // adapters of the passes before
    for (int f0 = 0; f0 < F; f0 += CH) {
        const int n = min(CH, F - f0), tot = n * KV;
        const bool prevValid = f0 || carried;
        if (f0) {
            load_scores(f0, tot, tid);
            for (int i = tid; i < n * NW; i += SEL_THREADS) (&Y[0][0])[i] = 0;
            lds_barrier();
        }
        for (int i0 = tid, t = tid / KV, q = tid - t * KV;;) {
#pragma unroll
            for (int u = 0; u < LB; ++u) {
                unsigned bits = 0;
#pragma unroll
                for (int z = 0; z < VEC; ++z) bits |= (sv[u][z] >= theta ? 1u : 0u) << z;
                const int l = q * VEC;
                if (bits && i0 < tot) atomicOr((unsigned *)&Y[t][0] + (l >> 5), bits << (l & 31));
                i0 += SEL_THREADS; t += step_t; q += step_q;
                if (q >= KV) { q -= KV; ++t; }
            }
            if (i0 - tid >= tot) break;
            load_scores(f0, tot, i0);
        }
        lds_barrier();
        if (f0 == 0 && wave == SEL_WAVES - 1 && carried) {     // the carried set: context ids -> scan positions, and what it provides
            uint64_t s = __ballot(lane < M && ((carried_ids >> order[lane < M ? lane : 0]) & 1ull));
            if (lane == 0) prevS = s;
            uint64_t pv = 0;
            for (; s; s &= s - 1) pv |= cmask[__ffsll((unsigned long long)s) - 1][lane < KW ? lane : 0];
            if (lane < KW) prevP[lane] = pv;
        }
        // greedy cover of frame `tid`
        uint64_t y[NW];
        uint64_t sel = 0;
        bool same = false;                                     // the labels of the previous frame (or the carried ones) again
        if (tid < n) {
            uint64_t u[NW], pv[NW];
            int active = 0;
            bool eq = true;
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                y[j] = j < KW ? Y[tid][j] : 0ull;
                u[j] = y[j]; pv[j] = 0;
                active += __popcll(y[j]);
                if (j < KW) eq &= y[j] == (tid ? Y[tid - 1][j] : prevY[j]);
            }
            same = eq && (tid > 0 || prevValid);
            uint64_t cand = M == 64 ? ~0ull : (1ull << M) - 1;
            if (active <= FEW_LABELS) {
                cand = 0;
#pragma unroll
                for (int j = 0; j < NW; ++j)
                    for (uint64_t b = u[j]; b;) {              // (with one or two waves per SIMD four labels per round trip to LDS)
                        constexpr int ZL = SEL_THREADS > 512 ? 1 : 4;
                        int f[ZL];
#pragma unroll
                        for (int z = 0; z < ZL; ++z) {
                            f[z] = first[j * 64 + (ZL == 1 || b ? __ffsll((unsigned long long)b) - 1 : 0)];
                            if (ZL > 1 && !b) f[z] = 64;
                            b &= b - 1;
                        }
#pragma unroll
                        for (int z = 0; z < ZL; ++z)
                            if (f[z] < 64) cand |= 1ull << f[z];       // 64: provided by nobody
                    }
            }
            for (; cand; cand &= cand - 1) {
                const int pos = __ffsll((unsigned long long)cand) - 1;
                uint64_t m[NW], hit = 0;
#pragma unroll
                for (int j = 0; j < NW; ++j) { m[j] = j < KW ? cmask[pos][j] : 0ull; hit |= u[j] & m[j]; }
                if (hit) {
                    sel |= 1ull << pos;
#pragma unroll
                    for (int j = 0; j < NW; ++j) { u[j] &= ~m[j]; pv[j] |= m[j]; }
                }
            }
            S[tid] = sel;
#pragma unroll
            for (int j = 0; j < NW; ++j)
                if (j < KW) P[tid][j] = pv[j];
        }
        // own: this frame took its own greedy set
        bool own = true;
        if (sequential) {
            if (!context_copy) {
                own = !same;
            } else {
                __syncthreads();
                // first frame of the pass that the carried set does not serve
                bool brk = false;
                if (tid < n && !same) {
                    brk = tid == 0 && !prevValid;
#pragma unroll
                    for (int j = 0; j < NW; ++j)
                        if (j < KW) brk |= (y[j] & ~prevP[j]) != 0;
                }
                const uint64_t bm = __ballot(brk), cm = __ballot(tid < n && !same);
                if (lane == 0) { wmask[wave] = bm; fresh[wave] = cm; }
                if (tid < n) reach[tid] = 0;
                if (tid == 0) { reach[n] = 0; nxt[0][n] = nxt[1][n] = (uint16_t)n; }
                __syncthreads();
                // only frames with new labels end a run or take a set of their own
                if (tid < n) {
                    int t = n;
                    if (!same) {
                        uint64_t np[NW];
#pragma unroll
                        for (int j = 0; j < NW; ++j) np[j] = j < KW ? ~P[tid][j] : 0ull;
                        int w = wave;
                        for (uint64_t m = cm & (lane == 63 ? 0ull : ~0ull << (lane + 1));;) {
                            if (m == 0) {
                                if (++w >= SEL_WAVES) break;
                                m = fresh[w];
                                continue;
                            }
                            const int at = w * 64 + __ffsll((unsigned long long)m) - 1;
                            m &= m - 1;
                            bool hit = false;
#pragma unroll
                            for (int j = 0; j < NW; ++j)
                                if (j < KW) hit |= (Y[at][j] & np[j]) != 0;
                            if (hit) { t = at; break; }
                        }
                    }
                    nxt[0][tid] = (uint16_t)t;
                }
                if (tid == 0) {
                    for (int w = 0; w < SEL_WAVES; ++w)
                        if (wmask[w]) { reach[w * 64 + __ffsll((unsigned long long)wmask[w]) - 1] = 1; break; }
                }
                // after a round the chain is marked four times as far.  (A mark that a thread sees a round early is on the chain too.)
                int from = 0;
                for (int span = 1; span < n; span <<= 2, from ^= 1) {
                    __syncthreads();
                    if (tid < n) {
                        const int a = nxt[from][tid], b2 = nxt[from][a], c3 = nxt[from][b2];
                        nxt[from ^ 1][tid] = nxt[from][c3];
                        if (reach[tid]) reach[a] = reach[b2] = reach[c3] = 1;
                    }
                }
                __syncthreads();
                own = tid < n && reach[tid] != 0;
            }
        }
        // the last frame up to this one that took its own set (-1: the carried set still serves)
        const uint64_t om = __ballot(tid < n && own);
        if (lane == 0) wmask[wave] = om;
        __syncthreads();
        int last = -1;
        {
            const uint64_t upto = om & (~0ull >> (63 - lane));
            if (upto) last = wave * 64 + 63 - __clzll((long long)upto);
            else if (wave * 64 < n)
                for (int w = wave - 1; w >= 0; --w)
                    if (wmask[w]) { last = w * 64 + 63 - __clzll((long long)wmask[w]); break; }
        }
        int c = 0, uu = 0;
        if (tid < n) {
            sel = last >= 0 ? S[last] : prevS;
            c = __popcll(sel);
#pragma unroll
            for (int j = 0; j < NW; ++j)
                if (j < KW) uu += __popcll(y[j] & ~(last >= 0 ? P[last][j] : prevP[j]));
        }
        // exclusive scan of the set sizes: a count has at most seven bits, so seven ballots give a wave's prefix sums
        int before = 0, wsum = 0;
        const uint64_t below = (1ull << lane) - 1;
#pragma unroll
        for (int b = 0; b < 7; ++b) {
            const uint64_t m = __ballot((c >> b) & 1);
            before += __popcll(m & below) << b;
            wsum += __popcll(m) << b;
        }
        if (__ballot(uu != 0)) {                               // some label is provided by nobody
            for (int o = 32; o > 0; o >>= 1) uu += __shfl_xor(uu, o, 64);
            if (lane == 0) atomicAdd(&unc_s, uu);
        }
        if (lane == 0) wtot[wave] = wsum;
        __syncthreads();
        int upto_w = wtot[lane & (SEL_WAVES - 1)];             // prefix sums over the waves, in every row of 16 lanes
        upto_w += __builtin_amdgcn_update_dpp(0, upto_w, 0x111, 0xf, 0xf, true);       // row_shr 1, 2, 4, 8
        upto_w += __builtin_amdgcn_update_dpp(0, upto_w, 0x112, 0xf, 0xf, true);
        upto_w += __builtin_amdgcn_update_dpp(0, upto_w, 0x114, 0xf, 0xf, true);
        if (SEL_WAVES > 8) upto_w += __builtin_amdgcn_update_dpp(0, upto_w, 0x118, 0xf, 0xf, true);
        int o = running + before + (wave ? __builtin_amdgcn_readlane(upto_w, wave - 1) : 0);
        running += __builtin_amdgcn_readlane(upto_w, SEL_WAVES - 1);
        if (tid < n) {
            row_offsets[f0 + tid + 1] = o + c;
            for (uint64_t s = sel; s; s &= s - 1, ++o) {
                const int id = order[__ffsll((unsigned long long)s) - 1];
                if (o < cap) {
                    adapter_ids[o] = id;
                    if (fo.meta) { fo.frame_of_row[o] = f0 + tid; fo.adapter_of_row[o] = id; }
                }
            }
        }
        if (f0 + CH < F) {
            __syncthreads();                                   // everybody has read the carried values and this pass's arrays
            if (tid == n - 1) {
                prevS = sel;
#pragma unroll
                for (int j = 0; j < NW; ++j)
                    if (j < KW) { prevY[j] = y[j]; if (last >= 0) prevP[j] = P[last][j]; }
            }
        } else if (tid == n - 1 && state && !stalled) {        // the last frame's labels and set, for the next call
            uint64_t ids = 0;
            for (uint64_t s = sel; s; s &= s - 1) ids |= 1ull << order[__ffsll((unsigned long long)s) - 1];
            state->valid = 1;
            state->set_ids = ids;
#pragma unroll
            for (int j = 0; j < NW; ++j)
                if (j < KW) state->labels[j] = y[j];
        }
    }
    if (tid == 0) {
        counters[0] = running;
        counters[1] = F > 0 ? unc_s : 0;
        if (fo.meta) {                                         // ids and offsets are valid by construction; only the capacity can be exceeded
            const bool bad = running > cap || stalled;
            fo.meta->R = bad ? 0 : running;
            fo.meta->F_ok = bad ? 0 : F;
            fo.meta->status = stalled ? POLY_ESTALL : bad ? POLY_ERANGE : POLY_OK;
            if (fo.dev_status) *fo.dev_status = fo.meta->status;
        }
    }
    if (stalled) return;
    if (fo.carry)
        for (int i = tid; i < K; i += SEL_THREADS) fo.carry[i] = fo.carry_src[i];
}

}  // namespace

extern "C" size_t poly_select_state_bytes(int K)
{
    if (K <= 0) return 0;
    return 16 + 8 * (size_t)((K + 63) / 64);
}

int launch_select(const float *label_scores, int F, int K, const uint8_t *group_membership, int M, const poly_select_opts *opts, void *state,
                  int32_t *row_offsets, int32_t *adapter_ids, int cap, int32_t *counters, const SelectFollow &fo, hipStream_t st)
{
    if (!opts || !group_membership || !row_offsets || !counters) return POLY_EINVAL;
    if (F < 0 || K <= 0 || K > POLY_MAX_LABELS || M <= 0 || M > POLY_MAX_CONTEXTS || cap < 0) return POLY_EINVAL;
    if ((F > 0 && !label_scores) || (cap > 0 && !adapter_ids)) return POLY_EINVAL;
    const bool wide = K % 4 == 0 && ((uintptr_t)label_scores & 15) == 0;
#define SELECT_LAUNCH(NW, VEC, NT)                                                                                                       \
    POLY_LAUNCH(POLY_STAGE_SELECT, (select_kernel<NW, VEC, NT>), dim3(1), dim3(NT), st, label_scores, F, K, group_membership, M,            \
                opts->theta, opts->context_copy, opts->acc, opts->tau, (SelState *)state, row_offsets, adapter_ids, cap, counters, fo)
#define SELECT_CASE(NW)                    \
    do {                                   \
        if (wide) SELECT_LAUNCH(NW, 4, 1024); \
        else SELECT_LAUNCH(NW, 1, 1024);   \
    } while (0)
    // Few frames and contexts: eight waves.  Most phases are a chain of LDS round trips that every wave goes through, four waves on a SIMD one behind
    // the other; the set-up of many contexts wants the waves.  us of the kernel, 80 labels, eight waves / sixteen: 16 contexts, 1 frame 5.2 / 5.4,
    // 64 6.1 / 6.6, with context copy 8.0 / 9.5, 256 7.5 / 7.6, with copy 9.3 / 10.3; 45 contexts, 1 frame 7.7 / 7.0, 64 8.8 / 8.3, 256 10.2 / 9.4.
    if (wide && F <= 256 && K <= 128 && M <= 32) {
        if (K <= 64) SELECT_LAUNCH(1, 4, 512);
        else SELECT_LAUNCH(2, 4, 512);
    }
    else if (K <= 64) SELECT_CASE(1);
    else if (K <= 128) SELECT_CASE(2);
    else if (K <= 256) SELECT_CASE(4);
    else SELECT_CASE(16);
#undef SELECT_LAUNCH
#undef SELECT_CASE
    return hipGetLastError() == hipSuccess ? POLY_OK : POLY_EHIP;
}

extern "C" int poly_select(const float *label_scores, int F, int K, const uint8_t *group_membership, int M,
                           const poly_select_opts *opts, void *state, int32_t *row_offsets, int32_t *adapter_ids, int cap,
                           int32_t *counters, void *stream)
{
    return launch_select(label_scores, F, K, group_membership, M, opts, state, row_offsets, adapter_ids, cap, counters, SelectFollow{},
                         (hipStream_t)stream);
}
