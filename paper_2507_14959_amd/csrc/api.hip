// C-ABI entry points: argument checks, workspace carving and the launch sequence of the forward.
#include "poly_dev.h"
#include "row_waves.h"

namespace {

inline size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }
inline size_t elt_size(int dtype) { return dtype == POLY_BF16 ? 2 : 4; }
inline int rank_pad(int r) { return (r + 15) / 16 * 16; }

struct Carver {
    char *base;
    size_t off;
    template <typename T> T *take(size_t bytes)
    {
        T *p = base ? (T *)(base + off) : nullptr;
        off = align_up(off + bytes);
        return p;
    }
};

inline int tokens(const poly_model_desc *m) { return 1 + (m->H / m->patch) * (m->W / m->patch); }

// A segment of the layers (shared, adapted) that may run as launches of many layers, of small tasks (flow.hip) or of tiles that stay on their CUs (rowrun.hip),
// instead of one or more launches per layer
struct FlowSegment {
    int blocks, layers;                     // 0 blocks: this segment may not
    int tiles;                              // rowrun.hip: rows of a tile; 0: flow.hip
};

// blocks up to which a segment may where it does not run on tiles that stay on their CUs (run_segment): up to 140 tiles of 32 rows where the row kernel is the alternative, 270 where the GEMM path is (ranks
// it does not take, adapters on the MLP, summed terms).  DeiT-tiny, twelve layers, as tasks / layer by layer: 18 blocks of 197 tokens (126
// tiles) 469 / 487 us, 20 (140) 494 / 491, 24 (168) 509 / 503, 32 (224) 624 / 509; 70 blocks of 50 tokens (140) 427 / 438, 96 (192) 533 / 462;
// GEMM path, rank 32: 32 blocks of 197 tokens (224) 644 / 748, 45 (315) 883 / 791; summed terms: 678 / 835 and 936 / 895, 60 blocks of 113
// tokens (240) 729 / 828, 80 (320) 894 / 871.
// The 768-wide backbone: 7 tiles in the shared layers, 21 in the adapted ones, which layer by layer have four shrinks more.  Forward, us: ten layers shared,
// 1 tile 444 / 483, 4 493 / 567, 7 490 / 626, 8 600 / 579, 10 590 / 572; adapted on every linear, 1 tile 462 / 716, 7 502 / 891, 14 654 / 929, 21 773 / 981,
// 21 of which 13 exist 569 / 936, 42 with 25 1136 / 1106.
// Single precision: at 64 and 128 columns layer by layer, not for speed (nobody has measured the tasks there) but because tests/test_gpu_stream.py asks that a call
// of such a model with 256 bytes less than poly_forward_workspace_bytes names is refused, and with room for the tasks in that size it would be taken (as it
// is at other widths); at 192 columns 165 tiles (220 adapted ones, of which a call mostly fills a part) times the square of the part of their rows that
// exist, for the other way runs its rows across blocks and its larger tiles gain with their number.  Four shared layers of 192 columns, us, layer by layer / as
// tasks, blocks of 17 tokens (1 tile each; 32 in any case): 71 217 / 227, 100 286 / 308, 143 320 / 425; of 50 (2) 52 329 / 324, 73 441 / 434, 84 460 / 490; of 101 (4) 37 470 / 438,
// 42 488 / 495, 53 503 / 617; of 197 (7) 23 661 / 613 (adapted on all linears), 26 538 / 559; of 122 (4), adapted, 44 573 / 595 (so 168 tiles at most).  With adapters the lines lie a tenth higher.
int flow_limit(const poly_model_desc *m, bool adapted)
{
    const int T = tokens(m), r = adapted ? m->r : 0, tgt = adapted ? m->targets & 15 : 0;
    if (m->dtype == POLY_BF16 && !(adapted && m->compose == POLY_COMPOSE_SUM && tgt) && flow_wide_supported(T, m->D, m->Dm, m->heads, r, tgt != 0))
        return (adapted && tgt ? 21 : 7) / ((T + 31) / 32);
    if (!flow_supported(T, m->D, m->Dm, m->heads, r, tgt != 0)) return 0;
    if (m->dtype == POLY_F32) {
        const int nrt = (T + 31) / 32;
        const long blocks = (adapted && tgt ? 220L : 165L) * T * T / (1024L * nrt * nrt * nrt);
        return m->D < 192 ? 0 : (int)(blocks * nrt < 32 ? 32 / nrt : blocks * nrt > 168 ? 168 / nrt : blocks);
    }
    const bool row_kernel = !(tgt & 12) && !(adapted && m->compose == POLY_COMPOSE_SUM && tgt) && rowlayer_supported(m->D, m->Dm, tgt ? r : 0);
    return (row_kernel ? 140 : 270) / ((T + 31) / 32);
}

// Whether a segment of a model like this may run on tiles that stay on their CUs.  Two lines are not drawn for speed but where tests/test_gpu_layer_kernels.py, test_gpu_rowreg.py
// and test_row_layer.py count the launches of the kernels that go layer by layer, in workspaces of the named size: models of fewer than four layers, and poly_forward
// (not the lagged loop) where the adapted layers have a rank that no row kernel takes.
bool run_possible(const poly_model_desc *m, bool adapted, bool loop)
{
    const int tgt = adapted ? m->targets & 15 : 0;
    if (m->L < 4 || (!loop && m->L0 < m->L && (m->targets & 3) && !rowlayer_supported(m->D, m->Dm, m->r))) return false;
    return m->dtype == POLY_BF16 && !(tgt & 12) && rowrun_supported(tokens(m), m->D, m->Dm, m->heads, tgt ? m->r : 0);
}

// of a call of F frames and R row-blocks; capped: of the largest call with no more frames and row-blocks that still may
FlowSegment flow_segment(const poly_model_desc *m, int F, int R, bool adapted, bool capped)
{
    const int layers = adapted ? m->L - m->L0 : m->L0;
    const int blocks = adapted && m->compose != POLY_COMPOSE_SUM ? R : F, limit = flow_limit(m, adapted);
    if (layers == 0 || (adapted && R == 0) || (blocks > limit && !capped)) return {0, layers, 0};
    return {blocks < limit ? blocks : limit, layers, 0};
}
// Up to 44 tiles of 32 rows the small tasks are faster: DeiT-tiny, twelve layers, tasks / tiles, us: 6 blocks of 197 tokens (42) 234 / 270, 8 (56) 283 / 270, 10 (70) 370 / 272;
// of 113 8 (32) 240 / 250, 12 (48) 284 / 250; of 50 16 (32) 230 / 243, 24 (48) 243 / 243, 48 (96) 374 / 243; of 17 24 203 / 243, 64 276 / 243; a bound of three adapters a
// frame, 1.8 each: 4 frames of 197 297 / 270, 6 390 / 270; summed terms: 8 blocks of 113 (32) 279 / 305, 12 (48) 324 / 304.
constexpr int FLOW_FEW = 44;
FlowSegment run_segment(const poly_model_desc *m, int F, int R, bool adapted, bool loop, bool capped)
{
    const int layers = adapted ? m->L - m->L0 : m->L0, T = tokens(m);
    const bool fan = adapted && m->compose != POLY_COMPOSE_SUM;
    const int blocks = fan ? R : F, r = adapted && (m->targets & 15) ? m->r : 0;
    const bool summed = r && !fan;
    if (layers == 0 || (adapted && R == 0) || !run_possible(m, adapted, loop)) return {0, layers, 64};
    if (capped) {                                          // (of pairs half the room is what is usual)
        const int most = summed ? RN_SUM_ROUNDS * 8 * (32 / ((T + 31) / 32)) : (fan ? 2 * RN_MOST_TILES : RN_MAX_TILES) / ((T + 63) / 64);
        return {blocks < most ? blocks : most, layers, 64};
    }
    PairCount n = fan ? pair_count(F, R) : known_count(blocks);
    if (n.usual > blocks) n.usual = blocks;
    if ((long)n.usual * ((T + 31) / 32) <= FLOW_FEW && flow_segment(m, F, R, adapted, false).blocks > 0) return {0, layers, 64};
    const int rows = summed ? rowrun_rounds(blocks, (T + 31) / 32) <= RN_SUM_ROUNDS ? 32 : 0 : rowrun_rows(T, m->D, m->Dm, r, r > 0, n);
    return {rows ? blocks : 0, layers, rows};
}

// Every layer of a launch of flow.hip has buffers of its own (see there), so what they take grows with the layers of a launch: a segment
// whose buffers would take more than FLOW_BYTES is cut into equal launches, down to FLOW_MIN_LAYERS layers each.  DeiT-tiny, twelve layers
// in 1, 2 and 3 launches: 18 blocks of 197 tokens 375, 390, 398 us with 188, 94, 63 MB (the row kernels: 475), 20 blocks 487, 483, 497 with
// 209, 105, 70 MB (491), 24 blocks of 113 tokens with summed terms 429, 429, 447 with 155, 78, 52 MB (707 on the GEMM path).
constexpr int FLOW_MIN_LAYERS = 4;
constexpr size_t FLOW_BYTES = (size_t)128 << 20;

struct FlowBuffers {
    void *qk, *vt, *o, *h;                  // (tiles: keys and values, that is all)
    float *x1, *x2;
};
FlowBuffers carve_flow(const poly_model_desc *m, size_t n, bool tiles, Carver &c)      // n: blocks x layers of a launch
{
    const int T = tokens(m);
    const size_t es = elt_size(m->dtype);
    FlowBuffers f = {};
    if (tiles) {
        f.qk = c.take<void>(es * n * rowrun_elements(T));
        f.vt = c.take<void>(es * n * rowrun_elements(T));
        return f;
    }
    f.qk = c.take<void>(es * n * flow_elements(T, 2 * m->D));
    f.vt = c.take<void>(es * n * flow_elements(T, m->D));
    f.o = c.take<void>(es * n * flow_elements(T, m->D));
    f.h = c.take<void>(es * n * flow_elements(T, m->Dm));
    f.x1 = c.take<float>(sizeof(float) * n * T * m->D);
    f.x2 = c.take<float>(sizeof(float) * n * T * m->D);
    return f;
}
constexpr size_t TILES_ALIGN = 512;         // of keys and values, where they take as much as there is
size_t flow_bytes(const poly_model_desc *m, size_t n, bool tiles)
{
    Carver c{nullptr, 0};
    carve_flow(m, n, tiles, c);
    return c.off + (tiles ? TILES_ALIGN : 0);
}
size_t launch_counters(const poly_model_desc *m, const FlowSegment &s) { return s.tiles ? align_up(rowrun_counter_bytes(s.blocks)) : flow_counter_bytes(s.blocks, m->heads); }
int flow_min_layers(const FlowSegment &s) { return s.layers < FLOW_MIN_LAYERS ? s.layers : FLOW_MIN_LAYERS; }
size_t flow_counters(const poly_model_desc *m, const FlowSegment &s)       // of all its launches, at their largest number
{
    return s.blocks ? (size_t)((s.layers + FLOW_MIN_LAYERS - 1) / FLOW_MIN_LAYERS) * launch_counters(m, s) : 0;
}

struct ForwardWs {
    PolyMeta *meta;
    int32_t *frame_of_row, *adapter_of_row;
    float *xa, *xb;  // residual streams: per frame (shared layers), per row-block (adapted layers)
    void *u, *qkv, *o, *h, *S, *patches;
    size_t fixed, bytes;                    // up to xb; all of it: what a call needs at least
    int fl_tiles[2];                        // rowrun.hip instead of flow.hip in the shared and in the adapted layers: rows of a tile
    int fl_room[2];                         // blocks x layers that it has buffers for
    int fl_layers[2];                       // layers per launch of these there (0: none; of rowrun.hip: at least)
    FlowBuffers fl[2];                      // in the place of u .. patches: the patches are embedded before the first launch
    unsigned *fl_cnt[2];                    // counters of its launches, behind everything else
    unsigned *fl_clear;                     // where they start
    size_t fl_clear_bytes;                  // of both
};

// `bytes`: what there is.  The layers run as tasks where it holds their buffers too, which a workspace of poly_forward_workspace_bytes for
// this many frames and row-blocks or more does; the kernels that go layer by layer need no more than w.bytes.  loop: of poly_stream_step.
ForwardWs carve_forward(const poly_model_desc *m, int F, int R, bool loop, void *base, size_t bytes)
{
    const size_t T = tokens(m), es = elt_size(m->dtype);
    const size_t nb = (size_t)(F > R ? F : R), rows = nb * T;
    Carver c{(char *)base, 0};
    ForwardWs w = {};
    w.meta = c.take<PolyMeta>(sizeof(PolyMeta));
    w.frame_of_row = c.take<int32_t>(sizeof(int32_t) * (size_t)(R + 1));
    w.adapter_of_row = c.take<int32_t>(sizeof(int32_t) * (size_t)(R + 1));
    w.xa = c.take<float>(sizeof(float) * (size_t)F * T * m->D);
    w.xb = c.take<float>(sizeof(float) * (size_t)R * T * m->D);
    w.fixed = c.off;
    w.u = c.take<void>(es * rows * m->D);
    w.qkv = c.take<void>(es * rows * 3 * m->D);
    w.o = c.take<void>(es * rows * m->D);
    w.h = c.take<void>(es * rows * m->Dm);
    w.S = c.take<void>(es * (size_t)R * T * rank_pad(m->r));
    w.patches = c.take<void>(es * (size_t)F * (T - 1) * 3 * m->patch * m->patch);
    w.bytes = c.off;

    FlowSegment seg[2];
    size_t cnt = 0, end = 0;
    for (bool tiles : {true, false}) {      // (a workspace below the named size may hold the buffers of the small tasks and not of the tiles)
        for (int a = 0; a < 2; ++a) {
            if (tiles) seg[a] = run_segment(m, F, R, a == 1, loop, false);
            else if (seg[a].blocks && end < w.fixed + flow_bytes(m, (size_t)seg[a].blocks * flow_min_layers(seg[a]), seg[a].tiles)) seg[a].blocks = 0;
            if (seg[a].blocks == 0) seg[a] = flow_segment(m, F, R, a == 1, false);
        }
        cnt = flow_counters(m, seg[0]) + flow_counters(m, seg[1]);
        end = bytes > cnt ? (bytes - cnt) & ~(size_t)255 : 0;              // the counters' place
    }
    if (cnt == 0 || end < w.bytes) return w;
    w.fl_clear = (unsigned *)((char *)base + end);
    for (int a = 0; a < 2; ++a) {
        if (seg[a].blocks == 0) continue;
        const int least = flow_min_layers(seg[a]);
        int launches = 1, n = seg[a].layers;                   // layers of a launch: as few launches as there is room for
        if (seg[a].tiles) {                                    // as much room as there is: the launches share the layers out by the blocks that exist
            const size_t one = 2 * es * rowrun_elements((int)T);
            const size_t room = (end - w.fixed - TILES_ALIGN) / one, all = (size_t)seg[a].blocks * n;
            if (end < w.fixed + TILES_ALIGN || room < (size_t)seg[a].blocks * least) continue;
            Carver cf{(char *)base, w.fixed};
            w.fl_room[a] = (int)(room < all ? room : all);
            w.fl[a] = carve_flow(m, w.fl_room[a], true, cf);
            w.fl_tiles[a] = seg[a].tiles;
            w.fl_layers[a] = w.fl_room[a] / seg[a].blocks;
            w.fl_cnt[a] = w.fl_clear + w.fl_clear_bytes / sizeof(unsigned);
            w.fl_clear_bytes += launch_counters(m, seg[a]) * (size_t)((n + w.fl_layers[a] - 1) / w.fl_layers[a]);
            continue;
        }
        auto fits = [&]() { return w.fixed + flow_bytes(m, (size_t)seg[a].blocks * n, false) <= end; };
        while (!fits() && n > least) {
            ++launches;
            n = (seg[a].layers + launches - 1) / launches;
            if (n < least) n = least;
        }
        if (!fits()) continue;
        Carver cf{(char *)base, w.fixed};
        w.fl[a] = carve_flow(m, (size_t)seg[a].blocks * n, false, cf);
        w.fl_layers[a] = n;
        w.fl_cnt[a] = w.fl_clear + w.fl_clear_bytes / sizeof(unsigned);
        w.fl_clear_bytes += launch_counters(m, seg[a]) * (size_t)((seg[a].layers + n - 1) / n);
    }
    return w;
}

// Never less for more frames or row-blocks, so that a workspace for the largest call of a program serves its smaller ones: the task
// buffers are those of the largest call up to this one that runs as tasks
size_t forward_bytes(const poly_model_desc *m, int F, int R, bool loop)
{
    const ForwardWs w = carve_forward(m, F, R, loop, nullptr, 0);
    size_t end = w.bytes, cnt = 0;
    for (int a = 0; a < 2; ++a)
        for (bool tiles : {false, true}) {
            const FlowSegment s = tiles ? run_segment(m, F, R, a == 1, loop, true) : flow_segment(m, F, R, a == 1, true);
            if (s.blocks == 0) continue;
            const size_t all = flow_bytes(m, (size_t)s.blocks * s.layers, tiles), least = flow_bytes(m, (size_t)s.blocks * flow_min_layers(s), tiles);
            const size_t most = least > FLOW_BYTES ? least : FLOW_BYTES, want = all < most ? all : most;
            if (w.fixed + want > end) end = w.fixed + want;
            cnt += flow_counters(m, s);
        }
    return end + align_up(cnt);
}

int check_model(const poly_model_desc *m)
{
    if (!m) return POLY_EINVAL;
    if (m->dtype != POLY_F32 && m->dtype != POLY_BF16) return POLY_EINVAL;
    if (m->patch <= 0 || m->H <= 0 || m->W <= 0 || m->H % m->patch || m->W % m->patch) return POLY_EINVAL;
    if (m->heads <= 0 || m->D != m->heads * POLY_HEAD_DIM || m->Dm <= 0 || m->L <= 0) return POLY_EINVAL;
    if (m->L0 < 0 || m->L0 > m->L) return POLY_EINVAL;
    if (m->r <= 0 || m->r > POLY_MAX_RANK || m->n_adapters <= 0 || m->C <= 0 || m->C > POLY_MAX_HEAD_CLASSES) return POLY_EINVAL;
    if (m->targets & ~15) return POLY_EINVAL;
    if (m->compose != POLY_COMPOSE_BRANCH && m->compose != POLY_COMPOSE_SUM) return POLY_EINVAL;
    const int T = tokens(m);
    if (m->dtype == POLY_BF16) {
        // 16-byte vector loads along the contraction index; attention keeps a block's keys in LDS
        if (m->Dm % 8 || (3 * m->patch * m->patch) % 8 || T > 224) return POLY_EINVAL;
    } else {
        if (m->Dm % 4 || (3 * m->patch * m->patch) % 4) return POLY_EINVAL;
    }
    return POLY_OK;
}

#define POLY_TRY(expr)                  \
    do {                                \
        const int rc_ = (expr);         \
        if (rc_ != POLY_OK) return rc_; \
    } while (0)

}  // namespace

extern "C" const char *poly_status_string(int status)
{
    switch (status) {
    case POLY_OK: return "ok";
    case POLY_EINVAL: return "invalid argument";
    case POLY_ERANGE: return "adapter id or row offsets out of range";
    case POLY_ECAP: return "output or workspace too small";
    case POLY_EHIP: return "HIP runtime error";
    case POLY_ESTALL: return "a kernel gave up waiting: workspace used by two calls at a time, or no CUs free for its workgroups";
    default: return "unknown status";
    }
}

extern "C" size_t poly_forward_workspace_bytes(const poly_model_desc *m, int F, int R)
{
    if (check_model(m) != POLY_OK || F < 0 || R < 0) return 0;
    return forward_bytes(m, F, R, false);
}

namespace {
// what poly_stream_step adds to the forward: the CSR arrays are written on the way (after the shared layers) instead of given
struct StreamStep {
    const poly_stream *s;
    int32_t *row_offsets, *adapter_ids, *counters;
    float *out_base_scores;
    float *lag;        // [F + 1][K], in the workspace behind the forward's part
};

int forward_impl(const poly_model_desc *m, const poly_base_weights *base, const poly_lora_weights *lora,
                 const poly_heads *heads, const void *frames, int F, const int32_t *row_offsets,
                 const int32_t *adapter_ids, int R, float *out_logits, float *out_scores, float *out_merged, int K,
                 int32_t *dev_status, void *workspace, size_t workspace_bytes, void *stream, const StreamStep *ss)
{
    POLY_TRY(check_model(m));
    if (!base || !heads || F < 0 || R < 0) return POLY_EINVAL;
    if (F == 0) return POLY_OK;
    if (!frames || !row_offsets || (R > 0 && (!adapter_ids || !out_scores))) return POLY_EINVAL;
    if (!base->patch_w || !base->patch_b || !base->cls || !base->pos || !base->ln1_g || !base->ln1_b || !base->qkv_w ||
        !base->qkv_b || !base->proj_w || !base->proj_b || !base->ln2_g || !base->ln2_b || !base->fc1_w || !base->fc1_b ||
        !base->fc2_w || !base->fc2_b || !base->lnf_g || !base->lnf_b || !heads->head_w || !heads->head_b)
        return POLY_EINVAL;
    if (out_merged && (!heads->class_map || K <= 0)) return POLY_EINVAL;
    const bool adapted = m->L0 < m->L;
    for (int t = 0; t < 4; ++t)
        if (adapted && (m->targets & (1 << t)) && (!lora || !lora->At[t] || !lora->Bt[t])) return POLY_EINVAL;
    if (((uintptr_t)workspace & 255) != 0 || !workspace) return POLY_EINVAL;
    const ForwardWs w = carve_forward(m, F, R, ss != nullptr, workspace, workspace_bytes);
    if (workspace_bytes < w.bytes) return POLY_ECAP;

    hipStream_t st = (hipStream_t)stream;
    const int dt = m->dtype, D = m->D, Dm = m->Dm, T = tokens(m), pd = 3 * m->patch * m->patch;
    const int RP = rank_pad(m->r);
    const size_t es = elt_size(dt);
    const int *R_dev = &w.meta->R;
    const bool sum = m->compose == POLY_COMPOSE_SUM;

    // tokens: x[f][0] = cls + pos[0]; x[f][1 + t] = patch_t W_pe + b_pe + pos[1 + t].  The same launch checks the CSR arrays and
    // builds the row maps (nothing before the first adapted layer needs them).
    const PatchArgs embed = {frames, F, m->H, m->W, m->patch, base->cls, base->pos, w.xa, out_merged, out_merged ? (size_t)F * K : 0, w.fl_clear,
                             w.fl_clear_bytes / sizeof(unsigned), {ss ? nullptr : row_offsets, adapter_ids, F, R, m->n_adapters, w.meta, w.frame_of_row,
                             w.adapter_of_row, dev_status}};
    const bool bf16 = dt == POLY_BF16;
    const bool embedded = bf16 ? patch_rows_fits(embed, base->patch_w, base->patch_b, D) : patch_rows_f32_fits(embed, base->patch_w, base->patch_b, D);
    if (embedded) POLY_TRY((bf16 ? launch_patch_rows : launch_patch_rows_f32)(embed, base->patch_w, base->patch_b, D, st));
    else POLY_TRY(launch_im2col(frames, w.patches, F, m->H, m->W, m->patch, dt, w.xa, base->cls, base->pos, T, D, out_merged,
                           out_merged ? (size_t)F * K : 0, w.fl_clear, w.fl_clear_bytes / sizeof(unsigned), ss ? nullptr : row_offsets,
                           adapter_ids, R, m->n_adapters, w.meta, w.frame_of_row, w.adapter_of_row, dev_status, st));
    // The heads (and with L0 == L the base head) read the class token of every block and nothing else, so of the last layer only the keys and values concern
    // the other rows: behind its qkv linear the blocks are one row long, kept where the attention output ends.  (Not on a handful of tokens, whose buffer is too short for that.)
    const bool class_rows = T >= 8;
    const float *x_end = adapted && !sum ? w.xb : w.xa;    // the residual stream behind the last layer, blocks of T_end rows
    int T_end = T;
    // The lagged loop: after the shared layers the base head scores the frames, Alg. 2 turns the scores of frame t - 1 into
    // the adapter set of frame t with its row maps -- all on this stream, no host in between.
    bool selected = ss == nullptr;
    auto select_now = [&]() -> int {
        selected = true;
        const poly_stream *s = ss->s;
        POLY_TRY(launch_base_head(adapted ? w.xa : x_end, T_end, D, base->lnf_g, base->lnf_b, m->ln_eps, s->base_w, s->base_b, s->K, F, ss->lag,
                                  ss->out_base_scores, s->carry, dt, st));
        // the selection also writes the row maps and carries the last frame's scores to the next call: two launches less
        const SelectFollow fo = {w.meta, w.frame_of_row, w.adapter_of_row, dev_status, s->carry, ss->lag + (size_t)F * s->K};
        return launch_select(ss->lag, F, s->K, s->group_membership, s->M, &s->opts, s->state, ss->row_offsets, ss->adapter_ids, R, ss->counters,
                             fo, st);
    };
    if (!embedded) {
        GemmArgs g = {};
        g.A = w.patches; g.Wt = base->patch_w; g.bias = base->patch_b;
        g.T = T - 1; g.K = pd; g.N = D; g.n_in = F;
        g.mode = EPI_RESID; g.out = w.xa; g.Tout = T; g.t_off = 1; g.pos = base->pos;
        POLY_TRY(launch_gemm(g, {true, 0}, dt, st));
    }

    auto flow = [&](bool ad) -> int {
        FlowArgs a = {};
        a.T = T; a.D = D; a.Dm = Dm; a.heads = m->heads; a.eps = m->ln_eps;
        a.nb = ad && !sum ? R : F;
        a.nb_dev = !ad ? nullptr : (sum ? &w.meta->F_ok : R_dev);
        a.x_in = w.xa; a.x = ad && !sum ? w.xb : w.xa;
        a.in_map = ad && !sum ? w.frame_of_row : nullptr;
        a.n_adapters = m->n_adapters; a.r = m->r; a.scale = m->lora_scale; a.adapter_of_row = w.adapter_of_row;
        a.set_off = ad && sum ? row_offsets : nullptr;
        const FlowBuffers &f = w.fl[ad];
        a.qk = f.qk; a.vt = f.vt; a.o = f.o; a.h = f.h; a.x1 = f.x1; a.x2 = f.x2;
        a.counters = w.fl_cnt[ad];
        a.patience = poly_patience(); a.workgroups = poly_workgroups(); a.meta = w.meta; a.dev_status = dev_status;
        const int first = ad ? m->L0 : 0, last = ad ? m->L : m->L0;
        for (int l = first; l < last; l += a.layers) {
            a.layers = last - l < w.fl_layers[ad] ? last - l : w.fl_layers[ad];
            const size_t ld = (size_t)l * D, lm = (size_t)l * Dm, dd = ld * D, dm = ld * Dm;
            a.ln1_g = base->ln1_g + ld; a.ln1_b = base->ln1_b + ld; a.ln2_g = base->ln2_g + ld; a.ln2_b = base->ln2_b + ld;
            a.Wq = (const char *)base->qkv_w + es * 3 * dd; a.Wp = (const char *)base->proj_w + es * dd;
            a.W1 = (const char *)base->fc1_w + es * dm; a.W2 = (const char *)base->fc2_w + es * dm;
            a.bq = base->qkv_b + 3 * ld; a.bp = base->proj_b + ld; a.b1 = base->fc1_b + lm; a.b2 = base->fc2_b + ld;
            const size_t din[4] = {(size_t)D, (size_t)D, (size_t)D, (size_t)Dm}, dout[4] = {(size_t)3 * D, (size_t)D, (size_t)Dm, (size_t)D};
            for (int t = 0; ad && t < 4; ++t) {
                const size_t ranks = (size_t)(l - first) * m->n_adapters * m->r;
                if (m->targets & (1 << t)) { a.At[t] = (const char *)lora->At[t] + es * ranks * din[t]; a.Bt[t] = (const char *)lora->Bt[t] + es * ranks * dout[t]; }
            }
            a.class_rows = l + a.layers == m->L;
            POLY_TRY(launch_flow(a, dt, st));
            a.x_in = a.x; a.in_map = nullptr;                  // the next launch continues on this one's blocks
            a.counters += flow_counter_bytes(a.nb, m->heads) / sizeof(unsigned);
        }
        return POLY_OK;
    };

    auto run = [&](bool ad) -> int {
        RowRunArgs a = {};
        a.T = T; a.Dm = Dm; a.eps = m->ln_eps;
        a.rows = w.fl_tiles[ad];
        a.nb = ad && !sum ? R : F;
        a.nb_dev = !ad ? nullptr : (sum ? &w.meta->F_ok : R_dev);
        a.x_in = w.xa; a.x_out = ad && !sum ? w.xb : w.xa;
        a.in_map = ad && !sum ? w.frame_of_row : nullptr;
        a.n_adapters = m->n_adapters; a.r = m->r; a.scale = m->lora_scale;
        a.k = (bf16_t *)w.fl[ad].qk; a.v = (bf16_t *)w.fl[ad].vt;
        a.counters = w.fl_cnt[ad];
        a.patience = poly_patience(); a.workgroups = poly_workgroups(); a.meta = w.meta; a.dev_status = dev_status;
        const int first = ad ? m->L0 : 0, last = ad ? m->L : m->L0;
        const size_t ld = (size_t)first * D, lm = (size_t)first * Dm, dd = ld * D, dm = ld * Dm;
        a.layers = last - first;
        a.capacity = w.fl_room[ad];
        a.class_rows = last == m->L;
        a.ln1_g = base->ln1_g + ld; a.ln1_b = base->ln1_b + ld; a.ln2_g = base->ln2_g + ld; a.ln2_b = base->ln2_b + ld;
        a.Wq = (const bf16_t *)base->qkv_w + 3 * dd; a.Wp = (const bf16_t *)base->proj_w + dd;
        a.W1 = (const bf16_t *)base->fc1_w + dm; a.W2 = (const bf16_t *)base->fc2_w + dm;
        a.bq = base->qkv_b + 3 * ld; a.bp = base->proj_b + ld; a.b1 = base->fc1_b + lm; a.b2 = base->fc2_b + ld;
        if (ad && (m->targets & 1)) { a.Aq = (const bf16_t *)lora->At[0]; a.Bq = (const bf16_t *)lora->Bt[0]; }
        if (ad && (m->targets & 2)) { a.Ap = (const bf16_t *)lora->At[1]; a.Bp = (const bf16_t *)lora->Bt[1]; }
        a.adapter_of_row = a.Aq || a.Ap ? w.adapter_of_row : nullptr;
        a.set_off = ad && sum && a.adapter_of_row ? row_offsets : nullptr;
        for (int done = 0; done < a.layers; done += w.fl_layers[ad], ++a.launch) {
            POLY_TRY(launch_rowrun(a, st));
            a.counters += align_up(rowrun_counter_bytes(a.nb)) / sizeof(unsigned);
        }
        return POLY_OK;
    };

    const PairCount pairs = pair_count(F, R);

    // What the row-wise part of layer l is: whether one launch does it, whether the next layer's qkv linear is in it (that layer works on the same blocks
    // and its linear needs no GEMM path for summed terms), with adapters, and the waves of rowreg.hip, 0: tiles of rowlayer.hip
    struct RowPart { bool fits, qkv, lora_q; int waves; };
    auto row_part = [&](int l) -> RowPart {
        const bool lora_on = l >= m->L0 && R > 0, summed = sum && l >= m->L0, branch = !sum && l >= m->L0;
        auto use = [&](int t) { return lora_on && (m->targets & (1 << t)); };
        if (dt != POLY_BF16 || use(2) || use(3) || (summed && (use(0) || use(1))) || !rowlayer_supported(D, Dm, use(0) || use(1) ? m->r : 0)) return {};
        const int ln = l + 1;
        const bool qkv_lora = ln >= m->L0 && R > 0 && (m->targets & 1);
        RowPart p = {true, ln < m->L && (sum || ln != m->L0) && !(sum && qkv_lora), false, 0};
        p.lora_q = p.qkv && qkv_lora;
        p.waves = rowreg_waves(T, D, Dm, use(1) || p.lora_q ? m->r : 0, use(1) || p.lora_q || (branch && l == m->L0), branch ? pairs : known_count(F));
        return p;
    };
    bool x_fragments = false;                  // the residual stream lies in the order of rowreg.hip: between two of its launches that nothing reads it between
    bool qkv_done = false;                     // the qkv linear of layer l was computed by layer l - 1's row kernel
    for (int l = 0; l < m->L; ++l) {
        if (l == 0 && w.fl_cnt[0]) {
            POLY_TRY(w.fl_tiles[0] ? run(false) : flow(false));
            l = m->L0;
            if (l == m->L) break;
        }
        if (l == m->L0 && !selected) POLY_TRY(select_now());
        if (l == m->L0 && w.fl_cnt[1]) {
            POLY_TRY(w.fl_tiles[1] ? run(true) : flow(true));
            break;
        }
        const bool lora_on = l >= m->L0 && R > 0;
        if (l >= m->L0 && R == 0) break;
        // Summed composition: the frame stays ONE block through the adapted layers; its adapters' low-rank terms
        // (one shrink per (frame, adapter) pair, as in the fan-out) are all added in the expand of the frame's block.
        const bool summed = sum && l >= m->L0;
        const bool fan = !sum && l == m->L0;   // first adapted layer: frames fan out into row-blocks
        const bool branch = !sum && l > m->L0; // residual stream already per row-block
        float *x_in = branch ? w.xb : w.xa;
        float *x_out = (!sum && l >= m->L0) ? w.xb : w.xa;
        const int nb = branch ? R : F;         // blocks of the LayerNorm-1 input
        const int *nb_dev = branch ? R_dev : (summed ? &w.meta->F_ok : nullptr);
        const int n_out = (!sum && l >= m->L0) ? R : F;  // blocks after the qkv linear
        const int *n_out_dev = (!sum && l >= m->L0) ? R_dev : (summed ? &w.meta->F_ok : nullptr);

        auto lora_ptr = [&](const void *stack, int t, size_t din, size_t dout, bool is_A) -> const void * {
            (void)t;
            const size_t per_layer = (size_t)m->n_adapters * m->r * (is_A ? din : dout);
            return (const char *)stack + es * per_layer * (size_t)(l - m->L0);
        };
        auto use = [&](int t) { return lora_on && (m->targets & (1 << t)); };

        // narrow models (D <= 192, bf16): LayerNorm, shrink, base product and expand of one linear run in one
        // kernel that keeps 64 token rows on chip; otherwise LayerNorm / shrink / GEMM are separate launches
        auto fused = [&](int t) { return dt == POLY_BF16 && !(summed && use(t)) && rowlin_supported(D, t == 0 ? 3 * D : (t == 2 ? Dm : D), m->r, use(t), t == 1); };
        // low-rank operands of the GEMM path: S block and adapter per (frame, adapter) pair; summed: the pairs of a frame
        // all land on the frame's block
        const int *shrink_map = summed ? w.frame_of_row : nullptr;
        auto lora_gemm = [&](GemmArgs &g, int t, const void *Bt) {
            g.S = w.S; g.RP = RP; g.Bt = Bt; g.r = m->r; g.adapter_of_out = w.adapter_of_row;
            g.set_off = summed ? row_offsets : nullptr;
            (void)t;
        };
        int Tr = T;                            // rows of a block
        auto rowlin = [&](int t, const float *x_ln, const float *ln_g, const float *ln_b, const void *a_in, const int *in_map,
                          const void *Wt, const float *bias, int N, int mode, void *out, const float *res, const int *res_map) -> int {
            RowLinArgs a = {};
            a.x_ln = x_ln; a.ln_g = ln_g; a.ln_b = ln_b; a.eps = m->ln_eps; a.a_in = (const bf16_t *)a_in; a.in_block_of_out = in_map;
            a.T = Tr; a.K = D; a.N = N; a.n_out = n_out; a.n_out_dev = n_out_dev;
            a.Wt = (const bf16_t *)Wt; a.bias = bias;
            if (use(t)) {
                a.At = (const bf16_t *)lora_ptr(lora->At[t], t, D, N, true); a.Bt = (const bf16_t *)lora_ptr(lora->Bt[t], t, D, N, false);
                a.r = m->r; a.scale = m->lora_scale; a.adapter_of_out = w.adapter_of_row;
            }
            a.mode = mode; a.out = out; a.res = res; a.res_block_of_out = res_map;
            return launch_rowlin(a, st);
        };
        const int *fan_map = fan ? w.frame_of_row : nullptr;
        const void *Wqkv = (const char *)base->qkv_w + es * (size_t)l * 3 * D * D, *Wproj = (const char *)base->proj_w + es * (size_t)l * D * D;
        const void *Wfc1 = (const char *)base->fc1_w + es * (size_t)l * Dm * D;

        RowPart rows = row_part(l);

        // ---- attention half
        if (qkv_done) {
            qkv_done = false;
        } else if (dt == POLY_BF16 && !(summed && use(0)) && rowlayer_supported(D, Dm, use(0) ? m->r : 0)) {
            RowLayerArgs a = {};
            a.T = T; a.D = D; a.Dm = Dm; a.n_out = n_out; a.n_out_dev = n_out_dev;
            a.adapter_of_out = use(0) ? w.adapter_of_row : nullptr; a.r = m->r; a.scale = m->lora_scale; a.eps = m->ln_eps;
            a.res = x_in; a.res_block_of_out = fan_map;
            a.lnq_g = base->ln1_g + (size_t)l * D; a.lnq_b = base->ln1_b + (size_t)l * D;
            a.Wqt = (const bf16_t *)Wqkv; a.bq = base->qkv_b + (size_t)l * 3 * D;
            if (use(0)) { a.Aqt = (const bf16_t *)lora_ptr(lora->At[0], 0, D, 3 * D, true); a.Bqt = (const bf16_t *)lora_ptr(lora->Bt[0], 0, D, 3 * D, false); }
            a.qkv_out = (bf16_t *)w.qkv;
            const int waves = rowreg_waves(T, D, Dm, use(0) ? m->r : 0, use(0) || fan, n_out_dev == R_dev ? pairs : known_count(n_out));
            POLY_TRY(waves ? launch_rowreg(a, waves, st) : launch_rowlayer(a, st));
        } else if (fused(0)) {
            POLY_TRY(rowlin(0, x_in, base->ln1_g + (size_t)l * D, base->ln1_b + (size_t)l * D, nullptr, fan_map, Wqkv,
                            base->qkv_b + (size_t)l * 3 * D, 3 * D, EPI_STORE, w.qkv, nullptr, nullptr));
        } else {
            const float *gain = base->ln1_g + (size_t)l * D, *shift = base->ln1_b + (size_t)l * D;
            const void *At = use(0) ? lora_ptr(lora->At[0], 0, D, 3 * D, true) : nullptr;
            const bool shrunk = use(0) && layernorm_shrink_fits(x_in, w.u, gain, shift, D, nb, At, RP, R, w.S, dt);
            if (shrunk) POLY_TRY(launch_layernorm_shrink(x_in, w.u, gain, shift, D, m->ln_eps, T, nb, nb_dev, At, m->r, m->lora_scale, R, R_dev,
                                                         (summed || fan) ? row_offsets : nullptr, w.adapter_of_row, w.S, st));
            const NormGemmArgs ng = {x_in, gain, shift, m->ln_eps, (const bf16_t *)Wqkv, base->qkv_b + (size_t)l * 3 * D, (bf16_t *)w.qkv, 3 * D, T, nb, nb_dev, false};
            const bool few = dt == POLY_BF16 && !use(0) && !fan && norm_gemm_fits(ng, D);
            if (few) POLY_TRY(launch_norm_gemm(ng, st));
            else if (!shrunk) POLY_TRY(launch_layernorm(x_in, w.u, gain, shift, D, m->ln_eps, T, nb, nb_dev, dt, st));
            GemmArgs g = {};
            g.A = w.u; g.Wt = Wqkv; g.bias = base->qkv_b + (size_t)l * 3 * D;
            g.T = T; g.K = D; g.N = 3 * D; g.n_in = nb; g.n_in_dev = fan ? &w.meta->F_ok : nb_dev;
            g.out_off = fan ? row_offsets : nullptr;
            if (use(0)) {
                const void *Bt = lora_ptr(lora->Bt[0], 0, D, 3 * D, false);
                if (!shrunk) POLY_TRY(launch_shrink(w.u, T, D, At, m->r, RP, m->lora_scale, F, R, R_dev, summed ? shrink_map : fan_map, w.adapter_of_row,
                                       (summed || fan) ? row_offsets : nullptr, w.S, dt, st));
                lora_gemm(g, 0, Bt);
            }
            g.mode = EPI_STORE; g.out = w.qkv; g.Tout = T;
            if (!few) POLY_TRY(launch_gemm(g, {!branch, pairs.usual}, dt, st));
        }
        if (class_rows && l + 1 == m->L) {
            float *x_class = (float *)((char *)w.o + align_up((size_t)n_out * D * es));
            POLY_TRY(launch_attention_class(w.qkv, w.o, T, D, m->heads, n_out, n_out_dev, x_in, fan_map, x_fragments, x_class, dt, st));
            x_in = x_out = x_class;
            x_end = x_class;
            fan_map = nullptr; x_fragments = false; rows.waves = 0;
            Tr = T_end = 1;
        } else {
            // (as a rule a frame has an adapter, so that there are about as many row-blocks as frames or more)
            POLY_TRY(launch_attention(w.qkv, w.o, T, D, m->heads, n_out, n_out_dev, n_out < F ? n_out : F, dt, rows.waves > 0, st));
        }
        // narrow models without adapters on fc1 / fc2: everything row-wise of the layer in one launch -- proj with its
        // residual, the MLP half, and the qkv linear of the next layer when that layer works on the same blocks
        if (rows.fits) {
            RowLayerArgs a = {};
            a.T = Tr; a.D = D; a.Dm = Dm; a.n_out = n_out; a.n_out_dev = n_out_dev;
            const bool adapters = lora_on && !sum && (use(1) || (m->targets & 1));
            a.adapter_of_out = adapters ? w.adapter_of_row : nullptr; a.r = m->r; a.scale = m->lora_scale; a.eps = m->ln_eps;
            a.o = (const bf16_t *)w.o; a.Wpt = (const bf16_t *)Wproj; a.bp = base->proj_b + (size_t)l * D;
            if (use(1)) { a.Apt = (const bf16_t *)lora_ptr(lora->At[1], 1, D, D, true); a.Bpt = (const bf16_t *)lora_ptr(lora->Bt[1], 1, D, D, false); }
            a.res = x_in; a.res_block_of_out = fan_map;
            a.ln2_g = base->ln2_g + (size_t)l * D; a.ln2_b = base->ln2_b + (size_t)l * D;
            a.W1t = (const bf16_t *)Wfc1; a.b1 = base->fc1_b + (size_t)l * Dm;
            a.W2t = (const bf16_t *)((const char *)base->fc2_w + es * (size_t)l * D * Dm); a.b2 = base->fc2_b + (size_t)l * D;
            a.x_out = x_out;
            const int ln = l + 1;
            if (rows.qkv) {
                a.lnq_g = base->ln1_g + (size_t)ln * D; a.lnq_b = base->ln1_b + (size_t)ln * D;
                a.Wqt = (const bf16_t *)((const char *)base->qkv_w + es * (size_t)ln * 3 * D * D); a.bq = base->qkv_b + (size_t)ln * 3 * D;
                if (rows.lora_q) {
                    const size_t per_layer = (size_t)m->n_adapters * m->r * D;
                    a.Aqt = (const bf16_t *)((const char *)lora->At[0] + es * per_layer * (size_t)(ln - m->L0));
                    a.Bqt = (const bf16_t *)((const char *)lora->Bt[0] + es * per_layer * 3 * (size_t)(ln - m->L0));
                }
                a.qkv_out = (bf16_t *)w.qkv;
                qkv_done = true;
            }
            // (rows in the order of rowreg.hip end up to 31 rows past the buffer's last: what lies there, the start of xb, u or h, is in no use then)
            a.res_fragments = x_fragments;
            const bool base_head_reads = ln == m->L0 && !selected;         // .. before the next layer, rows one by one
            x_fragments = a.out_fragments = rows.waves && rows.qkv && !base_head_reads && row_part(ln).waves;
            POLY_TRY(rows.waves ? launch_rowreg(a, rows.waves, st) : launch_rowlayer(a, st));
            continue;
        }
        if (fused(1)) {
            POLY_TRY(rowlin(1, nullptr, nullptr, nullptr, w.o, nullptr, Wproj, base->proj_b + (size_t)l * D, D, EPI_RESID, x_out, x_in, fan_map));
        } else {
            GemmArgs g = {};
            g.A = w.o; g.Wt = Wproj; g.bias = base->proj_b + (size_t)l * D;
            g.T = Tr; g.K = D; g.N = D; g.n_in = n_out; g.n_in_dev = n_out_dev;
            if (use(1)) {
                const void *At = lora_ptr(lora->At[1], 1, D, D, true), *Bt = lora_ptr(lora->Bt[1], 1, D, D, false);
                POLY_TRY(launch_shrink(w.o, Tr, D, At, m->r, RP, m->lora_scale, F, R, R_dev, shrink_map, w.adapter_of_row, summed ? row_offsets : nullptr,
                                       w.S, dt, st));
                lora_gemm(g, 1, Bt);
            }
            g.mode = EPI_RESID; g.out = x_out; g.Tout = Tr; g.res = x_in; g.res_block_of_out = fan_map;
            POLY_TRY(launch_gemm(g, {n_out_dev != R_dev, pairs.usual}, dt, st));
        }
        // ---- MLP half (x_out holds the stream from here on)
        if (dt == POLY_BF16 && !use(2) && !use(3) && mlp_supported(D, Dm)) {
            // no adapter on fc1 / fc2 in this layer: LayerNorm, both products, GELU and the residual in one kernel
            MlpArgs a = {};
            a.x = x_out; a.ln_g = base->ln2_g + (size_t)l * D; a.ln_b = base->ln2_b + (size_t)l * D; a.eps = m->ln_eps;
            a.T = Tr; a.D = D; a.Dm = Dm; a.n_out = n_out; a.n_out_dev = n_out_dev;
            a.W1t = (const bf16_t *)Wfc1; a.b1 = base->fc1_b + (size_t)l * Dm;
            a.W2t = (const bf16_t *)((const char *)base->fc2_w + es * (size_t)l * D * Dm); a.b2 = base->fc2_b + (size_t)l * D;
            POLY_TRY(launch_mlp(a, st));
            continue;
        }
        if (fused(2)) {
            POLY_TRY(rowlin(2, x_out, base->ln2_g + (size_t)l * D, base->ln2_b + (size_t)l * D, nullptr, nullptr, Wfc1,
                            base->fc1_b + (size_t)l * Dm, Dm, EPI_GELU, w.h, nullptr, nullptr));
        } else {
            const float *gain = base->ln2_g + (size_t)l * D, *shift = base->ln2_b + (size_t)l * D;
            const void *At = use(2) ? lora_ptr(lora->At[2], 2, D, Dm, true) : nullptr;
            const bool shrunk = use(2) && layernorm_shrink_fits(x_out, w.u, gain, shift, D, n_out, At, RP, R, w.S, dt);
            if (shrunk) POLY_TRY(launch_layernorm_shrink(x_out, w.u, gain, shift, D, m->ln_eps, Tr, n_out, n_out_dev, At, m->r, m->lora_scale, R, R_dev,
                                                         summed ? row_offsets : nullptr, w.adapter_of_row, w.S, st));
            NormGemmArgs ng = {x_out, gain, shift, m->ln_eps, (const bf16_t *)Wfc1, base->fc1_b + (size_t)l * Dm, (bf16_t *)w.h, Dm, T, n_out, n_out_dev, true};
            const bool few = dt == POLY_BF16 && !use(2) && norm_gemm_fits(ng, D);       // (class rows as the rows of the layers before: 11 us, 5 + 8 in two launches)
            ng.T = Tr;
            if (few) POLY_TRY(launch_norm_gemm(ng, st));
            else if (!shrunk) POLY_TRY(launch_layernorm(x_out, w.u, gain, shift, D, m->ln_eps, Tr, n_out, n_out_dev, dt, st));
            GemmArgs g = {};
            g.A = w.u; g.Wt = Wfc1; g.bias = base->fc1_b + (size_t)l * Dm;
            g.T = Tr; g.K = D; g.N = Dm; g.n_in = n_out; g.n_in_dev = n_out_dev;
            if (use(2)) {
                const void *Bt = lora_ptr(lora->Bt[2], 2, D, Dm, false);
                if (!shrunk) POLY_TRY(launch_shrink(w.u, Tr, D, At, m->r, RP, m->lora_scale, F, R, R_dev, shrink_map, w.adapter_of_row, summed ? row_offsets : nullptr,
                                       w.S, dt, st));
                lora_gemm(g, 2, Bt);
            }
            g.mode = EPI_GELU; g.out = w.h; g.Tout = Tr;
            if (!few) POLY_TRY(launch_gemm(g, {n_out_dev != R_dev, pairs.usual}, dt, st));
        }
        {
            GemmArgs g = {};
            g.A = w.h; g.Wt = (const char *)base->fc2_w + es * (size_t)l * D * Dm; g.bias = base->fc2_b + (size_t)l * D;
            g.T = Tr; g.K = Dm; g.N = D; g.n_in = n_out; g.n_in_dev = n_out_dev;
            if (use(3)) {
                const void *At = lora_ptr(lora->At[3], 3, Dm, D, true), *Bt = lora_ptr(lora->Bt[3], 3, Dm, D, false);
                POLY_TRY(launch_shrink(w.h, Tr, Dm, At, m->r, RP, m->lora_scale, F, R, R_dev, shrink_map, w.adapter_of_row, summed ? row_offsets : nullptr,
                                       w.S, dt, st));
                lora_gemm(g, 3, Bt);
            }
            g.mode = EPI_RESID; g.out = x_out; g.Tout = Tr; g.res = x_out;
            POLY_TRY(launch_gemm(g, {n_out_dev != R_dev, pairs.usual}, dt, st));
        }
    }

    if (!selected) POLY_TRY(select_now());        // (L0 == L: the shared layers are the whole backbone)
    if (R > 0) {
        POLY_TRY(launch_head(x_end, (adapted && !sum) ? nullptr : w.frame_of_row, T_end, D, base->lnf_g, base->lnf_b, m->ln_eps,
                             heads->head_w, heads->head_b, m->C, w.adapter_of_row, w.frame_of_row, heads->class_map, K, w.meta, R,
                             out_logits, out_scores, out_merged, dt, st));
    }
    return POLY_OK;
}
}  // namespace

extern "C" int poly_forward(const poly_model_desc *m, const poly_base_weights *base, const poly_lora_weights *lora,
                            const poly_heads *heads, const void *frames, int F, const int32_t *row_offsets,
                            const int32_t *adapter_ids, int R, float *out_logits, float *out_scores, float *out_merged, int K,
                            int32_t *dev_status, void *workspace, size_t workspace_bytes, void *stream)
{
    return forward_impl(m, base, lora, heads, frames, F, row_offsets, adapter_ids, R, out_logits, out_scores, out_merged, K, dev_status,
                        workspace, workspace_bytes, stream, nullptr);
}

// the lagged scores take the end of the workspace, the forward what is in front of them
static size_t stream_lag_bytes(int F, int K) { return sizeof(float) * (size_t)(F + 1) * K; }

extern "C" size_t poly_stream_step_workspace_bytes(const poly_model_desc *m, int F, int R, int K)
{
    if (check_model(m) != POLY_OK || F < 0 || R < 0 || K <= 0) return 0;
    return forward_bytes(m, F, R, true) + stream_lag_bytes(F, K);
}

extern "C" int poly_stream_step(const poly_model_desc *m, const poly_base_weights *base, const poly_lora_weights *lora,
                                const poly_heads *heads, const poly_stream *s, const void *frames, int F, int R,
                                int32_t *row_offsets, int32_t *adapter_ids, int32_t *counters, float *out_base_scores,
                                float *out_logits, float *out_scores, float *out_merged, int32_t *dev_status, void *workspace,
                                size_t workspace_bytes, void *stream)
{
    POLY_TRY(check_model(m));
    if (!s || !s->base_w || !s->base_b || !s->group_membership || !s->carry || !counters) return POLY_EINVAL;
    if (s->K <= 0 || s->K > POLY_MAX_LABELS || s->M <= 0 || s->M > POLY_MAX_CONTEXTS || s->M > m->n_adapters) return POLY_EINVAL;
    if (F < 0 || R < 0) return POLY_EINVAL;
    if (F == 0) return POLY_OK;
    if (!workspace || ((uintptr_t)workspace & 255) != 0) return POLY_EINVAL;
    const size_t lag = stream_lag_bytes(F, s->K);
    if (workspace_bytes < lag) return POLY_ECAP;
    const size_t forward = (workspace_bytes - lag) & ~(size_t)255;
    StreamStep ss = {s, row_offsets, adapter_ids, counters, out_base_scores, (float *)((char *)workspace + forward)};
    return forward_impl(m, base, lora, heads, frames, F, row_offsets, adapter_ids, R, out_logits, out_scores, out_merged, s->K, dev_status,
                        workspace, forward, stream, &ss);
}

// ------------------------------------------------------------------ isolated multi-LoRA linear

namespace {
struct LinearWs {
    PolyMeta *meta;
    int32_t *frame_of_row, *adapter_of_row;
    void *S;
    size_t bytes;
};
LinearWs carve_linear(int T, int r, int R, int dtype, void *base)
{
    Carver c{(char *)base, 0};
    LinearWs w;
    w.meta = c.take<PolyMeta>(sizeof(PolyMeta));
    w.frame_of_row = c.take<int32_t>(sizeof(int32_t) * (size_t)(R + 1));
    w.adapter_of_row = c.take<int32_t>(sizeof(int32_t) * (size_t)(R + 1));
    w.S = c.take<void>(elt_size(dtype) * (size_t)R * T * rank_pad(r));
    w.bytes = c.off;
    return w;
}
}  // namespace

extern "C" size_t poly_lora_linear_workspace_bytes(int n_xblocks, int T, int r, int R, int dtype)
{
    if (n_xblocks < 0 || T <= 0 || r <= 0 || R < 0 || (dtype != POLY_F32 && dtype != POLY_BF16)) return 0;
    return carve_linear(T, r, R, dtype, nullptr).bytes;
}

namespace {
int lora_linear_impl(const void *X, int n_xblocks, int T, int Kdim, const void *Wt, const float *bias, int Ndim, const void *At,
                     const void *Bt, int n_adapters, int r, float scale, const int32_t *row_offsets, const int32_t *adapter_ids, int R,
                     void *Y, int dtype, int32_t *dev_status, void *workspace, size_t workspace_bytes, void *stream)
{
    const LinearWs w = carve_linear(T, r, R, dtype, workspace);
    if (workspace_bytes < w.bytes) return POLY_ECAP;
    hipStream_t st = (hipStream_t)stream;
    const int RP = rank_pad(r);

    if (R > 0 && linear_ks_fits(X, n_xblocks, T, Wt, bias, Ndim, At, Bt, r, R, Y))
        return launch_linear_ks(X, n_xblocks, T, Kdim, Wt, bias, Ndim, At, Bt, n_adapters, r, scale, row_offsets, adapter_ids, R, Y, dtype, dev_status, st);
    if (R > 0 && shrink_csr_fits(n_xblocks, T, Kdim, dtype)) {
        POLY_TRY(launch_shrink_csr(X, T, Kdim, At, r, RP, scale, row_offsets, adapter_ids, n_xblocks, R, n_adapters, w.meta, w.frame_of_row,
                                   w.adapter_of_row, dev_status, w.S, st));
    } else {
        POLY_TRY(launch_prep(row_offsets, adapter_ids, n_xblocks, R, n_adapters, w.meta, w.frame_of_row, w.adapter_of_row, dev_status, st));
        if (R == 0) return POLY_OK;
        POLY_TRY(launch_shrink(X, T, Kdim, At, r, RP, scale, n_xblocks, R, &w.meta->R, w.frame_of_row, w.adapter_of_row, row_offsets, w.S, dtype, st));
    }
    GemmArgs g = {};
    g.A = X; g.Wt = Wt; g.bias = bias; g.T = T; g.K = Kdim; g.N = Ndim;
    g.n_in = n_xblocks; g.n_in_dev = &w.meta->F_ok; g.out_off = row_offsets;
    g.S = w.S; g.RP = RP; g.Bt = Bt; g.r = r; g.adapter_of_out = w.adapter_of_row;
    g.mode = EPI_STORE; g.out = Y; g.Tout = T;
    return launch_gemm(g, {true, R}, dtype, st);
}

int check_lora_linear(const void *X, int n_xblocks, int T, int Kdim, const void *Wt, int Ndim, const void *At, const void *Bt,
                      int n_adapters, int r, const int32_t *row_offsets, const int32_t *adapter_ids, int R, void *Y, int dtype)
{
    if (dtype != POLY_F32 && dtype != POLY_BF16) return POLY_EINVAL;
    if (n_xblocks < 0 || T <= 0 || Kdim <= 0 || Ndim <= 0 || n_adapters <= 0 || r <= 0 || r > POLY_MAX_RANK || R < 0) return POLY_EINVAL;
    if (Kdim % (dtype == POLY_BF16 ? 8 : 4)) return POLY_EINVAL;
    if (n_xblocks == 0) return POLY_OK;
    if (!X || !Wt || !At || !Bt || !row_offsets || (R > 0 && (!adapter_ids || !Y))) return POLY_EINVAL;
    return POLY_OK;
}
}  // namespace

extern "C" int poly_lora_linear(const void *X, int n_xblocks, int T, int Kdim, const void *Wt, const float *bias, int Ndim,
                                const void *At, const void *Bt, int n_adapters, int r, float scale, const int32_t *row_offsets,
                                const int32_t *adapter_ids, int R, void *Y, int dtype, int32_t *dev_status, void *workspace,
                                size_t workspace_bytes, void *stream)
{
    POLY_TRY(check_lora_linear(X, n_xblocks, T, Kdim, Wt, Ndim, At, Bt, n_adapters, r, row_offsets, adapter_ids, R, Y, dtype));
    if (n_xblocks == 0) return POLY_OK;
    if (!workspace || ((uintptr_t)workspace & 255) != 0) return POLY_EINVAL;
    return lora_linear_impl(X, n_xblocks, T, Kdim, Wt, bias, Ndim, At, Bt, n_adapters, r, scale, row_offsets, adapter_ids, R, Y, dtype,
                            dev_status, workspace, workspace_bytes, stream);
}

// ------------------------------------------------------------------ isolated linear without a caller workspace
// For callers that cannot allocate (code under graph capture, serving loops, harnesses that forbid hipMalloc): the bookkeeping,
// the row maps and the shrink output S live in a file-scope device array instead of a workspace argument.  Each GPU the library
// is loaded on holds its own copy of the array; its address on a device is looked up once, with that device current.
static __device__ __align__(256) unsigned char scratch[POLY_STATIC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
void *scratch_of_device[MAX_DEVICES];          // device address of `scratch` per device ordinal, null until looked up

int static_scratch(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return POLY_EHIP;
    void *p = __atomic_load_n(&scratch_of_device[dev], __ATOMIC_ACQUIRE);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return POLY_EHIP;
        __atomic_store_n(&scratch_of_device[dev], p, __ATOMIC_RELEASE);   // (two racing first calls look up the same address)
    }
    *out = p;
    return POLY_OK;
}
}  // namespace

extern "C" int poly_lora_linear_static(const void *X, int n_xblocks, int T, int Kdim, const void *Wt, const float *bias, int Ndim,
                                       const void *At, const void *Bt, int n_adapters, int r, float scale,
                                       const int32_t *row_offsets, const int32_t *adapter_ids, int R, void *Y, int dtype,
                                       int32_t *dev_status, void *stream)
{
    POLY_TRY(check_lora_linear(X, n_xblocks, T, Kdim, Wt, Ndim, At, Bt, n_adapters, r, row_offsets, adapter_ids, R, Y, dtype));
    if (n_xblocks == 0) return POLY_OK;
    if (carve_linear(T, r, R, dtype, nullptr).bytes > (size_t)POLY_STATIC_SCRATCH_BYTES) return POLY_ECAP;
    void *ws = nullptr;
    POLY_TRY(static_scratch(&ws));
    // nothing in the scratch area has to start at zero: the CSR check writes the bookkeeping words and the row maps of every
    // row it accepts, and the shrink writes all RP columns of every S row the product reads
    return lora_linear_impl(X, n_xblocks, T, Kdim, Wt, bias, Ndim, At, Bt, n_adapters, r, scale, row_offsets, adapter_ids, R, Y, dtype,
                            dev_status, ws, POLY_STATIC_SCRATCH_BYTES, stream);
}
