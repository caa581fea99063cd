// C ABI of libasynclm: sequence state machine, argument checking, memory, launch order.
#include "../../include/asynclm.h"
#include "common.h"
#include "launch.h"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <vector>

using namespace asynclm;

// Host-side builder of the row table of one pass.
struct PassBuilder {
    ChunkTable t{};
    int G = 1, Hkv = 1, max_keys = 0, batch_rows = CHUNK_BATCH_ROWS;
    long long block_tiles = 0;          // key tiles of 32 over all task blocks
    void clear() { t.rows = t.ngroups = t.ntasks = t.nhead = t.nblocks = t.npieces = 0; max_keys = 0; block_tiles = 0; }
    int tiles_of(int n) const { return (G * n + 31) / 32; }
    // batched steps: rows, attention tasks, and the attention's partial results (task x kv head x at least 4 key splits) all fit one pass
    bool fits(int n) const {
        return t.rows + n <= batch_rows && t.ntasks + tiles_of(n) <= CHUNK_BATCH_TASKS &&
               (long long)(t.ntasks + tiles_of(n)) * Hkv * 4 <= CHUNK_ATTN_MAX_UNITS;
    }
    // Appends a group of n rows to sequence `seq` (length before: pos0).  forced: the first row's token if >= 0, -1: the greedy
    // token of the sequence's logits, -2: `rest` holds the tokens of all n rows (else of the n - 1 behind the first).
    void add(int seq, int pos0, int n, int forced, const int32_t* rest, bool want_head) {
        const int row0 = t.rows;
        for (int r = 0; r < n; ++r) {
            ChunkRow& R = t.row[row0 + r];
            R = ChunkRow{};
            R.token = forced == -2 ? rest[r] : (r == 0 ? forced : rest[r - 1]);      // -1: chosen on the device
            R.seq = seq; R.pos = pos0 + r; R.row0 = row0; R.n = n; R.group = r == 0 && forced != -2 ? t.ngroups : -1;
        }
        ChunkGroup& Gp = t.group[t.ngroups++];
        Gp = ChunkGroup{};
        Gp.seq = seq; Gp.row0 = row0; Gp.n = n; Gp.pos0 = pos0; Gp.head = want_head ? t.nhead++ : -1;
        for (int tile = 0; tile < tiles_of(n); ++tile) {
            if (tile % 4 == 0) { t.block[t.nblocks++] = ChunkTaskBlock{t.ntasks, std::min(4, tiles_of(n) - tile)}; block_tiles += (pos0 + n + 31) / 32; }
            ChunkTask& T = t.task[t.ntasks++];
            T = ChunkTask{};
            T.seq = seq; T.row0 = row0; T.n = n; T.pos0 = pos0; T.tile = tile;
        }
        t.rows += n;
        max_keys = std::max(max_keys, pos0 + n);
    }
};


struct asynclm_ctx {
    asynclm_config cfg{};
    Geom g{};
    hipStream_t stream = nullptr;
    hipStream_t stream2 = nullptr;      // library-owned: every other kernel of a two-stream decoding step
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    bool pipe_ok = false;               // two workgroups of every single-row kernel fit one compute unit
    unsigned long long* pipe_stamps = nullptr;   // per kernel of the step: see pipe_stamp
    unsigned long long* stamp_done = nullptr;    // [pipe_kernels_max][STAMP_DONE_SLOTS]: see step_stamp_done
    int pipe_kernels = 0;               // kernels of the last step that left time stamps (two streams, or stamp mode); else 0
    int opt_step_stamps = 0;            // stamp mode: one-stream steps run as plain launches and leave time stamps
    bool stamp_now = false;             // the pass being enqueued is such a step
    bool last_step_stamp_mode = false;  // the last step was one
    int pipe_kernels_max = 0;
    unsigned* pipe_go = nullptr;        // [PIPE_REGIONS][PIPE_MAX_WORKGROUPS] hand-over words, one per cache line
    unsigned* pipe_counters = nullptr;  // [pipe_kernels_max] arrival counters, one per cache line
    int device = 0, n_cu = 0;
    bool poisoned = false;
    hipError_t last_hip = hipSuccess;

    const void* embed = nullptr; const float* final_norm = nullptr; const void* lm_head = nullptr;
    std::vector<const float*> attn_norm, ffn_norm;
    std::vector<const void*> wqkv, wo, wgate_up, wdown;

    std::vector<void*> allocs;          // everything from hipMalloc
    void* kv = nullptr;                 // [seq][layer][k|v][Hkv][max_pos][dh] in cfg.dtype
    float* logits = nullptr;            // [max_seqs][V]
    DecodeBuffers b{};
    ChunkBuffers cb{};
    bool chunk_ok = false;              // the matrix-core append path supports this model
    int pass_rows = CHUNK_BATCH_ROWS;   // rows that one of its passes can hold (CHUNK_BATCH_ROWS .. CHUNK_MAX; fewer: PASS_ROWS_UNALIGNED)
    RowsBuffers rb{};                   // the other models: several rows per pass through the vector-unit kernels
    int rows_pass = ROWS_MAX;           // ... this many at most (what the buffers hold)
    int wide_rows = 0;                  // ... or this many on the matrix cores (forward_wide_rows); 0: not this model
    SmallBuffers small{};               // decoding step of small models; null: not this model
    FusedPlan fused{};                  // single-kernel decoding step
    void* layers_dev = nullptr;         // per-layer pointer table of the fused step
    unsigned* bar = nullptr;            // its grid-barrier counters
    unsigned long long* trace = nullptr; // its optional phase time stamps
    bool want_trace = false;
    std::vector<unsigned long long> last_trace;  // raw stamps [stamp][workgroup] of the last profiled fused step
    int last_trace_stamps = 0;
    int32_t* token_host = nullptr;      // pinned, 16 ints: [0..1] staging of read-backs, [4..5] token and number of the running step (TokenWord)
    uint32_t tok_serial = 0;            // number of the last decoding step
    bool tok_early = false;             // the last decoding step leaves its token in that word as soon as it is chosen
    hipEvent_t tok_event = nullptr;     // behind the kernel that chooses it (long steps), see wait_token
    bool tok_marked = false;            // ... recorded there in the last step

    std::vector<int32_t> len;           // host mirror of the sequence lengths
    std::vector<int32_t> nban;          // host mirror of the number of banned token ids per sequence
    std::vector<char> choice_stale;     // the ban list changed after the sequence's greedy token was computed
    PassBuilder pass;                   // row table of the append-chunk pass being built
    // pinned staging of what the host uploads on the hot path (a pageable source would make the copy wait for the
    // stream): two copies of the row table and a small ring of ban-list rows, each reused once its event has passed
    unsigned char* tab_host[2] = {nullptr, nullptr};
    hipEvent_t tab_ev[2] = {nullptr, nullptr};
    int tab_next = 0;
    static constexpr int BAN_RING = 4;
    int32_t* ban_host = nullptr;        // [BAN_RING][1 + BAN_MAX]
    hipEvent_t ban_ev[BAN_RING] = {};
    int ban_next = 0;
    std::vector<char> batch_seen;       // scratch of asynclm_step_batch (sized at create)
    std::vector<int> batch_owner;

    // options
    int opt_chunk = CHUNK_MAX /* as long as the buffers allow */, opt_graph = 1, opt_attn_split = 0, opt_chunk_split = 0, opt_fused = 0, opt_attn_mfma_min = 1;
    int opt_pipeline = 0;

    std::map<int, hipGraphExec_t> graphs;   // captured decoding steps by graph_key(), all instantiated by rebuild_graphs()

    // profiling of one step
    bool prof = false;
    std::vector<hipEvent_t> prof_events;
    std::vector<int> prof_class;
};

namespace {

const char* const kClassNames[KC_COUNT] = {
    "begin_step", "embed", "qkv_rope_kvwrite", "attn_decode", "o_proj_residual", "gate_up_swiglu",
    "down_residual", "lm_head", "argmax", "chunk_prep", "chunk_gemm", "chunk_attn", "chunk_misc",
    "fused_step_kernel", "fused:qkv", "fused:qkv_barrier", "fused:attn", "fused:attn_barrier", "fused:merge",
    "fused:merge_barrier", "fused:o_proj", "fused:o_proj_barrier", "fused:gate_up", "fused:gate_up_barrier",
    "fused:down", "fused:down_barrier", "fused:lm_head", "fused:lm_head_barrier"};

// With ASYNCLM_VERBOSE set in the environment, HIP failures are reported on stderr.
void report_hip(const char* where, hipError_t e) {
    if (std::getenv("ASYNCLM_VERBOSE")) std::fprintf(stderr, "[asynclm] %s: %s\n", where, hipGetErrorString(e));
}

int fail_device(asynclm_ctx* c, hipError_t e) {
    report_hip("device call failed", e);
    c->poisoned = true;
    c->last_hip = e;
    return ASYNCLM_E_DEVICE;
}

#define HIPCK(c, expr)                                         \
    do {                                                       \
        hipError_t _e = (expr);                                \
        if (_e != hipSuccess) return fail_device((c), _e);     \
    } while (0)

template <class F>
hipError_t run(asynclm_ctx* c, int kc, F&& f) {
    if (!c->prof) return f();
    hipEvent_t e0, e1;
    hipError_t e;
    if ((e = hipEventCreate(&e0)) != hipSuccess) return e;
    if ((e = hipEventCreate(&e1)) != hipSuccess) return e;
    c->prof_events.push_back(e0); c->prof_events.push_back(e1); c->prof_class.push_back(kc);
    if ((e = hipEventRecord(e0, c->stream)) != hipSuccess) return e;
    if ((e = f()) != hipSuccess) return e;
    return hipEventRecord(e1, c->stream);
}

size_t elem_bytes(const asynclm_ctx* c) { return c->cfg.dtype == ASYNCLM_DTYPE_FP32 ? 4 : 2; }

void* kv_layer_ptr(const asynclm_ctx* c, int layer) {
    return (char*)c->kv + (size_t)layer * c->g.kv_layer_stride * elem_bytes(c);
}

// Attention splits for a context of len_after tokens.  Up to 2048 tokens: at most MERGE_MAX_SPLIT splits, which
// the O projection merges while it stages its input (no merge step at all).  Longer: up to ATTN_MAX_SPLIT
// splits with a merge step of their own.
struct SplitPlan { int nsplit; bool merge_in_oproj; bool mfma; bool small = false /* forward_single_small */; };

SplitPlan pick_nsplit(const asynclm_ctx* c, int len_after, bool single_row_kernel = false) {
    const bool no_v_rows = c->g.kv_v_offset == 0;      // the single-row kernel has nothing to read: matrix cores at any length
    if (!single_row_kernel && c->chunk_ok && (no_v_rows || (c->opt_attn_mfma_min > 0 && len_after >= c->opt_attn_mfma_min))) {
        // attention on the matrix cores: 96 key splits at every length (a wave takes one tile of 32 keys up to 3072 keys,
        // more beyond; waves without keys leave at once), so one captured graph serves every context length.  Measured
        // optima were one tile per wave up to about 96 tiles and 96 splits beyond (more only lengthen the merge).
        int n = 96;
        if (c->opt_attn_split > 0) n = std::max(4, std::min((c->opt_attn_split + 3) / 4 * 4, CHUNK_ATTN_MAX_SPLIT));
        return {n, false, true};
    }
    if (c->opt_attn_split > 0) {
        const int n = c->opt_attn_split < ATTN_MAX_SPLIT ? c->opt_attn_split : ATTN_MAX_SPLIT;
        return {n, n <= 8, false};
    }
    // up to 2048 tokens: a split per 64 positions, at most the 8 that the O projection merges; beyond: a split per
    // 256 positions (one pass of the kernel's inner loop), merged by the last workgroup of each kv head
    const bool merged = len_after <= 2048;
    const int want = merged ? (len_after + 63) / 64 : (len_after + 255) / 256, cap = merged ? 8 : ATTN_MAX_SPLIT;
    int n = 1;
    while (n < want && n < cap) n *= 2;
    return {n, merged, false};
}

// The plan of a decoding step.  Small models with few keys, where it pays: forward_single_small.
SplitPlan pick_step_plan(const asynclm_ctx* c, int len_after, bool pipelined) {
    if (c->small.parts && !pipelined && c->opt_attn_split == 0 && small_step_supported(c->cfg.dtype, c->g) && small_step_pays(c->cfg.dtype, c->g, c->cfg.n_layers, len_after))
        return {1, false, false, true};
    return pick_nsplit(c, len_after, pipelined);
}

// Such a step of few launches is issued launch by launch: a graph starts later than a launch.  Tiny preset with 1 / 2 / 3 / 4 / 6 layers: 28.2 / 40.5 /
// 52.8 / 65.6 / 92 us per step as a graph, 22.7 / 37.2 / 52.0 / 67.8 / 97 launch by launch, where the host becomes the slower side.
bool small_direct(const asynclm_ctx* c, SplitPlan sp) { return sp.small && c->cfg.n_layers <= SMALL_DIRECT_LAYERS; }

// Step of a small model behind its first kernel (launch_small_first, which is launched with sequence and forced token as arguments):
// see decode_small.hip.  The residual stream alternates between two vectors, because the workgroup that writes it is not the only one
// that reads it.
hipError_t forward_single_small(asynclm_ctx* c, bool with_head) {
    const int dt = c->cfg.dtype, nl = c->cfg.n_layers;
    const Geom& g = c->g;
    hipStream_t s = c->stream;
    float* xb[2] = {c->b.x, c->b.x2};
    hipError_t e;
    for (int l = 0; l < nl; ++l) {
        void* kvl = kv_layer_ptr(c, l);
        if (l > 0 && (e = run(c, KC_QKV, [&] { return launch_small_qkv(dt, c->wqkv[l], c->attn_norm[l], kvl, c->small, c->b, g, xb[(l - 1) & 1], xb[l & 1], s); }))) return e;
        if ((e = run(c, KC_ATTN, [&] { return launch_small_attn_o(dt, kvl, c->wo[l], c->small, c->b, g, l == 0, s); }))) return e;
        if ((e = run(c, KC_GATEUP, [&] { return launch_small_mlp(dt, c->wgate_up[l], c->wdown[l], c->ffn_norm[l], xb[l & 1], c->small, g, s); }))) return e;
    }
    return with_head ? run(c, KC_LMHEAD, [&] { return launch_small_head(dt, c->lm_head, c->final_norm, c->logits, c->small, c->b, g, xb[(nl - 1) & 1], s); }) : hipSuccess;
}

// One forward pass of a single row whose token/position are already in the step descriptor.
hipError_t forward_single(asynclm_ctx* c, int seq, bool with_head, SplitPlan sp) {
    const int dt = c->cfg.dtype;
    const Geom& g = c->g;
    hipStream_t s = c->stream;
    hipError_t e;
    // stamp mode (matrix-core attention plans): every kernel gets six stamp words, six kernels per layer, then the head
    const bool stamps = c->stamp_now && c->pipe_stamps && c->stamp_done;
    int idx = 0;
    PipeSync ps{};
    auto next = [&]() -> const PipeSync* {
        if (!stamps) return nullptr;
        ps.stamps = c->pipe_stamps + (size_t)idx * 6;
        ps.done_wg = c->stamp_done + (size_t)idx * STAMP_DONE_SLOTS;
        ++idx;
        return &ps;
    };
    if (stamps && (e = launch_stamp_init(c->stamp_done, c->pipe_kernels, s))) return e;
    for (int l = 0; l < c->cfg.n_layers; ++l) {
        void* kvl = kv_layer_ptr(c, l);
        const PipeSync* st = next();
        if ((e = run(c, KC_QKV, [&] { return launch_qkv(dt, c->wqkv[l], c->attn_norm[l], kvl, c->b, g, s, st); }))) return e;
        if (sp.mfma) {
            unsigned long long* sw = stamps ? c->pipe_stamps + (size_t)idx * 6 : nullptr;
            unsigned long long* dw = stamps ? c->stamp_done + (size_t)idx * STAMP_DONE_SLOTS : nullptr;
            idx += stamps ? 2 : 0;
            if ((e = run(c, KC_ATTN, [&] { return launch_decode_attn_mfma(c->cb, kvl, sp.nsplit, c->b, g, s, sw, dw); }))) return e;
        } else if ((e = run(c, KC_ATTN, [&] { return launch_attn_decode(dt, kvl, sp.nsplit, sp.merge_in_oproj, c->b, g, s); }))) return e;
        st = next();
        if ((e = run(c, KC_OPROJ, [&] { return launch_oproj(dt, c->wo[l], sp.merge_in_oproj ? sp.nsplit : 0, c->b, g, s, st); }))) return e;
        st = next();
        if ((e = run(c, KC_GATEUP, [&] { return launch_gateup(dt, c->wgate_up[l], c->ffn_norm[l], c->b, g, s, st); }))) return e;
        st = next();
        if ((e = run(c, KC_DOWN, [&] { return launch_down(dt, c->wdown[l], c->b, g, s, st); }))) return e;
    }
    if (with_head) {
        // logits of every sequence live in one array; the kernels pick the row from the descriptor
        const PipeSync* st = next();
        if ((e = run(c, KC_LMHEAD, [&] { return launch_lmhead(dt, c->lm_head, c->final_norm, c->logits, c->b, g, s, st); }))) return e;
    }
    return hipSuccess;
}

// The same pass with its kernels alternating between two streams, so that two neighbouring kernels run at the same
// time: while kernel n streams its weights and finishes, kernel n + 1 is already resident, has its first weight tiles
// in flight, and waits for kernel n's hand-over counter (PipeSync) before it reads kernel n's output.  Kernel n + 2
// follows kernel n on the same stream, so at most two kernels are in flight; two workgroups of any of them fit one
// compute unit (pipe_ok) and none launches more workgroups than there are compute units, so all workgroups of both
// are resident whatever the order of dispatch and no wait can starve the kernel it waits for.  The attention is the
// single-row kernel with at most 8 key splits, merged by the O projection while it stages its input.
// Visibility without fences (a device-scope release / acquire pair per workgroup writes back and invalidates a whole
// L2 and costs about 10 us once 256 workgroups do it): producers store their results write-through and signal after
// the stores have completed; a consumer reads them with ordinary loads, which cannot hit a stale line, because its
// die's L2 was invalidated when the consumer was dispatched, after every earlier reader of those buffers had ended,
// and nothing reads them again before the producer writes: no vector is updated in place (the residual stream
// alternates between b.x and b.x2), and before its hand-over a kernel reads nothing but weights.
// Measured on the 8B shape (time stamps of asynclm_profile_trace): a hand-over takes about 1 us, but the step is
// slower than the one-stream step (3.7 against 3.4 ms per token): what follows a hand-over - the input vector's round
// trip to memory, the last tiles, the write-through of the results, the counter, the hand-over words - is a chain of
// five to six memory round trips per kernel during which little is streamed, where a kernel of the one-stream step
// overlaps the same chain with its own first 32 MB of weights.  Kept as an option ("pipeline"), off by default.
hipError_t forward_single_pipelined(asynclm_ctx* c, int seq, bool with_head, SplitPlan sp) {
    const int dt = c->cfg.dtype;
    const Geom& g = c->g;
    hipStream_t sa = c->stream, sb = c->stream2;
    hipError_t e;
    if ((e = launch_embed(dt, c->embed, c->b, g, sa))) return e;
    if ((e = hipEventRecord(c->ev_fork, sa))) return e;
    if ((e = hipStreamWaitEvent(sb, c->ev_fork, 0))) return e;
    int idx = 0;
    hipStream_t s = sa;
    PipeSync ps{};
    // kernel k: arrival counter k, signals region k % PIPE_REGIONS, waits on region (k - 1) % PIPE_REGIONS
    auto next = [&]() {
        const size_t region = (size_t)PIPE_MAX_WORKGROUPS * PIPE_LINE_WORDS;
        ps.go_wait = idx > 0 ? c->pipe_go + (size_t)((idx - 1) % PIPE_REGIONS) * region : nullptr;
        ps.go_signal = c->pipe_go + (size_t)(idx % PIPE_REGIONS) * region;
        ps.counter = c->pipe_counters + (size_t)idx * PIPE_LINE_WORDS;
        ps.abort = c->b.pipe_abort;
        ps.error_word = c->b.token_log + 1;
        ps.step = c->b.step;
        ps.wait_kernel = (unsigned)(idx > 0 ? idx - 1 : 0); ps.my_kernel = (unsigned)idx;
        ps.stamps = c->pipe_stamps ? c->pipe_stamps + (size_t)idx * 6 : nullptr;
        s = (idx & 1) ? sb : sa;
        ++idx;
    };
    for (int l = 0; l < c->cfg.n_layers; ++l) {
        void* kvl = kv_layer_ptr(c, l);
        next(); if ((e = launch_qkv(dt, c->wqkv[l], c->attn_norm[l], kvl, c->b, g, s, &ps))) return e;
        next(); if ((e = launch_attn_decode(dt, kvl, sp.nsplit, true, c->b, g, s, &ps))) return e;
        next(); if ((e = launch_oproj(dt, c->wo[l], sp.nsplit, c->b, g, s, &ps, c->b.x2))) return e;
        next(); if ((e = launch_gateup(dt, c->wgate_up[l], c->ffn_norm[l], c->b, g, s, &ps, c->b.x2))) return e;
        next(); if ((e = launch_down(dt, c->wdown[l], c->b, g, s, &ps, c->b.x2))) return e;
    }
    if (with_head) {
        next(); if ((e = launch_lmhead(dt, c->lm_head, c->final_norm, c->logits, c->b, g, s, &ps))) return e;
    }
    if ((e = hipEventRecord(c->ev_join, sb))) return e;
    if ((e = hipStreamWaitEvent(sa, c->ev_join, 0))) return e;
    if (with_head && (e = launch_argmax(c->logits, c->b, g, sa))) return e;
    return hipSuccess;
}

bool use_pipeline(const asynclm_ctx* c, int len_after) {
    // (contexts beyond what 8 key splits of the single-row attention cover take the one-stream step)
    return c->opt_pipeline && c->pipe_ok && !c->prof && c->opt_attn_split == 0 && len_after <= 2048 &&
           5 * c->cfg.n_layers + 1 <= c->pipe_kernels_max && decode_gemv_grid() <= c->n_cu && decode_gemv_grid() <= PIPE_MAX_WORKGROUPS &&
           c->g.Hkv * 8 <= PIPE_MAX_WORKGROUPS;      // at most 8 key splits reach this step
}

// Captured steps.  The kernels read token, position and sequence from the step descriptor, so a graph depends only on
// the launch geometry: the attention plan, whether the pass ends with the output head, one or two streams.
int graph_key(SplitPlan sp, bool with_head, bool pipelined) {
    return (((((sp.nsplit << 1 | (sp.merge_in_oproj ? 1 : 0)) << 1 | (sp.mfma ? 1 : 0)) << 1 | (with_head ? 1 : 0)) << 1) | (pipelined ? 1 : 0)) << 1 | (sp.small ? 1 : 0);
}

hipError_t capture_step(asynclm_ctx* c, SplitPlan sp, bool with_head, bool pipelined, hipGraphExec_t* out) {
    hipError_t e;
    hipGraph_t graph = nullptr;
    if ((e = hipStreamBeginCapture(c->stream, hipStreamCaptureModeRelaxed))) return e;
    if (pipelined) e = forward_single_pipelined(c, 0, with_head, sp);
    else if (sp.small) e = forward_single_small(c, with_head);
    else {
        // stamp mode: the captured kernels carry their stamp words (the graphs are rebuilt when the option changes)
        c->stamp_now = c->opt_step_stamps && sp.mfma;
        if (c->stamp_now) c->pipe_kernels = 6 * c->cfg.n_layers + (with_head ? 1 : 0);
        e = forward_single(c, 0, with_head, sp);
        c->stamp_now = false;
    }
    hipError_t e2 = hipStreamEndCapture(c->stream, &graph);
    if (e) { if (graph) hipGraphDestroy(graph); return e; }
    if (e2) return e2;
    e = hipGraphInstantiate(out, graph, nullptr, nullptr, 0);
    hipGraphDestroy(graph);
    return e;
}

// Instantiates every graph that a decoding step can need under the current options (all attention plans that occur
// up to max_positions), so that no decoding step captures, instantiates or allocates.  Called by asynclm_create and by
// the options that change the launch geometry.
hipError_t rebuild_graphs(asynclm_ctx* c) {
    for (auto& kv : c->graphs) hipGraphExecDestroy(kv.second);
    c->graphs.clear();
    if (!c->opt_graph || !c->stream || c->opt_fused) return hipSuccess;
    const bool was_prof = c->prof;
    c->prof = false;
    hipError_t e = hipSuccess;
    for (int len_after = 1; len_after <= c->cfg.max_positions && !e; ++len_after) {
        const bool pipelined = use_pipeline(c, len_after);
        const SplitPlan sp = pick_step_plan(c, len_after, pipelined);
        for (int with_head = 0; with_head < 2 && !e; ++with_head) {
            const int key = graph_key(sp, with_head != 0, pipelined);
            if (c->graphs.count(key)) continue;
            hipGraphExec_t exec = nullptr;
            if (small_direct(c, sp)) continue;
            if ((e = capture_step(c, sp, with_head != 0, pipelined, &exec)) == hipSuccess) c->graphs.emplace(key, exec);
        }
    }
    c->prof = was_prof;
    return e;
}

// The greedy token of a sequence is computed when a forward pass ends; if the ban list changed since, it is
// recomputed from the (unchanged) logits before it is used.
hipError_t refresh_choice(asynclm_ctx* c, int seq) {
    if (!c->choice_stale[seq]) return hipSuccess;
    c->choice_stale[seq] = 0;
    return launch_argmax(c->logits, c->b, c->g, c->stream, seq);
}

// Is a decoding step expected to take less than SHORT_STEP_US (six launches a layer and the weights at the memory rate)?  An event behind
// its first kernel is a marker packet of its own, 3 us between two launches of such a step (tiny preset 41.0 -> 38.1 us as a graph without
// it); nothing at the 8B shape, where the queue is never empty.
constexpr int SHORT_STEP_US = 200, TOKEN_SPIN_US = 300;
bool short_step(const asynclm_ctx* c) {
    const Geom& g = c->g;
    const double layer = ((2.0 * g.Hq + 2.0 * g.Hkv) * g.dh + 3.0 * g.F) * g.d;
    return 20.0 * c->cfg.n_layers + (layer * c->cfg.n_layers + (double)g.V * g.d) * elem_bytes(c) / 6.6e6 < SHORT_STEP_US;
}

// Waits for the word that the first kernel of the running step writes.  Long steps have an event behind that kernel, whose wait is the
// runtime's own (with its scheduling flags).  In short steps the host looks at the word, for TOKEN_SPIN_US at most: with more in front of the step,
// a prompt for instance, it waits for an event behind all of it, which is a short step late.  `seen` false: the stream has run dry or
// failed without the word (take the token the long way).
hipError_t wait_token(asynclm_ctx* c, int32_t* token, bool* seen) {
    const unsigned long long* word = reinterpret_cast<const unsigned long long*>(c->token_host + 4);
    auto look = [&] {
        const unsigned long long v = __atomic_load_n(word, __ATOMIC_ACQUIRE);
        if ((uint32_t)(v >> 32) != c->tok_serial) return false;
        *token = (int32_t)(uint32_t)v;
        return *seen = true;
    };
    hipError_t e;
    if (!c->tok_marked) {
        const auto end = std::chrono::steady_clock::now() + std::chrono::microseconds(TOKEN_SPIN_US);
        do {
            for (int i = 0; i < 64; ++i) {
                if (look()) return hipSuccess;
                __builtin_ia32_pause();
            }
        } while (std::chrono::steady_clock::now() < end);
        if ((e = hipEventRecord(c->tok_event, c->stream))) return e;
    }
    if ((e = hipEventSynchronize(c->tok_event))) return e;
    look();
    return hipSuccess;
}

hipError_t step_one_token(asynclm_ctx* c, int seq, int forced, bool with_head) {
    hipError_t e;
    c->tok_early = false;
    if (forced < 0 && (e = refresh_choice(c, seq))) return e;
    if (c->opt_fused && c->nban[seq] == 0) {      // the single-kernel step has no token mask
        FusedLaunch L{};
        L.layers_dev = c->layers_dev; L.n_layers = c->cfg.n_layers;
        L.embed = c->embed; L.final_norm = c->final_norm; L.lm_head = c->lm_head;
        L.seq = seq; L.forced = forced; L.with_head = with_head;
        {
            SplitPlan sp = pick_nsplit(c, c->len[seq] + 1);
            if (!sp.merge_in_oproj) sp.nsplit = c->fused.nsplit;          // long context: every workgroup takes a split
            if (sp.nsplit > c->fused.nsplit) sp.nsplit = c->fused.nsplit;
            L.nsplit = sp.nsplit; L.merge_in_stage = sp.merge_in_oproj;
        }
        L.logits = c->logits + (size_t)seq * c->g.V; L.bar = c->bar; L.trace = c->want_trace ? c->trace : nullptr;
        if ((e = launch_decode_fused(c->cfg.dtype, c->fused, L, c->b, c->g, c->stream))) return e;
        c->len[seq] += 1;
        return hipSuccess;
    }
    const bool pipelined = use_pipeline(c, c->len[seq] + 1);
    const SplitPlan sp = pick_step_plan(c, c->len[seq] + 1, pipelined);
    // the chosen token also goes to pinned host memory: asynclm_decode_step waits for that word only, so the host has the token while
    // the forward pass is still running
    const TokenWord tok{reinterpret_cast<unsigned long long*>(c->token_host + 4), ++c->tok_serial};
    if (sp.small) {
        if ((e = run(c, KC_QKV, [&] { return launch_small_first(c->cfg.dtype, c->embed, c->wqkv[0], c->attn_norm[0], kv_layer_ptr(c, 0), c->b, c->g, seq,
                                                                forced, tok, c->b.x, c->stream); }))) return e;
    } else if ((e = run(c, KC_BEGIN, [&] { return launch_begin_step(c->cfg.dtype, c->embed, c->b, c->g, seq, forced, tok, c->stream); }))) return e;
    c->tok_marked = !c->prof && !short_step(c);
    if (c->tok_marked && (e = hipEventRecord(c->tok_event, c->stream))) return e;
    c->tok_early = !c->prof;
    c->pipe_kernels = pipelined ? 5 * c->cfg.n_layers + (with_head ? 1 : 0) : 0;
    const bool stamp_mode = c->opt_step_stamps && !pipelined && sp.mfma && !c->prof;
    if (stamp_mode) c->pipe_kernels = 6 * c->cfg.n_layers + (with_head ? 1 : 0);
    c->last_step_stamp_mode = stamp_mode;
    auto g_it = (c->opt_graph && !c->prof) ? c->graphs.find(graph_key(sp, with_head, pipelined)) : c->graphs.end();
    if (g_it != c->graphs.end()) e = hipGraphLaunch(g_it->second, c->stream);
    else if (pipelined) e = forward_single_pipelined(c, seq, with_head, sp);
    else if (sp.small) e = forward_single_small(c, with_head);
    else {
        c->stamp_now = stamp_mode;
        e = forward_single(c, seq, with_head, sp);
        c->stamp_now = false;
    }
    if (e) return e;
    c->len[seq] += 1;
    return hipSuccess;
}

template <class T>
hipError_t dev_alloc(asynclm_ctx* c, T** p, size_t count) {
    void* v = nullptr;
    hipError_t e = hipMalloc(&v, count * sizeof(T) > 0 ? count * sizeof(T) : 16);
    if (e != hipSuccess) return e;
    c->allocs.push_back(v);
    *p = (T*)v;
    return hipSuccess;
}

// Buffers of forward_wide_rows, for the models that it takes.  An error leaves none of them and wide_rows = 0.
hipError_t alloc_wide_rows(asynclm_ctx* c) {
    const Geom& g = c->g;
    const size_t qd = (size_t)g.Hq * g.dh, nqkv = qd + 2 * (size_t)g.Hkv * g.dh;
    if (c->cfg.dtype != ASYNCLM_DTYPE_BF16 || g.d % 128 || g.F % 128 || qd % 128 || (2 * g.Hkv * g.dh) % 128 || g.d > 8192) return hipSuccess;
    ChunkBuffers& cb = c->cb;
    const size_t had = c->allocs.size(), M = std::min(WIDE_ROWS_MAX, g.max_pos), wide = std::max(nqkv, (size_t)g.d);
    // partial planes: one of the widest product that writes any for the longest pass, every split of it for 128 rows (a down product of
    // the 8B shape over 203 rows with room for one part only: 245 us, with four parts 75)
    cb.part_capacity = std::max(M, (size_t)128 * CHUNK_GEMM_MAX_SPLIT) * wide;
    const size_t plane_elems = 3 * M * ((size_t)g.d + qd + g.F);
    bf16_t* planes = nullptr;
    hipError_t e = chunk_init_wide();
    if (!e) e = dev_alloc(c, &cb.tab_mem, CHUNK_TAB_BYTES);
    if (!e) e = dev_alloc(c, &cb.x, M * g.d);
    if (!e) e = dev_alloc(c, &cb.part, cb.part_capacity);
    if (!e) e = dev_alloc(c, &planes, plane_elems);
    // rows beyond the current pass are multiplied into discarded columns only, but must stay finite
    if (!e) e = hipMemset(planes, 0, plane_elems * sizeof(bf16_t));
    if (e) {
        for (size_t i = had; i < c->allocs.size(); ++i) hipFree(c->allocs[i]);
        c->allocs.resize(had);
        cb = ChunkBuffers{};
        return e;
    }
    auto take = [&](size_t n) { bf16_t* q = planes; planes += n; return q; };
    for (bf16_t** q : {&cb.nrm_hi, &cb.nrm_lo, &cb.nrm_lo2}) *q = take(M * g.d);
    for (bf16_t** q : {&cb.att_hi, &cb.att_lo, &cb.att_lo2}) *q = take(M * qd);
    for (bf16_t** q : {&cb.act_hi, &cb.act_lo, &cb.act_lo2}) *q = take(M * g.F);
    c->pass.G = g.Hq / g.Hkv; c->pass.Hkv = g.Hkv;
    c->wide_rows = (int)M;
    return hipSuccess;
}

bool config_ok(const asynclm_config* k) {
    if (k->n_layers <= 0 || k->d_model <= 0 || k->n_q_heads <= 0 || k->n_kv_heads <= 0 || k->ffn <= 0 || k->vocab <= 0) return false;
    if (k->head_dim != 64 && k->head_dim != 128) return false;
    if (k->n_q_heads % k->n_kv_heads) return false;
    const int grp = k->n_q_heads / k->n_kv_heads;
    if (grp != 1 && grp != 2 && grp != 4 && grp != 8) return false;
    if (k->d_model % 8 || k->ffn % 8) return false;
    if (k->dtype != ASYNCLM_DTYPE_FP32 && k->dtype != ASYNCLM_DTYPE_BF16) return false;
    if (k->max_seqs < 1 || k->max_positions < 1) return false;
    if (k->kv_format != ASYNCLM_KV_AUTO &&
        !((k->kv_format == ASYNCLM_KV_BF16 || k->kv_format == ASYNCLM_KV_PAIR_ROWS) && k->dtype == ASYNCLM_DTYPE_BF16)) return false;
    if (!(k->rms_eps >= 0.f) || !(k->rope_theta > 0.f)) return false;
    return true;
}

int check_seq(const asynclm_ctx* c, int32_t seq) {
    if (!c) return ASYNCLM_E_INVAL;
    if (c->poisoned) return ASYNCLM_E_DEVICE;
    if (seq < 0 || seq >= c->cfg.max_seqs) return ASYNCLM_E_INVAL;
    return ASYNCLM_OK;
}

int check_tokens(const asynclm_ctx* c, const int32_t* t, int32_t n) {
    if (!t || n <= 0) return ASYNCLM_E_INVAL;
    for (int i = 0; i < n; ++i)
        if (t[i] < 0 || t[i] >= c->cfg.vocab) return ASYNCLM_E_INVAL;
    return ASYNCLM_OK;
}

// Plans of the four products of a layer.
struct ChunkPlans { GemmPlan qkv, o, gu, down; };

// A product with N output rows and K columns over MT row tiles.  Up to four row tiles: (N / 128) S workgroups, one per
// compute unit at a time: S = the split that comes closest to one workgroup per unit, with at least two 128-column blocks
// per workgroup.  More: workgroups of nt weight-row tiles x 256 rows run in rounds of one per compute unit; a k-block costs
// nt + 1 (the activations' share; 0.6 us each), a workgroup's start and end about 8, and a partial plane of 512 x 4096 floats,
// written and read back, about 7.5.  Measured in a pass, down product of the 8B shape: 2048 rows nt 8 in 2 parts 372 us,
// nt 4 unsplit 395; 1019 rows 210 (8, 4 parts) and 206 (4, 2 parts).  All within the capacity of the partial planes.  `swiglu`: pairs of gate and up rows, no split.
GemmPlan pick_gemm_plan(const asynclm_ctx* c, int N, int K, int MT, bool swiglu = false) {
    const int nblk = K / 128;
    const int smax = std::min(CHUNK_GEMM_MAX_SPLIT, std::max(1, nblk / 2));
    auto fits = [&](int s) { return s == 1 || (size_t)s * MT * 32 * N <= c->cb.part_capacity; };
    if (MT <= 4) {
        const int tiles = N / 128;
        int s = std::max(1, std::min((c->n_cu + tiles / 2) / tiles, smax));
        if (MT == 4) {          // bound by the matrix cores rather than the weight stream: whole rounds, few planes
            s = 1;
            double best = 0;
            const double plane = 0.9 * ((double)MT * 32 * N) / (512.0 * 4096.0);
            for (int k = 1; k <= smax; ++k) {
                const int rounds = (tiles * k + c->n_cu - 1) / c->n_cu;
                const double cost = rounds * ((double)nblk / k + 1.5) + plane * (k - 1);
                if (k == 1 || cost < best) { best = cost; s = k; }
            }
        }
        if (c->opt_chunk_split > 0) s = std::min(c->opt_chunk_split, std::max(1, nblk));
        if (swiglu) s = 1;
        while (!fits(s)) --s;
        return {s, 4};
    }
    const int my = (MT + 7) / 8;
    GemmPlan best{1, 4};
    double best_cost = 0;
    const double plane = 7.5 * ((double)MT * 32 * N) / (512.0 * 4096.0);
    int s0 = 1, s1 = swiglu ? 1 : smax;
    if (!swiglu && c->opt_chunk_split > 0) { s0 = s1 = std::min(c->opt_chunk_split, std::max(1, nblk)); while (!fits(s1)) --s1; s0 = s1; }
    bool any = false;
    for (int s = s0; s <= s1; ++s) {
        if (!fits(s)) break;
        for (int nt = 8; nt >= 4; --nt) {
            const int tiles = (N / 32 + nt - 1) / nt * my * s;
            const int rounds = (tiles + c->n_cu - 1) / c->n_cu;
            const double cost = rounds * ((double)((nblk + s - 1) / s) * (nt + 1.0) + 8.0) + (swiglu ? 0.0 : plane * s);
            if (!any || cost < best_cost) { any = true; best_cost = cost; best = {s, nt}; }
        }
    }
    return best;
}

ChunkPlans chunk_plans(const asynclm_ctx* c, int MT) {
    const Geom& g = c->g;
    // the gate/up product of a wide pass is never split (unless forced): split-K would lose its SwiGLU epilogue
    GemmPlan gu = pick_gemm_plan(c, 2 * g.F, g.d, MT, MT > 3 && c->opt_chunk_split == 0);
    if (MT > 4 && gu.s == 1) gu = pick_gemm_plan(c, 2 * g.F, g.d, MT, true);
    return {pick_gemm_plan(c, (g.Hq + 2 * g.Hkv) * g.dh, g.d, MT), pick_gemm_plan(c, g.d, g.Hq * g.dh, MT), gu,
            pick_gemm_plan(c, g.d, g.F, MT)};
}

// Key splits of the chunk attention: about two 32-key tiles per wave, a multiple of 4, no more than fill the
// device eight waves deep (a large pass has enough tasks: more splits only add partial results to write and
// merge), within the capacity of the partial-result buffers.
int pick_chunk_attn_split(const asynclm_ctx* c, int max_keys, int ntasks) {
    const int tiles = (max_keys + 31) / 32;
    int n = ((tiles + 1) / 2 + 3) / 4 * 4;
    n = std::max(4, std::min(n, CHUNK_ATTN_MAX_SPLIT));
    const long long groups = (long long)ntasks * c->g.Hkv;
    const int fill = (int)std::max(4LL, 8LL * c->n_cu / groups / 4 * 4);
    n = std::min(n, fill);
    while (n > 4 && groups * n > CHUNK_ATTN_MAX_UNITS) n -= 4;
    return n;
}

// Key splits of every task, and the workgroups of the shared-key attention (`wide`), into the table.
// One sequence: `nsplit` parts of every block of tasks; with one part, longest first, and where all workgroups are resident at once (two per compute unit), those
// of the second half go the other way round, so that a unit gets a long and a short one.  70B shape, two layers, prompt of 4096 tokens 12.59 ->
// 12.37 ms; 8B shape, two layers, 700 / 1500 / 2048 tokens 1002 -> 993, 1593 -> 1587, 1998 -> 1973 us, 1019 (four layers) 2693 -> 2665, 16384 18.36 -> 18.08 ms, which
// is within what two runs differ by.  (Cutting the long blocks of a prompt as well: the same.)
// Several sequences: parts of at most `per` key tiles each, as few tiles as keep the workgroups to two per compute unit, because with
// one number of parts for all the longest sequence decides.  Four layers: 16 sequences of 512 to 4096 1181 -> 1137 us (attention 80 -> 74 a
// layer), 12 of up to 3400 1049 -> 1015, 8 of 128 to 4096 1224 -> 1202; four per compute unit 1154, 1035, 1276.
void plan_attention(const asynclm_ctx* c, ChunkTable& t, bool wide, int nsplit) {
    const int Hkv = c->g.Hkv;
    t.npieces = 0;
    if (!wide) {
        for (int i = 0; i < t.ntasks; ++i) { t.task[i].nsplit = nsplit; t.task[i].unit0 = i * nsplit; }
        return;
    }
    const int slots = 2 * c->n_cu;
    int tiles[CHUNK_MAX_GROUPS], longest = 1;           // of the keys that matter to a block, as the kernel counts them
    for (int b = 0; b < t.nblocks; ++b) {
        const ChunkTaskBlock& B = t.block[b];
        const ChunkTask& T = t.task[B.task0];
        tiles[b] = (T.pos0 + std::min((32 * T.tile) % T.n + 32 * B.n, T.n) + 31) / 32;
        longest = std::max(longest, tiles[b]);
    }
    auto parts = [&](int b, int per) { return (tiles[b] + per - 1) / per; };
    int per = 0;
    if (t.ngroups > 1) {                                // the fewest tiles that fit: what fits with some fits with more (120 sequences of 16k: 198 us of the host one by one)
        auto fits = [&](int p) {
            long long n = 0, units = 0;
            int most = 0;
            for (int b = 0; b < t.nblocks; ++b) { const int k = parts(b, p); n += k; units += (long long)k * t.block[b].n; most = std::max(most, k); }
            return n * Hkv <= slots && units * Hkv <= CHUNK_ATTN_MAX_UNITS && most <= CHUNK_ATTN_MAX_SPLIT;
        };
        per = 2;
        for (int hi = longest; per < hi;) { const int mid = (per + hi) / 2; if (fits(mid)) hi = mid; else per = mid + 1; }
    }
    int unit = 0;
    for (int b = 0; b < t.nblocks; ++b) {
        const int k = per ? parts(b, per) : nsplit;
        for (int i = 0; i < t.block[b].n; ++i) { ChunkTask& T = t.task[t.block[b].task0 + i]; T.nsplit = k; T.unit0 = unit; unit += k; }
    }
    for (int b = 0, e = 0; b < t.nblocks; b = e) {      // the blocks of one sequence that read the same keys next to each other: one XCD, its L2
        int most = 0;
        auto splits = [&](int i) { return t.task[t.block[i].task0].nsplit; };
        for (e = b; e < t.nblocks && t.task[t.block[e].task0].row0 == t.task[t.block[b].task0].row0; ++e) most = std::max(most, splits(e));
        for (int s = 0; s < most; ++s)
            for (int i = b; i < e; ++i)
                if (s < splits(i)) t.piece[t.npieces++] = ChunkPiece{(int16_t)i, (int16_t)s};
    }
    if (t.ngroups == 1 && nsplit == 1) {
        std::stable_sort(t.piece, t.piece + t.npieces, [&](const ChunkPiece& x, const ChunkPiece& y) { return tiles[x.block] > tiles[y.block]; });
        const int first = c->n_cu / Hkv;                // pieces that give every compute unit its first workgroup
        if (t.npieces > first && t.npieces * Hkv <= slots) std::reverse(t.piece + first, t.piece + t.npieces);
    }
}

// Layer `l` and the output head for one row of a pass, x its residual stream, whose position and sequence are in the step
// descriptor: the kernels of a decoding step.
hipError_t last_row_layer(asynclm_ctx* c, int l, float* x, int len_after) {
    const int dt = c->cfg.dtype;
    const Geom& g = c->g;
    hipStream_t s = c->stream;
    const SplitPlan sp = pick_nsplit(c, len_after);
    void* kvl = kv_layer_ptr(c, l);
    DecodeBuffers b = c->b;
    b.x = x;
    hipError_t e;
    if ((e = run(c, KC_QKV, [&] { return launch_qkv(dt, c->wqkv[l], c->attn_norm[l], kvl, b, g, s); }))) return e;
    if (sp.mfma) { if ((e = run(c, KC_ATTN, [&] { return launch_decode_attn_mfma(c->cb, kvl, sp.nsplit, b, g, s); }))) return e; }
    else if ((e = run(c, KC_ATTN, [&] { return launch_attn_decode(dt, kvl, sp.nsplit, sp.merge_in_oproj, b, g, s); }))) return e;
    if ((e = run(c, KC_OPROJ, [&] { return launch_oproj(dt, c->wo[l], sp.merge_in_oproj ? sp.nsplit : 0, b, g, s); }))) return e;
    if ((e = run(c, KC_GATEUP, [&] { return launch_gateup(dt, c->wgate_up[l], c->ffn_norm[l], b, g, s); }))) return e;
    if ((e = run(c, KC_DOWN, [&] { return launch_down(dt, c->wdown[l], b, g, s); }))) return e;
    return run(c, KC_LMHEAD, [&] { return launch_lmhead(dt, c->lm_head, c->final_norm, c->logits, b, g, s); });
}

// The used part of a pass's row table, through pinned memory: the copy is asynchronous and the host goes on enqueuing the pass.
hipError_t upload_table(asynclm_ctx* c, const ChunkTable& t) {
    ChunkBuffers& cb = c->cb;
    hipError_t e;
    const int i = c->tab_next;
    if ((e = hipEventSynchronize(c->tab_ev[i]))) return e;         // the upload that last used this copy has finished
    size_t bytes = 0;
    auto put = [&](const void* src, size_t n) {
        const size_t at = bytes;
        std::memcpy(c->tab_host[i] + at, src, n);
        bytes += (n + 31) / 32 * 32;
        return cb.tab_mem + at;
    };
    cb.tab.group = (const ChunkGroup*)put(t.group, sizeof(ChunkGroup) * t.ngroups);
    cb.tab.task = (const ChunkTask*)put(t.task, sizeof(ChunkTask) * t.ntasks);
    cb.tab.block = (const ChunkTaskBlock*)put(t.block, sizeof(ChunkTaskBlock) * t.nblocks);
    cb.tab.piece = (const ChunkPiece*)put(t.piece, sizeof(ChunkPiece) * t.npieces);
    cb.tab.row = (const ChunkRow*)put(t.row, sizeof(ChunkRow) * t.rows);
    if ((e = hipMemcpyAsync(cb.tab_mem, c->tab_host[i], bytes, hipMemcpyHostToDevice, c->stream))) return e;
    if ((e = hipEventRecord(c->tab_ev[i], c->stream))) return e;
    c->tab_next = i ^ 1;
    return hipSuccess;
}

// One forward pass over the rows of `pb` (1..pass_rows rows in any number of groups).  Groups that want logits
// get them from the single-row head kernels (one group) or from one more product on the matrix cores (several).
hipError_t forward_chunk(asynclm_ctx* c, PassBuilder& pb) {
    const Geom& g = c->g;
    ChunkBuffers& cb = c->cb;
    hipStream_t s = c->stream;
    ChunkTable& t = pb.t;
    const int rows = t.rows, MT = (rows + 31) / 32;
    const ChunkPlans sp = chunk_plans(c, MT);
    const int nqkv = (g.Hq + 2 * g.Hkv) * g.dh, qd = g.Hq * g.dh;
    const int asplit = pick_chunk_attn_split(c, pb.max_keys, t.ntasks);
    // Four waves on one tile of keys (k_chunk_attn_wide) or a wave of its own for every task and split (k_chunk_attn): the
    // first loads a tile once for up to four tasks and issues its loads from four waves, the second starts sooner and runs
    // more waves of small work.  8B shape, 4 layers, whole call, shared-key / other kernel, us: 24 rows (3 tasks) into 500 keys 627 / 621, 1.1k 632 / 627,
    // 2.1k 653 / 643, 4.2k 668 / 685, 16.4k 733 / 773; 48 rows (6 tasks) into 500 697 / 695, 1.1k 697 / 700, 2.1k 713 / 728, 16.4k 827 / 873.
    // Key splits of the first, one sequence: two workgroups per compute unit, at least two tiles each (one tile each: 1 % slower at 1.1k;
    // four workgroups per compute unit: 4 % slower at 16.4k, more partial results).  One split, which needs no merge, where
    // the blocks alone fill the units and the keys are few: 1019 tokens (4 layers) 2792 -> 2771 us, 2000 (2 layers) 1968 -> 1956,
    // 1300 tokens and 1024 rows after 1000 no difference; beyond, the second workgroup is worth more (1024 rows after
    // 4000 tokens 1588 against 1646 us, after 15000 2200 against 2331).  Several sequences are cut by plan_attention, each by its own length;
    // of them wsplit only says how long the longest one's chain of tiles would be with one count for all (`even`).
    const long long wgs = (long long)t.nblocks * g.Hkv, slots = 2LL * c->n_cu;
    int wsplit = (int)std::max(1LL, std::min<long long>((slots + (t.ngroups > 1 && t.ntasks < 2 * t.nblocks ? 0 : wgs - 1)) / wgs, ((pb.max_keys + 31) / 32 + 1) / 2));
    if (wgs >= c->n_cu && pb.max_keys <= 2048) wsplit = 1;
    wsplit = std::min(wsplit, CHUNK_ATTN_MAX_SPLIT);
    while (wsplit > 1 && (long long)t.ntasks * g.Hkv * wsplit > CHUNK_ATTN_MAX_UNITS) --wsplit;
    // k_chunk_attn has one split count for all sequences of a pass, and four times as many waves that each walk a chain of their own.
    // `even` dates from when the shared-key kernel had one count for all too, so that a sequence much longer than the others was a chain of
    // tiles that a quarter as many waves walked: at most 20 tiles over the average load of a workgroup slot.  plan_attention
    // cuts every sequence by its own length, which removes that reason: with the present cut the shared-key kernel is the faster one
    // or as fast wherever batches were compared, also where `even` sends one to the other kernel, and below 3072 keys, where the rule
    // sends most there.  8B shape, 4 layers, shared-key / other kernel, us: 16 sequences of 512 to 4096 with an interrupt of 24 1034 / 1118; 8 of 128 to 4096 787 / 842; 12 of 128
    // to 3400 with an interrupt 889 / 944; 16 of 500 to 900 774 / 810; 16 of 2000 to 2500 899 / 956, with an interrupt 994 / 1059; 4 of 1000 to 1500 695 / 692; 2 of 300 to
    // 500 655 / 648.  Before single blocks' keys were streamed: one sequence of 16k
    // and n of 500 tokens, n = 2 825 / 864, 4 841 / 880, 5 848 / 908, 7 860 / 955, 11 889 / 1039, 15 917 / 1089, 31 980 / 1390; one of 4k and 5, 7, 11, 15 768 / 807,
    // 778 / 844, 804 / 857, 827 / 880; 16 of 2900 1013 / 1036.
    const int chain = ((pb.max_keys + 31) / 32 + wsplit - 1) / wsplit;
    const bool even = t.ngroups == 1 || t.ntasks <= 4 || chain <= pb.block_tiles * g.Hkv / slots + 20;
    const bool wide_attn = ((pb.max_keys >= 3072 || t.ntasks >= 4 * t.ngroups) && even) || (t.ntasks >= 16 && t.ntasks >= 3 * t.nblocks);
    const int dt = c->cfg.dtype;
    hipError_t e;
    plan_attention(c, t, wide_attn, wide_attn ? wsplit : asplit);
    if ((e = upload_table(c, t))) return e;
    // A pass over one sequence: after the last layer's keys and values nothing but its last row is needed any more, so that
    // row finishes the pass through the single-row kernels (fp32 activations; its own key and value are formed once more
    // there), and a pass that wants no logits ends with the keys and values.  One layer of n: 3 % of a prompt's time at 32
    // layers.  Several sequences (a batched step: few rows) stay together to the end.
    const bool tail = t.ngroups == 1;
    const GemmPlan kv_plan = pick_gemm_plan(c, 2 * g.Hkv * g.dh, g.d, MT);
    for (int l = 0; l < c->cfg.n_layers; ++l) {
        void* kvl = kv_layer_ptr(c, l);
        if (l == 0) { if ((e = run(c, KC_CHUNK_PREP, [&] { return launch_chunk_embed_norm(c->embed, cb, c->attn_norm[0], rows, c->b, g, s); }))) return e; }
        else if ((e = run(c, KC_CHUNK_PREP, [&] { return launch_chunk_resid_norm(cb, sp.down.s, MT, c->attn_norm[l], rows, g, s); }))) return e;
        if (tail && l == c->cfg.n_layers - 1) {
            const char* wkv = (const char*)c->wqkv[l] + (size_t)qd * g.d * elem_bytes(c);
            if ((e = run(c, KC_CHUNK_GEMM, [&] { return launch_chunk_gemm(wkv, 2 * g.Hkv * g.dh, g.d, cb.nrm_hi, cb.nrm_lo, cb, kv_plan, rows, s); }))) return e;
            if ((e = run(c, KC_CHUNK_PREP, [&] { return launch_chunk_rope_kv(cb, kv_plan.s, kvl, c->b, rows, MT, g, s, true); }))) return e;
            if (t.nhead > 0 && (e = last_row_layer(c, l, cb.x + (size_t)(rows - 1) * g.d, pb.max_keys))) return e;
            break;
        }
        if ((e = run(c, KC_CHUNK_GEMM, [&] { return launch_chunk_gemm(c->wqkv[l], nqkv, g.d, cb.nrm_hi, cb.nrm_lo, cb, sp.qkv, rows, s); }))) return e;
        if ((e = run(c, KC_CHUNK_PREP, [&] { return launch_chunk_rope_kv(cb, sp.qkv.s, kvl, c->b, rows, MT, g, s); }))) return e;
        if (wide_attn) { if ((e = run(c, KC_CHUNK_ATTN, [&] { return launch_chunk_attn_wide(cb, kvl, t.npieces > t.nblocks, t.ntasks, t.npieces, g, s); }))) return e; }
        else if ((e = run(c, KC_CHUNK_ATTN, [&] { return launch_chunk_attn(cb, kvl, asplit, t.ntasks, g, s); }))) return e;
        if ((e = run(c, KC_CHUNK_GEMM, [&] { return launch_chunk_gemm(c->wo[l], g.d, qd, cb.att_hi, cb.att_lo, cb, sp.o, rows, s); }))) return e;
        if ((e = run(c, KC_CHUNK_PREP, [&] { return launch_chunk_resid_norm(cb, sp.o.s, MT, c->ffn_norm[l], rows, g, s); }))) return e;
        if (sp.gu.s == 1) {                 // no split-K: the SwiGLU is the product's epilogue
            if ((e = run(c, KC_CHUNK_GEMM, [&] { return launch_chunk_gemm_swiglu(c->wgate_up[l], g.F, g.d, cb.nrm_hi, cb.nrm_lo, cb, sp.gu, rows, s); }))) return e;
        } else {
            if ((e = run(c, KC_CHUNK_GEMM, [&] { return launch_chunk_gemm(c->wgate_up[l], 2 * g.F, g.d, cb.nrm_hi, cb.nrm_lo, cb, sp.gu, rows, s); }))) return e;
            if ((e = run(c, KC_CHUNK_PREP, [&] { return launch_chunk_swiglu(cb, sp.gu.s, MT, rows, g, s); }))) return e;
        }
        if ((e = run(c, KC_CHUNK_GEMM, [&] { return launch_chunk_gemm(c->wdown[l], g.d, g.F, cb.act_hi, cb.act_lo, cb, sp.down, rows, s); }))) return e;
    }
    const bool head_on_mfma = t.nhead > 1 && g.V % 128 == 0 && (size_t)((t.nhead + 31) / 32) * 32 * g.V <= cb.part_capacity;
    if (head_on_mfma) {
        if ((e = run(c, KC_CHUNK_MISC, [&] { return launch_chunk_head_rows(cb, sp.down.s, MT, c->final_norm, t.ngroups, g, s); }))) return e;
        if ((e = run(c, KC_LMHEAD, [&] { return launch_chunk_gemm(c->lm_head, g.V, g.d, cb.nrm_hi, cb.nrm_lo, cb, GemmPlan{1, 4}, t.nhead, s); }))) return e;
        if ((e = run(c, KC_ARGMAX, [&] { return launch_chunk_logits(cb, c->logits, c->b, t.ngroups, g, s); }))) return e;
    } else if (!tail) {
        for (int gi = 0; gi < t.ngroups; ++gi) {
            if (t.group[gi].head < 0) continue;
            const int seq = t.group[gi].seq;
            if ((e = run(c, KC_CHUNK_MISC, [&] { return launch_chunk_last_row(cb, sp.down.s, MT, gi, c->b, g, s); }))) return e;
            if ((e = run(c, KC_LMHEAD, [&] { return launch_lmhead(dt, c->lm_head, c->final_norm, c->logits, c->b, g, s); }))) return e;
        }
    }
    for (int gi = 0; gi < t.ngroups; ++gi) c->len[t.group[gi].seq] = t.group[gi].pos0 + t.group[gi].n;
    return hipSuccess;
}

// Split of K of a product of forward_wide_rows: parts so that the workgroups (one per 128 weight rows, part and four row tiles) come
// closest to whole rounds of one per compute unit; a 128-column block is one unit of time, a workgroup's start and end 1.5, a partial
// plane 0.9 per 512 x 4096 floats written and read back (as in pick_gemm_plan for four row tiles).
int pick_wide_split(const asynclm_ctx* c, int N, int K, int MT) {
    const int nblk = K / 128, tiles = N / 128 * ((MT + 3) / 4);
    const double plane = 0.9 * ((double)MT * 32 * N) / (512.0 * 4096.0);
    int best = 1;
    double best_cost = 0;
    for (int s = 1; s <= std::min(CHUNK_GEMM_MAX_SPLIT, std::max(1, nblk / 2)) && (size_t)s * MT * 32 * N <= c->cb.part_capacity; ++s) {
        const double cost = (tiles * s + c->n_cu - 1) / c->n_cu * ((double)nblk / s + 1.5) + plane * (s - 1);
        if (s == 1 || cost < best_cost) { best_cost = cost; best = s; }
    }
    return best;
}

// Key splits of the attention of n rows, merged by the last workgroup of a (row, kv head): a power of two, as many as the partial
// results hold.  A workgroup takes 256 keys per pass of its inner loop, about 15 us; a merge makes every workgroup publish its part with a
// device-wide fence, which costs 0.07 us per workgroup of the whole launch (they queue up for it) and twice that, however many the
// splits, for each (row, kv head) beyond 192.  Hence the split with the least sum of both: with one split per 256 keys, as it was, the merge took most
// of the time (200 rows at any context 550 us a layer, all but 40 to 150 of it fences).  Whole call, two layers of the 8B shape,
// single-plane cache, us with 1 / 2 / 4 / 8 / 16 splits: context 300, 24 rows 463 / 479 / 496 / 558 / 675, 256 rows 756 / 1361;
// context 1000, 8 rows 493 / 474 / 459 / 466 / 512, 64 rows 603 / 678 / 768 / 946; context 4000, 2 rows 685 / 562 / 493 / 463 / 456,
// 16 rows 709 / 598 / 541 / 557 / 613, 64 rows 795 / 804 / 849 / 988; context 16000, 16 rows 1498 / 998 / 756 / 734 / 807, 128 rows
// 2226 / 2009 / 1991.  The 15 us are that shape's (four heads per kv head, head_dim 128).  Other shapes with the same constants, four layers of
// d 512, whole call: with one head per kv head and head_dim 64 a pass over 256 keys takes 3.5 us, and the rule cuts too far (24 rows at 2000, eight kv heads, 407
// us with two splits, 256 with one; 32 kv heads, 8 rows at 4000 771 / 436); with eight heads on one kv head not far enough (24 rows at 2000 325 with two, 260 with
// eight).  One split per 256 keys is slower than the rule on all but the last (these: 608, 2625 and 260).
int pick_rows_split(const asynclm_ctx* c, int keys, int n) {
    const int most = std::min(ATTN_MAX_SPLIT, std::max(1, ROWS_MAX * ATTN_MAX_SPLIT / n));
    if (c->opt_attn_split > 0) return std::min(c->opt_attn_split, most);
    const int passes = (keys + 255) / 256, units = n * c->g.Hkv;
    int best = 1;
    double best_cost = 15.0 * passes;
    for (int s = 2; s <= most && s / 2 < passes; s *= 2) {
        const double cost = 15.0 * ((passes + s - 1) / s) + 0.07 * s * units + 0.14 * std::max(0, units - 192);
        if (cost < best_cost) { best_cost = cost; best = s; }
    }
    return best;
}

// One forward pass over n = 2..wide_rows rows of one sequence: bf16 models that keep the cache row by row (the single-plane format,
// head_dim 64), sizes multiples of 128.  Their activations are fp32 and stay so: the products take them as three bf16 planes, which
// together are the fp32 value, on the matrix cores (three products per weight, fp32 sums), and everything between the products is
// fp32.  The attention is the one of the other rows path (k_attn_decode), one workgroup per (row, kv head, key split).
// 8B shape with the single-plane cache, two layers, rows appended at a context of 64 or more, whole call: 2 rows 427 us against 461 in
// passes of eight rows through the vector units, 8 rows 417 / 464, 24 rows 422 / 1067, 64 rows 493 / 2630, 200 rows 693 / 8358; a session
// (203 + 24 tokens appended, 16 steps) 14.7 -> 6.9 ms.  Short passes of smaller models stay with forward_rows (rows_are_faster).
// Error against 64 bits of that session, rms over 40 seeds: 1.35e-4 before, 1.34e-4 now.
hipError_t forward_wide_rows(asynclm_ctx* c, int seq, const int32_t* tokens, int n, bool with_head) {
    const int dt = c->cfg.dtype;
    const Geom& g = c->g;
    ChunkBuffers& cb = c->cb;
    hipStream_t s = c->stream;
    const RowsPass p{seq, c->len[seq], n};
    const int MT = (n + 31) / 32, nqkv = (g.Hq + 2 * g.Hkv) * g.dh, nkv = 2 * g.Hkv * g.dh, qd = g.Hq * g.dh;
    const int nsplit = pick_rows_split(c, p.pos0 + n, n);
    const int s_qkv = pick_wide_split(c, nqkv, g.d, MT), s_kv = pick_wide_split(c, nkv, g.d, MT), s_o = pick_wide_split(c, g.d, qd, MT),
              s_down = pick_wide_split(c, g.d, g.F, MT);
    PassBuilder& pb = c->pass;
    pb.clear();
    pb.add(seq, p.pos0, n, -2, tokens, with_head);
    hipError_t e;
    if ((e = upload_table(c, pb.t))) return e;
    for (int l = 0; l < c->cfg.n_layers; ++l) {
        void* kvl = kv_layer_ptr(c, l);
        if (l == 0) { if ((e = run(c, KC_CHUNK_PREP, [&] { return launch_chunk_embed_norm(c->embed, cb, c->attn_norm[0], n, c->b, g, s, 3); }))) return e; }
        else if ((e = run(c, KC_CHUNK_PREP, [&] { return launch_chunk_resid_norm(cb, s_down, MT, c->attn_norm[l], n, g, s, 3); }))) return e;
        if (l == c->cfg.n_layers - 1) {         // as in forward_chunk: keys and values of all rows, the rest for the last row only
            const char* wkv = (const char*)c->wqkv[l] + (size_t)qd * g.d * elem_bytes(c);
            if ((e = run(c, KC_CHUNK_GEMM, [&] { return launch_wide_gemm(wkv, nkv, g.d, cb.nrm_hi, cb.nrm_lo, cb.nrm_lo2, cb, s_kv, n, s); }))) return e;
            if ((e = run(c, KC_CHUNK_PREP, [&] { return launch_rows_rope_kv(cb, s_kv, MT, kvl, c->rb, c->b, p, g, s, true); }))) return e;
            if (with_head && (e = last_row_layer(c, l, cb.x + (size_t)(n - 1) * g.d, p.pos0 + n))) return e;
            break;
        }
        if ((e = run(c, KC_CHUNK_GEMM, [&] { return launch_wide_gemm(c->wqkv[l], nqkv, g.d, cb.nrm_hi, cb.nrm_lo, cb.nrm_lo2, cb, s_qkv, n, s); }))) return e;
        if ((e = run(c, KC_CHUNK_PREP, [&] { return launch_rows_rope_kv(cb, s_qkv, MT, kvl, c->rb, c->b, p, g, s, false); }))) return e;
        if ((e = run(c, KC_ATTN, [&] { return launch_rows_attn(dt, kvl, nsplit, c->rb, p, g, s, &cb); }))) return e;
        if ((e = run(c, KC_CHUNK_GEMM, [&] { return launch_wide_gemm(c->wo[l], g.d, qd, cb.att_hi, cb.att_lo, cb.att_lo2, cb, s_o, n, s); }))) return e;
        if ((e = run(c, KC_CHUNK_PREP, [&] { return launch_chunk_resid_norm(cb, s_o, MT, c->ffn_norm[l], n, g, s, 3); }))) return e;
        if ((e = run(c, KC_CHUNK_GEMM, [&] { return launch_wide_gemm_swiglu(c->wgate_up[l], g.F, g.d, cb.nrm_hi, cb.nrm_lo, cb.nrm_lo2, cb, n, s); }))) return e;
        if ((e = run(c, KC_CHUNK_GEMM, [&] { return launch_wide_gemm(c->wdown[l], g.d, g.F, cb.act_hi, cb.act_lo, cb.act_lo2, cb, s_down, n, s); }))) return e;
    }
    c->len[seq] += n;
    return hipSuccess;
}

// One forward pass over n = 2..rows_pass rows of one sequence (models outside the matrix-core paths).
hipError_t forward_rows(asynclm_ctx* c, int seq, const int32_t* tokens, int n, bool with_head) {
    const int dt = c->cfg.dtype;
    const Geom& g = c->g;
    hipStream_t s = c->stream;
    const RowsPass p{seq, c->len[seq], n};
    const int nsplit = pick_rows_split(c, p.pos0 + n, n);
    hipError_t e;
    for (int r0 = 0; r0 < n; r0 += ROWS_MAX) {
        RowsTokens tk{};
        const int m = std::min(ROWS_MAX, n - r0);
        for (int r = 0; r < m; ++r) tk.t[r] = tokens[r0 + r];
        if ((e = run(c, KC_EMBED, [&] { return launch_rows_embed(dt, c->embed, tk, r0, m, c->rb, c->b, p, g, s); }))) return e;
    }
    for (int l = 0; l < c->cfg.n_layers; ++l) {
        void* kvl = kv_layer_ptr(c, l);
        if ((e = run(c, KC_QKV, [&] { return launch_rows_qkv(dt, c->wqkv[l], c->attn_norm[l], kvl, c->rb, c->b, p, g, s); }))) return e;
        if ((e = run(c, KC_ATTN, [&] { return launch_rows_attn(dt, kvl, nsplit, c->rb, p, g, s); }))) return e;
        if ((e = run(c, KC_OPROJ, [&] { return launch_rows_oproj(dt, c->wo[l], c->rb, p, g, s); }))) return e;
        if ((e = run(c, KC_GATEUP, [&] { return launch_rows_gateup(dt, c->wgate_up[l], c->ffn_norm[l], c->rb, p, g, s); }))) return e;
        if ((e = run(c, KC_DOWN, [&] { return launch_rows_down(dt, c->wdown[l], c->rb, p, g, s); }))) return e;
    }
    if (with_head) {
        DecodeBuffers b = c->b;
        b.x = c->rb.x + (size_t)(n - 1) * g.d;
        if ((e = run(c, KC_LMHEAD, [&] { return launch_lmhead(dt, c->lm_head, c->final_norm, c->logits, b, g, s); }))) return e;
    }
    c->len[seq] += n;
    return hipSuccess;
}

// Of the models that both forward_wide_rows and forward_rows take: is forward_rows the faster one for a pass of n rows?  It has five
// launches a layer against eight (and a table to upload), but its time grows with the weights of every group of eight rows.  Whole call in
// us, wide / rows, after a context of 200 (d model, layers, Mi weights per layer): 2 and 8 rows: d 256, 2 layers (0.8) 110 / 78, 117 / 89; d 512,
// 8 layers (2.1) 440 / 248, 475 / 294; d 2048, 4 layers (11) 286 / 198, 304 / 219; d 1024, 6 layers (14.5) 385 / 318, 431 / 370; d 2048, 8 layers (48)
// 681 / 617, 749 / 715, but 2 layers 176 / 173, 188 / 198, because the wide pass ends with its last row; d 2048, 16 layers (58) 1340 / 1291, 1519 / 1511;
// the 8B shape, 2 layers (208) 292 / 333, 295 / 342.  Contexts up to 16000 move the crossing little (8 rows at 16000: d 1024, 4 layers (5.5) 435 / 376;
// d 2048, 8 layers (48) 1510 / 1478; d 1024, 2 layers (14.5) 215 / 233).  More rows, where all products are small: 16, 24 and 32 rows at d 256, 4 layers
// 267 / 211, 310 / 273, 291 / 256; d 512, 4 layers 259 / 190, 273 / 228, 298 / 262, but 2 layers 127 / 109, 133 / 128, 138 / 141; d 1024, 4 layers (5.5)
// 306 / 253, 356 / 350, 345 / 354; d 1920, 4 layers (8.9) 353 / 346, 399 / 487; 48 rows at d 512, 4 layers 388 / 365, d 1024, 4 layers 475 / 521.
bool rows_are_faster(const asynclm_ctx* c, int n) {
    const Geom& g = c->g;
    const long long Mi = 1 << 20, nl = c->cfg.n_layers, groups = (n + ROWS_MAX - 1) / ROWS_MAX;
    const long long weights = ((long long)(2 * g.Hq + 2 * g.Hkv) * g.dh + 3LL * g.F) * g.d;      // of a layer
    if (n <= ROWS_MAX) return weights <= std::min(48LL, 16 * nl) * Mi;
    return n <= 32 && n <= std::min(c->rows_pass, rows_per_pass(c->cfg.dtype, g)) && nl >= 4 && groups * weights <= 12 * Mi;
}

// Append n >= 1 tokens to a sequence and leave logits for the token after them.
int append_tokens(asynclm_ctx* c, int seq, const int32_t* tokens, int n) {
    // the one-kernel and the two-stream step are asked for by option: then every token takes such a step
    const bool rows_path = !c->chunk_ok && !c->opt_fused && !c->opt_pipeline && rows_supported(c->cfg.dtype, c->g);
    const bool wide_path = c->wide_rows > 0 && !c->opt_fused && !c->opt_pipeline;
    const int chunk = c->chunk_ok ? std::min(c->opt_chunk, c->pass_rows) : wide_path ? std::min(c->opt_chunk, c->wide_rows) :
                      rows_path ? std::min({c->opt_chunk, c->rows_pass, rows_per_pass(c->cfg.dtype, c->g)}) : 1;
    int i = 0;
    while (i < n) {
        const int rows = std::min(chunk, n - i);
        const bool last = i + rows == n;
        if (rows == 1) {
            HIPCK(c, step_one_token(c, seq, tokens[i], last));
        } else if (wide_path && !(rows_path && rows_are_faster(c, rows))) {
            HIPCK(c, forward_wide_rows(c, seq, tokens + i, rows, last));
        } else if (!c->chunk_ok) {
            HIPCK(c, forward_rows(c, seq, tokens + i, rows, last));
        } else {
            PassBuilder& pb = c->pass;
            pb.clear();
            pb.add(seq, c->len[seq], rows, -2, tokens + i, last);
            HIPCK(c, forward_chunk(c, pb));
        }
        i += rows;
    }
    return ASYNCLM_OK;
}

}  // namespace

static int create_ctx(asynclm_ctx** out, const asynclm_config* cfg, const asynclm_weights* w, void* hip_stream, int max_rows, int* pass_rows);

// The product of more than 128 rows moves the weights from memory straight to LDS, 16 bytes a lane, which is only known to work
// on addresses that are multiples of 16; the products of up to 128 rows load them to registers, from any address.
constexpr int PASS_ROWS_UNALIGNED = 128;
static bool weights_aligned(const asynclm_config* cfg, const asynclm_weights* w) {
    uintptr_t bits = 0;     // (the output head has at most 128 rows)
    for (int l = 0; l < cfg->n_layers; ++l) bits |= (uintptr_t)w->wqkv[l] | (uintptr_t)w->wo[l] | (uintptr_t)w->wgate_up[l] | (uintptr_t)w->wdown[l];
    return bits % 16 == 0;
}

extern "C" {

int asynclm_create(asynclm_ctx** out, const asynclm_config* cfg, const asynclm_weights* w, void* hip_stream) {
    if (out) *out = nullptr;
    if (!out || !cfg || !w) return ASYNCLM_E_INVAL;
    // where memory is too short for the buffers of large passes, the smallest ones (none, for models of forward_wide_rows) do; what does not fit may also be a graph or
    // another object of the runtime, which reports a device error
    int pass_rows = 0;
    const int r = create_ctx(out, cfg, w, hip_stream, CHUNK_MAX, &pass_rows);
    if (r == ASYNCLM_OK || pass_rows <= CHUNK_BATCH_ROWS) return r;
    (void)hipGetLastError();
    return create_ctx(out, cfg, w, hip_stream, CHUNK_BATCH_ROWS, &pass_rows);
}

}  // extern "C"

static int create_ctx(asynclm_ctx** out, const asynclm_config* cfg, const asynclm_weights* w, void* hip_stream, int max_rows, int* pass_rows) {
    if (!config_ok(cfg)) return ASYNCLM_E_INVAL;
    if (!w->embed || !w->final_norm || !w->lm_head || !w->attn_norm || !w->wqkv || !w->wo || !w->ffn_norm ||
        !w->wgate_up || !w->wdown)
        return ASYNCLM_E_INVAL;
    for (int l = 0; l < cfg->n_layers; ++l)
        if (!w->attn_norm[l] || !w->wqkv[l] || !w->wo[l] || !w->ffn_norm[l] || !w->wgate_up[l] || !w->wdown[l])
            return ASYNCLM_E_INVAL;

    asynclm_ctx* c = new (std::nothrow) asynclm_ctx();
    if (!c) return ASYNCLM_E_NOMEM;
    hipError_t e0;
    c->cfg = *cfg;
    c->stream = (hipStream_t)hip_stream;
    if (!c->stream) c->opt_graph = 0;   // the null stream cannot be captured
    if ((e0 = hipGetDevice(&c->device)) != hipSuccess) { report_hip("hipGetDevice", e0); delete c; return ASYNCLM_E_DEVICE; }
    if ((e0 = hipDeviceGetAttribute(&c->n_cu, hipDeviceAttributeMultiprocessorCount, c->device)) != hipSuccess || c->n_cu < 1) {
        report_hip("hipDeviceGetAttribute", e0); delete c; return ASYNCLM_E_DEVICE;
    }

    c->embed = w->embed; c->final_norm = w->final_norm; c->lm_head = w->lm_head;
    for (int l = 0; l < cfg->n_layers; ++l) {
        c->attn_norm.push_back(w->attn_norm[l]); c->ffn_norm.push_back(w->ffn_norm[l]);
        c->wqkv.push_back(w->wqkv[l]); c->wo.push_back(w->wo[l]);
        c->wgate_up.push_back(w->wgate_up[l]); c->wdown.push_back(w->wdown[l]);
    }

    Geom& g = c->g;
    g.d = cfg->d_model; g.Hq = cfg->n_q_heads; g.Hkv = cfg->n_kv_heads; g.dh = cfg->head_dim;
    g.F = cfg->ffn; g.V = cfg->vocab; g.max_pos = (cfg->max_positions + 31) / 32 * 32; g.eps = cfg->rms_eps;
    g.scale = (float)(1.0 / std::sqrt((double)cfg->head_dim));
    {
        const bool pair = cfg->dtype == ASYNCLM_DTYPE_BF16 && cfg->kv_format != ASYNCLM_KV_BF16;
        // the matrix-core append path: bf16 weights, paired cache, head_dim 128, 128-aligned inner sizes
        c->chunk_ok = pair && g.dh == 128 && g.d % 128 == 0 && g.F % 128 == 0 && g.d <= 8192;
        const size_t plane = (size_t)g.max_pos * g.dh * g.Hkv;
        g.kv_head_stride = (size_t)g.max_pos * g.dh;
        // row-major values: every model but those of the append path, whose attention (decoding steps included) reads
        // the transposed planes only; PAIR_ROWS keeps both
        const bool v_rows = !c->chunk_ok || cfg->kv_format == ASYNCLM_KV_PAIR_ROWS;
        g.kv_lo_offset = pair ? plane : 0;
        g.kv_v_offset = v_rows ? (pair ? 2 * plane : plane) : 0;
        const size_t row_planes = (pair ? 2 : 1) * (v_rows ? 2 : 1);
        g.kv_vt_offset = c->chunk_ok ? row_planes * plane : 0;
        g.kv_layer_stride = (row_planes + (c->chunk_ok ? 2 : 0)) * plane;
        g.kv_seq_stride = g.kv_layer_stride * cfg->n_layers;
    }
    c->len.assign(cfg->max_seqs, 0);
    c->nban.assign(cfg->max_seqs, 0);
    c->choice_stale.assign(cfg->max_seqs, 0);

    auto bail = [&](int code) { asynclm_destroy(c); return code; };
    hipError_t e;
#define ALLOC(ptr, count) if ((e = dev_alloc(c, &(ptr), (count))) != hipSuccess) { report_hip("hipMalloc " #ptr, e); return bail(e == hipErrorOutOfMemory ? ASYNCLM_E_NOMEM : ASYNCLM_E_DEVICE); }
    {
        char* kvp = nullptr;
        ALLOC(kvp, g.kv_seq_stride * (size_t)cfg->max_seqs * elem_bytes(c));
        c->kv = kvp;
    }
    ALLOC(c->logits, (size_t)cfg->max_seqs * g.V);
    ALLOC(c->b.step, 1);
    ALLOC(c->b.seq_state, (size_t)cfg->max_seqs);
    ALLOC(c->b.token_log, 2);        // [0] chosen token, [1] set when a fused step gave up at a grid barrier
    ALLOC(c->b.x, (size_t)g.d);
    ALLOC(c->b.x2, (size_t)g.d);
    ALLOC(c->b.q, (size_t)g.Hq * g.dh);
    ALLOC(c->b.o, (size_t)g.Hq * g.dh);
    ALLOC(c->b.a, (size_t)g.F);
    ALLOC(c->b.part_acc, (size_t)g.Hq * ATTN_MAX_SPLIT * g.dh);
    ALLOC(c->b.part_ml, (size_t)g.Hq * ATTN_MAX_SPLIT * 2);
    ALLOC(c->b.attn_counters, (size_t)g.Hkv);
    ALLOC(c->b.amax_v, (size_t)ARGMAX_MAX_BLOCKS);
    ALLOC(c->b.amax_i, (size_t)ARGMAX_MAX_BLOCKS);
    ALLOC(c->b.amax_counter, 1);
    ALLOC(c->b.banned, (size_t)cfg->max_seqs * (1 + BAN_MAX));
    c->pipe_kernels_max = 6 * cfg->n_layers + 2;      // two-stream step: 5 per layer; stamp mode of the one-stream step: 6
    ALLOC(c->b.pipe_abort, (size_t)PIPE_LINE_WORDS);
    ALLOC(c->pipe_go, (size_t)PIPE_REGIONS * PIPE_MAX_WORKGROUPS * PIPE_LINE_WORDS);
    ALLOC(c->pipe_counters, (size_t)c->pipe_kernels_max * PIPE_LINE_WORDS);
    ALLOC(c->pipe_stamps, (size_t)c->pipe_kernels_max * 6);
    ALLOC(c->stamp_done, (size_t)c->pipe_kernels_max * STAMP_DONE_SLOTS);
    if (c->chunk_ok) {
        ChunkBuffers& cb = c->cb;
        // Rows per pass: longer prompts take passes of up to 2048 rows (fewer partial planes, whole rounds of workgroups: a
        // 16384-token prompt of the 8B shape, 2 layers, 51.2 ms in passes of 512 rows and 44.0 ms in passes of 2048, the product
        // of more than 128 rows changed with it), as long as the context can be that long and the partial results of the
        // attention fit.
        c->pass_rows = std::max(CHUNK_BATCH_ROWS, std::min({max_rows, g.max_pos, CHUNK_ATTN_MAX_UNITS * 32 / g.Hq / 32 * 32,
                                                            CHUNK_MAX_TASKS * 32 / (g.Hq / g.Hkv)}));
        if (!weights_aligned(cfg, w)) c->pass_rows = c->pass.batch_rows = PASS_ROWS_UNALIGNED;
        *pass_rows = c->pass_rows;
        const size_t M = c->pass_rows, MB = CHUNK_BATCH_ROWS, qd = (size_t)g.Hq * g.dh;
        // split-K partial planes: every split of the widest product for passes of up to 96 rows (bound by the weight
        // stream: many splits), two of it for 512 rows, one of the widest product other than gate/up for the longest pass
        // (more than 128 rows write gate/up through SwiGLU, unless split), the output head for one row per group; larger
        // splits as far as pick_gemm_plan finds room here
        const size_t wmax = std::max(std::max((size_t)2 * g.F, (size_t)(g.Hq + 2 * g.Hkv) * g.dh), (size_t)g.d);
        const size_t wunsplit = std::max((size_t)(g.Hq + 2 * g.Hkv) * g.dh, (size_t)g.d);       // the widest product without SwiGLU
        cb.part_capacity = std::max({(size_t)96 * CHUNK_GEMM_MAX_SPLIT * wmax, 2 * MB * wmax, M * wunsplit, (size_t)CHUNK_MAX_GROUPS * g.V});
        if ((e = chunk_init()) != hipSuccess) { report_hip("chunk_init", e); return bail(ASYNCLM_E_DEVICE); }
        cb.q_cols = (g.Hq / g.Hkv) * c->pass_rows + 32;
        const size_t qn = (size_t)g.Hkv * cb.q_cols * g.dh;
        c->pass.G = g.Hq / g.Hkv; c->pass.Hkv = g.Hkv;
        ALLOC(cb.tab_mem, CHUNK_TAB_BYTES);
        ALLOC(cb.x, M * g.d);
        ALLOC(cb.nrm_hi, M * g.d); ALLOC(cb.nrm_lo, M * g.d);
        ALLOC(cb.att_hi, M * qd); ALLOC(cb.att_lo, M * qd);
        ALLOC(cb.act_hi, M * g.F); ALLOC(cb.act_lo, M * g.F);
        ALLOC(cb.q_hi, qn); ALLOC(cb.q_lo, qn);
        ALLOC(cb.part, cb.part_capacity);
        ALLOC(cb.attn_o, (size_t)CHUNK_ATTN_MAX_UNITS * g.dh * 32);
        ALLOC(cb.attn_ml, (size_t)CHUNK_ATTN_MAX_UNITS * 64);
        ALLOC(cb.amax_v, (size_t)CHUNK_MAX_GROUPS * CHUNK_LOGIT_SLICES); ALLOC(cb.amax_i, (size_t)CHUNK_MAX_GROUPS * CHUNK_LOGIT_SLICES);
        ALLOC(cb.amax_counters, (size_t)CHUNK_MAX_GROUPS);
        if (hipMemset(cb.amax_counters, 0, sizeof(int32_t) * CHUNK_MAX_GROUPS) != hipSuccess) return bail(ASYNCLM_E_DEVICE);
        // rows beyond the current chunk are multiplied into discarded columns only, but must stay finite
        if (hipMemset(cb.x, 0, M * g.d * 4) || hipMemset(cb.nrm_hi, 0, M * g.d * 2) ||
            hipMemset(cb.nrm_lo, 0, M * g.d * 2) || hipMemset(cb.att_hi, 0, M * qd * 2) || hipMemset(cb.att_lo, 0, M * qd * 2) ||
            hipMemset(cb.act_hi, 0, M * g.F * 2) || hipMemset(cb.act_lo, 0, M * g.F * 2) || hipMemset(cb.q_hi, 0, qn * 2) ||
            hipMemset(cb.q_lo, 0, qn * 2))
            return bail(ASYNCLM_E_DEVICE);
    }
    if (!c->chunk_ok) {
        if ((e = rows_init(cfg->dtype)) != hipSuccess) { report_hip("rows_init", e); return bail(ASYNCLM_E_DEVICE); }
        c->rows_pass = rows_per_pass(cfg->dtype, g);
        const size_t R = c->rows_pass, qd = (size_t)g.Hq * g.dh;
        ALLOC(c->rb.x, R * g.d); ALLOC(c->rb.o, R * qd); ALLOC(c->rb.a, R * g.F);
        ALLOC(c->rb.part_acc, ROWS_MAX * qd * ATTN_MAX_SPLIT);
        ALLOC(c->rb.part_ml, (size_t)ROWS_MAX * g.Hq * ATTN_MAX_SPLIT * 2);
        // where memory is too short for the buffers of larger passes (or was, see asynclm_create), passes of ROWS_MAX rows do
        if (max_rows > CHUNK_BATCH_ROWS && (e = alloc_wide_rows(c)) != hipSuccess) { report_hip("buffers of wide passes", e); (void)hipGetLastError(); }
        if (c->wide_rows) *pass_rows = max_rows;
        const size_t RP = std::max<size_t>(R, c->wide_rows);
        ALLOC(c->rb.q, RP * qd);
        ALLOC(c->rb.counters, RP * g.Hkv);
        if (hipMemset(c->rb.counters, 0, sizeof(int32_t) * RP * g.Hkv) != hipSuccess) return bail(ASYNCLM_E_DEVICE);
    }
    if (!c->chunk_ok && small_step_supported(cfg->dtype, g)) ALLOC(c->small.parts, (size_t)(g.Hkv + small_mlp_parts(g)) * g.d);
    // cache rows that were never written are read (and masked) by the chunk attention: keep them finite
    if (hipMemset(c->kv, 0, g.kv_seq_stride * (size_t)cfg->max_seqs * elem_bytes(c)) != hipSuccess) return bail(ASYNCLM_E_DEVICE);
    float *rc = nullptr, *rs = nullptr;
    const size_t half = g.dh / 2, rope_n = (size_t)g.max_pos * half;
    ALLOC(rc, rope_n);
    ALLOC(rs, rope_n);
#undef ALLOC
    c->b.rope_cos = rc; c->b.rope_sin = rs;

    // rotary table: angle(pos, i) = pos * theta^(-2i/dh), formed in double, stored as fp32
    {
        std::vector<float> hc(rope_n), hs(rope_n);
        std::vector<double> inv(half);
        for (size_t i = 0; i < half; ++i) inv[i] = std::pow((double)cfg->rope_theta, -2.0 * (double)i / (double)g.dh);
        for (int p = 0; p < g.max_pos; ++p)
            for (size_t i = 0; i < half; ++i) {
                const double ang = (double)p * inv[i];
                hc[(size_t)p * half + i] = (float)std::cos(ang);
                hs[(size_t)p * half + i] = (float)std::sin(ang);
            }
        if (hipMemcpy(rc, hc.data(), rope_n * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
            hipMemcpy(rs, hs.data(), rope_n * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
            return bail(ASYNCLM_E_DEVICE);
    }
    if (hipMemset(c->b.seq_state, 0, sizeof(SeqState) * cfg->max_seqs) != hipSuccess ||
        hipMemset(c->b.attn_counters, 0, sizeof(int32_t) * g.Hkv) != hipSuccess ||
        hipMemset(c->b.amax_counter, 0, sizeof(int32_t)) != hipSuccess ||
        hipMemset(c->b.banned, 0, sizeof(int32_t) * cfg->max_seqs * (1 + BAN_MAX)) != hipSuccess ||
        hipMemset(c->b.step, 0, sizeof(StepDesc)) != hipSuccess || hipMemset(c->b.token_log, 0, 2 * sizeof(int32_t)) != hipSuccess)
        return bail(ASYNCLM_E_DEVICE);
    if (hipHostMalloc((void**)&c->token_host, 64, hipHostMallocDefault) != hipSuccess) return bail(ASYNCLM_E_NOMEM);
    std::memset(c->token_host, 0, 64);
    if (hipEventCreateWithFlags(&c->tok_event, hipEventDisableTiming) != hipSuccess) return bail(ASYNCLM_E_DEVICE);
    if (hipMemset(c->b.pipe_abort, 0, sizeof(unsigned) * PIPE_LINE_WORDS) != hipSuccess ||
        hipMemset(c->pipe_go, 0xff, sizeof(unsigned) * PIPE_REGIONS * PIPE_MAX_WORKGROUPS * PIPE_LINE_WORDS) != hipSuccess ||
        hipMemset(c->pipe_counters, 0, sizeof(unsigned) * c->pipe_kernels_max * PIPE_LINE_WORDS) != hipSuccess)
        return bail(ASYNCLM_E_DEVICE);
    if (c->stream) {     // second stream of the two-stream decoding step (default priority, as every stream here)
        if (hipStreamCreateWithFlags(&c->stream2, hipStreamNonBlocking) != hipSuccess ||
            hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&c->ev_join, hipEventDisableTiming) != hipSuccess)
            return bail(ASYNCLM_E_DEVICE);
    }
    if (c->chunk_ok && hipHostMalloc((void**)&c->cb.chosen_host, sizeof(int32_t) * CHUNK_MAX_GROUPS, hipHostMallocDefault) != hipSuccess) return bail(ASYNCLM_E_NOMEM);
    for (int i = 0; i < 2; ++i)
        if (hipHostMalloc((void**)&c->tab_host[i], CHUNK_TAB_BYTES, hipHostMallocDefault) != hipSuccess ||
            hipEventCreateWithFlags(&c->tab_ev[i], hipEventDisableTiming) != hipSuccess)
            return bail(ASYNCLM_E_NOMEM);
    if (hipHostMalloc((void**)&c->ban_host, sizeof(int32_t) * asynclm_ctx::BAN_RING * (1 + BAN_MAX), hipHostMallocDefault) != hipSuccess) return bail(ASYNCLM_E_NOMEM);
    for (int i = 0; i < asynclm_ctx::BAN_RING; ++i)
        if (hipEventCreateWithFlags(&c->ban_ev[i], hipEventDisableTiming) != hipSuccess) return bail(ASYNCLM_E_DEVICE);
    c->batch_seen.assign(cfg->max_seqs, 0);
    c->batch_owner.reserve(CHUNK_MAX_GROUPS + 1);
    // fused decoding step: pointer table, barrier counters, launch plan
    {
        std::vector<const void*> tab;
        for (int l = 0; l < cfg->n_layers; ++l) {
            tab.push_back(c->attn_norm[l]); tab.push_back(c->wqkv[l]); tab.push_back(c->wo[l]);
            tab.push_back(c->ffn_norm[l]); tab.push_back(c->wgate_up[l]); tab.push_back(c->wdown[l]);
            tab.push_back(kv_layer_ptr(c, l));
        }
        char* tabd = nullptr;
        if ((e = dev_alloc(c, &tabd, tab.size() * sizeof(void*))) != hipSuccess) return bail(ASYNCLM_E_NOMEM);
        c->layers_dev = tabd;
        if ((e = dev_alloc(c, &c->bar, (size_t)FUSED_BAR_WORDS)) != hipSuccess) return bail(ASYNCLM_E_NOMEM);
        
        if (hipMemcpy(tabd, tab.data(), tab.size() * sizeof(void*), hipMemcpyHostToDevice) != hipSuccess ||
            hipMemset(c->bar, 0, FUSED_BAR_WORDS * sizeof(unsigned)) != hipSuccess)
            return bail(ASYNCLM_E_DEVICE);
        if ((e = fused_init(cfg->dtype, g, &c->fused)) != hipSuccess) { report_hip("fused_init", e); return bail(ASYNCLM_E_DEVICE); }
        if (g.kv_v_offset == 0) c->fused.supported = false;     // its attention reads the values row by row
        c->opt_fused = 0;      // opt-in (set_option "fused"): the per-operation kernels are currently faster
        if (c->fused.supported && (e = dev_alloc(c, &c->trace, (size_t)FUSED_TRACE_MAX * c->fused.grid)) != hipSuccess) return bail(ASYNCLM_E_NOMEM);
    }
    const int max_k = g.F > g.d ? (g.F > g.Hq * g.dh ? g.F : g.Hq * g.dh) : (g.d > g.Hq * g.dh ? g.d : g.Hq * g.dh);
    if ((e = decode_init(cfg->dtype, max_k)) != hipSuccess) { report_hip("decode_init", e); return bail(ASYNCLM_E_DEVICE); }
    c->pipe_ok = c->stream2 && g.kv_v_offset != 0 && decode_pipeline_fits(cfg->dtype, g, g.kv_lo_offset != 0);
    if (const char* pv = std::getenv("ASYNCLM_PIPELINE")) c->opt_pipeline = (std::atoi(pv) != 0 && c->pipe_ok) ? 1 : 0;
    if (std::getenv("ASYNCLM_VERBOSE")) std::fprintf(stderr, "[asynclm] two-stream step: fits %d, on %d\n", (int)c->pipe_ok, c->opt_pipeline);
    if ((e = rebuild_graphs(c)) != hipSuccess) { report_hip("capture of the decoding steps", e); return bail(ASYNCLM_E_DEVICE); }
    if ((e = hipDeviceSynchronize()) != hipSuccess) { report_hip("hipDeviceSynchronize", e); return bail(ASYNCLM_E_DEVICE); }
    *out = c;
    return ASYNCLM_OK;
}

extern "C" {

int asynclm_destroy(asynclm_ctx* c) {
    if (!c) return ASYNCLM_OK;
    hipStreamSynchronize(c->stream);
    for (auto& kv : c->graphs) hipGraphExecDestroy(kv.second);
    for (hipEvent_t ev : c->prof_events) hipEventDestroy(ev);
    for (void* p : c->allocs) hipFree(p);
    if (c->token_host) hipHostFree(c->token_host);
    if (c->tok_event) hipEventDestroy(c->tok_event);
    if (c->stream2) { hipStreamSynchronize(c->stream2); hipStreamDestroy(c->stream2); }
    if (c->ev_fork) hipEventDestroy(c->ev_fork);
    if (c->ev_join) hipEventDestroy(c->ev_join);
    if (c->cb.chosen_host) hipHostFree(c->cb.chosen_host);
    for (int i = 0; i < 2; ++i) {
        if (c->tab_host[i]) hipHostFree(c->tab_host[i]);
        if (c->tab_ev[i]) hipEventDestroy(c->tab_ev[i]);
    }
    if (c->ban_host) hipHostFree(c->ban_host);
    for (int i = 0; i < asynclm_ctx::BAN_RING; ++i)
        if (c->ban_ev[i]) hipEventDestroy(c->ban_ev[i]);
    delete c;
    return ASYNCLM_OK;
}

int asynclm_prefill(asynclm_ctx* c, int32_t seq, const int32_t* tokens, int32_t n) {
    int r = check_seq(c, seq);
    if (r) return r;
    if ((r = check_tokens(c, tokens, n))) return r;
    if (c->len[seq] != 0) return ASYNCLM_E_STATE;
    if (n > c->cfg.max_positions) return ASYNCLM_E_CAPACITY;
    return append_tokens(c, seq, tokens, n);
}

int asynclm_decode_step(asynclm_ctx* c, int32_t seq, int32_t forced_token, int32_t* token_out) {
    int r = check_seq(c, seq);
    if (r) return r;
    if (forced_token >= c->cfg.vocab) return ASYNCLM_E_INVAL;
    if (c->len[seq] == 0) return ASYNCLM_E_STATE;
    if (c->len[seq] + 1 > c->cfg.max_positions) return ASYNCLM_E_CAPACITY;
    HIPCK(c, step_one_token(c, seq, forced_token < 0 ? -1 : forced_token, true));
    if (token_out) {
        if (c->tok_early) {                         // per-operation step: wait for the choice only
            bool seen = false;
            HIPCK(c, wait_token(c, token_out, &seen));
            if (seen) return ASYNCLM_OK;
        }
        HIPCK(c, hipMemcpyAsync(c->token_host, c->b.token_log, 2 * sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
        HIPCK(c, hipStreamSynchronize(c->stream));
        if (c->token_host[1]) return fail_device(c, hipErrorLaunchFailure);
        *token_out = c->token_host[0];
    }
    return ASYNCLM_OK;
}

int asynclm_inject_interrupt(asynclm_ctx* c, int32_t seq, const int32_t* tokens, int32_t k) {
    int r = check_seq(c, seq);
    if (r) return r;
    if ((r = check_tokens(c, tokens, k))) return r;
    if (c->len[seq] == 0) return ASYNCLM_E_STATE;
    if ((int64_t)c->len[seq] + k > c->cfg.max_positions) return ASYNCLM_E_CAPACITY;
    return append_tokens(c, seq, tokens, k);
}

int asynclm_step_batch(asynclm_ctx* c, int32_t nseq, const int32_t* seqs, const int32_t* forced, const int32_t* intr_tokens,
                       const int32_t* intr_offsets, int32_t* tokens_out) {
    if (!c) return ASYNCLM_E_INVAL;
    if (c->poisoned) return ASYNCLM_E_DEVICE;
    if (nseq < 1 || nseq > c->cfg.max_seqs || !seqs) return ASYNCLM_E_INVAL;
    // everything is checked before anything is enqueued
    {
        std::vector<char>& seen = c->batch_seen;
        std::fill(seen.begin(), seen.end(), 0);
        for (int i = 0; i < nseq; ++i) {
            const int q = seqs[i];
            if (q < 0 || q >= c->cfg.max_seqs || seen[q]) return ASYNCLM_E_INVAL;
            seen[q] = 1;
            if (forced && forced[i] >= c->cfg.vocab) return ASYNCLM_E_INVAL;
            if (intr_offsets && intr_offsets[i + 1] < intr_offsets[i]) return ASYNCLM_E_INVAL;
        }
        if (intr_offsets && intr_offsets[0] < 0) return ASYNCLM_E_INVAL;
        if (intr_offsets && intr_offsets[nseq] > intr_offsets[0] && !intr_tokens) return ASYNCLM_E_INVAL;
        if (intr_offsets)
            for (int j = intr_offsets[0]; j < intr_offsets[nseq]; ++j)
                if (intr_tokens[j] < 0 || intr_tokens[j] >= c->cfg.vocab) return ASYNCLM_E_INVAL;
        for (int i = 0; i < nseq; ++i)
            if (c->len[seqs[i]] == 0) return ASYNCLM_E_STATE;
        for (int i = 0; i < nseq; ++i) {
            const int64_t k = intr_offsets ? intr_offsets[i + 1] - intr_offsets[i] : 0;
            if ((int64_t)c->len[seqs[i]] + 1 + k > c->cfg.max_positions) return ASYNCLM_E_CAPACITY;
        }
    }
    auto forced_of = [&](int i) { return forced && forced[i] >= 0 ? forced[i] : -1; };
    if (nseq == 1 && (!intr_offsets || intr_offsets[1] == intr_offsets[0]))
        return asynclm_decode_step(c, seqs[0], forced_of(0), tokens_out);      // one row: the single-row kernels

    if (!c->chunk_ok) {
        // models outside the matrix-core append path: the same result sequence by sequence through the single-row kernels
        for (int i = 0; i < nseq; ++i) {
            const int k = intr_offsets ? intr_offsets[i + 1] - intr_offsets[i] : 0;
            HIPCK(c, step_one_token(c, seqs[i], forced_of(i), k == 0));
            if (tokens_out) {
                HIPCK(c, hipMemcpyAsync(c->token_host, c->b.token_log, 2 * sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
                HIPCK(c, hipStreamSynchronize(c->stream));
                if (c->token_host[1]) return fail_device(c, hipErrorLaunchFailure);
                tokens_out[i] = c->token_host[0];
            }
            if (k > 0) {
                const int r = append_tokens(c, seqs[i], intr_tokens + intr_offsets[i], k);
                if (r) return r;
            }
        }
        return ASYNCLM_OK;
    }

    // One weight pass per batch_rows rows: groups are packed in the order given; a group that does not fit is
    // continued in the next pass (its later rows see its earlier ones through the cache).
    for (int i = 0; i < nseq; ++i)
        if (forced_of(i) < 0) HIPCK(c, refresh_choice(c, seqs[i]));
    PassBuilder& pb = c->pass;
    std::vector<int>& owner = c->batch_owner;   // group of the current pass -> index i whose token it chooses, or -1
    owner.clear();
    auto flush = [&]() -> int {
        if (pb.t.rows == 0) return ASYNCLM_OK;
        const int ng = pb.t.ngroups;
        HIPCK(c, forward_chunk(c, pb));
        if (tokens_out) {
            HIPCK(c, hipStreamSynchronize(c->stream));
            for (int gi = 0; gi < ng; ++gi)
                if (owner[gi] >= 0) tokens_out[owner[gi]] = c->cb.chosen_host[gi];
        }
        pb.clear();
        owner.clear();
        return ASYNCLM_OK;
    };
    pb.clear();
    for (int i = 0; i < nseq; ++i) {
        const int q = seqs[i];
        const int k = intr_offsets ? intr_offsets[i + 1] - intr_offsets[i] : 0;
        const int32_t* it = k ? intr_tokens + intr_offsets[i] : nullptr;
        int done = 0;                       // rows of this sequence already placed (the chosen token is row 0)
        const int total = 1 + k;
        while (done < total) {
            int space = pb.batch_rows - pb.t.rows;
            if (space == 0 || !pb.fits(1)) { const int r = flush(); if (r) return r; space = pb.batch_rows; }
            int n = std::min(space, total - done);
            while (n > 1 && !pb.fits(n)) --n;
            const int pos0 = c->len[q];     // rows placed by earlier passes are already counted
            if (done == 0) pb.add(q, pos0, n, forced_of(i), it, done + n == total);
            else pb.add(q, pos0, n, -2, it + (done - 1), done + n == total);
            owner.push_back(done == 0 ? i : -1);
            done += n;
            if (done < total) { const int r = flush(); if (r) return r; }
        }
    }
    return flush();
}

int asynclm_set_banned_tokens(asynclm_ctx* c, int32_t seq, const int32_t* ids, int32_t n) {
    int r = check_seq(c, seq);
    if (r) return r;
    if (n < 0 || n > BAN_MAX || (n > 0 && !ids)) return ASYNCLM_E_INVAL;
    for (int i = 0; i < n; ++i)
        if (ids[i] < 0 || ids[i] >= c->cfg.vocab) return ASYNCLM_E_INVAL;
    // through a pinned row (asynchronous copy; stream order puts it before later steps)
    const int slot = c->ban_next;
    HIPCK(c, hipEventSynchronize(c->ban_ev[slot]));
    int32_t* row = c->ban_host + (size_t)slot * (1 + BAN_MAX);
    std::memset(row, 0, sizeof(int32_t) * (1 + BAN_MAX));
    row[0] = n;
    for (int i = 0; i < n; ++i) row[1 + i] = ids[i];
    HIPCK(c, hipMemcpyAsync(c->b.banned + (size_t)seq * (1 + BAN_MAX), row, sizeof(int32_t) * (1 + BAN_MAX), hipMemcpyHostToDevice, c->stream));
    HIPCK(c, hipEventRecord(c->ban_ev[slot], c->stream));
    c->ban_next = (slot + 1) % asynclm_ctx::BAN_RING;
    c->nban[seq] = n;
    if (c->len[seq] > 0) c->choice_stale[seq] = 1;      // the next greedy choice is recomputed under the new list
    return ASYNCLM_OK;
}

// ---- K/V swap (trap handling) ---------------------------------------------------------------------------------

namespace {

struct SwapHeader {
    uint32_t magic, version;
    int32_t len, n_layers, n_planes, has_vt, elem_bytes, Hkv, dh, vocab, next_token, pad;
    uint64_t total_bytes;
};
constexpr uint32_t SWAP_MAGIC = 0x4b56414cu;     // "LAVK"

int swap_planes(const asynclm_ctx* c) {          // row-major planes per layer: K (+lo), and V (+lo) where it is kept
    return (c->g.kv_lo_offset ? 2 : 1) * (c->g.kv_v_offset ? 2 : 1);
}

size_t swap_bytes(const asynclm_ctx* c, int len) {
    const Geom& g = c->g;
    const size_t esz = elem_bytes(c);
    const size_t rows = (size_t)len * g.dh * g.Hkv * esz;                                  // one row-major plane
    const size_t vt = g.kv_vt_offset ? (size_t)((len + 31) / 32) * 32 * g.dh * g.Hkv * esz : 0;   // one tiled V^T plane
    return sizeof(SwapHeader) + (size_t)c->cfg.n_layers * (swap_planes(c) * rows + 2 * vt) + (size_t)g.V * sizeof(float);
}

// Copies every cached row of `seq` between the cache and the packed host image (direction by `out`).
hipError_t swap_copy(asynclm_ctx* c, int seq, int len, char* host, bool out) {
    const Geom& g = c->g;
    const size_t esz = elem_bytes(c);
    const size_t width = (size_t)len * g.dh * esz, pitch = g.kv_head_stride * esz;
    const size_t vt_width = (size_t)((len + 31) / 32) * 32 * g.dh * esz;
    const hipMemcpyKind kind = out ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice;
    char* h = host;
    hipError_t e;
    for (int l = 0; l < c->cfg.n_layers; ++l) {
        char* base = (char*)kv_layer_ptr(c, l) + (size_t)seq * g.kv_seq_stride * esz;
        size_t offs[4]; int np = 0;
        offs[np++] = 0;
        if (g.kv_lo_offset) offs[np++] = g.kv_lo_offset;
        if (g.kv_v_offset) {
            offs[np++] = g.kv_v_offset;
            if (g.kv_lo_offset) offs[np++] = g.kv_v_offset + g.kv_lo_offset;
        }
        for (int p = 0; p < np; ++p) {
            char* dev = base + offs[p] * esz;
            e = out ? hipMemcpy2DAsync(h, width, dev, pitch, width, g.Hkv, kind, c->stream)
                    : hipMemcpy2DAsync(dev, pitch, h, width, width, g.Hkv, kind, c->stream);
            if (e) return e;
            h += width * g.Hkv;
        }
        if (g.kv_vt_offset) {
            for (int p = 0; p < 2; ++p) {
                char* dev = base + (g.kv_vt_offset + (p ? g.kv_lo_offset : 0)) * esz;
                e = out ? hipMemcpy2DAsync(h, vt_width, dev, pitch, vt_width, g.Hkv, kind, c->stream)
                        : hipMemcpy2DAsync(dev, pitch, h, vt_width, vt_width, g.Hkv, kind, c->stream);
                if (e) return e;
                h += vt_width * g.Hkv;
            }
        }
    }
    float* lg = c->logits + (size_t)seq * g.V;
    e = out ? hipMemcpyAsync(h, lg, sizeof(float) * g.V, kind, c->stream) : hipMemcpyAsync(lg, h, sizeof(float) * g.V, kind, c->stream);
    return e;
}

}  // namespace

int asynclm_kv_bytes(asynclm_ctx* c, int32_t seq, uint64_t* bytes) {
    int r = check_seq(c, seq);
    if (r) return r;
    if (!bytes) return ASYNCLM_E_INVAL;
    if (c->len[seq] == 0) return ASYNCLM_E_STATE;
    *bytes = swap_bytes(c, c->len[seq]);
    return ASYNCLM_OK;
}

int asynclm_kv_swap_out(asynclm_ctx* c, int32_t seq, void* host_buf, uint64_t capacity) {
    int r = check_seq(c, seq);
    if (r) return r;
    if (!host_buf) return ASYNCLM_E_INVAL;
    if (c->len[seq] == 0) return ASYNCLM_E_STATE;
    const int len = c->len[seq];
    const size_t need = swap_bytes(c, len);
    if (capacity < need) return ASYNCLM_E_CAPACITY;
    HIPCK(c, refresh_choice(c, seq));           // the saved greedy token is the one under the current ban list
    SwapHeader hd{};
    hd.magic = SWAP_MAGIC; hd.version = 1; hd.len = len; hd.n_layers = c->cfg.n_layers; hd.n_planes = swap_planes(c);
    hd.has_vt = c->g.kv_vt_offset ? 1 : 0; hd.elem_bytes = (int32_t)elem_bytes(c); hd.Hkv = c->g.Hkv; hd.dh = c->g.dh;
    hd.vocab = c->g.V; hd.total_bytes = need;
    HIPCK(c, swap_copy(c, seq, len, (char*)host_buf + sizeof(SwapHeader), true));
    HIPCK(c, hipMemcpyAsync(c->token_host, &c->b.seq_state[seq].next_token, sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    HIPCK(c, hipStreamSynchronize(c->stream));
    hd.next_token = c->token_host[0];
    std::memcpy(host_buf, &hd, sizeof(hd));
    return ASYNCLM_OK;
}

int asynclm_kv_swap_in(asynclm_ctx* c, int32_t seq, const void* host_buf, uint64_t bytes) {
    int r = check_seq(c, seq);
    if (r) return r;
    if (!host_buf || bytes < sizeof(SwapHeader)) return ASYNCLM_E_INVAL;
    if (c->len[seq] != 0) return ASYNCLM_E_STATE;
    SwapHeader hd;
    std::memcpy(&hd, host_buf, sizeof(hd));
    if (hd.magic != SWAP_MAGIC || hd.version != 1 || hd.len < 1 || hd.n_layers != c->cfg.n_layers || hd.n_planes != swap_planes(c) ||
        hd.has_vt != (c->g.kv_vt_offset ? 1 : 0) || hd.elem_bytes != (int32_t)elem_bytes(c) || hd.Hkv != c->g.Hkv || hd.dh != c->g.dh ||
        hd.vocab != c->g.V || hd.next_token < 0 || hd.next_token >= c->g.V)
        return ASYNCLM_E_INVAL;
    if (hd.len > c->cfg.max_positions) return ASYNCLM_E_CAPACITY;
    if (hd.total_bytes != swap_bytes(c, hd.len) || bytes < hd.total_bytes) return ASYNCLM_E_INVAL;
    HIPCK(c, swap_copy(c, seq, hd.len, (char*)const_cast<void*>(host_buf) + sizeof(SwapHeader), false));
    SeqState st{hd.len, hd.next_token};
    HIPCK(c, hipMemcpyAsync(c->b.seq_state + seq, &st, sizeof(st), hipMemcpyHostToDevice, c->stream));
    HIPCK(c, hipStreamSynchronize(c->stream));   // the host image may be released when the call returns
    c->len[seq] = hd.len;
    c->choice_stale[seq] = c->nban[seq] > 0;     // the restored token was chosen under the saver's list
    return ASYNCLM_OK;
}

int asynclm_peek_token(asynclm_ctx* c, int32_t seq, int32_t* token_out) {
    int r = check_seq(c, seq);
    if (r) return r;
    if (!token_out) return ASYNCLM_E_INVAL;
    if (c->len[seq] == 0) return ASYNCLM_E_STATE;
    HIPCK(c, refresh_choice(c, seq));
    HIPCK(c, hipMemcpyAsync(c->token_host, &c->b.seq_state[seq].next_token, sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    HIPCK(c, hipStreamSynchronize(c->stream));
    *token_out = c->token_host[0];
    return ASYNCLM_OK;
}

int asynclm_logits(asynclm_ctx* c, int32_t seq, float* out_host, int32_t n) {
    int r = check_seq(c, seq);
    if (r) return r;
    if (!out_host || n != c->cfg.vocab) return ASYNCLM_E_INVAL;
    if (c->len[seq] == 0) return ASYNCLM_E_STATE;
    HIPCK(c, hipMemcpyAsync(out_host, c->logits + (size_t)seq * c->g.V, sizeof(float) * n, hipMemcpyDeviceToHost, c->stream));
    HIPCK(c, hipMemcpyAsync(c->token_host, c->b.token_log, 2 * sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    HIPCK(c, hipStreamSynchronize(c->stream));
    if (c->token_host[1]) return fail_device(c, hipErrorLaunchFailure);
    return ASYNCLM_OK;
}

int asynclm_logits_device(asynclm_ctx* c, int32_t seq, const float** out_dev) {
    int r = check_seq(c, seq);
    if (r) return r;
    if (!out_dev) return ASYNCLM_E_INVAL;
    *out_dev = c->logits + (size_t)seq * c->g.V;
    return ASYNCLM_OK;
}

int asynclm_seq_len(asynclm_ctx* c, int32_t seq, int32_t* len) {
    int r = check_seq(c, seq);
    if (r) return r;
    if (!len) return ASYNCLM_E_INVAL;
    *len = c->len[seq];
    return ASYNCLM_OK;
}

int asynclm_reset(asynclm_ctx* c, int32_t seq) {
    int r = check_seq(c, seq);
    if (r) return r;
    HIPCK(c, hipMemsetAsync(c->b.seq_state + seq, 0, sizeof(SeqState), c->stream));
    c->len[seq] = 0;
    c->choice_stale[seq] = 0;
    return ASYNCLM_OK;
}

int asynclm_synchronize(asynclm_ctx* c) {
    if (!c) return ASYNCLM_E_INVAL;
    if (c->poisoned) return ASYNCLM_E_DEVICE;
    HIPCK(c, hipStreamSynchronize(c->stream));
    return ASYNCLM_OK;
}

int asynclm_set_option(asynclm_ctx* c, const char* name, int32_t value) {
    if (!c || !name) return ASYNCLM_E_INVAL;
    if (!std::strcmp(name, "chunk")) { if (value < 0 || value > CHUNK_BATCH_ROWS) return ASYNCLM_E_INVAL; c->opt_chunk = value ? value : CHUNK_MAX; return ASYNCLM_OK; }
    if (!std::strcmp(name, "chunk_split")) { if (value < 0 || value > CHUNK_GEMM_MAX_SPLIT) return ASYNCLM_E_INVAL; c->opt_chunk_split = value; return ASYNCLM_OK; }
    // the options below change the launch geometry of a decoding step: its captured graphs are built again (this call allocates)
    auto regraph = [&]() -> int {
        HIPCK(c, hipStreamSynchronize(c->stream));
        HIPCK(c, rebuild_graphs(c));
        return ASYNCLM_OK;
    };
    if (!std::strcmp(name, "gemv_grid")) { if (value < 1 || value > 4096) return ASYNCLM_E_INVAL; decode_set_gemv_grid(value); return regraph(); }
    if (!std::strcmp(name, "fused")) { c->opt_fused = (value && c->fused.supported) ? 1 : 0; return regraph(); }
    if (!std::strcmp(name, "pipeline")) { c->opt_pipeline = (value && c->pipe_ok) ? 1 : 0; return regraph(); }
    if (!std::strcmp(name, "graph")) { c->opt_graph = (value && c->stream) ? 1 : 0; return regraph(); }
    if (!std::strcmp(name, "attn_mfma_min")) { if (value < 0) return ASYNCLM_E_INVAL; c->opt_attn_mfma_min = value; return regraph(); }
    if (!std::strcmp(name, "step_stamps")) { c->opt_step_stamps = value ? 1 : 0; return regraph(); }
    if (!std::strcmp(name, "attn_split")) { if (value < 0 || value > CHUNK_ATTN_MAX_SPLIT) return ASYNCLM_E_INVAL; c->opt_attn_split = value; return regraph(); }
    return ASYNCLM_E_INVAL;
}

int asynclm_profile_step(asynclm_ctx* c, int32_t seq, int32_t forced_token, const char* const** names_out,
                         float* ms_out, int32_t* launches_out, int32_t cap) {
    int r = check_seq(c, seq);
    if (r) return r;
    if (!ms_out || !launches_out || cap < KC_COUNT || forced_token < 0 || forced_token >= c->cfg.vocab) return ASYNCLM_E_INVAL;
    if (c->len[seq] == 0) return ASYNCLM_E_STATE;
    if (c->len[seq] + 1 > c->cfg.max_positions) return ASYNCLM_E_CAPACITY;
    for (hipEvent_t ev : c->prof_events) hipEventDestroy(ev);
    c->prof_events.clear(); c->prof_class.clear();
    for (int i = 0; i < KC_COUNT; ++i) { ms_out[i] = 0.f; launches_out[i] = 0; }
    if (c->opt_fused) {
        // one launch: HIP events around the kernel, and the kernel's own phase time stamps (100 MHz clock)
        const int nl = c->cfg.n_layers, n_stamps = 1 + 12 * nl + 2;
        if (n_stamps > FUSED_TRACE_MAX) return ASYNCLM_E_INVAL;
        hipEvent_t e0, e1;
        HIPCK(c, hipEventCreate(&e0)); HIPCK(c, hipEventCreate(&e1));
        c->prof_events.push_back(e0); c->prof_events.push_back(e1);
        HIPCK(c, hipEventRecord(e0, c->stream));
        c->want_trace = true;
        hipError_t e = step_one_token(c, seq, forced_token, true);
        c->want_trace = false;
        if (e) return fail_device(c, e);
        HIPCK(c, hipEventRecord(e1, c->stream));
        // stamps [i][workgroup]; a phase lasts from the latest start to the latest finish over the workgroups,
        // a barrier from the latest arrival to the latest release
        const size_t nw = (size_t)c->fused.grid;
        std::vector<unsigned long long> raw((size_t)n_stamps * nw), t(n_stamps);
        HIPCK(c, hipMemcpyAsync(raw.data(), c->trace, sizeof(unsigned long long) * raw.size(), hipMemcpyDeviceToHost, c->stream));
        HIPCK(c, hipStreamSynchronize(c->stream));
        for (int i = 0; i < n_stamps; ++i) t[i] = *std::max_element(raw.begin() + i * nw, raw.begin() + (i + 1) * nw);
        c->last_trace = raw; c->last_trace_stamps = n_stamps;
        float ms = 0.f;
        HIPCK(c, hipEventElapsedTime(&ms, e0, e1));
        ms_out[KC_F_TOTAL] = ms; launches_out[KC_F_TOTAL] = 1;
        auto add = [&](int kc, size_t i) { ms_out[kc] += (float)((double)(t[i] - t[i - 1]) * 1e-5); launches_out[kc] += 1; };
        for (int l = 0; l < nl; ++l) {
            const size_t b = 1 + 12 * (size_t)l;
            for (int k = 0; k < 12; ++k) add(KC_F_QKV + k, b + k);
        }
        add(KC_F_HEAD, 1 + 12 * (size_t)nl); add(KC_F_HEAD_WAIT, 2 + 12 * (size_t)nl);
        if (names_out) *names_out = kClassNames;
        return KC_COUNT;
    }
    c->prof = true;
    hipError_t e = step_one_token(c, seq, forced_token, true);
    c->prof = false;
    if (e) return fail_device(c, e);
    HIPCK(c, hipStreamSynchronize(c->stream));
    for (size_t i = 0; i < c->prof_class.size(); ++i) {
        float ms = 0.f;
        HIPCK(c, hipEventElapsedTime(&ms, c->prof_events[2 * i], c->prof_events[2 * i + 1]));
        ms_out[c->prof_class[i]] += ms;
        launches_out[c->prof_class[i]] += 1;
    }
    if (names_out) *names_out = kClassNames;
    return KC_COUNT;
}

int asynclm_profile_trace(asynclm_ctx* c, uint64_t* out_host, int32_t cap, int32_t* n_stamps, int32_t* n_workgroups) {
    if (!c || !n_stamps || !n_workgroups) return ASYNCLM_E_INVAL;
    if (c->pipe_kernels > 0 && !c->opt_fused) {
        // the last two-stream step (or one-stream step in stamp mode): per kernel, start / hand-over seen (input vector
        // staged) / done of its first and of its last workgroup
        *n_stamps = 3 * c->pipe_kernels; *n_workgroups = 2;
        if (out_host) {
            if (cap < 6 * c->pipe_kernels) return ASYNCLM_E_INVAL;
            std::vector<unsigned long long> raw((size_t)6 * c->pipe_kernels);
            HIPCK(c, hipStreamSynchronize(c->stream));
            HIPCK(c, hipMemcpy(raw.data(), c->pipe_stamps, raw.size() * sizeof(unsigned long long), hipMemcpyDeviceToHost));
            if (c->last_step_stamp_mode) {      // done: earliest and latest of the workgroups' own words
                std::vector<unsigned long long> done((size_t)c->pipe_kernels * STAMP_DONE_SLOTS);
                HIPCK(c, hipMemcpy(done.data(), c->stamp_done, done.size() * sizeof(unsigned long long), hipMemcpyDeviceToHost));
                for (int k = 0; k < c->pipe_kernels; ++k) {
                    unsigned long long lo = ~0ull, hi = 0;
                    for (int w = 0; w < STAMP_DONE_SLOTS; ++w) {
                        const unsigned long long t = done[(size_t)k * STAMP_DONE_SLOTS + w];
                        if (t) { lo = std::min(lo, t); hi = std::max(hi, t); }
                    }
                    raw[(size_t)k * 6 + 2] = hi ? lo : 0; raw[(size_t)k * 6 + 5] = hi;
                }
            }
            for (int k = 0; k < c->pipe_kernels; ++k)
                for (int w = 0; w < 2; ++w)
                    for (int j = 0; j < 3; ++j) out_host[(size_t)(3 * k + j) * 2 + w] = raw[(size_t)k * 6 + w * 3 + j];
        }
        return ASYNCLM_OK;
    }
    *n_stamps = c->last_trace_stamps;
    *n_workgroups = c->last_trace_stamps ? (int32_t)(c->last_trace.size() / c->last_trace_stamps) : 0;
    if (out_host) {
        if ((size_t)cap < c->last_trace.size()) return ASYNCLM_E_INVAL;
        for (size_t i = 0; i < c->last_trace.size(); ++i) out_host[i] = c->last_trace[i];
    }
    return ASYNCLM_OK;
}

// ---- greedy choice without any allocation -----------------------------------------------------------------------

namespace {

// Scratch of asynclm_greedy_token_static: per-block maxima, their indices, the arrival counter.  One copy per device
// that loads the library, held until the process ends.  In host code the array's name is not a device address: the
// address comes from hipGetSymbolAddress, once per device, and only that pointer is handed to kernels.
struct ArgmaxScratch { float part_v[ARGMAX_MAX_BLOCKS]; int32_t part_i[ARGMAX_MAX_BLOCKS]; int32_t counter; int32_t pad[63]; };
static __device__ __align__(256) unsigned char scratch[sizeof(ArgmaxScratch)];

constexpr int STATIC_MAX_DEVICES = 64;
void* g_scratch_ptr[STATIC_MAX_DEVICES] = {};      // per device: device address of `scratch`

}  // namespace

int asynclm_greedy_token_static(const float* logits_dev, int32_t n, const int32_t* banned_dev, int32_t n_banned,
                                int32_t* token_out_dev, void* hip_stream) {
    if (!logits_dev || !token_out_dev || n < 1 || n > ASYNCLM_STATIC_MAX_VOCAB) return ASYNCLM_E_INVAL;
    if (n_banned < 0 || n_banned > BAN_MAX || (n_banned > 0 && !banned_dev)) return ASYNCLM_E_INVAL;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= STATIC_MAX_DEVICES) return ASYNCLM_E_DEVICE;
    if (!g_scratch_ptr[dev]) {          // first call on this device (it is the current one)
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) { report_hip("hipGetSymbolAddress", e); return ASYNCLM_E_DEVICE; }
        g_scratch_ptr[dev] = p;
    }
    ArgmaxScratch* sc = (ArgmaxScratch*)g_scratch_ptr[dev];
    const hipError_t e = launch_argmax_flat(logits_dev, n, banned_dev, n_banned, sc->part_v, sc->part_i, &sc->counter, token_out_dev,
                                            (hipStream_t)hip_stream);
    if (e != hipSuccess) { report_hip("asynclm_greedy_token_static", e); return ASYNCLM_E_DEVICE; }
    return ASYNCLM_OK;
}

const char* asynclm_strerror(int code) {
    switch (code) {
        case ASYNCLM_OK: return "ok";
        case ASYNCLM_E_INVAL: return "invalid argument";
        case ASYNCLM_E_STATE: return "call not allowed in this sequence state";
        case ASYNCLM_E_CAPACITY: return "sequence would exceed max_positions";
        case ASYNCLM_E_NOMEM: return "out of memory";
        case ASYNCLM_E_DEVICE: return "HIP error (context unusable)";
        default: return "unknown error";
    }
}

const char* asynclm_version(void) { return "0.1.0"; }

}  // extern "C"
