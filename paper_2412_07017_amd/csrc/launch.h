// Host-callable launchers of the device code (one function per kernel class).
#pragma once

#include "common.h"

namespace asynclm {

constexpr int ARGMAX_MAX_BLOCKS = 256;
constexpr int BAN_MAX = 31;            // token ids per sequence that the greedy choice may be told to skip
constexpr int ATTN_MAX_SPLIT = 64;

// Device buffers of the single-row (decode) path.  All fp32 unless noted.
struct DecodeBuffers {
    StepDesc* step;
    SeqState* seq_state;      // [max_seqs]
    int32_t* token_log;       // last token chosen by k_begin_step
    float* x;                 // [d] residual stream
    float* x2;                // [d] the residual stream's other vector (two-stream step: after the attention block; short step: every second layer)
    float* q;                 // [Hq*dh]
    float* o;                 // [Hq*dh]
    float* a;                 // [F]
    float* part_acc;          // [Hq][ATTN_MAX_SPLIT][dh]
    float* part_ml;           // [Hq][ATTN_MAX_SPLIT][2]
    int32_t* attn_counters;   // [Hkv]
    float* amax_v;            // [ARGMAX_MAX_BLOCKS]
    int32_t* amax_i;
    int32_t* amax_counter;
    int32_t* banned;          // [max_seqs][1 + BAN_MAX]: count, then the ids the greedy choice of the sequence skips
    const float* rope_cos;    // [max_pos][dh/2]
    const float* rope_sin;
    unsigned* pipe_abort;     // give-up word of the two-stream step (see PipeSync)
};

constexpr int CHUNK_MAX = 2048;        // rows per forward pass of the append-chunk path (one sequence; see asynclm_ctx::pass_rows)
constexpr int CHUNK_MAX_TASKS = 512;   // attention tiles (32 query columns of one group) per pass
constexpr int CHUNK_MAX_GROUPS = 128;
constexpr int CHUNK_LOGIT_SLICES = 24; // workgroups per row of logits of a batched step (at most 64: merged by one wave)
// a batched step fills passes of at most this many rows and tiles
constexpr int CHUNK_BATCH_ROWS = 512, CHUNK_BATCH_TASKS = 128;
constexpr int CHUNK_ATTN_MAX_SPLIT = 128;
constexpr int CHUNK_ATTN_MAX_UNITS = 4096;   // (task, kv head, key split) partial results per pass
constexpr int CHUNK_GEMM_MAX_SPLIT = 8;

// What one pass of the append-chunk path processes: rows, grouped by sequence.  A group is a run of
// consecutive rows appended to one sequence: [chosen token] ++ [interrupt tokens], or plain tokens.
// The host fills the table; k_chunk_embed_norm resolves the tokens that are chosen on the device.
// row0, n: its group; token < 0 (first row of a group only): the greedy token of the sequence's current logits;
// group: number of the group whose chosen token this row carries, -1 for the other rows
struct ChunkRow { int32_t token, seq, pos, row0, n, group, pad1, pad2; };
struct ChunkGroup {
    int32_t seq, row0, n, pos0;
    int32_t head;       // row of this group in the output-head product, -1: no logits wanted
    int32_t pad0, pad1, pad2;
};
// query columns 32 tile .. 32 tile + 31 of a group; its attention has nsplit key splits, whose partial results start at unit0 (x kv heads)
struct ChunkTask { int32_t seq, row0, n, pos0, tile, nsplit, unit0, pad; };
// Every group has at least one task, so a batched pass holds at most CHUNK_MAX_GROUPS groups.  A pass uploads the used
// entries only, packed one after the other (ChunkTab): under 1 KB for an interrupt.
struct ChunkTaskBlock { int32_t task0, n; };   // up to four consecutive tasks of one group (they share keys and values)
struct ChunkPiece { int16_t block, split; };   // a workgroup (per kv head) of the shared-key attention
struct ChunkTable {
    int32_t rows, ngroups, ntasks, nhead, nblocks;
    ChunkGroup group[CHUNK_MAX_GROUPS];
    ChunkTask task[CHUNK_MAX_TASKS];
    ChunkTaskBlock block[CHUNK_MAX_GROUPS];     // at most four tasks each: as many as groups in a batched pass, tasks / 4 for one group
    int32_t npieces;
    ChunkPiece piece[CHUNK_ATTN_MAX_UNITS];
    ChunkRow row[CHUNK_MAX];
};

struct ChunkTab { const ChunkGroup* group; const ChunkTask* task; const ChunkTaskBlock* block; const ChunkPiece* piece; const ChunkRow* row; };
constexpr size_t CHUNK_TAB_BYTES = sizeof(ChunkGroup) * CHUNK_MAX_GROUPS + sizeof(ChunkTask) * CHUNK_MAX_TASKS +
                                   (sizeof(ChunkTaskBlock) * CHUNK_MAX_GROUPS + 31) / 32 * 32 + sizeof(ChunkPiece) * CHUNK_ATTN_MAX_UNITS + sizeof(ChunkRow) * CHUNK_MAX;

// Device buffers of the append-chunk path (bf16 models).  "hi/lo" are the two bf16 planes of a value.
struct ChunkBuffers {
    unsigned char* tab_mem;   // [CHUNK_TAB_BYTES]
    ChunkTab tab;             // the running pass's entries in it
    int32_t* chosen_host;     // pinned, [CHUNK_MAX_GROUPS]: token chosen for the first row of each group
    float* x;                 // [pass rows][d] residual stream
    // inputs of the products, as many rows each, stored in matrix-core operand order (tiled planes); the third plane
    // (lo2, the remainder of the other two) exists for the models of forward_wide_rows only
    bf16_t *nrm_hi, *nrm_lo, *nrm_lo2;  // d columns:     normalised input of the QKV, gate/up and output-head products
    bf16_t *att_hi, *att_lo, *att_lo2;  // Hq*dh columns: attention output
    bf16_t *act_hi, *act_lo, *act_lo2;  // F columns:     SwiGLU output
    // rotated, scaled queries [Hkv][q_cols][dh]: the columns of a group are [q head within the kv group][row]
    bf16_t *q_hi, *q_lo;
    int q_cols;               // G * pass rows + 32 (a tile may read up to 31 columns past its group)
    float* part;              // split-K partial planes of the current product
    size_t part_capacity;     // floats in `part`
    float* attn_o;            // [unit][dh][32]      unit = the task's unit0 * Hkv + kv head * its nsplit + split
    float* attn_ml;           // [unit][2][32]
    float* amax_v;            // [CHUNK_MAX_GROUPS][CHUNK_LOGIT_SLICES]
    int32_t* amax_i;
    int32_t* amax_counters;   // [CHUNK_MAX_GROUPS], zero between launches
};

// Several rows of one sequence per pass through the vector-unit kernels (decode_rows.hip): models outside the matrix-core
// append path.  Eight rows: the vectors of 4096 columns fill 128 of the 160 KiB of LDS, and the 2 x 8 products per weight
// element take the vector units about two thirds of the time that the weight stream takes.
constexpr int ROWS_MAX = 8;
constexpr int ROWS_PASS_SMALL = 128;    // rows per pass of a model whose products are all small (k_rows_small)
constexpr int WIDE_ROWS_MAX = 512;      // rows per pass of forward_wide_rows
struct RowsTokens { int32_t t[ROWS_MAX]; };
struct RowsPass { int32_t seq, pos0, n; };
struct RowsBuffers {        // R rows: as many as a pass can have (ROWS_MAX or ROWS_PASS_SMALL; q and the counters: those of forward_wide_rows too)
    float* x;               // [R][d]
    float* q;               // [R][Hq*dh]
    float* o;               // [R][Hq*dh]
    float* a;               // [R][F]
    float* part_acc;        // [ROWS_MAX * ATTN_MAX_SPLIT rows x splits][Hq][dh]
    float* part_ml;         // [ROWS_MAX * ATTN_MAX_SPLIT][Hq][2]
    int32_t* counters;      // [R][Hkv], zero between launches
};
// whether the vectors and the parked results of every product fit LDS with the present number of workgroups
bool rows_supported(int dtype, const Geom& g);
// rows per pass: ROWS_MAX, or ROWS_PASS_SMALL where all products are small
int rows_per_pass(int dtype, const Geom& g);
hipError_t rows_init(int dtype);
// Rows row0 .. row0 + n - 1 of the pass (n <= ROWS_MAX: their tokens travel in the kernel's arguments).
hipError_t launch_rows_embed(int dtype, const void* E, const RowsTokens& tk, int row0, int n, const RowsBuffers& rb, const DecodeBuffers& b, const RowsPass& p,
                             const Geom& g, hipStream_t s);
hipError_t launch_rows_qkv(int dtype, const void* wqkv, const float* gain, void* kv_layer, const RowsBuffers& rb, const DecodeBuffers& b,
                           const RowsPass& p, const Geom& g, hipStream_t s);
// planes: null, or the buffers whose att planes take the output as three bf16 planes (any number of rows; rows x nsplit bounded
// by the partial results' size as long as there is more than one split)
hipError_t launch_rows_attn(int dtype, const void* kv_layer, int nsplit, const RowsBuffers& rb, const RowsPass& p, const Geom& g, hipStream_t s,
                            const ChunkBuffers* planes = nullptr);
// bf16 models: sums the partial planes of a QKV product (kv_only: of its key and value rows), rotates, writes the row-major cache and rb.q
hipError_t launch_rows_rope_kv(const ChunkBuffers& c, int S, int MT, void* kv_layer, const RowsBuffers& rb, const DecodeBuffers& b, const RowsPass& p,
                               const Geom& g, hipStream_t s, bool kv_only);
hipError_t launch_rows_oproj(int dtype, const void* wo, const RowsBuffers& rb, const RowsPass& p, const Geom& g, hipStream_t s);
hipError_t launch_rows_gateup(int dtype, const void* wgu, const float* gain, const RowsBuffers& rb, const RowsPass& p, const Geom& g, hipStream_t s);
hipError_t launch_rows_down(int dtype, const void* wd, const RowsBuffers& rb, const RowsPass& p, const Geom& g, hipStream_t s);

// Decoding step of small models with partial vectors between the kernels (decode_small.hip).
constexpr size_t SMALL_O_BYTES = 128 * 1024;    // columns of the O projection that belong to one kv head: read by one compute unit
constexpr int SMALL_MAX_KV_HEADS = 16, SMALL_MAX_D = 512;
constexpr int SMALL_MAX_KEYS = 384;             // see small_step_pays
constexpr int SMALL_DIRECT_LAYERS = 3;          // up to this many layers a step's launches are issued one by one, see small_direct
struct SmallBuffers { float* parts; };          // [Hkv + small_mlp_parts][d]
bool gemv_all_small(int dtype, const Geom& g);  // every product of a step, output head included, is one of k_gemv_small
bool small_step_supported(int dtype, const Geom& g);
// whether such a step over so many keys is faster than the kernels of the other models
bool small_step_pays(int dtype, const Geom& g, int n_layers, int keys);
int small_mlp_parts(const Geom& g);
// First kernel of such a step: the token (forced, or the sequence's greedy one) and what k_begin_step does for it, its embedding, the first layer's QKV product.
// The position is read from the device, as everywhere in a decoding step: a step that the caller has captured goes on with every replay.
hipError_t launch_small_first(int dtype, const void* E, const void* wqkv, const float* gain, void* kv_layer, const DecodeBuffers& b, const Geom& g, int seq,
                              int forced, TokenWord token_early, float* x_out, hipStream_t s);
// QKV product of a later layer: x_in + all partial vectors -> x_out
hipError_t launch_small_qkv(int dtype, const void* wqkv, const float* gain, void* kv_layer, const SmallBuffers& sb, const DecodeBuffers& b, const Geom& g,
                            const float* x_in, float* x_out, hipStream_t s);
// first_layer: the sequence grows by the step's token
hipError_t launch_small_attn_o(int dtype, const void* kv_layer, const void* wo, const SmallBuffers& sb, const DecodeBuffers& b, const Geom& g, bool first_layer, hipStream_t s);
hipError_t launch_small_mlp(int dtype, const void* wgu, const void* wdown, const float* gain, const float* x, const SmallBuffers& sb, const Geom& g, hipStream_t s);
hipError_t launch_small_head(int dtype, const void* wout, const float* gain, float* logits_base, const SmallBuffers& sb, const DecodeBuffers& b, const Geom& g,
                             const float* x_in, hipStream_t s);

// Fused (persistent, single-kernel) decoding step.
struct FusedPlan {
    bool supported;
    int grid;           // workgroups = compute units
    int nsplit;         // largest number of attention splits per kv head
    int xs_groups;      // LDS capacity of the staged vector
    int done_cap;       // finished units a wave can park in LDS
    size_t lds_bytes;
};
struct FusedLaunch {
    const void* layers_dev;     // device array, 7 pointers per layer: attn_norm, wqkv, wo, ffn_norm, wgate_up, wdown, kv_layer
    int n_layers;
    const void* embed; const float* final_norm; const void* lm_head;
    int seq, forced; bool with_head;
    int nsplit; bool merge_in_stage;   // attention splits of this step; merged by the O projection's staging if set
    float* logits;              // of this sequence
    unsigned* bar;              // FUSED_BAR_WORDS words, zero at create
    void* trace;                // optional device buffer of 64-bit time stamps [FUSED_TRACE_MAX][grid]
};
constexpr int FUSED_TRACE_MAX = 4096;
constexpr int FUSED_BAR_WORDS = 8 + 1024;   // barrier header + one flag per workgroup
hipError_t fused_init(int dtype, const Geom& g, FusedPlan* plan);
hipError_t launch_decode_fused(int dtype, const FusedPlan& plan, const FusedLaunch& L, const DecodeBuffers& b, const Geom& g,
                               hipStream_t s);

hipError_t decode_init(int dtype, int max_k);
void decode_set_gemv_grid(int grid);
int decode_gemv_grid();
hipError_t chunk_init();         // dynamic LDS of the append path's kernels
hipError_t chunk_init_wide();    // ... of those of forward_wide_rows
// planes: 2, or 3 (see forward_wide_rows)
hipError_t launch_chunk_embed_norm(const void* E, const ChunkBuffers& c, const float* gain, int rows, const DecodeBuffers& b, const Geom& g,
                                   hipStream_t s, int planes = 2);
hipError_t launch_chunk_resid_norm(const ChunkBuffers& c, int S, int MT, const float* gain, int rows,
                                   const Geom& g, hipStream_t s, int planes = 2);
// residual stream of the last row of group `group` -> the single-row path's x (and its sequence -> the step descriptor)
hipError_t launch_chunk_last_row(const ChunkBuffers& c, int S, int MT, int group, const DecodeBuffers& b, const Geom& g,
                                 hipStream_t s);
// last rows of all groups that want logits: residual + final norm -> rows 0..nhead-1 of the nrm planes
hipError_t launch_chunk_head_rows(const ChunkBuffers& c, int S, int MT, const float* gain, int ngroups, const Geom& g,
                                  hipStream_t s);
// rows of the head product -> logits of their sequences, greedy argmax -> next_token
hipError_t launch_chunk_logits(const ChunkBuffers& c, float* logits_base, const DecodeBuffers& b, int ngroups,
                               const Geom& g, hipStream_t s);
hipError_t launch_chunk_swiglu(const ChunkBuffers& c, int S, int MT, int rows, const Geom& g, hipStream_t s);
// kv_only: the product held the key and value rows only
hipError_t launch_chunk_rope_kv(const ChunkBuffers& c, int S, void* kv_layer, const DecodeBuffers& b, int rows, int MT,
                                const Geom& g, hipStream_t s, bool kv_only = false);
// How a product of the append path is cut: split of K into s parts with partial planes of their own, nt weight-row tiles of 32
// per workgroup (passes of more than four row tiles only).
struct GemmPlan { int s, nt; };
hipError_t launch_chunk_gemm(const void* W, int N, int K, const bf16_t* xhi, const bf16_t* xlo, const ChunkBuffers& c,
                             GemmPlan pl, int rows, hipStream_t s);
hipError_t launch_chunk_gemm_swiglu(const void* W, int F, int K, const bf16_t* xhi, const bf16_t* xlo, const ChunkBuffers& c,
                                    GemmPlan pl, int rows, hipStream_t s);
// The same products with inputs of three planes (xlo2 / c.act_lo2 the third), any number of row tiles.
hipError_t launch_wide_gemm(const void* W, int N, int K, const bf16_t* xhi, const bf16_t* xlo, const bf16_t* xlo2, const ChunkBuffers& c, int S,
                            int rows, hipStream_t s);
hipError_t launch_wide_gemm_swiglu(const void* W, int F, int K, const bf16_t* xhi, const bf16_t* xlo, const bf16_t* xlo2, const ChunkBuffers& c,
                                   int rows, hipStream_t s);
hipError_t launch_chunk_attn(const ChunkBuffers& c, const void* kv_layer, int nsplit, int ntasks, const Geom& g, hipStream_t s);
// The key splits of every task are in the table; merge: some task has more than one.
hipError_t launch_chunk_attn_wide(const ChunkBuffers& c, const void* kv_layer, bool merge, int ntasks, int npieces, const Geom& g, hipStream_t s);
// single-row decoding attention on the matrix cores (long contexts): b.q -> b.o through the chunk attention
// stamps / done_wg: null, or the stamp words (2 x 6) and finishing-time words (2 x STAMP_DONE_SLOTS) of the attention
// kernel and of its merge kernel (see step_stamp_done)
hipError_t launch_decode_attn_mfma(const ChunkBuffers& c, const void* kv_layer, int nsplit, const DecodeBuffers& b, const Geom& g,
                                   hipStream_t s, unsigned long long* stamps = nullptr, unsigned long long* done_wg = nullptr);
hipError_t launch_stamp_init(unsigned long long* done_wg, int kernels, hipStream_t s);
// token_early: pinned host word that also gets the chosen token
hipError_t launch_embed(int dtype, const void* E, const DecodeBuffers& b, const Geom& g, hipStream_t s);
hipError_t launch_begin_step(int dtype, const void* E, const DecodeBuffers& b, const Geom& g, int seq, int forced, TokenWord token_early,
                             hipStream_t s);
// sync (all single-row launchers): hand-over flags when the step's kernels alternate between two streams (see PipeSync)
hipError_t launch_qkv(int dtype, const void* wqkv, const float* gain, void* kv_layer, const DecodeBuffers& b,
                      const Geom& g, hipStream_t s, const PipeSync* sync = nullptr);
// merge_in_oproj: the attention only leaves per-split partials and the O projection merges them (nsplit <= 8)
hipError_t launch_attn_decode(int dtype, const void* kv_layer, int nsplit, bool merge_in_oproj, const DecodeBuffers& b,
                              const Geom& g, hipStream_t s, const PipeSync* sync = nullptr);
// x_out / x_in / res_in: the residual stream between the O projection and the down projection lives in a second
// vector when given (the two-stream step never updates a vector in place); default: b.x throughout
hipError_t launch_oproj(int dtype, const void* wo, int merge_nsplit, const DecodeBuffers& b, const Geom& g, hipStream_t s,
                        const PipeSync* sync = nullptr, float* x_out = nullptr);
hipError_t launch_gateup(int dtype, const void* wgu, const float* gain, const DecodeBuffers& b, const Geom& g,
                         hipStream_t s, const PipeSync* sync = nullptr, const float* x_in = nullptr);
hipError_t launch_down(int dtype, const void* wd, const DecodeBuffers& b, const Geom& g, hipStream_t s, const PipeSync* sync = nullptr,
                       const float* res_in = nullptr);
// logits_base: [sequences][V]; the kernel writes the row of the step descriptor's sequence and, except in a two-stream step,
// leaves the greedy choice (banned ids skipped) as its next token
hipError_t launch_lmhead(int dtype, const void* wout, const float* gain, float* logits_base, const DecodeBuffers& b,
                         const Geom& g, hipStream_t s, const PipeSync* sync = nullptr);
// True when two workgroups of every single-row kernel of this model fit one compute unit (registers, LDS), i.e. when
// the workgroups of two neighbouring kernels of a step can always all be resident: the condition for running the
// step on two streams.
bool decode_pipeline_fits(int dtype, const Geom& g, bool kv_pair);
// greedy choice (banned ids skipped) of sequence `seq`, or of the step descriptor's sequence when seq < 0
hipError_t launch_argmax(const float* logits_base, const DecodeBuffers& b, const Geom& g, hipStream_t s, int seq = -1);
// the same choice over caller-provided logits[n], skipping the nban ids in ban; part_v / part_i: ARGMAX_MAX_BLOCKS entries
// of scratch, counter: one word of scratch (cleared by the launch); the result goes to *out (device)
hipError_t launch_argmax_flat(const float* logits, int n, const int32_t* ban, int nban, float* part_v, int32_t* part_i,
                              int32_t* counter, int32_t* out, hipStream_t s);

}  // namespace asynclm
