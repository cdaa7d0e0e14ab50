// Host-side launchers of the gfx950 kernels.  Each launcher validates nothing: the C-ABI
// layer in eet_api.hip checks shapes and pointers before any launch.
#pragma once

#include "common.hpp"
#include "tile_rules.hpp"

namespace eet {

// ---- row-wise kernels (rowops.hip) ---------------------------------------------------------
// Words that a launch sets to zero on the side, one to a 128-byte line (counters of a later launch); layernorm_clears says where it can
constexpr int kClearStride = 32;
struct ClearLines {
    uint32_t* at;
    int lines;
};
bool layernorm_clears(int64_t rows, int width, int lines);
// LayerNorm of `rows` rows.  Row r is read from x[in_row_map ? in_row_map[r] : r] and written
// to y[r].  If bump_lens != nullptr, the block of row r < bump_count also does bump_lens[r] += 1
// (advances the per-sequence cache length after all readers of this step were enqueued).
hipError_t launch_layernorm(const half_t* x, const int32_t* in_row_map, const half_t* gamma,
                            const half_t* beta, half_t* y, int64_t rows, int width, float eps,
                            int32_t* bump_lens, int bump_count, hipStream_t s, ClearLines clear = {nullptr, 0});
hipError_t launch_bias_gelu(const half_t* x, const half_t* bias, half_t* y, int64_t rows, int width,
                            hipStream_t s);
hipError_t launch_bias_residual(const half_t* x, const half_t* bias, const half_t* res, half_t* y,
                                int64_t rows, int width, hipStream_t s);
// left_padded: the valid positions of sequence b are S-len[b] .. S-1 (the layout Algorithm 1 is printed for)
hipError_t launch_softmax_maskfree(half_t* scores, const SeqLens& lens, int batch, int heads, int S,
                                   float scale, hipStream_t s, bool left_padded = false);
// Index set-up of a prefill: device copies of the lengths, prefix sums, packed->padded row map,
// and zero fill of the pad rows of `out` ([batch, S, width]).
hipError_t launch_prefill_setup(const SeqLens& lens, int batch, int S, int width, int32_t* cache_lens,
                                int32_t* cu_seqlens, int32_t* row_map, half_t* out, hipStream_t s,
                                bool left_padded = false);
// The exchange area of decode_step.hip, for the launches that set the cache lengths: of every group's words the first kStepCtlWords
// become zero, the others all ones.  words == 0: none.
struct StepArea {
    unsigned long long* ctl;
    uint32_t words;
    int groups;
};
// The same together with the LayerNorm of the valid rows of x ([batch, S, width]) into the packed rows of y, where the width allows.
bool prefill_setup_takes_layernorm(int width);
hipError_t launch_prefill_setup_layernorm(const SeqLens& lens, int batch, int S, int width, int32_t* cache_lens, int32_t* cu_seqlens,
                                          int32_t* row_map, half_t* out, bool left_padded, const half_t* x, const half_t* gamma,
                                          const half_t* beta, half_t* y, float eps, StepArea step, hipStream_t s);

// cache_lens[b] = lens.len[b] for b < batch (DEVICE array of the layer's workspace)
hipError_t launch_set_cache_lens(const SeqLens& lens, int batch, int32_t* cache_lens, StepArea step, hipStream_t s);

// ---- operands of the launches that follow, pulled towards the memory-side cache -------------
// A latency-bound decode projection leaves CUs idle (64-128 workgroups on 256 CUs).  Extra workgroups of the same
// launch use them to touch one word of every 128-byte line of what the NEXT launches will read (weights; the K/V
// rows of the next attention): those launches then find their operands in the memory-side cache, at about half
// the latency of HBM.  Nothing depends on it: the data is read and dropped.
struct PrefetchArgs {
    const void* lin[2];         // linear ranges ...
    uint32_t lin_lines[2];      // ... in 128-byte lines
    const half_t* k_cache;      // K/V rows [0, lens[b]) of every (sequence, head); nullptr = none
    const half_t* v_cache;
    const int32_t* lens;        // DEVICE
    int kv_batch, kv_heads, kv_d, kv_capacity;
    int blocks;                 // extra workgroups that do nothing else; 0 = no prefetch
};

// The same for weights that the launches behind a prefill's attention read: linear ranges in 128-byte lines, touched by `blocks` extra
// workgroups (tile_rules.hpp: prefill_touches_weights has the rule).
struct WeightsAhead {
    const void* at[2];
    uint32_t lines[2];
    int blocks;                 // 0 = none
};

// ---- dense projections (gemm.hip) ------------------------------------------------------------
enum Epilogue : int { EPI_BIAS = 0, EPI_BIAS_GELU = 1, EPI_BIAS_RES = 2, EPI_QKV = 3 };
constexpr int EPI_PARTIAL = 4;   // inside gemm.hip only: the sums of one K range, unrounded (GemmArgs::part)

struct GemmArgs {
    const half_t* x;        // [M, K] activations, row-major
    const half_t* w;        // [N, K] weights, row-major
    const half_t* bias;     // [N]
    half_t* y;              // output [*, N] (EPI_QKV: the Q rows, [M, hidden])
    int M, N, K;
    // MFMA tile kernels only (launch_gemm refuses them elsewhere; see gemm_takes_row_strides): halfs between consecutive
    // rows of x and of y (0: K and N; multiples of 8, not below K and N; not with EPI_QKV)
    int lda, ldy;
    // EPI_BIAS_RES: residual row of output row m is res[res_row_map ? res_row_map[m] : m]
    const half_t* res;
    const int32_t* res_row_map;
    // output row of m is out_row_map ? out_row_map[m] : m   (scatter back to the padded layout)
    const int32_t* out_row_map;
    // EPI_QKV: columns [0,hidden) -> y, [hidden,2*hidden) -> K cache, [2*hidden,3*hidden) -> V cache.
    // Row m belongs to (b, pos): prefill: (row_map[m] / S, row_map[m] % S); decode: (m, lens[m]).
    half_t* k_cache;
    half_t* v_cache;
    const int32_t* tok_row_map;   // prefill: packed row -> b*S + pos ; nullptr in decode
    const int32_t* lens;          // decode: device cache lengths; prefill with left_pad: device prompt lengths
    int left_pad;                 // prefill: tokens of sequence b sit at rows S-len[b] .. S-1 of its block (position = row - (S-len[b]))
    int S, hidden, heads, d, max_seq;
    // weight-streaming kernel only (M <= 16): LayerNorm of x fused in front (nullptr = x is used as it is),
    // and n_b += 1 for the first bump_count sequences (nullptr = no)
    const half_t* ln_gamma;
    const half_t* ln_beta;
    float ln_eps;
    int32_t* bump_lens;
    int bump_count;
    PrefetchArgs pf;              // gemm_flat only
    // gemm_flat with EPI_BIAS_RES only (x_splits > 1): the activations are the decode attention's output still split
    // over key ranges, and the kernel merges the ranges while it loads them (x is not read).  Row m, head g = column
    // / d, range s: weighted values x_part_acc[((m*heads + g)*x_splits + s)*d ..+d], (maximum, sum) in the exp2
    // domain x_part_ml[((m*heads + g)*x_splits + s)*2 ..+2]; heads and d above give the layout.
    const float* x_part_acc;
    const float* x_part_ml;
    int x_splits;
    // gemm_stream with at most 16 rows only: the statistics of a LayerNorm handed from the projection that writes a row
    // (EPI_BIAS_RES, row_stats_out != nullptr) to the projection that normalises it (ln_gamma != nullptr, row_stats_in !=
    // nullptr), so that no launch stands between the two.  Every workgroup of the producer also writes, per row, the mean
    // and the sum of squared deviations of its own columns of the rounded output: row_stats_out[(group*16 + row)*2 ..+2].
    // The consumer merges the row_stats_groups groups of row_stats_cols columns each into mean and 1/std per row and
    // normalises the activation rows on their way to the matrix instructions; its x is the producer's output as it is.
    float* row_stats_out;
    const float* row_stats_in;
    int row_stats_groups, row_stats_cols;
    // gemm_stream and the weight stream of 17 to 128 rows: 1 = the weights are read with the non-temporal hint (common.hpp:
    // load_once).  Right when nothing could keep them cached until their next use anyway (a decode step that moves more than the
    // memory-side cache holds); wrong for a layer small enough to live in that cache from step to step, which the hint would keep
    // out of it.  Uncut projections of 65 rows and more take that stream with the hint only (tile_rules.hpp: rows_stream_uncut).
    int read_once;
    // EPI_BIAS_RES with 17 rows and more: room for the fp32 sums of the K ranges a narrow output is cut into, k_ranges of
    // them (gemm_cut_ranges says how many; <= 1 or part == nullptr: no cut).  [k_ranges][M][N], read by finish_rows.
    float* part;
    int k_ranges;
    // with k_ranges > 1 only: LayerNorm of the finished rows into fin_y[m] ([M, N]) by the same launch (nullptr = no), and
    // n_b += 1 for the first bump_count sequences (bump_lens above)
    const half_t* fin_gamma;
    const half_t* fin_beta;
    half_t* fin_y;
    float fin_eps;
    int fin_as_launch;            // 1: in the order of additions of launch_layernorm for as many rows, so that a row has the bits it would have from there
};
// For a bias+residual projection that launch_gemm would give to gemm_stream and that then can leave row statistics for
// `consumer` (which gemm_stream must take too): the layout of row_stats_out (workgroups, columns per workgroup); else false.
bool gemm_hands_row_stats(const GemmArgs& producer, const GemmArgs& consumer, Epilogue consumer_epi, int& groups, int& cols);
// true when launch_gemm can serve this problem with row strides (more than 16 rows: an MFMA tile kernel)
bool gemm_takes_row_strides(const GemmArgs& a);
// true when launch_gemm would give this projection of at most 16 rows, LayerNorm attached, to the small-layer kernel
bool gemm_takes_layernorm(const GemmArgs& a);
// true when it would give this bias+residual projection of at most 16 rows there: no other kernel has workgroups to prefetch with
bool gemm_takes_prefetch(const GemmArgs& a);
// true when launch_gemm would give this bias+residual projection to the kernel that can merge the key ranges itself
bool gemm_merges_attention_ranges(const GemmArgs& a);

// Adds up the K ranges a.part of a cut projection (rowops.hip); N a multiple of 8, at most kFinishRowsMaxWidth.
// How many ranges the K of a bias + residual projection is worth cutting into (tile_rules.hpp: prompt_k_ranges for a call with row maps, gemm_k_ranges
// otherwise): the caller that has room for their sums ([ranges][M][N] floats) sets GemmArgs::part and k_ranges, for M up to kGemmCutMaxM.
int gemm_cut_ranges(const GemmArgs& a);
hipError_t launch_finish_rows(const GemmArgs& a, hipStream_t s);

// M > 16: MFMA tile kernel.  M <= 16 (decode): weight-streaming kernel.
hipError_t launch_gemm(const GemmArgs& a, Epilogue epi, hipStream_t s);

// ---- attention (attention.hip) -------------------------------------------------------------------
// Prefill: q rows of sequence b start at q_row0 + b*q_seq_stride (+ prefix sum of lens if packed).
struct AttnPrefillArgs {
    const half_t* q;        // row r, head g at q[r*hidden + g*d]
    half_t* ctx;            // same addressing as q
    const half_t* k_cache;  // [batch, heads, capacity, d]
    const half_t* v_cache;
    int batch, heads, d, capacity, hidden;
    int packed;             // 1: rows of sequence b start at sum(len[0..b)); 0: at b*S
    int S;                  // padded length (row stride between sequences when not packed)
    int max_len;            // max over lens (sizes the grid)
    int causal;             // 1: query i sees keys 0..i; 0: every valid query sees all L_b keys (encoder)
    WeightsAhead ahead;             // launch_attention_prefill only
    int chunk_pairs, chunk_tiles, tile_blocks;   // set by the launcher (callers leave 0): pipe::prefill_tile
};
hipError_t launch_attention_prefill(const AttnPrefillArgs& a, const SeqLens& lens, hipStream_t s);
// Unfused form (causal, not packed, S a multiple of 8): raw scores q.k into scores[batch, heads, S, S] for the tiles
// Algorithm 1 will look at; and ctx = probs . V from the probabilities Algorithm 1 left there.
hipError_t launch_attention_scores(const AttnPrefillArgs& a, const SeqLens& lens, half_t* scores, hipStream_t s);
hipError_t launch_attention_apply(const AttnPrefillArgs& a, const SeqLens& lens, const half_t* probs, hipStream_t s);

struct AttnDecodeArgs {
    const half_t* q;        // [batch, heads*d]
    half_t* ctx;            // [batch, heads*d]
    const half_t* k_cache;
    const half_t* v_cache;
    const int32_t* lens;    // DEVICE: number of visible keys minus `len_bias`
    int len_bias;           // keys visible = lens[b] + len_bias (1 inside a decode step: the new token)
    int batch, heads, d, capacity;
    int splits;             // key-range splits per (sequence, head)
    float* part_acc;        // [batch*heads*splits, d]   (splits > 1)
    float* part_ml;         // [batch*heads*splits, 2]
    uint32_t* arrived;      // splits > 1: a zeroed counter per pair, kClearStride apart: the pair's last workgroup merges its ranges, no merge launch (nullptr: there is one)
    int leave_ranges;       // 1: no merge launch, the projection that follows merges the ranges (GemmArgs::x_splits)
    int read_once;          // 1: K/V rows loaded with the non-temporal hint (see GemmArgs::read_once)
    int longest_first;      // set by the launcher
};
int attention_decode_splits(int batch, int heads, int capacity);
size_t attention_decode_scratch_bytes(int batch, int heads, int d, int splits);
hipError_t launch_attention_decode(const AttnDecodeArgs& a, hipStream_t s);

// ---- all layers of a decode step in one launch (decode_step.hip) ----------------------------------
constexpr int kStepLayers = 32;          // layers per launch (their pointers travel as kernel arguments)
constexpr int kStepCtlWords = 32;        // ctl[0]: next item (and kStepGaveUp), layer number; ctl[16]: items that have reset their part; a line each
constexpr uint32_t kStepGaveUp = 1u << 31;
constexpr int kStepGroups = 8;           // groups of rows that a step may have, each with control words and exchange sets of its own
struct StepLayer {
    const half_t *ln1_g, *ln1_b, *w_qkv, *b_qkv, *w_o, *b_o, *ln2_g, *ln2_b, *w_fc1, *b_fc1, *w_fc2, *b_fc2;
    half_t *k_cache, *v_cache;
};
struct StepBuffer {                      // part of an exchange set (words): blocks of 2^log_cols columns, one producer each
    uint32_t at, block;
    int log_cols;
};
// Where the input of a decode step comes from when it is not handed over: row m = wte[ids[m]] + wpe[lens[m]] (launch_embedding's rows, its NaN
// included), which the launch also leaves in `rows`
struct StepTokens {
    const int32_t* ids;                  // nullptr: StepArgs::x
    const half_t *wte, *wpe;
    half_t* rows;
    int vocab, max_pos;
};
struct StepArgs {
    const half_t* x;                     // [M, H] input of the first layer
    StepTokens tok;
    half_t* out;                         // [M, H] output of the last
    unsigned long long* ctl;             // per group kStepCtlWords words, then two exchange sets
    uint32_t set_words;                  // words of a set: decode_step_set_words of the layer's configuration, whatever M is
    int32_t* lens;                       // DEVICE: cached keys; += 1 by the launch when bump
    float eps;
    int bump, M, H, F, heads, max_seq, n_layers;
    // set by the launcher
    StepBuffer bx, bqkv, bctx, by, bf;
    int d, splits, groups, rows, n_qkv, n_att, n_out, n_ffn1, per_layer, items;     // rows: of a group; items: of a group
    StepLayer layer[kStepLayers];
};
// Rows and widths the kernel takes, of a stack of so many layers (1: a layer on its own).
bool decode_step_fits(int rows, int hidden, int heads, int ffn, int max_seq, int layers);
// ... and whether it is the faster way with `visible` keys in all (decode_step.hip has the figures).
bool decode_step_fits_keys(int rows, int heads, int d, size_t visible);
// Words of an exchange set that holds a step of any number of rows up to max_rows that the kernel takes (0: it takes none).  A set has
// this size, is set up (by the launches that set the cache lengths: launch_prefill_setup_layernorm, launch_set_cache_lens) and is
// emptied whole, whatever the rows of a step: a caller may have recorded a step of another number of sequences than those
// of the latest prefill or of the step before, and replay it now.
uint32_t decode_step_set_words(int max_rows, int hidden, int heads, int ffn, int max_seq);
int decode_step_groups(int max_rows, int hidden, int heads, int ffn, int max_seq);     // groups of a step of up to max_rows rows
hipError_t launch_decode_layers(StepArgs& a, bool read_once, hipStream_t s);

// ---- all layers of a short prefill in one launch (prompt_step.hip) ---------------------------------
constexpr int kPromptStepRows = 512;     // rows of the largest prompt
constexpr int kPromptStepK = 1024;       // longest K of an item: hidden, and the range of ffn that an item of the second feed-forward projection takes
constexpr int kPromptStepRanges = 4;
struct PromptShape {
    int row_tiles;                       // of 16 rows
    int ranges, range_units;             // ranges of ffn, units of 64 of each
    int counters;                        // per row tile
    uint32_t ctl_words;                  // number of the next item, then the counters, kClearStride apart
    uint32_t at_ctl, at_f, at_q, at_ctx, at_y, at_part, bytes;   // what the launch hands on
};
struct PromptArgs : PromptShape {
    const half_t* tokens;                // [padded_rows, H] input of the first layer
    half_t* x;                           // [padded_rows, H] between layers (may be tokens or out: a row tile reads and writes its own rows only)
    half_t* out;                         // [padded_rows, H] output of the last
    half_t *q, *ctx, *y, *f;             // packed rows
    float* part;
    uint32_t* ctl;
    const int32_t *lens, *cu, *row_map;  // DEVICE, left by launch_prompt_setup
    StepArea step;                       // of the decode steps to come: where a wait given up is said (no groups: nowhere)
    float eps;
    int T, padded_rows, S, batch, max_len, H, F, heads, max_seq, n_layers, causal, left_pad;
    // set by the launcher
    int d, n_qkv, n_att, n_out, n_ffn1, per_layer, items;
    StepLayer layer[kStepLayers];
};
bool prompt_step_fits(int64_t rows, int64_t padded_rows, int batch, int max_len, int hidden, int heads, int ffn);
PromptShape prompt_step_shape(int rows, int hidden, int ffn);
size_t prompt_step_bytes_up_to(int64_t max_rows, int hidden, int heads, int ffn);
// Lengths, prefix sums and row map, pad rows of a.out, the counters, and the exchange area of the decode steps to come (not where an earlier
// launch of the same prefill has done that, and may have said something there)
hipError_t launch_prompt_setup(const SeqLens& lens, const PromptArgs& a, int32_t* cache_lens, int32_t* cu, int32_t* row_map, StepArea step, hipStream_t s);
hipError_t launch_prompt_layers(PromptArgs& a, bool read_once, hipStream_t s);

// ---- what comes behind the last layer, in one launch (head.hip) --------------------------------------
constexpr int kHeadMaxRows = 16, kHeadMaxK = 1792, kHeadGroups = 256;
struct HeadArgs {
    const half_t* x;            // row m is x[row_map ? row_map[m] : m]
    const int32_t* row_map;
    const half_t *gamma, *beta; // of the final LayerNorm
    const half_t* w;            // [N, K] the table
    half_t* logits;             // [M, N]
    int32_t* next_ids;          // [M]: first maximum of columns [0, vocab); nullptr: no choice, and the two below are not looked at
    unsigned long long* best;   // room for [M, kHeadGroups]
    uint32_t* arrived;          // zero; left zero
    int M, N, K, vocab;
    float eps;
    int x_rows;                 // set by the launcher
};
bool head_takes(int rows, int width, int columns);
hipError_t launch_head(HeadArgs a, hipStream_t s);

// ---- operators around the stack (model.hip) ------------------------------------------------------
// out[b*S + i] = wte[ids[b*S + i]] + wpe[i - first] for first <= i < first + lens.len[b] (first = 0, or S - lens.len[b]
// when left_padded), zeros for pad rows (positions == nullptr);
// or, with S == 1, out[b] = wte[ids[b]] + wpe[positions[b]] (positions on the DEVICE).  Rows whose id or position
// is outside its table become NaN.  last_row (optional, DEVICE [batch]): row index of each sequence's last valid token.
hipError_t launch_embedding(const int32_t* ids, const SeqLens& lens, const int32_t* positions, int batch, int S, int width,
                            int vocab, int max_pos, const half_t* wte, const half_t* wpe, half_t* out, int32_t* last_row,
                            hipStream_t s, bool left_padded = false);
// out[r] = first maximum of logits[r*ld + 0 .. vocab)   (ld % 8 == 0)
hipError_t launch_argmax(const half_t* logits, int rows, int vocab, int ld, int32_t* out, hipStream_t s);

}  // namespace eet
