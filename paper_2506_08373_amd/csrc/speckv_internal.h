// Internal plan shared by the host API and the gfx950 kernels of libspeckv.
// Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstdlib>
#include <cstring>

#include "speckv.h"

namespace speckv {

constexpr int kMaxSeqs = SPECKV_MAX_SEQS;

// Per-sequence prefix tables, passed to kernels by value (kernarg segment).
struct SeqTab {
  int32_t n_seqs;
  int32_t cu[kMaxSeqs + 1];   // token prefix sums
  int32_t ck[kMaxSeqs + 1];   // prefix sums of n_keep_s
  int32_t cc[kMaxSeqs + 1];   // prefix sums of the unmasked key chunks (scoring grid)
  int32_t tail0[kMaxSeqs];    // first key of the masked tail: keys below it are visible to every row
};

struct Dims {
  int32_t L, S, Hq, Hkv, G, D, elt;       // elt = bytes per element (2 bf16 / f16, 4 f32)
  int32_t dt;                              // speckv_dtype of q, k, v
  int32_t w, a, R, M;                      // M = G * R rows per KV group
  int32_t pool_k, c_max;
  int32_t reduce_max;                      // 1: max over the rows of a head instead of the sum
  int32_t head_max;                        // 1: heads (and layers) combined by max instead of sum
  int32_t pool_avg;                        // 1: zero-padded mean instead of the clipped max
  int32_t weight_rows;                     // 1: window row i scaled by (i + 1) / n_window (Alg. 2)
  float sm_scale;
  int64_t q_sl, q_ss, q_sr, q_sh;          // element strides
  int64_t kv_sl, kv_st, kv_sh;
  int64_t T, KT;                           // total tokens, total kept rows
  const int32_t *n_dev;                    // device-side token count of a one-sequence call, or null
};

// Geometry of the scoring launches (Alg. 1 CrossAttention + reduce).
struct ScoreGeom {
  int32_t MB;         // 32-row blocks per wave
  int32_t NW;         // waves per workgroup
  int32_t RSB;        // rows per workgroup = NW * MB * 32
  int32_t RS;         // row super-blocks per KV group
  int32_t Rp;         // observation rows per head, padded to a multiple of 32
  int32_t HPS;        // whole heads per super-block (when a head fits), else 1
  int32_t PPH;        // super-blocks per head (1 when a head fits)
  int32_t pitch;      // rows from one head's first row to the next one's: Rp, or R where rows are packed (pack_rows)
  uint32_t pitch_inv; // 2^32 / pitch, rounded up: row / pitch is the high word of row * pitch_inv (rows stay below 2^13)
  int32_t packed;     // row blocks of the group where rows are packed, spread evenly over the super-blocks; else 0
  int32_t KC;         // keys per chunk (multiple of the LDS tile)
  int32_t short_log;  // when not 0: chunks have fewer keys if the length that is read on the device says so; log2 of a tile's keys (chunk_keys)
  int32_t n_fast_chunks;   // unmasked chunks over all sequences = cc[S]
  int32_t n_chunks;        // n_fast_chunks + one masked tail chunk per sequence
};

struct Plan {
  Dims d;
  SeqTab t;
  ScoreGeom g;
  // workspace carve-up (byte offsets, 256-aligned): carve_workspace
  int32_t one_row, sel_kept;               // prompt tokens: one output row for all layers and heads, tokens kept in it
  int64_t room_chunks, most_chunks;        // unmasked chunks that there is room for; the most of any prompt no longer than this one
  size_t off_part, off_lse, off_planes, off_pooled, off_pooled2, off_sel, total;
  size_t off_ada_hist, off_ada_state, total_ada;   // extra scratch of the shared-budget selection
  // selection of long rows in calls with few rows: parts per row (1: not split), keys per part, scratch
  int32_t sel_parts, sel_part_len, most_sel_parts;       // most_sel_parts: of any prompt
  size_t off_sel_hist, off_sel_state;
  // pruned scoring (score_prune.hip): sample step of every sequence; the pairs, in the pooled scores' place; scratch behind everything else
  int32_t chunk_of[kMaxSeqs], order[kMaxSeqs];     // see PruneArgs
  int32_t item_keys, prune_keep;                   // prune_keep: of prompt tokens, else 0
  size_t off_prune_items, off_prune_rows, off_prune_pairs, off_squares, off_row_extra, total_pruned;
  // first-digit histograms of the pooled rows (2048 counters per row), filled by the pooling kernel
  // of a fused call so that selection starts at the second read; hist0_words == 0: not used
  size_t off_hist0;
  int64_t hist0_words;
};

// Keys per chunk of a prompt with `keys` unmasked keys in a call that longer chunks would not spread over the CUs (see
// build_plan): as few tiles as make at most kShortChunks chunks, and not more than `longest`.
constexpr int kShortChunks = 20;
inline __host__ __device__ int short_chunk(uint32_t keys, int tile_log, int longest) {
  const int tiles = (int)(((keys >> tile_log) + kShortChunks - 1) / (uint32_t)kShortChunks);
  const int c = (tiles > 1 ? tiles : 1) << tile_log;
  return c < longest ? c : longest;
}
// Keys per chunk, given the first key of the masked tail as the kernels see it (straight code: a branch here, never taken, cost
// the sweeps of small calls 1 %).
inline __host__ __device__ int chunk_keys(const ScoreGeom &g, int tail0) {
  const int c = short_chunk((uint32_t)tail0, g.short_log, g.KC);
  return g.short_log == 0 ? g.KC : c;
}

inline __host__ __device__ int64_t align_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// Tokens of sequence s as the kernels see them.  Normally the host's length; with a device-side
// count (one-sequence calls only) that count, clamped to [max(1, n_window), host length].  The
// host length stays the row stride of every layout and the bound of every grid.
__device__ inline int live_len(const Dims &d, const SeqTab &t, int s) {
  const int n_host = t.cu[s + 1] - t.cu[s];
  if (d.n_dev == nullptr) return n_host;
  const int lo = d.w > 1 ? d.w : 1;
  const int v = *d.n_dev;
  return v < lo ? lo : (v > n_host ? n_host : v);
}
// First key of the masked tail for a live length n: keys below it are whole LDS tiles (kt keys)
// that every observation row may see (key <= n - n_window).
__device__ inline int live_tail0(const Dims &d, const SeqTab &t, int s, int n, int kt) {
  if (d.n_dev == nullptr) return t.tail0[s];
  const int visible = n - d.w + 1 < n ? n - d.w + 1 : n;
  return visible / kt * kt;
}

// Lays out the workspace of a call with up to `chunks` unmasked chunks; pooled: the least bytes for pooled scores.
void carve_workspace(Plan *pl, int64_t chunks, size_t pooled = 0);

// Raises a kernel's dynamic LDS limit; the runtime call is made once per (device, kernel, size)
// and remembered (score.hip).
hipError_t allow_dynamic_lds(const void *kernel, size_t bytes);

// Kernel launchers (each returns the hipError of its launches).
hipError_t launch_compact(const Plan &pl, const void *k, const void *v, const int32_t *idx,
                          void *k_out, void *v_out, hipStream_t st);
// `events`, when not null, holds 4 hipEvent_t recorded before pass 1, before the merge of the
// row statistics, before pass 2 and after pass 2.
// `lse_in`, when not null, holds natural-log row normalisers [L][S][R][Hq]; the row-statistics
// sweep is skipped and only the column reduction runs.
// `clear`, when not null, is scratch of clear_words 32-bit words that the call leaves zeroed (done
// by the kernel between the sweeps or by the column sweep: the fused calls need zeroed counters for the pooling
// kernel and must not use a memset, which a captured graph may not contain).
// ints behind the partial pairs of the row-statistics sweep (one short list per chunk workgroup)
int64_t score_fail_words(const Dims &d, const ScoreGeom &g, int64_t n_fast_chunks);
// Workgroups of one scoring sweep: chunk workgroups ((layer, head, chunk) items rounded up to a
// multiple of 8, times the row super-blocks) plus one masked tail per (unit, sequence).
inline int64_t score_chunk_workgroups(const Dims &d, const ScoreGeom &g, int64_t n_fast_chunks) {
  return (n_fast_chunks * d.L * d.Hkv + 7) / 8 * 8 * g.RS;
}
// True when the key-tile row-statistics sweep sums against fixed reference exponents and a repair
// launch follows it.  That pays when the sweep runs for several rounds of workgroups; in a
// one-round sweep the repair launch (a few microseconds when it has nothing to do, a segment's
// duration when it has) costs about what the first sweep gains.  Scoring at the 8B shape, 128 rows per head, us
// fixed / online by workgroups of a sweep: 136 (one layer of 8K keys) 52.5-55 / 51-52.5; 240 (32K) 93 / 92.5;
// 256 (128K) 275-279 / 279-285; 288 (3 layers x 40K) 326 / 335; 432 (6 x 32K) 488 / 505; 528 (2 x 128K) 576 / 594;
// 640 (16 x 16K) 583 / 603.  They cross near one round, below the line, which dates from kernels before the reference
// came from a whole tile.
// The environment can override the choice (read on every call so that a test can switch it):
// SPECKV_ROW_STATISTICS=fixed (always) or online (never); with either, fused calls are not pruned.
inline bool score_rows_fixed_reference(const Dims &d, const ScoreGeom &g) {
  const char *e = std::getenv("SPECKV_ROW_STATISTICS");
  if (e != nullptr && std::strcmp(e, "fixed") == 0) return true;
  if (e != nullptr && std::strcmp(e, "online") == 0) return false;
  return score_chunk_workgroups(d, g, g.n_fast_chunks) + (int64_t)d.L * d.Hkv * g.RS * d.S > 2 * 256;
}
hipError_t launch_score(const Plan &pl, const void *q, const void *k, float2 *part, float *lse,
                        float *planes, hipStream_t st, hipEvent_t *events = nullptr,
                        const float *lse_in = nullptr, uint32_t *clear = nullptr, int64_t clear_words = 0);
// True when sweep `pass` (1 row statistics, 2 column reduction) over the unmasked chunks of this
// plan runs in the Q-stationary kernel (score_qs.hip) rather than the tile-streaming one
// (score_sweep.h); diagnostics only.
bool score_uses_qs(const Plan &pl, int pass);
// Row blocks of super-block `rs`; *first: the group's row blocks before it (PPH == 1).
__host__ __device__ inline int super_block_blocks(const Dims &d, const ScoreGeom &g, int rs, int *first) {
  if (g.PPH != 1) {
    const int rows = d.R - (rs % g.PPH) * g.RSB;
    *first = 0;
    return ((rows < g.RSB ? rows : g.RSB) + 31) / 32;
  }
  if (g.packed != 0) {
    const int base = g.packed / g.RS, more = g.packed % g.RS;
    *first = rs * base + (rs < more ? rs : more);
    return base + (rs < more ? 1 : 0);
  }
  const int heads = d.G - rs * g.HPS;
  *first = rs * g.HPS * (g.Rp / 32);
  return (heads < g.HPS ? heads : g.HPS) * (g.Rp / 32);
}
// Row `lr` of super-block `rs` -> (head in group, observation row); false for padding rows.
// A super-block holds a run of the group's row blocks, or one of the PPH slices of a single head.  Each head's R rows are padded
// to Rp, so that heads never share a 32-row block, unless rows are packed.
__host__ __device__ inline bool decode_row(const Dims &d, const ScoreGeom &g, int rs, int lr, int *hh, int *i) {
  int first;
  const int n = super_block_blocks(d, g, rs, &first);
  if (g.PPH == 1) {
    const int row = first * 32 + lr;
    *hh = (int)(((uint64_t)(uint32_t)row * g.pitch_inv) >> 32);
    *i = row - *hh * g.pitch;
    return lr < n * 32 && *hh < d.G && *i < d.R;
  }
  *hh = rs / g.PPH;
  *i = (rs % g.PPH) * g.RSB + lr;
  return *i < d.R;
}
// Which wavefronts compute a super-block's n row blocks in the key-tile sweeps.  The first `full` blocks belong to one wavefront
// each (block b to wave b % NW, as its row block b / NW), which loads the four SIMDs of a CU (wave w runs on SIMD w % 4) evenly
// if `full` is a multiple of four.  One or two blocks beyond that are shared by the next four waves, `per` = 4 or 2 waves a block,
// each of which takes every per-th 32-key block; per = 1: every block belongs to one wave.
struct BlockSplit { int n, full, per; };
__host__ __device__ inline BlockSplit split_blocks(int n, bool share) {
  BlockSplit b = {n, n, 1};
  const int rest = n & 3;
  if (share && (rest == 1 || rest == 2)) { b.full = n - rest; b.per = 4 / rest; }
  return b;
}
// Block that slot s (= row block * NW + wave) computes.
__host__ __device__ inline int block_of_slot(const BlockSplit &b, int s) { return s < b.full ? s : b.full + (s - b.full) / b.per; }

// ---- pruned scoring (score_prune.hip, prune.hip) ----
// What the pruned sweeps know of an output row (layer, seq, head).
struct PruneRow {
  float bound;       // keys whose bound from the sweep is below this are not listed (negative: every key is)
  int32_t digit;     // first digit of the scores that cannot come from an unlisted key; smaller digits are not counted
  int32_t listed;    // keys in the row's list
  int32_t failed;    // 1: fewer than c_max scores reached the digit, every key is computed
  int32_t layer_digit;   // shared budget: the digit that the layer's threshold will reach
  int32_t pad[3];
};
// An item of a listed sweep holds at most Plan::item_keys keys, and at least this many but for the last of a row.
constexpr int kPruneItemMin = 512, kPruneItemMax = 2048;
inline __host__ __device__ int prune_step(int32_t chunk_of) { return chunk_of & 7; }
// Keys of a sample's tile: Operand::KT of the scoring kernels.
inline int prune_tile_keys(const Plan &pl) { return pl.d.D == 64 && pl.g.MB == 2 ? 256 : 128; }
// Turns the plan of a fused call into one of a pruned call where that is faster; false: it is not.
// ada: for a shared budget (scratch behind that of the selection).  keep: 0, or the tokens kept by a call for prompt tokens, whose
// layers and heads have one output row.
bool prune_plan(Plan *pl, int32_t keep = 0, bool ada = false);
// Bytes of workspace with which such a call is pruned, and every one with prompts no longer (0: it is not).
size_t prune_workspace(const Plan &pl, int32_t keep, bool ada);
// Row statistics over the sample, then the sweep over the other keys (bounds into the planes), then the normalisers
// (clear: see launch_score).
hipError_t launch_prune_rows(const Plan &pl, const void *q, const void *k, void *ws, hipStream_t st, hipEvent_t *events,
                             uint32_t *clear, int64_t clear_words);
// Column sums of the sample and the masked tails; thresholds and lists; column sums of the listed keys.
// c_floor, from 0 on: of a shared budget.
hipError_t launch_prune_columns(const Plan &pl, const void *q, const void *k, void *ws, hipStream_t st, int32_t c_floor = -1);
// The same for prompt tokens, with the merged planes' pooling.  scratch: kRowScratchWords words, as launch_select_row_parts reads them.
hipError_t launch_prune_token_columns(const Plan &pl, const void *q, const void *k, void *ws, uint32_t *scratch, hipStream_t st);
hipError_t launch_prune_token_repeat(const Plan &pl, const void *q, const void *k, void *ws, uint32_t *scratch, hipStream_t st);
// After the pooling of these: column sums of all keys, and pooling, of the rows that failed.
hipError_t launch_prune_repeat(const Plan &pl, const void *q, const void *k, void *ws, uint32_t *hist0, hipStream_t st,
                               int32_t c_floor = -1);
// counts: of a shared budget, 2048 words per row of scratch.
hipError_t launch_prune_thresholds(const Plan &pl, const float *planes, const float *row_extra, PruneRow *rows, int32_t *n_items,
                                   hipStream_t st, int32_t c_floor = -1, uint32_t *counts = nullptr);
hipError_t launch_prune_list(const Plan &pl, const float *planes, PruneRow *rows, int32_t *list, int2 *items, int32_t *n_items,
                             hipStream_t st);
// hist0: the pooled scores' first digits.  Lists every key of the rows that failed.
hipError_t launch_prune_check(const Plan &pl, const uint32_t *hist0, PruneRow *rows, int32_t *list, int2 *items, int32_t *n_items,
                              hipStream_t st, int32_t c_floor = -1);

// out rows = (layer, seq, head): pooled/raw in the "scores" layout from RS planes.
// prune, when not null: smaller digits than a row's are not counted; repeat: only the rows that failed, only the smaller digits.
// hist0, when not null: [rows][2048] zeroed counters; the kernel adds the first-digit histogram of
// every row's pooled scores (the non-window entries), for launch_select.
hipError_t launch_reduce_pool(const Plan &pl, const float *planes, float *raw, float *pooled,
                              hipStream_t st, uint32_t *hist0 = nullptr, uint32_t *arrived = nullptr,
                              const PruneRow *prune = nullptr, bool repeat = false);
// Pooling and selection of a fused call's short rows in one launch, where pool_select_fused says so.
bool pool_select_fused(const Plan &pl);
hipError_t launch_pool_select(const Plan &pl, const float *planes, int32_t *idx, hipStream_t st);
// single output row merging every plane of a one-sequence call (prompt-token selection), pooled with pool_k (1: not at
// all); leaves clear[0..clear_words) zeroed
hipError_t launch_reduce_pool_all(const Plan &pl, const float *planes, float *pooled, int32_t pool_k, uint32_t *clear,
                                  int32_t clear_words, hipStream_t st, const PruneRow *if_failed = nullptr);
// max-pool (kernel pool_k, clipped to [0, n_in - n_window)) of one row of n_in scores; hist0, arrived: see launch_reduce_pool
hipError_t launch_pool_row(const Plan &pl, const float *in, float *out, int32_t pool_k, uint32_t *hist0, uint32_t *arrived,
                           hipStream_t st, const PruneRow *prune = nullptr, bool repeat = false);
// hist0, when not null: the rows' first-digit histograms from launch_reduce_pool.  With them, and with list (a word per
// score, laid out like pooled) and counters (kPartsWords per row: an arrival counter, which launch_reduce_pool zeroes, and from
// word 64 on 2 * P counts; rows whose counters share a cache line would wait for each other's atomics), several workgroups
// share a row where select_parts_of says so.
constexpr int kPartsWords = 256;
struct SelectParts { int32_t P, part_len; };
SelectParts select_parts_of(const Plan &pl);
hipError_t launch_select(const Plan &pl, const float *pooled, int32_t *idx, uint32_t *hist, uint32_t *state,
                         hipStream_t st, const uint32_t *hist0 = nullptr, uint32_t *list = nullptr,
                         uint32_t *counters = nullptr);
// Shared layer budget: head offsets from a layer-wide threshold, then per-head selection.
// hist: L*S*Hkv*2048 uint32, state: L*S*(2 + 3*Hkv) uint32 of scratch.
hipError_t launch_select_ada(const Plan &pl, int32_t c_floor, const float *pooled, int32_t *idx,
                             int32_t *head_off, uint32_t *hist, uint32_t *state, hipStream_t st);
hipError_t launch_compact_ada(const Plan &pl, const void *k, const void *v, const int32_t *idx,
                              const int32_t *head_off, void *k_out, void *v_out, hipStream_t st);
// The same by several workgroups (row_parts_of: P > 1).  scratch: kRowScratchWords words, the row's first-digit histogram from
// launch_pool_row and the arrival counter it zeroed; list: a word per score.
constexpr int kRowScratchWords = 2048 + kPartsWords;
SelectParts row_parts_of(int32_t m, int32_t count, size_t scratch_bytes);
hipError_t launch_select_row_parts(const float *row, int32_t m, int32_t count, int32_t *sel, const SelectParts &sp,
                                   uint32_t *list, uint32_t *scratch, hipStream_t st);
hipError_t launch_select_row(const float *pooled_row, int32_t m, int32_t count, int32_t *sel,
                             hipStream_t st);
hipError_t launch_expand(const int32_t *sel, int32_t count, int32_t n_in, int32_t n_window,
                         int32_t n_neighbor, const int32_t *token_ids, int32_t *idx_out,
                         int32_t *ids_out, int32_t *count_out, hipStream_t st);

}  // namespace speckv
