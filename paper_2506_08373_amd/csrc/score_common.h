// Definitions shared by the scoring kernels (Sec. 3.1 Eq. 1; Alg. 1 CrossAttention and reduce
// steps): MFMA wrappers per number type, the swizzled 16-byte-chunk row layout used for operand
// tiles in LDS, and the argument block of the sweeps.  Not part of the C ABI.
#pragma once

#include "speckv_internal.h"

namespace speckv {

// Argument block of the scoring sweeps.
struct ScoreArgs {
  Dims d;
  SeqTab t;
  ScoreGeom g;
  const char *q;
  const char *k;
  float2 *part;     // [unit][chunk][RSB] (max2, sum) per row, unit = (layer, head, row super-block)
  int norm_from;    // where the column sweep takes its row normalisers from: kNorm... below
  int share;        // the key-tile sweeps let waves share row blocks (split_blocks)
  float *lse;       // [layer][head][seq][RS*RSB] (kNormMerged)
  const float *lse_in;   // optional caller-supplied natural-log normalisers [L][S][R][Hq]
  float *planes;    // [RS][layer][Hkv*T]
  uint32_t *clear;  // optional scratch (clear_words words) that is zeroed on the way: by the kernel between the sweeps
                    // where there is one, else by the column sweep
  int64_t clear_words;
  int chunk_blocks; // whole-sweep launches: workgroups that run unmasked chunks; the masked tails follow them
  int32_t *fail;    // row-statistics sweep: kFailWords ints per chunk workgroup (see score_sweep.h)
};

// Which of a chunk's keys a sweep visits.  A pruned call (score_prune.hip) has a sample, every 2^step_log-th tile of a sequence's
// unmasked keys, the others, and lists of single keys.
constexpr int kAllKeys = 0, kSampleKeys = 1, kOtherKeys = 2, kListedKeys = 3;

// Argument block of a pruned call's sweeps.
struct PruneArgs : ScoreArgs {
  int32_t chunk_of[kMaxSeqs];   // keys per chunk of the sequence + step_log (prune_step); step_log 0: every key is in the sample
  int32_t order[kMaxSeqs];      // the sequences, those with the longest chunks first
  int32_t item_keys;
  float *squares;               // [unit][chunk][RSB]: sums of the squared terms of the samples' pairs
  float *row_extra;             // laid out like lse: what a row's sample and tail are of its first reference, later log2(first reference /
                                // normaliser)
  const int32_t *list;          // [layer][Hkv*T], laid out like the scores: a row's listed keys
  const PruneRow *rows;
  int32_t one_row;              // 1: one output row for all layers and heads (prompt tokens): every unit computes its list
  const int2 *items;            // (row, place): up to item_keys listed keys of the row from this place on
  const int32_t *n_items;
};

// Row normalisers of the column sweep: merged by a kernel between the sweeps, merged from the partial pairs by every
// workgroup of the column sweep for its own rows, or the caller's.
constexpr int kNormMerged = 0, kNormPairs = 1, kNormCaller = 2;

namespace {

// Super-block of chunk workgroup `bid` of a pruned call.
__device__ __forceinline__ int prune_super_block(const PruneArgs &A, int bid) { return bid % (8 * A.g.RS) >> 3; }
// Chunk workgroup `bid` of a pruned call (unit < 0: it has none).  The workgroups of all layers and heads take a chunk of a sequence
// before those of the next chunk, the longest chunks first.  For the super-blocks of a group see score_sweep.h.
struct PruneChunk { int unit, s, chunk, key_begin, key_end; };
__device__ __forceinline__ PruneChunk prune_chunk(const PruneArgs &A, int bid) {
  PruneChunk c;
  const int groups = A.d.L * A.d.Hkv, per_group = 8 * A.g.RS;
  const int item = bid / per_group * 8 + (bid % per_group & 7);
  c.unit = -1;
  if (item >= A.g.n_fast_chunks * groups) return c;
  int rank = item / groups, i = 0;
  c.unit = item % groups * A.g.RS + prune_super_block(A, bid);
  int s = A.order[0];
  for (;;) {
    const int n = A.t.cc[s + 1] - A.t.cc[s];
    if (rank < n) break;
    rank -= n;
    s = A.order[++i];
  }
  c.s = s;
  const int kc = A.chunk_of[c.s] - prune_step(A.chunk_of[c.s]);
  c.chunk = A.t.cc[c.s] + rank;
  c.key_begin = rank * kc;
  c.key_end = c.key_begin + kc < A.t.tail0[c.s] ? c.key_begin + kc : A.t.tail0[c.s];
  return c;
}
// The tile-th tile of a chunk that is not in the sample, among all of the chunk's.
__device__ __forceinline__ int other_tile(int tile, int step_log) {
  return tile + 1 + (int)((unsigned)tile / ((1u << step_log) - 1u));
}

// Zeroes A.clear (if any), the work spread over every thread of the grid; id: the thread's number in it.
__device__ inline void clear_scratch(const ScoreArgs &A, int64_t id, int64_t n_threads) {
  if (A.clear == nullptr) return;
  for (int64_t i = id; i < A.clear_words; i += n_threads) A.clear[i] = 0u;
}

// The pairs of a row are merged in one order, wherever that is done: a length that is read on the device may come with the
// chunks, and so the place, of a longer prompt, and gives the bits that the same length on the host gives.  merge_slices
// threads per row take every such entry of the row's list: the first kMergeFirst entries together, then kMergeNext each.  The first
// thread adds the others' pairs.  Entry 0 is the pair of the sequence's masked tail, entry e that of its e-th chunk; entries
// of empty chunks, (kNegBig, 0), change nothing.
constexpr int merge_slices(int MB) { return 2 / MB; }
constexpr int kMergeFirst = 32, kMergeNext = 8;

// Adds N (reference, sum) pairs to the pair (top, sum).  (Fused by hand: every copy rounds alike.)
template <int N>
__device__ __forceinline__ void merge_pairs(float &top, float &sum, const float2 *in) {
  const float before = top;
#pragma unroll
  for (int u = 0; u < N; ++u) top = fmaxf(top, in[u].x);
  sum *= __builtin_amdgcn_exp2f(before - top);
#pragma unroll
  for (int u = 0; u < N; ++u) sum = __builtin_fmaf(in[u].y, __builtin_amdgcn_exp2f(in[u].x - top), sum);
}
template <int N>
__device__ __forceinline__ void merge_pairs(float &top, float &sum, const float2 (&in)[N]) { merge_pairs<N>(top, sum, &in[0]); }

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // one 128-bit lane access

constexpr float kNegBig = -1.0e30f;    // finite stand-in for "no key seen yet"
// Row statistics against a fixed reference (score_sweep.h): a segment of kAnchorTiles tiles after
// which a row sum has reached 2^126 (or is not a number) is repeated with the online step.
constexpr int kAnchorTiles = 2;
// the sum's exponent is carried into the reference when it has grown by this many binary orders
constexpr int kAnchorGrowth = 4;
// What each wavefront of a chunk workgroup of the row-statistics sweep leaves for the repair
// launch: [0] the number of segments to repeat, [1 .. kFailListed] the first ones by number,
// [kFailWords - 1] the segment from which on every segment is to be repeated when there are more
// than that.  A workgroup has kFailWaves such lists (the most waves a workgroup has).
constexpr int kFailWords = 8, kFailListed = 6, kFailWaves = 8;
constexpr float kAnchorLimit = 8.507059e37f;
// The sweep of a pruned call over the keys that are not in the sample sums 2^(score - e - kPruneShift) along rows and columns, with
// e the log2 normaliser that the sample and the masked tail give the row.  A score may exceed e by 126 + kPruneShift binary
// orders (140 nats) before the sum of a segment of kPruneSegment tiles overflows and is left to the repair launch; a column sum is
// a bound as long as what underflows in it does not matter beside the threshold (prune_floor).
// An exponent near -kPruneShift is rounded to 2^-18, where one beside a running maximum is to 2^-22 or so.  It does not show: the error
// of a score, the normaliser in it, against 64 bits is as without pruning or smaller (logits of standard deviation 1, 5.5, 10, rms
// 1.0e-7, 1.1e-6, 1.4e-6, all scores 1.1e-7, 1.5e-6, 2.3e-6), since the products' own rounding and the stored normaliser's are larger.
// Without the shift, keys that stand out by 100 nats overflow segment after segment: 32 layers x 128K 5600 -> 6680 us, 32 x 16K,
// maximum, 861 -> 1140.
// The references are multiples of 1 / kPruneGrain and grow by such, so that they are exact.
constexpr float kPruneShift = 76.f, kPruneGrain = 8.f;
// Segments that wavefronts leave out are listed as kFailWords says, but with the row blocks from bit kFailBlocks on.
constexpr int kPruneSegment = 8, kFailBlocks = 28;


// x + (x of the lane 32 away), in every lane, without going through LDS (v_permlane32_swap).
__device__ inline float add_other_half(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}


__device__ inline float max_other_half(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Number types (values of speckv_dtype) and their element size.
constexpr int kBf16 = SPECKV_BF16, kF32 = SPECKV_F32, kF16 = SPECKV_F16;
constexpr int elt_bytes(int dt) { return dt == kF32 ? 4 : 2; }

// One 16-byte chunk of the head dimension per lane half: 8 bf16/f16 or 4 f32 products per row pair.
template <int DT>
__device__ inline f32x16 mma_chunk(u32x4 a, u32x4 b, f32x16 acc);

template <>
__device__ inline f32x16 mma_chunk<kBf16>(u32x4 a, u32x4 b, f32x16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

template <>
__device__ inline f32x16 mma_chunk<kF16>(u32x4 a, u32x4 b, f32x16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                __builtin_bit_cast(f16x8, b), acc, 0, 0, 0);
}

template <>
__device__ inline f32x16 mma_chunk<kF32>(u32x4 a, u32x4 b, f32x16 acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
  return acc;
}

template <int ELT, int D>
struct Tile {
  static constexpr int ROWB = D * ELT;          // bytes per key / query row
  static constexpr int C16 = ROWB / 16;         // 16-byte chunks per row
  static constexpr int NCS = C16 / 2;           // chunk steps (each lane half owns NCS chunks)
  static constexpr int ALIGN = ROWB <= 128 ? 256 : ROWB <= 256 ? 128 : 64;     // chunks and masked tails start at multiples of this many keys
  static constexpr int RPB = ROWB >= 256 ? 1 : 256 / ROWB;   // rows per 256-byte bank sweep
  static constexpr int SWZ = (C16 < 16 ? C16 : 16) - 1;      // xor mask applied to the chunk index
  __device__ static inline int swizzle(int row) { return (row / RPB) & SWZ; }
};

}  // namespace

// Column-reduction and row-statistics sweeps over the unmasked chunks with the group's query
// rows stationary in LDS and each wave streaming its own keys through registers (score_qs.hip).
// Returns false when the geometry is outside what that kernel is built for; then nothing was
// launched and the caller uses the tile-streaming kernel.
// The two sweeps over all chunks and masked tails of a call (score_rows.hip, score_cols.hip).
hipError_t launch_row_statistics_sweep(const ScoreArgs &A, hipStream_t st);
hipError_t launch_column_sweep(const ScoreArgs &A, hipStream_t st);
// Merges the partial pairs of every row into A.lse; row_extra: not null in a pruned call, see there (score.hip).
hipError_t launch_lse_combine(const ScoreArgs &A, float *row_extra, hipStream_t st);
// First references of a pruned call, into A.lse and A.row_extra; the samples' pairs join the tails' (prune.hip).
hipError_t launch_prune_references(const PruneArgs &A, int tile_keys, hipStream_t st);
bool qs_supported(const ScoreArgs &A, int pass);
hipError_t launch_qs_sweep(const ScoreArgs &A, int pass, hipStream_t st);

}  // namespace speckv
