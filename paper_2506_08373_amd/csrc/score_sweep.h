// Importance scoring on the gfx950 matrix cores (Sec. 3.1 Eq. 1; Alg. 1 CrossAttention and
// reduce steps; App. C.2 for the GQA group).
//
// For one (layer, sequence, KV head) the logits are S = Qg . K^T with Qg the M = G*R stacked
// observation rows of the G query heads that share the KV head (row r = head_in_group*R + i)
// and K the n_in prompt keys of that head.  The importance of key j is the column sum of the
// row softmax of sm_scale*S.  A column sum needs every row's normaliser first, so S is
// computed twice and never stored:
//
//   pass 1  row statistics: per row a pair (reference exponent, sum of 2^(c*S - reference)) over
//           the keys of one chunk, the reference either the running maximum or fixed per chunk
//           (see score_body); a small kernel, or pass 2 itself, merges the chunks into
//           lse2[row] = log2 sum_j 2^(c*S[row,j]), c = sm_scale*log2(e).
//   pass 2  column sums: raw[j] = sum_rows 2^(c*S[row,j] - lse2[row]).
//
// Work split: a workgroup owns RSB = NW*MB*32 rows (all of them when M <= RSB) and one chunk of
// keys.  Each wave keeps the MFMA fragments of its MB 32-row blocks of Q in registers for the
// whole sweep; K tiles of KT keys stream HBM -> LDS directly (global_load_lds, double buffered,
// no staging registers; fp32 tiles pass through registers, where they are split, see Operand).  The LDS tile is unpadded; the 16-byte chunks of a row are stored at
// slot = chunk ^ swizzle(row) so that the 128-bit fragment reads of 16 consecutive keys hit 16
// different bank groups.  Every wave reads all K fragments of a tile.
// Pass 1 multiplies with K as the A operand, so a lane holds 16 keys of ONE query row and the
// row statistics stay in two registers per row block; pass 2 multiplies with Q as the A operand,
// so a lane holds 16 rows of ONE key and the column sum is an in-lane add, one cross-half add and
// a cross-wave add through LDS.  No atomics anywhere: results are bit-reproducible.
//
// MFMA operand layout used (v_mfma_f32_32x32x16_bf16, v_mfma_f32_32x32x16_f16; v_mfma_f32_32x32x2_f32
// for fp32 blocks whose scores are not finite): lane l holds
// row (A) or column (B) l%32 and the k-slice selected by l/32; the result register i of lane l
// is element (8*(i/4) + 4*(l/32) + i%4, l%32).  Both operands take their k-slices from the same
// 16-byte chunks of the head dimension (half l/32 reads the chunks of its parity: the two halves' loads of a query row
// then fall into one cache line, and the loads of a workgroup's query rows, which are bound by the lines they
// touch, take half the time), so the
// contraction is over all d channels whatever order the hardware assigns inside a slice.
//
// This header holds the sweep kernels and their launcher, compiled into two translation units, one per
// sweep (score_rows.hip, score_cols.hip).
#pragma once
#include <type_traits>
#include <utility>

#include "score_common.h"

namespace speckv {
namespace {


// Column partials of a tile are complete one unit into the next tile and are read a tile later
// (see do_tile): three tiles' worth is alive at a time, kept modulo four.
constexpr int kCsumBuffers = 4;

// (Out of its generic caller, in which an asm statement may not name its variable.)
__device__ __forceinline__ void add_squares(float &q, float scale, float squares) {
  q = fmaf(q * scale, scale, squares);
  asm volatile("" : "+v"(q));
}

// Has the compiler compute x where this stands.
__device__ __forceinline__ void stay_here(float (&x)[16]) {
#pragma unroll
  for (int i = 0; i < 16; i += 4) asm volatile("" : "+v"(x[i]), "+v"(x[i + 1]), "+v"(x[i + 2]), "+v"(x[i + 3]));
}

// Row blocks (bit mask) of the rows whose lanes, as add_over_lanes has them, are set in `lanes`.
template <int MB>
__device__ __forceinline__ int row_blocks_of(uint64_t lanes) {
  if (MB == 1) return lanes != 0 ? 1 : 0;
  return ((lanes & 0x0000ffff0000ffffull) != 0 ? 1 : 0) | ((lanes & 0xffff0000ffff0000ull) != 0 ? 2 : 0);
}

// Sums 16 MB values per lane over the 32 lanes of its half; lane l gets the sum of value l % 16 of row block l / 16 (MB = 1: of
// value l % 16).  At each step a lane hands half of its values to another lane of the half and adds what it gets for the others.
template <int MB>
__device__ __forceinline__ float add_over_lanes(const float (&v)[MB][16]) {
  const int lane = threadIdx.x;
  float a[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if constexpr (MB == 2) {        // lanes 0 .. 15 keep row block 0
      const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[0][i]), __float_as_uint(v[1][i]), false, false);
      a[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else {
      a[i] = v[0][i];
    }
  }
  auto halve = [&](auto n_c, auto ctrl_c) {            // n values left; the other lane's number differs in bit n
    constexpr int n = decltype(n_c)::value, ctrl = decltype(ctrl_c)::value;
    const bool high = (lane & n) != 0;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const float keep = high ? a[i + n] : a[i], give = high ? a[i] : a[i + n];
      a[i] = keep + __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(give), ctrl, 0xf, 0xf, false));
    }
  };
  halve(std::integral_constant<int, 8>{}, std::integral_constant<int, 0x128>{});     // row_ror:8, lane ^ 8
  halve(std::integral_constant<int, 4>{}, std::integral_constant<int, 0x141>{});     // row_half_mirror, lane ^ 7
  halve(std::integral_constant<int, 2>{}, std::integral_constant<int, 0x4e>{});      // quad_perm [2, 3, 0, 1], lane ^ 2
  halve(std::integral_constant<int, 1>{}, std::integral_constant<int, 0xb1>{});      // quad_perm [1, 0, 3, 2], lane ^ 1
  if constexpr (MB == 1) {
    const unsigned u = __float_as_uint(a[0]);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    a[0] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  return a[0];
}

// How a sweep holds its operands.  bf16 and f16 rows are used as they are.  An fp32 row becomes three
// bf16 rows ("planes") that add up to it exactly, v = v0 + v1 + v2 with each part the remainder of the ones
// before it, rounded to bf16's 8 significant bits: |v1| <= 2^-8 |v|, |v2| <= 2^-17 |v|, and what is left after
// three parts of a 24-bit number is zero (numbers near the ends of the range: see split_chunk).  A product of
// two rows becomes eight products of planes; only v2 w2, below 2^-34 of a term, is left out.  (v1 w2 and v2 w1
// reach 2^-25 of a term each, half the rounding of an fp32 sum: without them the error of rows with few
// non-zero channels grew.)  The seven lower products are summed in an accumulator of their own and added to the
// sum of the leading ones v0 w0 with one fp32 addition: the matrix instruction keeps only a few bits below the
// last place of the largest number it adds, so that lower products summed into the leading ones lose by it.
// Error of a logit against 64-bit sums, in 2^-24 of its size, rms / largest, fp32 instruction -> here (4096 keys x
// 32 rows with the given number of non-zero channels at d = 128): 1 channel 0.49 / 1.05 -> 0.49 / 1.05, 2 channels
// 0.50 / 1.5 -> 0.45 / 1.1, 4 channels 0.61 / 1.9 -> 0.47 / 1.0, 128 channels of one sign 3.0 / 13 -> 0.46 / 0.9,
// of both signs 2.7 / 11 -> 1.1 / 4.6.  One channel with six products: 0.66 / 2.1; with eight in one accumulator,
// smallest first: 0.64 / 1.54.
// The fp32 matrix instruction runs at 1/16 of the bf16 rate (4096 cycles per 32x32 block at d = 128), eight
// bf16 products take 2048.  Calls measured with it -> here: 4 layers x 16K keys, 32 heads of 128, 128 rows 1092 ->
// 845 us; 4 layers x 32K keys, 32 heads of 64, 128 rows 1279 -> 874 us; 8 layers x 16K keys, heads of 64, 32 rows
// 348 -> 310 us.
template <int DT, int D, int MB>
struct Operand {
  static constexpr bool SPLIT = DT == kF32;
  static constexpr int PLANES = SPLIT ? 3 : 1;
  static constexpr int MMA_DT = SPLIT ? kBf16 : DT;            // type of the operands the matrix cores see
  using TL = Tile<2, D>;                                      // LDS layout of one plane
  static constexpr int ALIGN = Tile<elt_bytes(DT), D>::ALIGN;
  // Keys per LDS tile: 32 KiB of keys, except where a row is 128 bytes and a wave has one row block.  The column
  // sweep of 8 such waves has 101 registers, and with 16 KiB tiles (48 KiB of LDS in all) two workgroups share
  // a CU and one works while the other waits at its tile barrier: prompt-token selection, 16 layers x 64K keys 917 us
  // with 256-key tiles, 874 with 128; 16 layers x 40K, 4 heads x 64 rows 580 and 561 us.  With two row blocks a
  // wave has 151 to 160 registers and one workgroup the CU either way, so that the smaller tile only doubles
  // the barriers: prompt compression, 8 layers x 32K keys, 346 us with 256-key tiles, 363 with 128; 4 layers x 100K,
  // 4 heads x 80 rows, max 603 and 633 us, sum the same.
  static constexpr int KT = ALIGN == 256 && MB == 1 ? 128 : ALIGN;
  static constexpr int PLANE_BYTES = KT * TL::ROWB, TILE_BYTES = PLANES * PLANE_BYTES;
};

// fp32 with two row blocks per wave (d = 64): three planes of query fragments for both blocks leave no
// registers for the blocks' row normalisers in the column sweep (with them 10 spilled inside the loop, 28 before
// recompute_unless_finite made its addresses on the spot), so each wave keeps them in LDS and reads the 16 of
// a block beside its products.  4 layers x 32K keys, 4 heads x 128 rows per group: 892 -> 874 us; 2 layers, 8
// heads: 162 -> 154 us.  One row block per wave and two super-blocks measure 896 and 151 us, with twice the planes
// in the workspace.
template <int DT, int MB>
constexpr bool normalisers_in_lds() { return DT == kF32 && MB == 2; }

template <int DT, int D, int MB, int NW>
constexpr size_t score_lds_bytes(bool row_sums = false) {
  using OP = Operand<DT, D, MB>;
  return (size_t)2 * OP::TILE_BYTES + (size_t)kCsumBuffers * NW * MB * OP::KT * sizeof(float) +
         (normalisers_in_lds<DT, MB>() ? 1 : row_sums ? 3 : 0) * NW * MB * 32 * sizeof(float) +
         (OP::SPLIT ? NW * MB * 32 * sizeof(int64_t) : 0);        // row_off
}

// Bits of 2^-103.  The last bit of a smaller number lies below 2^-126, where a plane's numbers end.
constexpr unsigned kSplitMin = (127u - 103u) << 23;

// Eight fp32 values (two 16-byte chunks) as one 16-byte chunk per bf16 plane.  A number that three planes do
// not hold (between 0 and 2^-103 in size; infinite, NaN or nearer to 2^128 than to the largest bf16 number)
// makes its chunk's leading plane, and with it every score of its row, NaN: see recompute_unless_finite.  (Two
// vector instructions a number; with them the calls take 0 to 3 % longer.)
__device__ __forceinline__ void split_chunk(u32x4 lo, u32x4 hi, u32x4 (&plane)[3]) {
  unsigned least = ~0u;               // of 2 * bits - 1, which is largest for zero
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float r0 = __uint_as_float(j < 2 ? lo[2 * j] : hi[2 * j - 4]);
    float r1 = __uint_as_float(j < 2 ? lo[2 * j + 1] : hi[2 * j - 3]);
    least = min(least, min(2 * __float_as_uint(r0) - 1, 2 * __float_as_uint(r1) - 1));
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const bf16x2 b = {(__bf16)r0, (__bf16)r1};               // round to nearest even, v_cvt_pk_bf16_f32
      const unsigned u = __builtin_bit_cast(unsigned, b);
      plane[p][j] = u;
      r0 -= __uint_as_float(u << 16);
      r1 -= __uint_as_float(u & 0xffff0000u);
    }
  }
  plane[0][0] |= least < 2 * kSplitMin - 1 ? 0x7fffu : 0u;
}

// Whether a column sweep's waves take neighbouring row blocks (see `paired` below).
template <int RED, int MB, int NW>
__device__ __forceinline__ bool sweep_pairs_blocks(const ScoreArgs &A, int nblk) {
  const int blocks_per_head = (A.g.PPH != 1 ? NW * MB * 32 : A.g.packed != 0 ? 32 : A.g.Rp) / 32;
  return RED == 1 && MB == 2 && nblk == NW * MB && (blocks_per_head % 2 == 0 || A.g.packed != 0);
}

constexpr int kAskPairs = -1;

// One workgroup's sweep over a chunk of keys; bid = its index among the workgroups of its kind.
//   PASS    1: row statistics, 2: column reduction
//   RED     (pass 2) 0: sum over the rows of a head, 1: max over the rows of a head;
//           (pass 1) 0: online step on every key block, 1: fixed reference exponents with a
//           repair launch behind the sweep (see below; for sweeps of several rounds of workgroups)
//   MASKED  false: every tile of the chunk is complete and visible to every row (key <= m), the
//           loop body is straight-line code without any bounds or mask logic;
//           true: the tail of a sequence (keys that window rows may not see, end of sequence)
//   REPAIR  (pass 1, unmasked) false: the whole chunk against fixed references; every wavefront
//           leaves the segments (kAnchorTiles tiles) in which one of its sums overflowed out of
//           its pairs and lists them in A.fail;  true: segment `seg` alone with the online step,
//           its pairs merged into the ones already written; wavefronts that do not take part
//           (the segment is not on their list) only help to load the key tiles
//   MAY_SHARE  the code for row blocks that waves share (split_blocks)
//   KEYS    which of a chunk's keys: all, or for a pruned call (score_prune.hip) its sample, the others or a list.
//           Pass 2 over the others also sums the rows, in segments of kPruneSegment tiles.
//   PAIRED  what sweep_pairs_blocks says, where that is known (0, 1); kAskPairs: it is asked
template <int DT, int D, int MB, int NW, int PASS, int RED, bool MASKED, bool REPAIR = false, bool MAY_SHARE = true,
          int KEYS = kAllKeys, int PAIRED = kAskPairs, typename Args = ScoreArgs>
__device__ __forceinline__ void score_body(const Args &A, const int bid, const int seg = 0,
                                           const bool wave_takes_part = true) {
  static_assert(!REPAIR || (PASS == 1 && !MASKED && KEYS == kAllKeys), "only the row-statistics sweep is repaired");
  static_assert(KEYS == kAllKeys || (DT != kF32 && !MASKED), "pruned calls: 16-bit rows, unmasked keys");
  // What prune_plan has decided: one head a super-block or more, sums or maxima of a head's rows added up over heads, the host's
  // length, normalisers merged beforehand.
  constexpr bool PRUNED = KEYS != kAllKeys;
  if constexpr (PRUNED) __builtin_assume(A.g.PPH == 1);
  constexpr bool ROW_SUMS = PASS == 2 && KEYS == kOtherKeys;
  constexpr bool SQUARES = PASS == 1 && KEYS == kSampleKeys;             // also sums of squared terms (prune_reference_kernel)
  static_assert(KEYS != kOtherKeys || !MAY_SHARE, "with the code for shared blocks the row sums do not fit the registers");
  constexpr int ELT = elt_bytes(DT);
  using OP = Operand<DT, D, MB>;
  using TL = typename OP::TL;
  constexpr bool SPLIT = OP::SPLIT;
  constexpr int ROWB = TL::ROWB, NCS = TL::NCS, KT = OP::KT, TILE_BYTES = OP::TILE_BYTES;
  constexpr int PLANE_BYTES = OP::PLANE_BYTES, PLANES = OP::PLANES;
  constexpr int RSB = NW * MB * 32;
  constexpr int SEG_PER_WAVE = TILE_BYTES / 1024 / NW;   // 1 KiB (one wave-wide 128-bit load) segments
  constexpr int RPS = 1024 / ROWB;                        // tile rows per segment
  constexpr int SPLIT_CHUNKS = KT * (D / 8) / (NW * 64);   // fp32: groups of 8 channels a thread splits per tile
  static_assert(TILE_BYTES % (1024 * NW) == 0, "tile load must divide evenly over the waves");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  unsigned char *kbuf = smem;
  float *csum = reinterpret_cast<float *>(smem + 2 * TILE_BYTES);

  const Dims &d = A.d;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  int unit, s, chunk, key_begin, key_end;
  if (MASKED) {
    const int units = d.L * d.Hkv * A.g.RS;
    unit = bid % units;
    s = bid / units;
    chunk = A.g.n_fast_chunks + s;
  } else if constexpr (KEYS == kListedKeys) {
    const int per_item = A.one_row != 0 ? d.L * d.Hkv * A.g.RS : A.g.RS;
    const int2 item = A.items[bid / per_item];
    const int layer_seq = item.x / d.Hkv;
    s = layer_seq % d.S;
    unit = (layer_seq / d.S * d.Hkv + item.x % d.Hkv) * A.g.RS + bid % per_item;
    chunk = 0;
    key_begin = item.y;                                   // places in the row's list, not keys
    key_end = min(item.y + A.item_keys, A.rows[item.x].listed);
  } else if constexpr (KEYS != kAllKeys) {
    const PruneChunk c = prune_chunk(A, bid);
    if (c.unit < 0) return;
    unit = c.unit;
    s = c.s;
    chunk = c.chunk;
    key_begin = c.key_begin;
    key_end = c.key_end;
  } else {
    // 1-D grid.  Workgroups go to the 8 XCDs round-robin by their linear id and each XCD has its
    // own L2, so the RS row super-blocks that sweep the SAME keys of a (layer, head) get ids 8
    // apart: same XCD, dispatched together, and the keys come from HBM once instead of RS times.
    const int per_group = 8 * A.g.RS;
    const int grp = bid / per_group, within = bid % per_group;
    const int item = grp * 8 + (within & 7);            // (layer, head, chunk), chunk fastest
    if (item >= A.g.n_fast_chunks * d.L * d.Hkv) return;
    chunk = item % A.g.n_fast_chunks;
    unit = (item / A.g.n_fast_chunks) * A.g.RS + (within >> 3);
    s = 0;
    while (s + 1 < d.S && A.t.cc[s + 1] <= chunk) ++s;
  }
  const int n_host = A.t.cu[s + 1] - A.t.cu[s];          // row stride of the score layouts
  const int n_s = PRUNED ? n_host : live_len(d, A.t, s);  // tokens that exist (device-side count honoured)
  const int tail0 = PRUNED ? A.t.tail0[s] : live_tail0(d, A.t, s, n_s, OP::ALIGN);
  if (MASKED) {
    key_begin = tail0;
    key_end = n_s;
  } else if constexpr (KEYS == kAllKeys) {
    const int kc = chunk_keys(A.g, tail0);
    key_begin = (chunk - A.t.cc[s]) * kc;
    key_end = min(tail0, key_begin + kc);                 // a chunk past a shorter live prompt is empty
  }
  const int rs = unit % A.g.RS;
  const int g = (unit / A.g.RS) % d.Hkv;
  const int layer = unit / (A.g.RS * d.Hkv);
  const int m = n_s - d.w;
  const int chunk_tiles = (key_end - key_begin + KT - 1) / KT;
  int step_log = 0;                                       // the sample: every 2^step_log-th tile of a chunk
  if constexpr (KEYS == kSampleKeys || KEYS == kOtherKeys) step_log = prune_step(A.chunk_of[s]);
  const int sampled = (chunk_tiles + (1 << step_log) - 1) >> step_log;
  const int ntiles = KEYS == kSampleKeys ? sampled : KEYS == kOtherKeys ? chunk_tiles - sampled : chunk_tiles;
  // a tile's first key (place in the list)
  auto tile_key = [&](int tile) {
    if constexpr (KEYS == kSampleKeys) tile <<= step_log;
    if constexpr (KEYS == kOtherKeys) tile = other_tile(tile, step_log);
    return key_begin + tile * KT;
  };
  const float c2 = d.sm_scale * 1.4426950408889634f;

  // Which of the super-block's row blocks this wave computes (see split_blocks): `nact` of its own, row blocks 0 .. nact-1 of
  // the wave, and, if `sharing`, every per-th 32-key block (the ones of number `phase` modulo `per`, counted from the
  // chunk's first) of the block that is its row block number nact.
  int first_block;
  const int nblk = super_block_blocks(d, A.g, rs, &first_block);
  const BlockSplit split = split_blocks(nblk, MAY_SHARE && A.share != 0);
  const int share_w0 = split.full % NW;                   // waves share_w0 .. share_w0 + 3 share
  const int nact = wave_takes_part ? __builtin_amdgcn_readfirstlane(max(0, min(MB, (split.full - wv + NW - 1) / NW))) : 0;
  const bool sharing = MAY_SHARE && wave_takes_part && split.per > 1 && wv >= share_w0 && wv < share_w0 + 4;
  const int per = MAY_SHARE ? split.per : 1, phase = (wv - share_w0) & (per - 1);
  // Maximum over the query rows, full super-block, an even number of blocks per head (or heads that are combined by
  // maximum as well): the wave
  // takes two neighbouring blocks (2 wv and 2 wv + 1, the same head) instead, merges their
  // column maxima in registers and hands one value per key to the flush, not two.  A maximum
  // does not depend on the order, so the result is the same bit for bit.
  const int blocks_per_head = (A.g.PPH != 1 ? RSB : A.g.packed != 0 ? 32 : A.g.Rp) / 32;
  const bool paired = PASS == 2 && !MASKED && (PAIRED == kAskPairs ? sweep_pairs_blocks<RED, MB, NW>(A, nblk) : PAIRED == 1);
  // ... and where heads are combined by maximum too, a wave merges whatever blocks it has.
  const bool merged = paired || (PASS == 2 && RED == 1 && !MASKED && !PRUNED && d.head_max != 0);
  auto block_of = [&](int rb) { return paired ? wv * MB + rb : block_of_slot(split, rb * NW + wv); };
  // row r32 of the wave's row block rb: its head and observation row; false for padding
  auto row_at = [&](int rb, int r32, int &hh, int &i) { return decode_row(d, A.g, rs, block_of(rb) * 32 + r32, &hh, &i); };

  // ---- K tile staging: each wave issues SEG_PER_WAVE wave-wide 128-bit loads that land in LDS
  // at lds_base + lane*16; the lane picks the global chunk that belongs in its (row, slot).
  const char *kbase = A.k + ((int64_t)layer * d.kv_sl + (int64_t)A.t.cu[s] * d.kv_st + (int64_t)g * d.kv_sh) * ELT;
  const int64_t tokb = d.kv_st * ELT;
  const int st_row = (lane * 16) / ROWB, st_slot = ((lane * 16) % ROWB) / 16;
  // unmasked sweep: the lane's byte offset inside a tile never changes, only the (uniform) tile
  // base moves, so the loads use a scalar base plus a 32-bit lane offset; where registers are short, one offset for all
  // segments (d = 128, 4 layers x 60K, a caller's normalisers: 244.9 us with an offset a segment, 247.8 with one)
  static_assert(SPLIT || NW * RPS / TL::RPB % (TL::SWZ + 1) == 0, "a wave's segments of a tile are swizzled alike");
  constexpr int OFFSETS = KEYS == kAllKeys ? SEG_PER_WAVE : 1;
  uint32_t loff[OFFSETS];
#pragma unroll
  for (int it = 0; it < OFFSETS; ++it) {
    const int r_ = (it * NW + wv) * RPS + st_row;
    loff[it] = (KEYS == kListedKeys ? 0u : (uint32_t)r_ * (uint32_t)tokb) + (uint32_t)((st_slot ^ TL::swizzle(r_)) * 16);
  }
  // listed keys: the lane's keys of the next tile to be loaded, requested one tile ahead
  const int32_t *list = nullptr;
  int next_key[SEG_PER_WAVE];
  auto request_keys = [&](int tile) {
    if constexpr (KEYS == kListedKeys) {
#pragma unroll
      for (int it = 0; it < SEG_PER_WAVE; ++it)      // places past the end repeat the last key; they are not written
        next_key[it] = list[min(key_begin + tile * KT + (it * NW + wv) * RPS + st_row, key_end - 1)];
    }
  };
  if constexpr (KEYS == kListedKeys) {
    list = A.list;
    if (A.one_row == 0) list += (int64_t)layer * d.Hkv * d.T + (int64_t)d.Hkv * A.t.cu[s] + (int64_t)g * n_host;
    request_keys(0);
  }
#define SPECKV_LOAD_TILE(tile_, buf_)                                                         \
  {                                                                                           \
    const int k0_ = tile_key(tile_);                                                          \
    const char *tbase_ = kbase + (int64_t)k0_ * tokb;                                         \
    _Pragma("unroll") for (int it = 0; it < SEG_PER_WAVE; ++it) {                             \
      const int seg_ = it * NW + wv;                                                          \
      const char *src_;                                                                       \
      if (MASKED) {                                                                           \
        const int r_ = seg_ * RPS + st_row;                                                   \
        /* rows past the end of the sequence re-read its last key; they are masked later */   \
        src_ = kbase + (int64_t)min(k0_ + r_, n_s - 1) * tokb + (st_slot ^ TL::swizzle(r_)) * 16; \
      } else if (KEYS == kListedKeys) {                                                       \
        src_ = kbase + (int64_t)next_key[it] * tokb + loff[0];                                \
      } else {                                                                                \
        src_ = OFFSETS > 1 ? tbase_ + loff[it % OFFSETS]                                      \
                           : tbase_ + (int64_t)(it * NW * RPS) * tokb + loff[0];              \
      }                                                                                       \
      __builtin_amdgcn_global_load_lds(                                                       \
          (const __attribute__((address_space(1))) void *)src_,                               \
          (__attribute__((address_space(3))) void *)(kbuf + (buf_) * TILE_BYTES + seg_ * 1024), 16, 0, 0); \
    }                                                                                         \
    request_keys((tile_) + 1);                                                                \
  }
  // fp32: the tile passes through registers, split into its planes on the way.  SPECKV_FETCH_TILE
  // requests it, SPECKV_STORE_TILE (before the barrier that hands the tile over) splits and stores it.
  u32x4 raw[SPLIT ? SPLIT_CHUNKS : 1][2];
#define SPECKV_FETCH_TILE(tile_)                                                              \
  _Pragma("unroll") for (int it = 0; it < SPLIT_CHUNKS; ++it) {                               \
    const int e_ = it * NW * 64 + tid, r_ = e_ / (D / 8), c_ = e_ % (D / 8);                  \
    const int k_ = key_begin + (tile_) * KT + r_;                                             \
    /* rows past the end of the sequence re-read its last key; they are masked later */       \
    const char *src_ = kbase + (int64_t)(MASKED ? min(k_, n_s - 1) : k_) * tokb + c_ * 32;    \
    raw[it][0] = *reinterpret_cast<const u32x4 *>(src_);                                      \
    raw[it][1] = *reinterpret_cast<const u32x4 *>(src_ + 16);                                 \
  }
#define SPECKV_STORE_TILE(buf_)                                                               \
  _Pragma("unroll") for (int it = 0; it < SPLIT_CHUNKS; ++it) {                               \
    const int e_ = it * NW * 64 + tid, r_ = e_ / (D / 8), c_ = e_ % (D / 8);                  \
    u32x4 part_[3];                                                                           \
    split_chunk(raw[it][0], raw[it][1], part_);                                               \
    _Pragma("unroll") for (int p = 0; p < 3; ++p)                                             \
      *reinterpret_cast<u32x4 *>(kbuf + (buf_) * TILE_BYTES + p * PLANE_BYTES + r_ * ROWB +   \
                                 ((c_ ^ TL::swizzle(r_)) * 16)) = part_[p];                   \
  }
  // Column sweep, normalisers merged here (in the order of merge_pairs): one thread (or RSB_SLICES of them) per row.
  // The first entries are requested before everything else: loads return in the order they were issued.
  constexpr int RSB_SLICES = NW * 64 / RSB, BATCH = kMergeFirst / RSB_SLICES;
  static_assert(RSB_SLICES == merge_slices(MB), "threads per row");
  const int norm_row = tid % RSB, norm_slice = tid / RSB, n_entries = A.t.cc[s + 1] - A.t.cc[s] + 1;
  const float2 *pairs_of_row = A.part + (int64_t)unit * A.g.n_chunks * RSB + norm_row;
  auto entry = [&](int e) {
    return e < n_entries ? pairs_of_row[(int64_t)(e == 0 ? A.g.n_fast_chunks + s : A.t.cc[s] + e - 1) * RSB] : make_float2(kNegBig, 0.f);
  };
  float2 first_pairs[BATCH];
  if (PASS == 2 && !PRUNED && A.norm_from == kNormPairs) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u) first_pairs[u] = entry(norm_slice + u * RSB_SLICES);
  }
  // the first tile is requested before the other loads, so that its latency overlaps
  // with the Q fragment and row normaliser loads below
  const int first_tile = REPAIR ? 1 + seg * kAnchorTiles : 0;
  if (ntiles > first_tile) {
    if constexpr (SPLIT) SPECKV_FETCH_TILE(first_tile)
    else SPECKV_LOAD_TILE(first_tile, 0)
  }

  // ---- Q fragments of this wave's row blocks, resident for the whole sweep
  u32x4 qf[MB][PLANES * NCS];
  // fp32: where the wave's query rows lie (-1: padding), for recompute_unless_finite, which would keep everything that goes
  // into these offsets in scalar registers (with rows packed, more than there are)
  int64_t *row_off = reinterpret_cast<int64_t *>(csum + (size_t)kCsumBuffers * NW * MB * KT + (normalisers_in_lds<DT, MB>() ? RSB : 0));
#pragma unroll
  for (int rb = 0; rb < MB; ++rb) {
    int hh, i;
    const bool valid = row_at(rb, l32, hh, i);
    const int64_t off = ((int64_t)layer * d.q_sl + (int64_t)s * d.q_ss + (int64_t)(valid ? i : 0) * d.q_sr +
                         (int64_t)(g * d.G + (valid ? hh : 0)) * d.q_sh) * ELT;
    const char *qp = A.q + off + half * 8 * ELT;                     // chunk 0 of the lane's share of query row l32
    if (SPLIT && half == 0) row_off[(rb * NW + wv) * 32 + l32] = valid ? off : -1;
#pragma unroll
    for (int cs = 0; cs < NCS; ++cs) {
      if constexpr (SPLIT) {
        u32x4 part[3];
        split_chunk(valid ? *reinterpret_cast<const u32x4 *>(qp + cs * 64) : (u32x4)(0u),
                    valid ? *reinterpret_cast<const u32x4 *>(qp + cs * 64 + 16) : (u32x4)(0u), part);
#pragma unroll
        for (int p = 0; p < 3; ++p) qf[rb][p * NCS + cs] = part[p];
      } else {
        qf[rb][cs] = valid ? *reinterpret_cast<const u32x4 *>(qp + cs * 32) : (u32x4)(0u);
      }
    }
  }

  // ---- per-pass row state
  float mrun[MB], lrun[MB];          // pass 1: lane = one query row per row block
  float qrun[SQUARES ? MB : 1];
  // Pass 2 with row sums: what a wave knows of its rows between segments lies in LDS, [NW][MB][32] each: the row's negated
  // reference, its sum, and the sum over the sample and the tail.  A lane keeps the row own_slot() for this:
  // row l32 % 16, counted as in nlse, of row block l32 / 16 (MB = 1: lanes from 16 on repeat the others).
  float *own_ref = csum + (size_t)kCsumBuffers * NW * MB * KT, *own_sum = own_ref + RSB, *own_first = own_sum + RSB;
  auto own_slot = [&]() {
    int l = lane;
    asm volatile("" : "+v"(l));        // made where it is used, not kept in a register
    return wv * MB * 32 + (MB == 2 ? l & 16 : 0) * 2 + 8 * ((l & 15) >> 2) + 4 * (l >> 5) + (l & 3);
  };
  constexpr bool LSE_LDS = PASS == 2 && normalisers_in_lds<DT, MB>();
  float nlse[LSE_LDS ? 1 : MB][16];  // pass 2: lane = 16 rows per row block
  float *lds_lse = csum + (size_t)kCsumBuffers * NW * MB * KT;                     // ... or in LDS, [RSB]
  // masked sweep: last key each row may see (window row i sees keys <= m + i, a lookahead row the whole prompt),
  // computed once instead of per score
  int last1[MB];                     // pass 1: the lane's own query row per row block
  int last2[MASKED ? MB : 1][16];    // pass 2: the 16 rows a lane holds per row block
  if (PASS == 1) {
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
      mrun[rb] = kNegBig;
      lrun[rb] = 0.f;
      if constexpr (SQUARES) qrun[rb] = 0.f;
      if (MASKED) {
        int hh, io;
        (void)row_at(rb, l32, hh, io);
        last1[rb] = io < d.w ? m + io : n_s - 1;
      }
    }
  } else {
    // The normalisers of the workgroup's rows go through LDS.  Merging
    // the chunks' pairs here instead of in a kernel between the sweeps saves that launch (see launch_score).
    float2 *pairs = reinterpret_cast<float2 *>(csum);                                  // [RSB_SLICES][RSB]
    float *norm = LSE_LDS ? lds_lse : csum + 2 * NW * 64;                             // [RSB]
    int *row_last = reinterpret_cast<int *>(csum + 2 * NW * 64 + RSB);                // [RSB], masked: last key a row may see
    static_assert((size_t)kCsumBuffers * NW * MB * KT >= (size_t)2 * NW * 64 + 2 * RSB, "scratch of the merge");
    const int lr = norm_row, slice = norm_slice;
    int hh, io;
    const bool valid = decode_row(d, A.g, rs, lr, &hh, &io);
    float v = 0.f;                                        // log2 normaliser of row lr
    if (!PRUNED && A.norm_from == kNormPairs) {
      float top = kNegBig, sum = 0.f;
      merge_pairs(top, sum, first_pairs);
      for (int e0 = slice + BATCH * RSB_SLICES; e0 < n_entries; e0 += RSB_SLICES * kMergeNext) {
        float2 in[kMergeNext];
#pragma unroll
        for (int u = 0; u < kMergeNext; ++u) in[u] = entry(e0 + u * RSB_SLICES);
        merge_pairs(top, sum, in);
      }
      if constexpr (RSB_SLICES > 1) {
        pairs[slice * RSB + lr] = make_float2(top, sum);
        __syncthreads();
        if (slice == 0) {
          float2 in[RSB_SLICES - 1];
#pragma unroll
          for (int u = 1; u < RSB_SLICES; ++u) in[u - 1] = pairs[u * RSB + lr];
          merge_pairs(top, sum, in);
        }
      }
      v = top + log2f(sum);
    } else if (!PRUNED && A.norm_from == kNormCaller) {
      if (valid) v = A.lse_in[(((int64_t)layer * d.S + s) * d.R + io) * d.Hq + g * d.G + hh] * 1.4426950408889634f;
    } else {
      v = A.lse[(((int64_t)layer * d.Hkv + g) * d.S + s) * ((int64_t)A.g.RS * RSB) + rs * RSB + lr];
    }
    if (slice == 0) {
      v = -v;
      if constexpr (ROW_SUMS) v = ceilf(v * kPruneGrain) / kPruneGrain - kPruneShift;      // see kPruneShift
      if (!PRUNED && d.weight_rows && valid && io < d.w) v += log2f((float)(io + 1) / (float)d.w);     // row weight folded in
      norm[lr] = valid ? v : -INFINITY;                   // padded rows contribute 2^-inf = 0
      if (MASKED) row_last[lr] = io < d.w ? m + io : n_s - 1;
    }
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < MB; ++rb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = block_of(rb) * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
        if constexpr (!LSE_LDS) nlse[rb][i] = norm[r];
        if constexpr (MASKED) last2[rb][i] = row_last[r];
      }
    if constexpr (ROW_SUMS) {
      const int own = own_slot();
      own_ref[own] = norm[block_of((own >> 5) & (MB - 1)) * 32 + (own & 31)];
      own_sum[own] = 0.f;
      const int own_row = block_of((own >> 5) & (MB - 1)) * 32 + (own & 31);
      own_first[own] = __builtin_amdgcn_exp2f(-kPruneShift) *
                       A.row_extra[(((int64_t)layer * d.Hkv + g) * d.S + s) * ((int64_t)A.g.RS * RSB) + rs * RSB + own_row];
    }
    __syncthreads();
    // slots of skipped blocks must read as zero when the tile partials are merged
    if (MASKED || split.full < NW || per > 1 || (RED == 1 && nblk != NW * MB))
      for (int x = tid; x < kCsumBuffers * NW * MB * KT; x += NW * 64) csum[x] = 0.f;
  }
  // the negated normalisers of the lane's 16 rows in row block rb
  auto load_lse = [&](int rb, float (&nl)[16]) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if constexpr (LSE_LDS) nl[i] = lds_lse[block_of(rb) * 32 + 8 * (i >> 2) + 4 * half + (i & 3)];
      else nl[i] = nlse[rb][i];
    }
  };

  // per-lane LDS offsets of the fragment chunks of key row l32 (same for every 32-key block)
  uint32_t foff[NCS];
#pragma unroll
  for (int cs = 0; cs < NCS; ++cs) foff[cs] = l32 * ROWB + (((2 * cs + half) ^ TL::swizzle(l32)) * 16);
  // chunk cs of key block kb_ in plane p_ (fp32: the smallest plane comes first)
#define SPECKV_FRAG(buf_, p_, kb_, cs_) \
  (*reinterpret_cast<const u32x4 *>(kbuf + (buf_) * TILE_BYTES + (p_) * PLANE_BYTES + (kb_) * 32 * ROWB + foff[cs_]))
#define SPECKV_LOAD_BFRAG(dst_, buf_, kb_) \
  _Pragma("unroll") for (int cs = 0; cs < NCS; ++cs) dst_[cs] = SPECKV_FRAG(buf_, PLANES - 1, kb_, cs);
  // adds the product of key chunk bf (chunk cs of some plane) and plane qp of row block rb to the scores x
  auto add_product = [&](f32x16 &x, const u32x4 &bf, int qp, int rb, int cs) {
    x = PASS == 1 ? mma_chunk<OP::MMA_DT>(bf, qf[rb][qp * NCS + cs], x) : mma_chunk<OP::MMA_DT>(qf[rb][qp * NCS + cs], bf, x);
  };
  // fp32: the same for every plane of the rows that goes with key plane kp, the leading pair left out
  auto add_lower_products = [&](f32x16 &x, const u32x4 &bf, int kp, int rb, int cs) {
#pragma unroll
    for (int qp = kp == PLANES - 1 ? PLANES - 2 : PLANES - 1; qp >= (kp == 0 ? 1 : 0); --qp) add_product(x, bf, qp, rb, cs);
  };
  // Numbers that three planes do not hold (see split_chunk) and overflowing sums leave NaN or infinity where
  // fp32 products might not: a block with a score that is not finite is computed again from memory with the fp32
  // instruction (one multiply-add per score to look for it, beside 32 or 64 MFMAs).  key0: the block's first key.
  auto recompute_unless_finite = [&](f32x16 &x, int rb, int key0) {
    if constexpr (SPLIT) {
      float probe = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) probe = fmaf(x[i], 0.f, probe);       // NaN if any score is infinite or NaN
      if (__builtin_amdgcn_ballot_w64(!(probe == 0.f)) != 0) {
        int r32 = l32;
        asm volatile("" : "+v"(r32));  // the addresses are made here, not kept in registers through the sweep
        const int64_t off = row_off[(rb * NW + wv) * 32 + r32];
        const bool valid = off >= 0;
        const char *qp = A.q + (valid ? off : 0) + half * (D / 2) * ELT;
        const char *kp = kbase + (int64_t)min(key0 + r32, n_s - 1) * tokb + half * (D / 2) * ELT;
        x = (f32x16){0};
#pragma unroll 1
        for (int cs = 0; cs < D / 8; ++cs) {
          const u32x4 kc = *reinterpret_cast<const u32x4 *>(kp + cs * 16);
          const u32x4 qc = valid ? *reinterpret_cast<const u32x4 *>(qp + cs * 16) : (u32x4)(0u);
          x = PASS == 1 ? mma_chunk<kF32>(kc, qc, x) : mma_chunk<kF32>(qc, kc, x);
        }
      }
    }
  };

  // cross-wave merge of the column partials of one finished tile (pass 2)
  float *plane_out = nullptr;
  if (PASS == 2)
    plane_out = A.planes + ((int64_t)rs * d.L + layer) * d.Hkv * d.T + (int64_t)d.Hkv * A.t.cu[s] + (int64_t)g * n_host;
  const bool head_max = !PRUNED && d.head_max != 0;
  const int slots_per_head = paired && blocks_per_head > 1 ? blocks_per_head / 2 : blocks_per_head;
  // sum, unmasked: a wave with a block of its own keeps the column sums of the one it shares in a second slot
  const bool share_slots = per > 1 && split.full >= NW;
#define SPECKV_FLUSH_TILE(tile_)                                                             \
  if (tid < KT) {                                                                            \
    const int key_ = tile_key(tile_) + tid;                                                  \
    if (key_ < key_end) {                                                                    \
      const float *cp_ = csum + (size_t)((tile_) % kCsumBuffers) * NW * MB * KT + tid;                  \
      float total_ = 0.f;                                                                    \
      if (RED == 0) {                                                                        \
        _Pragma("unroll") for (int w2 = 0; w2 < NW; ++w2) total_ += cp_[w2 * KT];            \
        if (MB == 2 && share_slots) {                                                        \
          _Pragma("unroll") for (int w2 = 0; w2 < 4; ++w2) total_ += cp_[(NW + share_w0 + w2) * KT]; \
        }                                                                                    \
      } else if (head_max) {                                                                 \
        /* one slot per wave (masked: per block), and those of a shared block */             \
        _Pragma("unroll") for (int b2 = 0; b2 < NW * MB; ++b2)                               \
          if (MASKED || b2 < NW || share_slots) total_ = fmaxf(total_, cp_[b2 * KT]);        \
      } else {                                                                               \
        /* per block (or block pair) maxima: max within a head, then heads added */          \
        float cur_ = 0.f;                                                                    \
        int in_head_ = 0;                                                                    \
        _Pragma("unroll") for (int b2 = 0; b2 < NW * MB; ++b2) {                             \
          if (paired && b2 >= NW) break;                                                     \
          if (in_head_ == slots_per_head) {                                                  \
            total_ += cur_;                                                                  \
            cur_ = 0.f;                                                                      \
            in_head_ = 0;                                                                    \
          }                                                                                  \
          cur_ = fmaxf(cur_, cp_[b2 * KT]);                                                  \
          ++in_head_;                                                                        \
        }                                                                                    \
        total_ += cur_;                                                                      \
      }                                                                                      \
      if constexpr (KEYS == kListedKeys) plane_out[list[key_]] = total_;                     \
      else plane_out[key_] = total_;                                                         \
    }                                                                                        \
  }

  if constexpr (SPLIT) {
    if (ntiles > first_tile) SPECKV_STORE_TILE(0)
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // Row statistics of an unmasked chunk.  The chunk's first tile gives each row its reference exponent
  // (its maximum, found by the online step); every later block only adds 2^(score - reference) to the
  // row's sum: no maximum search, no rescaling.  After a segment (kAnchorTiles tiles, counted from the
  // second tile) in which the sum has grown by 2^kAnchorGrowth or more its exponent moves into the
  // reference, which keeps the sum between 2^-shift and 2^(kAnchorGrowth-shift) with shift = 100 -
  // ceil(log2(keys per chunk)): a term that underflows (below 2^-126) beside it is less than 2^-25 /
  // (keys per chunk) of the sum, so all of a chunk's keys together stay below fp32 resolution, and a
  // score may exceed everything the row has seen before its segment by 126 + shift - kAnchorGrowth
  // binary orders (143 nats for 32K-key chunks) before the sum overflows.  An overflow is sticky
  // (infinity stays infinity), so it is looked for once per segment (kAnchorLimit; also NaN): the
  // wavefront then goes back to the pairs it had before the segment, notes the segment on its list in
  // A.fail and goes on; the repair launch behind this one (REPAIR) sweeps the noted segments with
  // the online step on every block and adds their pairs.  (The same second sweep as code inside
  // this kernel, inlined, outlined or as a compact loop, costs the first sweep the 3 % it is
  // there to gain.)
  constexpr bool kAnchored = PASS == 1 && !MASKED && !REPAIR && RED == 1;
  const int anchor_shift = 100 - (32 - __builtin_clz((unsigned)max(A.g.KC, 2) - 1u));
  float l_before[MB];                 // the sums at the start of the current segment
  int n_failed = 0;
  int listed[kFailListed + 1];        // uniform: lives in scalar registers
  if (kAnchored || ROW_SUMS) {
#pragma unroll
    for (int i = 0; i <= kFailListed; ++i) listed[i] = 0;
  }
  // The segment is over (every block of it is in the sums): keep it or leave it to the repair launch.
  // Usually the sums are still small and nothing but this comparison happens (2.5 % on the sweep
  // against moving the exponent after every segment).
  const float grown = __builtin_ldexpf(1.f, kAnchorGrowth - anchor_shift);
  // new_reference(rb, r): a reference for a row that has none yet (every score it has seen is -infinity, so that
  // r is below everything and the first segment with a finite score overflows); without it every segment
  // of the chunk would overflow.
  auto end_segment = [&](int segment, auto new_reference) {
    bool look = false;
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) look |= !(lrun[rb] < grown);
    if (__builtin_amdgcn_ballot_w64(look) != 0 || n_failed > kFailListed) {           // seldom
      bool out_of_range = false;
#pragma unroll
      for (int rb = 0; rb < MB; ++rb) out_of_range |= !(lrun[rb] < kAnchorLimit);
      // The decision is the wavefront's own (its rows are nobody else's): no barrier, no exchange.
      // (A full list: every later segment is left to the repair as well, overflowed or not.)
      if (__builtin_amdgcn_ballot_w64(out_of_range) != 0 || n_failed > kFailListed) {
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) {
          lrun[rb] = l_before[rb];
          if (!(l_before[rb] > 0.f)) mrun[rb] = new_reference(rb, mrun[rb]);
        }
#pragma unroll
        for (int i = 0; i <= kFailListed; ++i)
          if (i == n_failed) listed[i] = segment;
        ++n_failed;
      } else {                                         // the sum's exponent above 2^-shift goes into the reference
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) {
          const int up = lrun[rb] > 0.f ? max(__builtin_amdgcn_frexp_expf(lrun[rb]) + anchor_shift, 0) : 0;
          lrun[rb] = __builtin_ldexpf(lrun[rb], -up);
          mrun[rb] += (float)up;
        }
      }
    }
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) l_before[rb] = lrun[rb];
  };

  if constexpr (MASKED) {
    auto takes = [&](int rb, int kb) { return rb < nact || (sharing && rb == nact && (kb & (per - 1)) == phase); };
    for (int tile = 0; tile < ntiles; ++tile) {
      const int buf = tile & 1;
      if (tile + 1 < ntiles) {
        if constexpr (SPLIT) SPECKV_FETCH_TILE(tile + 1)
        else SPECKV_LOAD_TILE(tile + 1, buf ^ 1)
      }
      if (PASS == 2 && tile > 0) SPECKV_FLUSH_TILE(tile - 1)
      const int tk0 = key_begin + tile * KT;
      // Tail tiles: keys above m are hidden from some window rows; keys >= n_s do not exist.
#pragma unroll 1
      for (int kb = 0; kb < KT / 32; ++kb) {
        if (tk0 + kb * 32 >= key_end) break;               // nothing but padding from here on
        // scores of row block rb against key block kb
        u32x4 bf[NCS];
        if constexpr (!SPLIT) SPECKV_LOAD_BFRAG(bf, buf, kb)
        auto scores = [&](int rb) {
          f32x16 acc = {0}, low = {0};
          if constexpr (SPLIT) {
#pragma unroll
            for (int kp = PLANES - 1; kp >= 0; --kp) {
#pragma unroll
              for (int cs = 0; cs < NCS; ++cs) bf[cs] = SPECKV_FRAG(buf, kp, kb, cs);
#pragma unroll
              for (int cs = 0; cs < NCS; ++cs) add_lower_products(low, bf[cs], kp, rb, cs);
            }
          }
#pragma unroll
          for (int cs = 0; cs < NCS; ++cs) add_product(acc, bf[cs], 0, rb, cs);
          if constexpr (SPLIT) {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] += low[i];
          }
          recompute_unless_finite(acc, rb, tk0 + kb * 32);
          return acc;
        };
        if (PASS == 1) {
#pragma unroll
          for (int rb = 0; rb < MB; ++rb) {
            if (!takes(rb, tile * (KT / 32) + kb)) continue;
            f32x16 acc = scores(rb);
            // lane: query row (wv*MB+rb)*32 + l32; keys tk0 + kb*32 + 8*(i/4) + 4*half + i%4
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const int key = tk0 + kb * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
              if (key > last1[rb]) acc[i] = -INFINITY;
            }
            float tmax = acc[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, acc[i]);
            const float mnew = fmaxf(mrun[rb], tmax * c2);
            const float scale = __builtin_amdgcn_exp2f(mrun[rb] - mnew);
            const float nm = -mnew;
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(fmaf(acc[i], c2, nm));
            lrun[rb] = fmaf(lrun[rb], scale, sum);
            mrun[rb] = mnew;
          }
        } else {
          float colsum = 0.f;
          const int key = tk0 + kb * 32 + l32;
          float *dst = csum + (size_t)(tile % kCsumBuffers) * NW * MB * KT + kb * 32 + l32;
#pragma unroll
          for (int rb = 0; rb < MB; ++rb) {
            if (!takes(rb, tile * (KT / 32) + kb)) continue;
            f32x16 acc = scores(rb);
            // lane: key tk0 + kb*32 + l32; rows (wv*MB+rb)*32 + 8*(i/4) + 4*half + i%4
            float p[16], nl[16];
            load_lse(rb, nl);
#pragma unroll
            for (int i = 0; i < 16; ++i) p[i] = __builtin_amdgcn_exp2f(fmaf(acc[i], c2, nl[i]));
#pragma unroll
            for (int i = 0; i < 16; ++i)
              if (key > last2[rb][i]) p[i] = 0.f;
            if (RED == 0) {
#pragma unroll
              for (int i = 0; i < 16; ++i) colsum += p[i];
            } else {
              float cm = 0.f;
#pragma unroll
              for (int i = 0; i < 16; ++i) cm = fmaxf(cm, p[i]);
              dst[(rb * NW + wv) * KT] = max_other_half(cm);
            }
          }
          if (RED == 0) dst[wv * KT] = add_other_half(colsum);
        }
      }
      if constexpr (SPLIT) {
        if (tile + 1 < ntiles) SPECKV_STORE_TILE(buf ^ 1)
      }
      // the next tile must have landed in LDS, and every wave must be done with this one
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
    if (PASS == 2 && ntiles > 0) SPECKV_FLUSH_TILE(ntiles - 1)
  } else {
    // The unmasked sweep is software-pipelined in every wave (but see PIPELINED).  A unit is one 32-key x 32-row block: while
    // its chain of MFMAs runs (a chain on one accumulator issues at the full rate), the wave turns the
    // block of the unit before it into probabilities, so that each wave by itself keeps both pipes
    // busy.  (Without this the two waves of a SIMD, released together by the tile barrier, do
    // their matrix work together and then their vector work together.)  The last unit of a tile is
    // finished beside the first MFMAs of the next tile, where it also covers the latency of that tile's
    // first fragment reads.  The key fragments are reloaded in place, each as soon as its last MFMA of the
    // current key block is issued.
    // What bounds a 32x32 block at d = 128: an MFMA holds the vector issue port for about 8 cycles, an
    // exp2 8, a multiply-add or add 4, hence 8*8 + 16*(8 + 4 + 4) = 324 cycles of issue for 256 cycles of
    // matrix work.
    // Measured on 32 layers x 128K keys, 512 rows per KV head: 4.35 -> 4.07 ms (row statistics), 4.21 ->
    // 4.15 ms (column sums), 458 -> 416 and 436 -> 432 cycles per 32x32 block; the clock falls with the
    // stalls (power limit), so the time gains less than the cycles where calls follow each other.
    // Units of both row blocks at once (the next key block's 16 MFMAs beside 96 vector
    // instructions), 16x16x32 MFMAs and explicit instruction ratios measure the same or worse.
    // NACT = number of active row blocks of this wave (nact): the whole sweep is one straight piece of
    // code per number, so that the open block and the row state never move between registers
    // (1.7 % on the row statistics).
    constexpr int KB = KT / 32;
    // The column sweep of 8 waves x 1 row block at d = 128 is better off without: pipelined it needs 177 registers,
    // so one workgroup has the CU; a unit's block finished right behind its MFMAs leaves 123 and two workgroups
    // (80 KiB of LDS each), whose four waves a SIMD overlap by themselves.  32 layers x 16K keys, 4 heads x 64
    // rows 729 -> 709 us, 28 layers x 60K, 7 x 32 rows 1087 -> 1051 us, 5 x 32 rows 1162 -> 1114 us (before any
    // pipelining 727, 1085, 1140 us).
    constexpr bool PIPELINED = !(PASS == 2 && MB == 1 && NW == 8 && D == 128 && !SPLIT);
    // SHARED: the wave also has its part of row block NACT, done at the end of a tile: usually one 32-key block of four,
    // beside which the other wave of the SIMD has its own work.
    auto sweep = [&](auto nact_c, auto shared_c) {
      constexpr int NACT = decltype(nact_c)::value;
      constexpr bool SHARED = decltype(shared_c)::value;
      f32x16 acc[2];                   // blocks of the units: the open one in one, the next one in the other
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[1][i] = -INFINITY;    // nothing open: probabilities of 2^-inf = 0
      bool open = false;               // a unit waits in acc[1] (fp32: only then are its scores looked at)
      float top_before = 0.f;          // pass 1, fp32: largest score of the unit before a segment's last look
      float shared_top = 0.f;          // pass 1: largest score of the last unit of the shared block
      float colsum = 0.f;              // pass 2: the lane's key, over the row blocks of the current key block
      float row_sum[ROW_SUMS ? MB : 1][16];                 // over the keys that the lane has seen in this segment
      if constexpr (ROW_SUMS) {
#pragma unroll
        for (int rb = 0; rb < MB; ++rb)
#pragma unroll
          for (int i = 0; i < 16; ++i) row_sum[rb][i] = 0.f;
      }
      // The segment is over: its row sums, added up over the lanes, join the rows' sums.  A row block in which one overflowed is left
      // to the repair launch, as is everything once the list is full.
      auto end_row_segment = [&](int segment) {
        if constexpr (ROW_SUMS) {
          const float t = add_over_lanes<MB>(row_sum);
#pragma unroll
          for (int rb = 0; rb < MB; ++rb)
#pragma unroll
            for (int i = 0; i < 16; ++i) row_sum[rb][i] = 0.f;
          const uint64_t over = __builtin_amdgcn_ballot_w64(!(t < kAnchorLimit));
          if (over != 0 || n_failed > kFailListed) {           // seldom
            const int blocks = row_blocks_of<MB>(over);
#pragma unroll
            for (int i = 0; i <= kFailListed; ++i)
              if (i == n_failed) listed[i] = i < kFailListed ? segment | blocks << kFailBlocks : segment;
            ++n_failed;
          }
          if (n_failed <= kFailListed) {
            const int own = own_slot();
            const bool left_out = (row_blocks_of<MB>(over) >> (MB == 2 ? lane >> 4 & 1 : 0) & 1) != 0;
            float sum = own_sum[own] + (left_out ? 0.f : t), first = own_first[own];
            // A bound is as close as the row's reference is to its normaliser: the reference follows what has been seen, in steps
            // that are exact (kPruneGrain).
            const float up = floorf((__builtin_amdgcn_logf(sum + first) + kPruneShift) * kPruneGrain) / kPruneGrain;
            const bool grown = up > 0.f && up < 1024.f;
            if (grown) {
              const float scale = __builtin_amdgcn_exp2f(-0.5f * up);        // (its square may be too small for a number)
              sum = sum * scale * scale;
              own_first[own] = first * scale * scale;
              own_ref[own] -= up;
            }
            own_sum[own] = sum;
            if (__builtin_amdgcn_ballot_w64(grown) != 0) {
#pragma unroll
              for (int rb = 0; rb < MB; ++rb)
#pragma unroll
                for (int i = 0; i < 16; ++i) nlse[rb][i] = own_ref[(wv * MB + rb) * 32 + 8 * (i >> 2) + 4 * half + (i & 3)];
            }
          }
        }
      };

      // pass 2: sum (maximum) of the lane's 16 probabilities and `before`
      auto column_of = [&](const f32x16 &x, int rb, float before) {
        float p[16], nl[16];
        load_lse(rb, nl);
#pragma unroll
        for (int i = 0; i < 16; ++i) p[i] = __builtin_amdgcn_exp2f(fmaf(x[i], c2, nl[i]));
        if constexpr (ROW_SUMS) {
#pragma unroll
          for (int i = 0; i < 16; ++i) row_sum[rb][i] += p[i];
          stay_here(row_sum[rb]);        // (added later, the block's probabilities would be kept until then)
        }
        if (RED == 0)
          return before + ((((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]))) +
                           (((p[8] + p[9]) + (p[10] + p[11])) + ((p[12] + p[13]) + (p[14] + p[15]))));
        const float t0 = fmaxf(fmaxf(p[0], p[1]), p[2]), t1 = fmaxf(fmaxf(p[3], p[4]), p[5]);
        const float t2 = fmaxf(fmaxf(p[6], p[7]), p[8]), t3 = fmaxf(fmaxf(p[9], p[10]), p[11]);
        const float t4 = fmaxf(fmaxf(p[12], p[13]), p[14]);
        return fmaxf(fmaxf(before, fmaxf(fmaxf(t0, t1), t2)), fmaxf(fmaxf(t3, t4), p[15]));
      };
      // turns the scores x of row block rb into probabilities; pass 2: of key block kb, into partial buffer cbuf
      auto finish_unit = [&](const f32x16 &x, int rb, int kb, int cbuf, auto anchored_c) {
        if constexpr (PASS == 1 && decltype(anchored_c)::value) {
          const float nm = -mrun[rb];
          float sum = 0.f;
#pragma unroll
          for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(fmaf(x[i], c2, nm));
          lrun[rb] += sum;
          asm volatile("" : "+v"(lrun[rb]));      // stays in its unit (the compiler would sink it to the next use)
        } else if constexpr (PASS == 1) {
          // branch-free online softmax step for the lane's query row
          float tmax = fmaxf(fmaxf(x[0], x[1]), x[2]);
#pragma unroll
          for (int i = 3; i < 15; i += 2) tmax = fmaxf(fmaxf(tmax, x[i]), x[i + 1]);
          tmax = fmaxf(tmax, x[15]);
          const float mnew = fmaxf(mrun[rb], tmax * c2);
          const float scale = __builtin_amdgcn_exp2f(mrun[rb] - mnew);
          const float nm = -mnew;
          float sum = 0.f, squares = 0.f;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const float p = __builtin_amdgcn_exp2f(fmaf(x[i], c2, nm));
            sum += p;
            if (SQUARES) squares = fmaf(p, p, squares);
          }
          lrun[rb] = fmaf(lrun[rb], scale, sum);
          mrun[rb] = mnew;
          asm volatile("" : "+v"(lrun[rb]), "+v"(mrun[rb]));
          if constexpr (SQUARES) add_squares(qrun[rb], scale, squares);
        } else {
          if (rb == 0 || (RED == 1 && !merged)) colsum = 0.f;
          colsum = column_of(x, rb, colsum);
          // sum (or the maximum over a block pair): one value per wave, slot wv; otherwise one per 32-row
          // block, blocks of a head are merged at the flush.  Both halves write the same value.
          float *dst = csum + (size_t)cbuf * NW * MB * KT + kb * 32 + l32;
          if (RED == 0) {
            if (rb == NACT - 1) dst[wv * KT] = add_other_half(colsum);
          } else if (!merged || rb == NACT - 1) {
            dst[merged ? wv * KT : (rb * NW + wv) * KT] = max_other_half(colsum);
          }
          asm volatile("" : "+v"(colsum));
        }
      };

      // The wave's key blocks of a tile for the row block it shares.
      auto shared_units = [&](int tile, int buf, auto anchored_c) {
        constexpr bool anchored = decltype(anchored_c)::value;
        // A tile of two key blocks shared by four waves leaves two of them without any of the chunk's first tile, which gives
        // the rows their references: they take theirs from a key block that is another wave's.
        const bool reference_only = kAnchored && !anchored && KB < 4 && tile == 0 && phase >= KB;
#pragma unroll 1
        for (int kb = reference_only ? phase - KB : (phase - tile * KB) & (per - 1); kb < KB; kb += per) {
          f32x16 x = {0}, low = {0};
          u32x4 bf[NCS];
          if constexpr (SPLIT) {
#pragma unroll
            for (int kp = PLANES - 1; kp >= 0; --kp) {
#pragma unroll
              for (int cs = 0; cs < NCS; ++cs) bf[cs] = SPECKV_FRAG(buf, kp, kb, cs);
#pragma unroll
              for (int cs = 0; cs < NCS; ++cs) add_lower_products(low, bf[cs], kp, NACT, cs);
            }
          } else {
            SPECKV_LOAD_BFRAG(bf, buf, kb)
          }
#pragma unroll
          for (int cs = 0; cs < NCS; ++cs) add_product(x, bf[cs], 0, NACT, cs);
          if constexpr (SPLIT) {
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] += low[i];
            recompute_unless_finite(x, NACT, key_begin + tile * KT + kb * 32);
          }
          if constexpr (PASS == 1) {
            if constexpr (kAnchored) {
              float top = fmaxf(fmaxf(x[0], x[1]), x[2]);
#pragma unroll
              for (int i = 3; i < 15; i += 2) top = fmaxf(fmaxf(top, x[i]), x[i + 1]);
              shared_top = fmaxf(top, x[15]);
            }
            if (reference_only) mrun[NACT] = fmaxf(mrun[NACT], shared_top * c2);
            else finish_unit(x, NACT, kb, 0, anchored_c);
          } else {
            // (a block that heads share has no maximum of its own head: one slot per block is right for the flush)
            const float v = column_of(x, NACT, 0.f);
            float *dst = csum + (size_t)(tile % kCsumBuffers) * NW * MB * KT + kb * 32 + l32;
            dst[(NACT * NW + wv) * KT] = RED == 0 ? add_other_half(v) : max_other_half(v);
          }
        }
      };
      // the open unit (the last one of a tile: it always sits in acc[1])
      auto drain = [&](int last_tile, auto anchored_c) {
        if constexpr (NACT > 0 && PIPELINED) {
          if (SPLIT && open) recompute_unless_finite(acc[1], NACT - 1, key_begin + last_tile * KT + (KB - 1) * 32);
          finish_unit(acc[1], NACT - 1, KB - 1, last_tile % kCsumBuffers, anchored_c);
        }
        open = false;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[1][i] = -INFINITY;
      };
      // One tile of the sweep; the LDS buffer index is a compile-time constant so that every LDS
      // address below is a register plus an immediate.  Pass 2 flushes the tile before last: its last
      // column partials were written in the previous tile's first unit.
      // anchored: row statistics against the fixed reference (see above), else the online step
      auto do_tile = [&](int tile, auto buf_c, auto anchored_c) {
        constexpr int buf = decltype(buf_c)::value;
        constexpr bool anchored = decltype(anchored_c)::value;
        if (tile + 1 < ntiles) {
          if constexpr (SPLIT) SPECKV_FETCH_TILE(tile + 1)
          else SPECKV_LOAD_TILE(tile + 1, buf ^ 1)
        }
        if (PASS == 2 && tile > 1) SPECKV_FLUSH_TILE(tile - 2)
        // (here, where no fragment and only the open block is in registers)
        if (ROW_SUMS && buf == 0 && tile > 0 && tile % kPruneSegment == 0) {
          drain(tile - 1, anchored_c);
          end_row_segment(tile / kPruneSegment - 1);
        }
        if constexpr (NACT == 0 && SHARED && kAnchored && anchored && buf == 1) {
          if (tile > 1)
            end_segment((tile - 3) / kAnchorTiles, [&](int, float) { return fmaxf(shared_top * c2, kNegBig) + (float)anchor_shift; });
        }
        if constexpr (NACT > 0) {
          u32x4 bf[NCS];
          SPECKV_LOAD_BFRAG(bf, buf, 0)
#pragma unroll
          for (int u = 0; u < KB * NACT; ++u) {
            const int kb = u / NACT, rb = u % NACT;
            const int pu = (u + KB * NACT - 1) % (KB * NACT);      // the unit before (of the tile before for u = 0)
            // (where nothing is open its place is in the partial buffer that no tile uses now)
            const int pbuf = (u != 0 ? tile : ROW_SUMS && !open ? tile + 1 : tile + kCsumBuffers - 1) % kCsumBuffers;
            if constexpr (SPLIT) {
              // the open unit is finished beside the lower products, the leading ones then take its registers
              f32x16 low = {0};
#pragma unroll
              for (int kp = PLANES - 1; kp >= 0; --kp) {
#pragma unroll
                for (int cs = 0; cs < NCS; ++cs) {
                  add_lower_products(low, bf[cs], kp, rb, cs);
                  if (kp > 0) bf[cs] = SPECKV_FRAG(buf, kp - 1, kb, cs);
                }
              }
              f32x16 &x = acc[1];
              if (u > 0 || open)
                recompute_unless_finite(x, pu % NACT, key_begin + (u == 0 ? tile - 1 : tile) * KT + pu / NACT * 32);
              finish_unit(x, pu % NACT, pu / NACT, pbuf, anchored_c);
              if (kAnchored && NACT == 2 && u == 0) {              // see end_segment below
                top_before = x[0];
#pragma unroll
                for (int i = 1; i < 16; ++i) top_before = fmaxf(top_before, x[i]);
              }
              __builtin_amdgcn_sched_barrier(0);
              x = (f32x16){0};
#pragma unroll
              for (int cs = 0; cs < NCS; ++cs) {
                add_product(x, bf[cs], 0, rb, cs);
                if (rb < NACT - 1) bf[cs] = SPECKV_FRAG(buf, PLANES - 1, kb, cs);
                else if (kb + 1 < KB) bf[cs] = SPECKV_FRAG(buf, PLANES - 1, kb + 1, cs);
              }
#pragma unroll
              for (int i = 0; i < 16; ++i) x[i] += low[i];
            } else if constexpr (!PIPELINED) {
              f32x16 &x = acc[1];
              x = (f32x16){0};
#pragma unroll
              for (int cs = 0; cs < NCS; ++cs) {
                add_product(x, bf[cs], 0, rb, cs);
                if (rb == NACT - 1 && kb + 1 < KB) bf[cs] = SPECKV_FRAG(buf, 0, kb + 1, cs);
              }
              finish_unit(x, rb, kb, tile % kCsumBuffers, anchored_c);
            } else {
              f32x16 &x = acc[u & 1];
              x = (f32x16){0};
#pragma unroll
              for (int cs = 0; cs < NCS; ++cs) {
                add_product(x, bf[cs], 0, rb, cs);
                if (rb == NACT - 1 && kb + 1 < KB) bf[cs] = SPECKV_FRAG(buf, 0, kb + 1, cs);
              }
              finish_unit(acc[(u & 1) ^ 1], pu % NACT, pu / NACT, pbuf, anchored_c);
            }
            // the compiler may not move work of the neighbouring units across: without this it piles up
            // fragment reads and open blocks until the registers spill
            __builtin_amdgcn_sched_barrier(0);
            if (kAnchored && anchored && u == 0 && buf == 1 && tile > 1) {
              // scores at hand for a new reference: this unit's and those of the unit before it, the other row block's
              // where there are two (fp32: this unit has its registers by now, their maximum is kept)
              end_segment((tile - 3) / kAnchorTiles, [&](int rb_, float) {
                float top = top_before;
                if (SHARED && rb_ == NACT) {
                  top = shared_top;
                } else if (!SPLIT || rb_ == 0) {
                  const f32x16 &s_ = acc[SPLIT || rb_ != 0 ? 1 : 0];
                  top = s_[0];
#pragma unroll
                  for (int i = 1; i < 16; ++i) top = fmaxf(top, s_[i]);
                }
                return fmaxf(top * c2, kNegBig) + (float)anchor_shift;
              });
            }
          }
        }
        open = true;
        if constexpr (SHARED) shared_units(tile, buf, anchored_c);
        if constexpr (SPLIT) {
          if (tile + 1 < ntiles) SPECKV_STORE_TILE(buf ^ 1)
        }
        // the next tile must have landed in LDS, and every wave must be done with this one
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
      };
      // tiles [t0, t1); tile t0 sits in LDS buffer `buf`
      auto run_tiles = [&](int t0, int t1, auto buf_c, auto anchored_c) {
        constexpr int buf = decltype(buf_c)::value;
        for (int tile = t0; tile < t1; tile += 2) {
          do_tile(tile, std::integral_constant<int, buf>{}, anchored_c);
          if (tile + 1 < t1) do_tile(tile + 1, std::integral_constant<int, buf ^ 1>{}, anchored_c);
        }
      };
      using buf0 = std::integral_constant<int, 0>;
      using buf1 = std::integral_constant<int, 1>;
      if constexpr (REPAIR) {
        const int end = min(ntiles, first_tile + kAnchorTiles);
        run_tiles(first_tile, end, buf0{}, std::false_type{});
        drain(end - 1, std::false_type{});
      } else if constexpr (kAnchored) {
        if (ntiles > 0) {
          do_tile(0, buf0{}, std::false_type{});       // finds the references
          drain(0, std::false_type{});
#pragma unroll
          for (int rb = 0; rb < MB; ++rb) {            // moves them up for the blocks that follow
            lrun[rb] = __builtin_ldexpf(lrun[rb], -anchor_shift);
            mrun[rb] += (float)anchor_shift;
            l_before[rb] = lrun[rb];
          }
          run_tiles(1, ntiles, buf1{}, std::true_type{});
          drain(ntiles - 1, std::true_type{});
          if (ntiles > 1) end_segment((ntiles - 2) / kAnchorTiles, [](int, float r) { return r; });
        }
      } else if (ntiles > 0) {
        run_tiles(0, ntiles, buf0{}, std::false_type{});
        drain(ntiles - 1, std::false_type{});
        end_row_segment((ntiles - 1) / kPruneSegment);
        if (PASS == 2) {
          __syncthreads();
          if (ntiles > 1) SPECKV_FLUSH_TILE(ntiles - 2)
          SPECKV_FLUSH_TILE(ntiles - 1)
        }
      }
    };
    // (the barriers inside count wavefronts, whichever copy of the code they are in)
    auto sweep_shared = [&](auto nact_c) {
      if constexpr (MAY_SHARE) {
        if (sharing) return sweep(nact_c, std::true_type{});
      }
      sweep(nact_c, std::false_type{});
    };
    if (nact == MB) sweep(std::integral_constant<int, MB>{}, std::false_type{});
    else if (MB > 1 && nact == 1) sweep_shared(std::integral_constant<int, MB - 1>{});
    else sweep_shared(std::integral_constant<int, 0>{});
    if constexpr (kAnchored || ROW_SUMS) {
      if (lane <= kFailListed + 1) {
        int32_t *mine = A.fail + ((int64_t)bid * NW + wv) * kFailWords;
        int v = n_failed;
#pragma unroll
        for (int i = 0; i <= kFailListed; ++i)
          if (lane == i + 1) v = listed[i];
        mine[lane] = v;                  // [0] count, [1 ..] segments, the last one the start of the rest
      }
    }
  }

  if constexpr (ROW_SUMS) {
    const int own = own_slot(), own_rb = (own >> 5) & (MB - 1);
    int e2;
    const float sum = own_sum[own], lf = __builtin_frexpf(sum, &e2);
    if (l32 < MB * 16)
      A.part[((int64_t)unit * A.g.n_chunks + chunk) * RSB + block_of(own_rb) * 32 + (own & 31)] =
          sum > 0.f ? make_float2((float)e2 - own_ref[own], lf) : make_float2(kNegBig, 0.f);
  }
  if (PASS == 1) {
    // an empty chunk (a sequence without masked tail) leaves the neutral pair (-big, 0)
    float2 *pp = A.part + ((int64_t)unit * A.g.n_chunks + chunk) * RSB;
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
      // A sum taken against a fixed reference can be many binary orders away from 1.  Its exponent
      // moves into the reference first, so that every pair handed on has a sum in [0.5, 1) (or 0)
      // and merging two pairs never multiplies a large sum by a factor that underflows.
      // (The reference of a sample's pair is the sample's maximum: prune_reference_kernel.  Its sum is no larger than its keys are many.)
      int e2 = 0;
      const float lf = SQUARES ? lrun[rb] : __builtin_frexpf(lrun[rb], &e2);
      const float mf = mrun[rb] + (float)e2;
      const float mo = __shfl_xor(mf, 32, 64), lo = __shfl_xor(lf, 32, 64);
      float mm = fmaxf(mf, mo);
      float ll = lf * __builtin_amdgcn_exp2f(mf - mm) + lo * __builtin_amdgcn_exp2f(mo - mm);
      float qq = 0.f;                        // in units of the pair's reference, squared
      if constexpr (SQUARES) {
        const float unit_ = __builtin_amdgcn_exp2f(mrun[rb] - mm), mine_ = qrun[rb] * unit_ * unit_;
        qq = mine_ + __shfl_xor(mine_, 32, 64);
      }
      // a block that waves share: the first of them adds the others' pairs
      const bool in_share = per > 1 && rb == split.full / NW && wv >= share_w0 && wv < share_w0 + 4;
      if (per > 1 && rb == split.full / NW) {
        float2 *others = reinterpret_cast<float2 *>(csum);
        float *others_qq = reinterpret_cast<float *>(others + 4 * 32);
        if (in_share && half == 0) others[(wv - share_w0) * 32 + l32] = make_float2(mm, ll);
        if (SQUARES && in_share && half == 0) others_qq[(wv - share_w0) * 32 + l32] = qq;
        __syncthreads();
        if (in_share && phase == 0) {
          for (int u = 1; u < per; ++u) {
            const float2 v = others[(wv - share_w0 + u) * 32 + l32];
            const float m2 = fmaxf(mm, v.x);
            const float f1 = __builtin_amdgcn_exp2f(mm - m2), f2 = __builtin_amdgcn_exp2f(v.x - m2);
            ll = ll * f1 + v.y * f2;
            if (SQUARES) qq = qq * f1 * f1 + others_qq[(wv - share_w0 + u) * 32 + l32] * f2 * f2;
            mm = m2;
          }
        }
      }
      if (half == 0 && (!in_share || phase == 0)) {
        float2 *slot = &pp[block_of(rb) * 32 + l32];
        if constexpr (SQUARES) A.squares[((int64_t)unit * A.g.n_fast_chunks + chunk) * RSB + block_of(rb) * 32 + l32] = qq;
        if (REPAIR) {                // add to what the first sweep (and earlier repairs) left there
          const float2 have = *slot;
          const float m2 = fmaxf(have.x, mm);
          *slot = make_float2(m2, have.y * __builtin_amdgcn_exp2f(have.x - m2) + ll * __builtin_amdgcn_exp2f(mm - m2));
        } else {
          *slot = make_float2(mm, ll);
        }
      }
    }
  }
}

#undef SPECKV_LOAD_TILE
#undef SPECKV_FETCH_TILE
#undef SPECKV_STORE_TILE
#undef SPECKV_FRAG
#undef SPECKV_LOAD_BFRAG
#undef SPECKV_FLUSH_TILE

// A kernel with TAIL_ONLY = false is a whole sweep in one launch: its first A.chunk_blocks
// workgroups run one unmasked chunk each, the ones behind them the sequences' masked tails (one per
// (unit, sequence)).  A tail is a short latency chain; behind the chunks it fills the CUs that the
// last round of chunk workgroups frees one by one (ragged batches: 1 % faster than tails in front,
// equal-length grids: the same).  TAIL_ONLY = true is the tails alone (calls without a complete
// chunk, and the tails behind a Q-stationary sweep).
// RED + kWhole: a sweep of fp32 without the code for row blocks that waves share, which costs the fp32 sweeps where no block is shared
// (sweeps with it / without: maximum, 8 heads of 400K keys, d = 128, 2 row blocks a group 710 / 643 us; sum, d = 64, 8 blocks, column sums 434 /
// 432, row statistics 444 / 429; two blocks a wave, 12 and 9 in two super-blocks, 1241 / 1149).  The 16-bit sweeps are level and have
// one kernel for both.  With blocks shared, calls of 2 fp32 layers x 30K keys take (with the code / all blocks whole): 1 row block a group
// 95 / 145 us, 5 blocks 172 / 204, 9 blocks in two super-blocks of d = 128 537 / 667, 9 and 13 blocks with two a wave 266 / 285 and 346 / 391.
// A super-block that shares beside a fuller one that does not gains nothing: 8 and 6 blocks 749 / 717.
// The maximum of two blocks a wave never shares: it would have 90 scalar registers spilled instead of 18 (19 layers x 27K keys 2660 and 3000 us).
constexpr int kWhole = 2;
template <int DT, int MB, int PASS>
bool shares_blocks(const ScoreArgs &A) {
  if (DT == kF32 && MB == 2 && PASS == 2 && A.d.reduce_max) return false;
  int first;
  return split_blocks(super_block_blocks(A.d, A.g, 0, &first), A.share != 0).per > 1;        // no super-block is fuller than the first
}

template <int DT, int D, int MB, int NW, int PASS, int RED, bool TAIL_ONLY>
__device__ __forceinline__ void score_dispatch(const ScoreArgs &A) {
  constexpr int R = RED & 1;
  constexpr bool SHARE = RED < kWhole;
  const int bid = blockIdx.x;
  if (PASS == 2 && A.norm_from != kNormMerged)
    clear_scratch(A, (int64_t)bid * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
  if (TAIL_ONLY) score_body<DT, D, MB, NW, PASS, R, true, false, SHARE>(A, bid);
  else if (bid < A.chunk_blocks) score_body<DT, D, MB, NW, PASS, R, false, false, SHARE>(A, bid);
  else score_body<DT, D, MB, NW, PASS, R, true, false, SHARE>(A, bid - A.chunk_blocks);
}

// The row-statistics sweep is compiled for exactly two waves per SIMD (the register allocator
// then schedules its softmax arithmetic more freely); the column sweep does better without.
template <int DT, int D, int MB, int NW, int PASS, int RED, bool TAIL_ONLY>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void score_kernel_rows(ScoreArgs A) {
  score_dispatch<DT, D, MB, NW, PASS, RED, TAIL_ONLY>(A);
}

template <int DT, int D, int MB, int NW, int PASS, int RED, bool TAIL_ONLY>
__global__ __launch_bounds__(NW * 64) void score_kernel_cols(ScoreArgs A) {
  score_dispatch<DT, D, MB, NW, PASS, RED, TAIL_ONLY>(A);
}

// The launch behind a row-statistics sweep: a chunk workgroup's twin reads the lists its wavefronts
// left and repeats the listed segments, in ascending order, with the online step (normally there
// are none and it returns).  Every thread walks all NW lists, so the order needs no exchange.
// (Compiled for one workgroup per CU, which its LDS allows: otherwise one fp32 variant spills.)
template <int DT, int D, int MB, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4))) void score_kernel_rows_repair(ScoreArgs A) {
  const int bid = blockIdx.x;
  const int per_group = 8 * A.g.RS;
  const int item = (bid / per_group) * 8 + ((bid % per_group) & 7);
  if (item >= A.g.n_fast_chunks * A.d.L * A.d.Hkv) return;        // padding of the grid: no lists written
  const int32_t *lists = A.fail + (int64_t)bid * NW * kFailWords;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  int count[NW], at[NW];
  int total = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) { count[w] = lists[w * kFailWords]; at[w] = 0; total += count[w]; }
  if (total == 0) return;
  auto listed = [&](int w, int i) {
    return i <= kFailListed ? lists[w * kFailWords + 1 + i] : lists[w * kFailWords + 1 + kFailListed] + (i - kFailListed);
  };
  for (;;) {
    int next = 0x7fffffff;
#pragma unroll
    for (int w = 0; w < NW; ++w)
      if (at[w] < count[w]) next = min(next, listed(w, at[w]));
    if (next == 0x7fffffff) break;
    bool mine = false;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const bool has = at[w] < count[w] && listed(w, at[w]) == next;
      if (has) ++at[w];
      if (w == wv) mine = has;
    }
    score_body<DT, D, MB, NW, 1, 0, false, true>(A, bid, next, mine);
    __syncthreads();
  }
}

template <typename K>
hipError_t launch_one(K kernel, const ScoreArgs &A, dim3 grid, dim3 block, size_t lds, hipStream_t st) {
  hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, grid, block, lds, st, A);
  return hipGetLastError();
}

template <int DT, int D, int MB, int NW, int PASS, int RED>
hipError_t launch_sweep(const ScoreArgs &A0, size_t lds, hipStream_t st) {
  ScoreArgs A = A0;
  const int64_t tails = (int64_t)A.d.L * A.d.Hkv * A.g.RS * A.d.S;
  if (tails > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 block(NW * 64);
  A.chunk_blocks = 0;
  if (A.g.n_fast_chunks > 0 && !qs_supported(A, PASS)) {
    const int64_t items = (int64_t)A.g.n_fast_chunks * A.d.L * A.d.Hkv;
    const int64_t chunk_wgs = (items + 7) / 8 * 8 * A.g.RS;
    if (chunk_wgs + tails > 0x7fffffffLL) return hipErrorInvalidValue;
    A.chunk_blocks = (int)chunk_wgs;
    const dim3 grid((unsigned)(chunk_wgs + tails));
    if constexpr (PASS == 1) {
      hipError_t e;
      if constexpr (NW == 8) e = launch_one(score_kernel_rows<DT, D, MB, NW, PASS, RED, false>, A, grid, block, lds, st);
      else e = launch_one(score_kernel_cols<DT, D, MB, NW, PASS, RED, false>, A, grid, block, lds, st);
      if (e != hipSuccess || (RED & 1) == 0) return e;
      return launch_one(score_kernel_rows_repair<DT, D, MB, NW>, A, dim3((unsigned)chunk_wgs), block, lds, st);
    } else {
      return launch_one(score_kernel_cols<DT, D, MB, NW, PASS, RED, false>, A, grid, block, lds, st);
    }
  }
  if (A.g.n_fast_chunks > 0) {
    const hipError_t e = launch_qs_sweep(A, PASS, st);
    if (e != hipSuccess) return e;
  }
  return launch_one(score_kernel_cols<DT, D, MB, NW, PASS, RED & 1, true>, A, dim3((unsigned)tails), block, lds, st);
}

// Sweep PASS (1 row statistics, 2 column reduction) for the number type, head dimension and
// workgroup geometry of A.
template <int DT, int D, int MB, int NW, int PASS>
hipError_t sweep_for_geometry(const ScoreArgs &A, hipStream_t st) {
  const size_t lds = score_lds_bytes<DT, D, MB, NW>();
  const bool red = PASS == 1 ? score_rows_fixed_reference(A.d, A.g) : A.d.reduce_max != 0;
  if constexpr (DT == kF32) {
    if (!shares_blocks<DT, MB, PASS>(A)) {
      ScoreArgs whole = A;                       // (the masked tails and the repair launch read it)
      whole.share = 0;
      return red ? launch_sweep<DT, D, MB, NW, PASS, 1 + kWhole>(whole, lds, st) : launch_sweep<DT, D, MB, NW, PASS, kWhole>(whole, lds, st);
    }
  }
  if constexpr (!(DT == kF32 && MB == 2 && PASS == 2)) {
    if (red) return launch_sweep<DT, D, MB, NW, PASS, 1>(A, lds, st);
  }
  return launch_sweep<DT, D, MB, NW, PASS, 0>(A, lds, st);
}

template <int DT, int D, int PASS>
hipError_t sweep_for_type(const ScoreArgs &A, hipStream_t st) {
  switch (A.g.NW * 10 + A.g.MB) {
    case 41: return sweep_for_geometry<DT, D, 1, 4, PASS>(A, st);
    case 81: return sweep_for_geometry<DT, D, 1, 8, PASS>(A, st);
    case 82:
      if constexpr (D * elt_bytes(DT) <= 256) return sweep_for_geometry<DT, D, 2, 8, PASS>(A, st);
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

template <int PASS>
hipError_t dispatch_sweep(const ScoreArgs &A, hipStream_t st) {
  switch (A.d.dt) {
    case SPECKV_BF16: return A.d.D == 128 ? sweep_for_type<kBf16, 128, PASS>(A, st) : sweep_for_type<kBf16, 64, PASS>(A, st);
    case SPECKV_F16: return A.d.D == 128 ? sweep_for_type<kF16, 128, PASS>(A, st) : sweep_for_type<kF16, 64, PASS>(A, st);
    default: return A.d.D == 128 ? sweep_for_type<kF32, 128, PASS>(A, st) : sweep_for_type<kF32, 64, PASS>(A, st);
  }
}

}  // namespace
}  // namespace speckv
