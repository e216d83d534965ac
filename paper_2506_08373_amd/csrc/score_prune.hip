// Pruned scoring: the sweeps of a fused call that needs the scores only to find the largest ones (Alg. 1 CrossAttention, reduce and
// "Select KVs" together), and their host entry.
//
// A column sum of the row softmax needs every row's normaliser first, so two sweeps over all keys multiply every key with every row
// twice (score_sweep.h).  A call that returns indices and rows, not scores, needs the exact scores of the best keys alone:
//
//   1  row statistics over a sample (every 2^step_log-th key tile) and the masked tails, and from them a cautious estimate e of a row's
//      normaliser (prune_reference_kernel)
//   2  one sweep over the other keys sums 2^(score - e) along rows, which completes the normalisers, and along columns: as far as e is
//      no larger than the normaliser, a column sum is an upper bound on the key's score.  e follows what a chunk has seen.
//   3  column sums of the sample with the normalisers; from them a threshold that more than c_max pooled scores will reach
//      (prune.hip), and the list of the other keys whose bound reaches it
//   4  column sums of the listed keys, by the same arithmetic as without pruning
//   5  pooling.  A score that is not known is below the threshold, and so is its stand-in, the bound: where c_max or more pooled
//      scores reach the threshold they and their order are exact.  Rows where fewer do are computed whole.
//
// The indices are those of all scores, whatever the data; only the time depends on them.
// One sweep instead of two is what there is to gain.  Sum of 32 layers x 128K keys, 4 heads x 128 rows, d = 128, us: the two sweeps
// 4260 + 4400; here sample 330, sweep 4410 (a block's 16 more additions and the row sums cost it 8 %), sample's columns 290,
// listed keys (4 %) 250, the rest 180.  Calls, all scores / pruned: that one 8540 / 5500, eight prompts of 4K to 64K, groups of 7,
// 28 layers 15860 / 10480, 32 layers x 16K, maximum 1010 / 775, 8 layers x 32K 590 / 470; d = 64, prompt tokens, 16 layers x 64K
// 844 / 694.
// Where nothing can be pruned (scores all alike, or a threshold under prune_floor) the listed sweep is a second whole one, a tenth
// slower than a column sweep, and the sample and the small launches come on top.  Calls of rows that attend to all keys alike, all
// scores / pruned: 32 layers x 128K 8470 / 9510, 8 layers x 32K 610 / 715, maximum, 32 x 16K 768 / 935; prompt tokens, whose score
// is a sum over all rows, also where the rows have nothing to do with each other, 16 x 64K 856 / 1013.
#include <algorithm>
#include <utility>

#include "score_sweep.h"

namespace speckv {
namespace {

template <int DT, int D, int MB, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void prune_sample_rows_kernel(PruneArgs A) {
  const int bid = blockIdx.x;
  if (bid < A.chunk_blocks) score_body<DT, D, MB, NW, 1, 0, false, false, true, kSampleKeys>(A, bid);
  else score_body<DT, D, MB, NW, 1, 0, true>(static_cast<const ScoreArgs &>(A), bid - A.chunk_blocks);
}

// (Four waves per SIMD, so that two workgroups share a CU, where the LDS has room for them.  The maximum of a head's rows by pairs of
// blocks and by single ones are two bodies: one that does either does not fit the registers at d = 128, where 12 were spilled into the
// loop.  Sweep over 32 layers x 128K keys 4760 us beside the sum's 4380, with two bodies 4270 beside 4410; call of 32 x 16K keys, 12
// blocks, 911 / 833.)
template <int DT, int D, int MB, int NW, int RED>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(D == 64 && MB == 1 ? 4 : 2)))
void prune_sweep_kernel(PruneArgs A) {
  if constexpr (RED == 1 && MB == 2) {
    const int rs = prune_super_block(A, blockIdx.x);
    int first;
    if (!sweep_pairs_blocks<RED, MB, NW>(A, super_block_blocks(A.d, A.g, rs, &first))) {
      score_body<DT, D, MB, NW, 2, RED, false, false, false, kOtherKeys, 0>(A, blockIdx.x);
      return;
    }
  }
  score_body<DT, D, MB, NW, 2, RED, false, false, false, kOtherKeys, RED == 1 && MB == 2>(A, blockIdx.x);
}

// The segments that wavefronts of the sweep left out of their sums, with the online step; one workgroup per wavefront's list
// (normally empty), whose eight wavefronts share a segment's keys and read them straight into fragments.  A segment is one chain
// of latencies: 8 tiles by the sweep's own workgroup shape (one wavefront working) take 30 us.
template <int DT, int D, int MB, int NW, int RED>
__global__ __launch_bounds__(512) void prune_repair_kernel(PruneArgs A) {
  using OP = Operand<DT, D, MB>;
  constexpr int NCS = OP::TL::NCS, KT = OP::KT, RSB = NW * MB * 32, WAVES = 8;
  __shared__ float2 pairs[WAVES][MB * 32];
  const int bid = blockIdx.x / NW, list = blockIdx.x % NW;
  const PruneChunk c = prune_chunk(A, bid);
  if (c.unit < 0) return;
  const int32_t *listed = A.fail + ((int64_t)bid * NW + list) * kFailWords;
  const int count = listed[0];
  if (count == 0) return;
  const Dims &d = A.d;
  const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int rs = c.unit % A.g.RS, g = c.unit / A.g.RS % d.Hkv, layer = c.unit / (A.g.RS * d.Hkv);
  const int step_log = prune_step(A.chunk_of[c.s]), tiles = (c.key_end - c.key_begin + KT - 1) / KT;
  const int others = tiles - ((tiles + (1 << step_log) - 1) >> step_log);
  const float c2 = d.sm_scale * 1.4426950408889634f;
  int first;
  const int nblk = super_block_blocks(d, A.g, rs, &first);
  const bool paired = sweep_pairs_blocks<RED, MB, NW>(A, nblk);
  auto block_of = [&](int rb) { return paired ? list * MB + rb : rb * NW + list; };
  u32x4 qf[MB][NCS];
#pragma unroll
  for (int rb = 0; rb < MB; ++rb) {
    int hh, i;
    const bool valid = decode_row(d, A.g, rs, block_of(rb) * 32 + l32, &hh, &i);
    const char *qp = A.q + ((int64_t)layer * d.q_sl + (int64_t)c.s * d.q_ss + (int64_t)(valid ? i : 0) * d.q_sr +
                            (int64_t)(g * d.G + (valid ? hh : 0)) * d.q_sh) * 2 + half * 16;
#pragma unroll
    for (int cs = 0; cs < NCS; ++cs) qf[rb][cs] = valid ? *reinterpret_cast<const u32x4 *>(qp + cs * 32) : (u32x4)(0u);
  }
  const char *kbase = A.k + ((int64_t)layer * d.kv_sl + (int64_t)A.t.cu[c.s] * d.kv_st + (int64_t)g * d.kv_sh) * 2 + half * 16;
  float top[MB], sum[MB];
#pragma unroll
  for (int rb = 0; rb < MB; ++rb) { top[rb] = kNegBig; sum[rb] = 0.f; }
  for (int n = 0; n < count; ++n) {
    const int entry = n < kFailListed ? listed[1 + n] : listed[1 + kFailListed] + (n - kFailListed);
    const int seg = entry & ((1 << kFailBlocks) - 1), blocks = n < kFailListed ? entry >> kFailBlocks : (1 << MB) - 1;
    const int b1 = min(others, (seg + 1) * kPruneSegment) * (KT / 32);
    u32x4 next[NCS];
    auto request = [&](int b) {
      const int bb = min(b, b1 - 1);
      const int key = c.key_begin + other_tile(bb / (KT / 32), step_log) * KT + bb % (KT / 32) * 32 + l32;
      const char *kp = kbase + (int64_t)key * d.kv_st * 2;
#pragma unroll
      for (int cs = 0; cs < NCS; ++cs) next[cs] = *reinterpret_cast<const u32x4 *>(kp + cs * 32);
    };
    const int b0 = seg * kPruneSegment * (KT / 32) + wave;
    request(b0);
    for (int b = b0; b < b1; b += WAVES) {
      u32x4 kf[NCS];
#pragma unroll
      for (int cs = 0; cs < NCS; ++cs) kf[cs] = next[cs];
      request(b + WAVES);
#pragma unroll
      for (int rb = 0; rb < MB; ++rb) {
        if ((blocks >> rb & 1) == 0) continue;
        f32x16 x = {0};
#pragma unroll
        for (int cs = 0; cs < NCS; ++cs) x = mma_chunk<DT>(kf[cs], qf[rb][cs], x);
        float t = x[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) t = fmaxf(t, x[i]);
        const float m = fmaxf(top[rb], t * c2);
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) s += __builtin_amdgcn_exp2f(fmaf(x[i], c2, -m));
        sum[rb] = fmaf(sum[rb], __builtin_amdgcn_exp2f(top[rb] - m), s);
        top[rb] = m;
      }
    }
  }
#pragma unroll
  for (int rb = 0; rb < MB; ++rb) {
    const float2 other = make_float2(__shfl_xor(top[rb], 32, 64), __shfl_xor(sum[rb], 32, 64));
    merge_pairs<1>(top[rb], sum[rb], &other);
    if (half == 0) pairs[wave][rb * 32 + l32] = make_float2(top[rb], sum[rb]);
  }
  __syncthreads();
  if (threadIdx.x < MB * 32) {
    const int r = threadIdx.x;
    float2 *slot = A.part + ((int64_t)c.unit * A.g.n_chunks + c.chunk) * RSB + block_of(r >> 5) * 32 + (r & 31);
    float2 have = *slot;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) merge_pairs<1>(have.x, have.y, &pairs[w][r]);
    *slot = have;
  }
}

template <int DT, int D, int MB, int NW, int RED>
__global__ __launch_bounds__(NW * 64) void prune_sample_columns_kernel(PruneArgs A) {
  const int bid = blockIdx.x;
  if (bid < A.chunk_blocks) score_body<DT, D, MB, NW, 2, RED, false, false, true, kSampleKeys>(A, bid);
  else score_body<DT, D, MB, NW, 2, RED, true>(static_cast<const ScoreArgs &>(A), bid - A.chunk_blocks);
}

template <int DT, int D, int MB, int NW, int RED>
__global__ __launch_bounds__(NW * 64) void prune_listed_kernel(PruneArgs A) {
  const int n = *A.n_items * A.g.RS * (A.one_row != 0 ? A.d.L * A.d.Hkv : 1);
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    score_body<DT, D, MB, NW, 2, RED, false, false, true, kListedKeys>(A, i);
    __syncthreads();
  }
}

enum class Sweep { SampleRows, Others, SampleColumns, Listed };

template <int DT, int D, int MB, int NW, int RED>
hipError_t launch_prune_sweep(Sweep which, const PruneArgs &A, hipStream_t st) {
  const unsigned chunks = (unsigned)A.chunk_blocks, tails = (unsigned)(A.d.L * A.d.Hkv * A.g.RS * A.d.S);
  const dim3 block(NW * 64);
  auto launch = [&](auto kernel, unsigned grid, bool row_sums = false) {
    const size_t lds = score_lds_bytes<DT, D, MB, NW>(row_sums);
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(grid), block, lds, st, A);
    return hipGetLastError();
  };
  switch (which) {
    case Sweep::SampleRows: return launch(prune_sample_rows_kernel<DT, D, MB, NW>, chunks + tails);
    case Sweep::Others: {
      const hipError_t e = launch(prune_sweep_kernel<DT, D, MB, NW, RED>, chunks, true);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL((prune_repair_kernel<DT, D, MB, NW, RED>), dim3(chunks * NW), dim3(512), 0, st, A);
      return hipGetLastError();
    }
    case Sweep::SampleColumns: return launch(prune_sample_columns_kernel<DT, D, MB, NW, RED>, chunks + tails);
    default: return launch(prune_listed_kernel<DT, D, MB, NW, RED>, 512);
  }
}

template <int DT, int D>
hipError_t launch_for_type(Sweep which, const PruneArgs &A, hipStream_t st) {
  const bool max = A.d.reduce_max != 0;
  if (A.g.MB == 2) return max ? launch_prune_sweep<DT, D, 2, 8, 1>(which, A, st) : launch_prune_sweep<DT, D, 2, 8, 0>(which, A, st);
  return max ? launch_prune_sweep<DT, D, 1, 8, 1>(which, A, st) : launch_prune_sweep<DT, D, 1, 8, 0>(which, A, st);
}

hipError_t launch(Sweep which, const PruneArgs &A, hipStream_t st) {
  if (A.d.dt == SPECKV_BF16) return A.d.D == 128 ? launch_for_type<kBf16, 128>(which, A, st) : launch_for_type<kBf16, 64>(which, A, st);
  return A.d.D == 128 ? launch_for_type<kF16, 128>(which, A, st) : launch_for_type<kF16, 64>(which, A, st);
}

int64_t prune_rows(const Plan &pl) { return pl.one_row ? 1 : (int64_t)pl.d.L * pl.d.S * pl.d.Hkv; }

// The buffers of a pruned call.
struct Buffers {
  PruneArgs A;
  float *planes;
  PruneRow *rows;
  int32_t *list, *n_items;            // n_items[0] of the first listing, [1] of the repeated one
  int2 *items;
  Buffers(const Plan &pl, const void *q, const void *k, void *workspace) {
    char *ws = static_cast<char *>(workspace);
    planes = reinterpret_cast<float *>(ws + pl.off_planes);
    rows = reinterpret_cast<PruneRow *>(ws + pl.off_prune_rows);
    n_items = reinterpret_cast<int32_t *>(rows + prune_rows(pl));
    items = reinterpret_cast<int2 *>(ws + pl.off_prune_items);
    list = reinterpret_cast<int32_t *>(ws + pl.off_pooled);      // written after the pairs, read before the pooled scores are written
    A.d = pl.d; A.t = pl.t; A.g = pl.g;
    A.q = (const char *)q; A.k = (const char *)k;
    A.part = reinterpret_cast<float2 *>(ws + pl.off_prune_pairs);
    A.lse = reinterpret_cast<float *>(ws + pl.off_lse);
    A.planes = planes; A.lse_in = nullptr; A.clear = nullptr; A.clear_words = 0;
    A.norm_from = kNormMerged;
    A.share = A.d.reduce_max == 0;
    A.chunk_blocks = (int)score_chunk_workgroups(A.d, A.g, A.g.n_fast_chunks);
    A.fail = reinterpret_cast<int32_t *>(A.part + (int64_t)A.d.L * A.d.Hkv * A.g.RS * A.g.n_chunks * A.g.RSB);
    std::memcpy(A.chunk_of, pl.chunk_of, sizeof(A.chunk_of));
    std::memcpy(A.order, pl.order, sizeof(A.order));
    A.item_keys = pl.item_keys;
    A.one_row = pl.prune_keep != 0;
    A.squares = reinterpret_cast<float *>(ws + pl.off_squares);
    A.row_extra = reinterpret_cast<float *>(ws + pl.off_row_extra);
    A.list = list; A.rows = rows; A.items = items; A.n_items = n_items;
  }
};

}  // namespace

// Of a sequence of m candidates, per cent of a whole sweep: the more of them are kept, the more have to be listed (2 to 8 % of the keys
// from 32 c_max on, 10 % at 16, 20 to 35 % at 7 c_max).
constexpr int kPruneLeast = 7;
static int prune_saving(int64_t m, int64_t c_max) {
  return m >= 32 * c_max ? 33 : m >= 16 * c_max ? 28 : m >= 11 * c_max ? 20 : m >= kPruneLeast * c_max ? 12 : 0;
}
// Keys of a chunk where there is no sample but every key is in it.
constexpr int kPruneAllSample = 4096;

// The most chunks a pruned call is cut into: about kPruneRounds rounds of the CUs, or chunks of kPruneLong keys, or what sequences
// that are all sample need.  Short chunks even out the end of the sweep, but in each the references begin anew with what the sample
// gives, and more keys are listed; and they take room in the workspace, whose size has to be that of the longest prompt whatever the
// number of chunks of a shorter one.  Calls, us, with up to 12 rounds / with this: 3 layers of 54K (53 chunks / 9) 486 / 341, 18 of
// 63K, one KV head, 928 / 784, 28 of 98K the same, shared budget 1671 / 1500, 26 of 57K, groups of 7, maximum 1724 / 1557; of 51
// random ones none slower.
constexpr int kPruneRounds = 4, kPruneLong = 16384, kPruneChunkMin = 512;
static int64_t prune_most_chunks(const Plan &pl) {
  const int64_t units = (int64_t)pl.d.L * pl.d.Hkv * pl.g.RS, c_max = pl.one_row ? pl.sel_kept : pl.d.c_max;
  int64_t of_min = 0, of_long = 0, whole = 0;
  for (int s = 0; s < pl.d.S; ++s) {
    const int64_t n = pl.t.tail0[s];
    of_min += (n + kPruneChunkMin - 1) / kPruneChunkMin;
    of_long += (n + kPruneLong - 1) / kPruneLong;
    whole += (std::min(n, kPruneLeast * c_max) + kPruneAllSample - 1) / kPruneAllSample;
  }
  return std::max({whole, of_long, std::min((kPruneRounds * 256 + units - 1) / units + pl.d.S - 1, of_min)});
}

// Chunks of a sequence when none is longer than kc: equal ones, of whole periods of the sample.  (Of a sequence that is all sample a
// workgroup has every key to do, and they should not be the last ones of the sample's sweep.)
struct Chunks { int count, keys; };
static Chunks prune_chunks(const Plan &pl, int s, int step, int64_t kc) {
  const int64_t n = pl.t.tail0[s];
  if (n == 0) return {0, prune_tile_keys(pl)};
  if (step == 0) kc = std::min<int64_t>(kc, std::max(kPruneAllSample, pl.g.KC));
  const int64_t count = (n + kc - 1) / kc;
  const int64_t keys = std::max<int64_t>(align_up((n + count - 1) / count, (int64_t)prune_tile_keys(pl) << step), kPruneChunkMin);
  return {(int)((n + keys - 1) / keys), (int)keys};
}

// The most keys of a chunk.  References grow with what a chunk has seen, so that longer chunks have closer bounds and fewer keys to
// list: the longest that costs the sweep little in CUs left idle at its end.
static int64_t prune_chunk_keys(const Plan &pl, const int *step, int64_t units) {
  constexpr int kCUs = 256, kSimulated = 16;
  constexpr double kCost = 190.;                        // of a workgroup, in keys
  int64_t longest = 0;
  for (int s = 0; s < pl.d.S; ++s)
    if (step[s] != 0) longest = std::max<int64_t>(longest, pl.t.tail0[s]);
  // The sweep's duration in key-times: the longest chunks first, each to the CU that is free first.  Beyond kSimulated sequences
  // the chunks are many and of all lengths: an even spread and half a short one.
  auto duration = [&](int64_t kc) {
    std::pair<double, int64_t> todo[kMaxSeqs];                              // keys and number of a sequence's workgroups
    int n_todo = 0;
    double total = 0., shortest = 1e30;
    for (int s = 0; s < pl.d.S; ++s) {
      if (step[s] == 0) continue;
      const Chunks c = prune_chunks(pl, s, step[s], kc);
      todo[n_todo++] = {std::min(c.keys, pl.t.tail0[s]) + kCost, c.count * units};
      total += todo[n_todo - 1].first * (double)todo[n_todo - 1].second;
      shortest = std::min(shortest, todo[n_todo - 1].first);
    }
    std::sort(todo, todo + n_todo, [](auto &a, auto &b) { return a.first > b.first; });
    if (n_todo > kSimulated) return std::max(todo[0].first, total / kCUs + 0.5 * shortest);
    std::pair<double, int64_t> free_at[kCUs + 1] = {{0., kCUs}};            // CUs by the time they are free, ascending; none empty
    int n_free = 1;
    for (int i = 0; i < n_todo; ++i) {
      for (int64_t n = todo[i].second; n > 0;) {
        const double done = free_at[0].first + todo[i].first;
        const int64_t k = std::min(free_at[0].second, n);
        n -= k;
        free_at[0].second -= k;
        if (free_at[0].second == 0) std::copy(free_at + 1, free_at + n_free--, free_at);
        int x = 0;
        while (x < n_free && free_at[x].first < done) ++x;
        if (x < n_free && free_at[x].first == done) {
          free_at[x].second += k;
        } else {
          std::copy_backward(free_at + x, free_at + n_free, free_at + n_free + 1);
          free_at[x] = {done, k};
          ++n_free;
        }
      }
    }
    return free_at[n_free - 1].first;
  };
  static const int parts[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 40, 48, 64, 96, 128};
  constexpr size_t kParts = sizeof(parts) / sizeof(parts[0]);
  const int64_t most = prune_most_chunks(pl);            // (at least as many as one chunk a sequence with a sample makes)
  double best = 1e30, took[kParts];
  size_t n = 0;
  for (; n < kParts; ++n) {
    const int64_t kc = (longest + parts[n] - 1) / parts[n];
    int64_t chunks = 0;
    for (int s = 0; s < pl.d.S; ++s) chunks += prune_chunks(pl, s, step[s], kc).count;
    if (n > 0 && chunks > most) break;
    best = std::min(best, took[n] = duration(kc));
  }
  size_t i = 0;
  while (took[i] > 1.03 * best) ++i;
  return (longest + parts[i] - 1) / parts[i];
}

// What pruning has to save of a whole sweep to pay for its additional launches, in blocks of 32 rows x keys.  All scores / pruned, us,
// d = 128: 3.5M (3 layers of 32K) 332 / 363, 5.5M (one of 128K) 311 / 343, (2 of 64K) 314 / 362, 6.6M (32 of 8K, 512 kept) 659 / 597,
// 9.4M (8 of 32K) 638 / 562; d = 64: 6.3M (12 layers of 66K, 2 heads) 309 / 259.  Below the line a call gains where its own sweeps fill
// the last round of the CUs badly: 5.9M (5 of 32K) 528 / 426, 4.1M (6 of 16K) 352 / 339.
// Every further sequence makes the chunks shorter and the launches less even: 12.6M (2 layers of 7 prompts) 864 / 838; with groups of 7
// 8.6M (2 of 6) 732 / 609, below the line.
constexpr int64_t kPruneMinSaving = 6000000, kPruneMinPerSeq = 700000;
// Half as much again where there are more launches (prompt tokens, shared budgets) or a whole sweep has two workgroups a CU (8 waves
// of one row block): 4.7M (shared budget, 4 layers of 32K) 353 / 397, 4.7M (d = 64, 9 of 25K, 64 rows) 233 / 252, 6.6M (prompt
// tokens, 9 of 41K) 350 / 348; 9.4M (shared budget, 8 of 32K) 664 / 613, 10M (25 of 19K, 64 rows) 675 / 654, 13.4M (prompt tokens,
// 16 of 64K) 856 / 728.
// Whether a call is pruned, each sequence's sample step and the keys of those that have one.
static bool prune_pays(const Plan &pl, int32_t keep, bool ada, int *step, int64_t *pruned) {
  const Dims &d = pl.d;
  const ScoreGeom &g = pl.g;
  if (d.elt != 2 || g.NW != 8 || g.PPH != 1 || d.pool_avg || d.head_max || d.pool_k > 16 || d.n_dev != nullptr ||
      (pl.one_row ? keep < 1 : d.c_max < 1))
    return false;
  const int64_t c_max = pl.one_row ? keep : d.c_max;
  int64_t saved = 0;
  *pruned = 0;
  for (int s = 0; s < d.S; ++s) {
    const int64_t m = pl.t.cu[s + 1] - pl.t.cu[s] - d.w;
    const int saving = prune_saving(m, c_max);
    // (the sum over all layers and heads has closer bounds: 7 % of 64K keys are listed with a sample of 1/4, 9 % with 1/8)
    step[s] = saving == 0 ? 0 : m < 24000 || (!pl.one_row && m < 16 * c_max) ? 2 : pl.one_row || m < 48 * c_max || m < 60000 ? 3 : 4;
    if (saving != 0) *pruned += pl.t.tail0[s];
    saved += (int64_t)pl.t.tail0[s] * saving / 100;
  }
  const int64_t least = kPruneMinSaving * (pl.one_row || ada || g.MB == 1 ? 3 : 2) / 2 + kPruneMinPerSeq * (d.S - 1);
  if (saved * d.L * d.Hkv * ((d.M + 31) / 32) < least) return false;
  const int64_t most = 0x7fffffff / 8, units = (int64_t)d.L * d.Hkv * g.RS;           // workgroups of a launch
  return score_chunk_workgroups(d, g, prune_most_chunks(pl)) <= most && units * d.S <= most && prune_rows(pl) * (d.T / 4096 + 1) <= most;
}

// Lays out the workspace of a pruned call of up to `chunks` unmasked chunks, in a workspace with room for `all` of a call that is not.  The
// pairs and the samples' squares are read for the last time before the lists are written, in the place of the pooled scores.
static void prune_carve(Plan *pl, bool ada, const int *step, int64_t chunks, int64_t all) {
  const Dims &d = pl->d;
  const ScoreGeom &g = pl->g;
  const size_t units = (size_t)d.L * d.Hkv * g.RS;
  const size_t pairs = (size_t)align_up((int64_t)(units * (chunks + d.S) * g.RSB * sizeof(float2) +
                                                  (size_t)score_fail_words(d, g, chunks) * sizeof(int32_t)), 256);
  carve_workspace(pl, all, pairs + units * chunks * g.RSB * sizeof(float));
  pl->off_prune_pairs = pl->off_pooled;
  pl->off_squares = pl->off_pooled + pairs;
  size_t off = ada ? pl->total_ada : pl->total;
  auto take = [&](size_t bytes) { size_t o = off; off = (size_t)align_up((int64_t)(off + bytes), 256); return o; };
  pl->off_row_extra = take(units * d.S * g.RSB * sizeof(float));
  pl->off_prune_rows = take((size_t)prune_rows(*pl) * sizeof(PruneRow) + 2 * sizeof(int32_t));
  int64_t items = 0;
  for (int s = 0; s < d.S; ++s)
    if (step[s] != 0) items += (pl->t.tail0[s] + kPruneItemMin - 1) / kPruneItemMin;
  pl->off_prune_items = take((size_t)(items * (pl->one_row ? 1 : d.L * d.Hkv)) * sizeof(int2));
  pl->total_pruned = off;
}

size_t prune_workspace(const Plan &pl, int32_t keep, bool ada) {
  int step[kMaxSeqs];
  int64_t pruned;
  if (!prune_pays(pl, keep, ada, step, &pruned)) return 0;
  Plan most = pl;
  most.sel_parts = pl.most_sel_parts;
  prune_carve(&most, ada, step, prune_most_chunks(pl), pl.most_chunks);
  return most.total_pruned;
}

// The environment's choices among the kernels that compute every score (score_uses_qs, score_rows_fixed_reference) are for fused
// calls, too.
static bool whole_kernels_asked_for() {
  const char *kernel = std::getenv("SPECKV_SCORE_KERNEL"), *rows = std::getenv("SPECKV_ROW_STATISTICS");
  return (kernel != nullptr && kernel[0] != '\0') || (rows != nullptr && rows[0] != '\0');
}

bool prune_plan(Plan *pl, int32_t keep, bool ada) {
  Dims &d = pl->d;
  ScoreGeom &g = pl->g;
  int step[kMaxSeqs];
  int64_t pruned;
  // (rows that are ranked in parts have no counts of first digits)
  if ((!pl->one_row && pl->hist0_words == 0) || whole_kernels_asked_for() || !prune_pays(*pl, keep, ada, step, &pruned)) return false;
  pl->prune_keep = pl->one_row ? keep : 0;
  const int64_t units = (int64_t)d.L * d.Hkv * g.RS;
  // About a tenth of the keys is listed: an item per CU, if that makes items short.  (Twice as many of half the size measure the same,
  // 8 layers x 32K, shared budget: 80 us for the listed sweep.)
  pl->item_keys = kPruneItemMax;
  while (pl->item_keys > kPruneItemMin && pl->item_keys * 1280ll >= pruned * units) pl->item_keys /= 2;
  const int64_t kc = prune_chunk_keys(*pl, step, units);
  int cc = 0;
  for (int s = 0; s < d.S; ++s) {
    const Chunks c = prune_chunks(*pl, s, step[s], kc);
    pl->t.cc[s] = cc;
    cc += c.count;
    pl->chunk_of[s] = c.keys + step[s];
    pl->order[s] = s;
  }
  // (a chunk that is all sample weighs less than one of as many keys: the sweep over the others has nothing to do for it)
  std::sort(pl->order, pl->order + d.S, [&](int a, int b) {
    return pl->chunk_of[a] != pl->chunk_of[b] ? pl->chunk_of[a] > pl->chunk_of[b] : a < b;
  });
  pl->t.cc[d.S] = cc;
  g.n_fast_chunks = cc;
  g.n_chunks = cc + d.S;
  prune_carve(pl, ada, step, cc, pl->room_chunks);
  return true;
}

hipError_t launch_prune_rows(const Plan &pl, const void *q, const void *k, void *ws, hipStream_t st, hipEvent_t *ev, uint32_t *clear,
                             int64_t clear_words) {
  Buffers b(pl, q, k, ws);
  hipError_t e;
  if (ev && (e = hipEventRecord(ev[0], st)) != hipSuccess) return e;
  if ((e = launch(Sweep::SampleRows, b.A, st)) != hipSuccess) return e;
  if ((e = launch_prune_references(b.A, prune_tile_keys(pl), st)) != hipSuccess) return e;
  if ((e = launch(Sweep::Others, b.A, st)) != hipSuccess) return e;
  if (ev && (e = hipEventRecord(ev[1], st)) != hipSuccess) return e;
  b.A.clear = clear;
  b.A.clear_words = clear != nullptr ? clear_words : 0;
  if ((e = launch_lse_combine(b.A, b.A.row_extra, st)) != hipSuccess) return e;
  if (ev && (e = hipEventRecord(ev[2], st)) != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_prune_columns(const Plan &pl, const void *q, const void *k, void *ws, hipStream_t st, int32_t c_floor) {
  Buffers b(pl, q, k, ws);
  hipError_t e;
  if ((e = launch(Sweep::SampleColumns, b.A, st)) != hipSuccess) return e;
  uint32_t *counts = c_floor >= 0 ? reinterpret_cast<uint32_t *>(static_cast<char *>(ws) + pl.off_ada_hist) : nullptr;
  if ((e = launch_prune_thresholds(pl, b.planes, b.A.row_extra, b.rows, b.n_items, st, c_floor, counts)) != hipSuccess) return e;
  if ((e = launch_prune_list(pl, b.planes, b.rows, b.list, b.items, b.n_items, st)) != hipSuccess) return e;
  return launch(Sweep::Listed, b.A, st);
}

hipError_t launch_prune_repeat(const Plan &pl, const void *q, const void *k, void *ws, uint32_t *hist0, hipStream_t st, int32_t c_floor) {
  Buffers b(pl, q, k, ws);
  b.A.n_items = b.n_items + 1;
  hipError_t e;
  if ((e = launch_prune_check(pl, hist0, b.rows, b.list, b.items, b.n_items + 1, st, c_floor)) != hipSuccess) return e;
  if ((e = launch(Sweep::Listed, b.A, st)) != hipSuccess) return e;
  float *pooled = reinterpret_cast<float *>(static_cast<char *>(ws) + pl.off_pooled);
  return launch_reduce_pool(pl, b.planes, nullptr, pooled, st, hist0, nullptr, b.rows, true);
}

hipError_t launch_prune_token_columns(const Plan &pl, const void *q, const void *k, void *ws, uint32_t *scratch, hipStream_t st) {
  Buffers b(pl, q, k, ws);
  float *merged = reinterpret_cast<float *>(static_cast<char *>(ws) + pl.off_pooled2);
  hipError_t e;
  if ((e = launch(Sweep::SampleColumns, b.A, st)) != hipSuccess) return e;
  if ((e = launch_reduce_pool_all(pl, b.planes, merged, 1, nullptr, 0, st)) != hipSuccess) return e;
  if ((e = launch_prune_thresholds(pl, merged, b.A.row_extra, b.rows, b.n_items, st)) != hipSuccess) return e;
  if ((e = launch_prune_list(pl, merged, b.rows, b.list, b.items, b.n_items, st)) != hipSuccess) return e;
  if ((e = launch(Sweep::Listed, b.A, st)) != hipSuccess) return e;
  if ((e = launch_reduce_pool_all(pl, b.planes, merged, 1, scratch, 2048, st)) != hipSuccess) return e;
  return launch_pool_row(pl, merged, reinterpret_cast<float *>(b.list), pl.d.pool_k, scratch, scratch + 2048, st, b.rows);
}

hipError_t launch_prune_token_repeat(const Plan &pl, const void *q, const void *k, void *ws, uint32_t *scratch, hipStream_t st) {
  Buffers b(pl, q, k, ws);
  float *merged = reinterpret_cast<float *>(static_cast<char *>(ws) + pl.off_pooled2);
  b.A.n_items = b.n_items + 1;
  hipError_t e;
  if ((e = launch_prune_check(pl, scratch, b.rows, b.list, b.items, b.n_items + 1, st)) != hipSuccess) return e;
  if ((e = launch(Sweep::Listed, b.A, st)) != hipSuccess) return e;
  if ((e = launch_reduce_pool_all(pl, b.planes, merged, 1, nullptr, 0, st, b.rows)) != hipSuccess) return e;
  return launch_pool_row(pl, merged, reinterpret_cast<float *>(b.list), pl.d.pool_k, scratch, nullptr, st, b.rows, true);
}

}  // namespace speckv
