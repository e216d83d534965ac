// Pruned scoring: which keys' column sums have to be computed (see score_prune.hip for the whole and the reasons).
//
// A pruned call knows, per output row (layer, sequence, head), the exact scores of a sample of its keys and a bound on the score
// of every other key.  The kernels here take a threshold from the sample and list the keys whose bound reaches it.
#include <algorithm>

#include "first_digit.h"
#include "score_common.h"

namespace speckv {
namespace {

// A bound counts as below a threshold only if it is by this much: the bound's own rounding (probabilities to 2^-13 where
// logits reach 1000, sums to 2^-20) stays inside half of it, and what underflows in the bound inside the other half.
constexpr float kPruneSlack = 1.f / 1024.f;
// Smallest threshold that prunes an output row to which `rows` rows add up (a group's, or all of a call for prompt tokens).  Each may
// lose a probability below 2^(kPruneShift - 126).
__device__ __forceinline__ float prune_floor(int rows) { return (float)rows * __builtin_exp2f(kPruneShift - 126.f) / (0.5f * kPruneSlack); }

__device__ __forceinline__ uint32_t key_of(float x) {            // the selection's ordered key
  const uint32_t u = __float_as_uint(x + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

struct RowAt { int layer, s, g, n, m, tail0; int64_t base; };
__device__ __forceinline__ RowAt row_at(const Dims &d, const SeqTab &t, int row) {
  RowAt r;
  r.g = row % d.Hkv;
  r.s = (row / d.Hkv) % d.S;
  r.layer = row / (d.Hkv * d.S);
  r.n = t.cu[r.s + 1] - t.cu[r.s];
  r.m = r.n - d.w;
  r.tail0 = t.tail0[r.s];
  r.base = (int64_t)r.layer * d.Hkv * d.T + (int64_t)d.Hkv * t.cu[r.s] + (int64_t)r.g * r.n;
  return r;
}

// With three deviations one of 256 rows of 128K falls short in every third call (100 us of 5500 to compute it whole), with three and a half
// seldom; a threshold lower by as much lists a tenth more keys (15 us).
constexpr float kThresholdDeviations = 3.5f;
// Of the sample's pooled scores, how many have to reach a threshold when `expected` of them are among the ones kept.
__device__ __forceinline__ uint32_t wanted_of(float expected, int pool_k) {
  return (uint32_t)ceilf(expected + kThresholdDeviations * sqrtf(expected * (float)pool_k));
}

// A row whose scores from `digit` on are to be found; over: log2 of what its bounds may be too small by; rows: see prune_floor.
__device__ __forceinline__ PruneRow row_from(int digit, float over, int rows) {
  int open;
  const uint32_t key = key_prefix_of((uint32_t)digit, &open);
  const float threshold = key >= 0x80000000u ? __uint_as_float(key ^ 0x80000000u) : 0.f;
  const float bound = threshold * __builtin_exp2f(-over);
  // (written so that a threshold that is not a number lists every key)
  if (bound < prune_floor(rows)) return {-1.f, 0, 0, 0, 0, {0, 0, 0}};
  return {bound * (1.f - kPruneSlack) * __builtin_exp2f(-kPruneShift), digit, 0, 0, 0, {0, 0, 0}};
}

struct Steps { int32_t log[kMaxSeqs]; };

// First references of the rows.  What the sample and the masked tail add up to, S + T, is a lower bound on a row's normaliser,
// but of a row that attends to many keys alike only the sample's share, and the bounds on scores are larger by as much.  The rest of
// such a row is expected from its sample, (ratio - 1) S with ratio = keys / keys in the sample, less four standard deviations,
// ratio sqrt(sum of squared terms), both without the largest term, which is often one key's that all rows attend to: nothing is left
// of it where a few keys make up the row.  A reference that turns out above its normaliser makes the bounds too small by as much,
// which prune_threshold_kernel allows for.  What was seen, S + T, takes the tail's place among the row's pairs.
// Keys listed of 32K with logits of standard deviation 1, a sample of 1/8: 84 % with S + T, 18 % with this; 2: 25 and 6 %; 3 to 8: level.
constexpr float kSampleDeviations = 4.f;
constexpr int kRefThreads = 256;
__global__ __launch_bounds__(kRefThreads) void prune_reference_kernel(PruneArgs A, int tile_keys) {
  const Dims &d = A.d;
  const int RSB = A.g.RSB, s = blockIdx.y;
  const int unit_row = blockIdx.x * kRefThreads + threadIdx.x, unit = unit_row / RSB, r = unit_row % RSB;
  if (unit >= d.L * d.Hkv * A.g.RS) return;
  const int first = A.t.cc[s], n = A.t.cc[s + 1] - first;
  float2 *pairs = A.part + (int64_t)unit * A.g.n_chunks * RSB + r;
  const float *squares = A.squares + (int64_t)unit * A.g.n_fast_chunks * RSB + r;
  const float2 tail = pairs[(int64_t)(A.g.n_fast_chunks + s) * RSB];
  float top = kNegBig, sum = 0.f, square = 0.f;            // of the sample, in units of its largest term
  for (int e0 = 0; e0 < n; e0 += kMergeNext) {
    float2 in[kMergeNext];
    float sq[kMergeNext];
#pragma unroll
    for (int u = 0; u < kMergeNext; ++u) {
      in[u] = e0 + u < n ? pairs[(int64_t)(first + e0 + u) * RSB] : make_float2(kNegBig, 0.f);
      sq[u] = e0 + u < n ? squares[(int64_t)(first + e0 + u) * RSB] : 0.f;
    }
    const float before = top;
    merge_pairs<kMergeNext>(top, sum, in);
    const float f = __builtin_amdgcn_exp2f(before - top);
    square *= f * f;
#pragma unroll
    for (int u = 0; u < kMergeNext; ++u) {
      const float fu = __builtin_amdgcn_exp2f(in[u].x - top);
      square = __builtin_fmaf(sq[u] * fu, fu, square);
    }
  }
  const int step = prune_step(A.chunk_of[s]), tiles = A.t.tail0[s] / tile_keys, sampled = (tiles + (1 << step) - 1) >> step;
  const float ratio = sampled > 0 ? (float)tiles / (float)sampled : 1.f;
  const float rest = (ratio - 1.f) * (sum - 1.f) - kSampleDeviations * ratio * sqrtf(fmaxf(square - 1.f, 0.f));
  const float m = fmaxf(top, tail.x), f1 = __builtin_amdgcn_exp2f(top - m);
  const float seen = sum * f1 + tail.y * __builtin_amdgcn_exp2f(tail.x - m), all = seen + (rest > 0.f ? rest * f1 : 0.f);
  const int rs = unit % A.g.RS, lh = unit / A.g.RS;
  const int64_t at = ((int64_t)lh * d.S + s) * ((int64_t)A.g.RS * RSB) + rs * RSB + r;
  A.lse[at] = m + log2f(all);
  A.row_extra[at] = seen / all;
  // the sample's pairs have served, and the chunks' places are free for those of the other keys
  pairs[(int64_t)(A.g.n_fast_chunks + s) * RSB] = make_float2(m, seen);
}

constexpr int kThrThreads = 1024, kThrEach = 8;

// A row's threshold: the lower end of the largest first digit that enough of the sample's pooled scores reach.  Neighbouring
// pooled scores are one key's, so that `expected` of them are about expected / pool_k independent draws; some standard
// deviations more are asked for, since a row that falls short is computed whole (launch_prune_repeat).
// Bound: the latency of two or three rounds of loads; one workgroup per row.
__global__ __launch_bounds__(kThrThreads) void prune_threshold_kernel(Dims d, SeqTab t, Steps steps, int tile_log, int n_planes,
                                                                      const float *__restrict__ planes,
                                                                      const float *__restrict__ row_extra, int group_rows,
                                                                      PruneRow *__restrict__ rows, int32_t *__restrict__ n_items,
                                                                      int c_floor, uint32_t *__restrict__ counts) {
  __shared__ float score[kThrThreads * kThrEach];
  __shared__ uint32_t hist[2048];
  __shared__ uint32_t wave_tot[kThrThreads / 64];
  __shared__ int digit;
  __shared__ float excess[kThrThreads / 64];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  if (row == 0 && tid < 2) n_items[tid] = 0;
  const RowAt r = row_at(d, t, row);
  const int step = steps.log[r.s], tile = 1 << tile_log;
  if (step == 0) {
    if (tid == 0) rows[row] = {-1.f, 0, 0, 0, 0, {0, 0, 0}};
    return;
  }
  hist[tid] = hist[tid + kThrThreads] = 0;
  if (tid == 0) digit = 0;
  const int n_tiles = ((r.tail0 >> tile_log) + (1 << step) - 1) >> step, n = n_tiles << tile_log;
  const int64_t plane = (int64_t)d.L * d.Hkv * d.T;
  const int before = d.pool_k / 2, after = (d.pool_k - 1) / 2;
  auto key_at = [&](int e) { return ((e >> tile_log) << (tile_log + step)) + (e & (tile - 1)); };
  for (int e0 = 0; e0 < n; e0 += kThrThreads * kThrEach) {            // (whole tiles at a time)
    float v[kThrEach];
#pragma unroll
    for (int u = 0; u < kThrEach; ++u) {
      const int e = e0 + u * kThrThreads + tid;
      v[u] = 0.f;
      if (e < n)
        for (int p = 0; p < n_planes; ++p) v[u] += planes[p * plane + r.base + key_at(e)];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kThrEach; ++u) score[u * kThrThreads + tid] = v[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kThrEach; ++u) {
      const int x = u * kThrThreads + tid, first = x & ~(tile - 1);
      if (e0 + x >= n || key_at(e0 + x) >= r.m) continue;
      const int lo = max(first, x - before), hi = min(first + tile - 1, x + after);
      float best = score[lo];
      for (int y = lo + 1; y <= hi; ++y) best = fmaxf(best, score[y]);
      atomicAdd(&hist[first_digit_of(key_of(best))], 1u);
    }
  }
  __syncthreads();
  // how far the largest reference of the group's rows is above its normaliser
  float over = 0.f;
  for (int x = tid; x < group_rows; x += kThrThreads)
    over = fmaxf(over, row_extra[(((int64_t)r.layer * d.Hkv + r.g) * d.S + r.s) * group_rows + x]);
  for (int o = 32; o > 0; o /= 2) over = fmaxf(over, __shfl_xor(over, o, 64));
  if (lane == 0) excess[tid >> 6] = over;
  const uint32_t wanted = wanted_of((float)(counts != nullptr ? min(c_floor, d.c_max) : d.c_max) * (float)n / (float)r.m, d.pool_k);
  // numbers of scores from digit b on, digits in descending order: thread i has digits 2047 - 2 i and 2046 - 2 i
  const uint32_t c0 = hist[2047 - 2 * tid], c1 = hist[2046 - 2 * tid];
  uint32_t sum = c0 + c1;
  for (int o = 1; o < 64; o *= 2) {
    const uint32_t x = __shfl_up(sum, o, 64);
    if (lane >= o) sum += x;
  }
  if (lane == 63) wave_tot[tid >> 6] = sum;
  __syncthreads();
  for (int w = 0; w < (tid >> 6); ++w) sum += wave_tot[w];
  const uint32_t upto1 = sum, upto0 = sum - c1, none = sum - c1 - c0;
  if (none < wanted && upto0 >= wanted) digit = 2047 - 2 * tid;
  else if (upto0 < wanted && upto1 >= wanted) digit = 2046 - 2 * tid;
  if (counts != nullptr) {
    counts[(int64_t)row * 2048 + 2047 - 2 * tid] = upto0;
    counts[(int64_t)row * 2048 + 2046 - 2 * tid] = upto1;
  }
  __syncthreads();
  if (tid != 0) return;
  for (int w = 0; w < kThrThreads / 64; ++w) over = fmaxf(over, excess[w]);
  if (counts != nullptr) rows[row] = {over, wanted == 0 ? 2047 : digit, 0, 0, 0, {0, 0, 0}};      // see prune_shared_threshold_kernel
  else rows[row] = row_from(digit, over, group_rows);
}

// Shared budget, one workgroup per (layer, sequence), after prune_threshold_kernel: the layer's digit is the largest that so many of the
// samples' scores reach, beyond the heads' floors, as the layer keeps; a head's is no larger, and no larger than the one of its floor.
// Whatever is kept then reaches its head's digit.
__global__ __launch_bounds__(kThrThreads) void prune_shared_threshold_kernel(Dims d, SeqTab t, Steps steps, int tile_log, int c_floor,
                                                                             int group_rows, PruneRow *__restrict__ rows,
                                                                             const uint32_t *__restrict__ counts) {
  __shared__ int layer_digit;
  const int ls = blockIdx.x, s = ls % d.S, tid = threadIdx.x;
  const int step = steps.log[s];
  if (step == 0) return;
  const int n_tiles = ((t.tail0[s] >> tile_log) + (1 << step) - 1) >> step, m = t.cu[s + 1] - t.cu[s] - d.w;
  const float share = (float)(n_tiles << tile_log) / (float)m;
  const int kept = min(d.c_max, m), floor_ = min(c_floor, kept);
  const float need = (float)wanted_of((float)d.Hkv * (float)(kept - floor_) * share, d.pool_k), in_floor = (float)floor_ * share;
  if (tid == 0) layer_digit = 0;
  __syncthreads();
  for (int b = tid; b < 2048; b += kThrThreads) {
    float beyond = 0.f;
    for (int h = 0; h < d.Hkv; ++h) beyond += fmaxf((float)counts[((int64_t)ls * d.Hkv + h) * 2048 + b] - in_floor, 0.f);
    if (beyond >= need) atomicMax(&layer_digit, b);
  }
  __syncthreads();
  if (tid >= d.Hkv) return;
  PruneRow *row = rows + (int64_t)ls * d.Hkv + tid;
  *row = row_from(min(layer_digit, row->digit), row->bound, group_rows);
  row->layer_digit = layer_digit;
}

constexpr int kListThreads = 512, kListEach = 8, kListKeys = kListThreads * kListEach;

// Adds `n` keys to a row's list: returns the place of the first, and makes the items that begin among them (in any order: an
// item's results depend neither on its place nor on the order of its keys).
__device__ __forceinline__ int reserve(PruneRow *rows, int row, int n, int item_keys, int2 *items, int32_t *n_items) {
  const int at = atomicAdd(&rows[row].listed, n);
  const int i0 = (at + item_keys - 1) / item_keys, i1 = (at + n + item_keys - 1) / item_keys;
  if (i1 > i0) {
    const int first = atomicAdd(n_items, i1 - i0);
    for (int i = i0; i < i1; ++i) items[first + i - i0] = make_int2(row, i * item_keys);
  }
  return at;
}

// Lists the keys outside the sample whose bound reaches the row's threshold, kListKeys of the row's keys a workgroup.
// Bound: reading the bounds once.
__global__ __launch_bounds__(kListThreads) void prune_list_kernel(Dims d, SeqTab t, Steps steps, int tile_log, int n_planes, int parts,
                                                                  int item_keys,
                                                                  const float *__restrict__ planes, PruneRow *__restrict__ rows,
                                                                  int32_t *__restrict__ list, int2 *__restrict__ items,
                                                                  int32_t *__restrict__ n_items) {
  __shared__ int wave_tot[kListThreads / 64];
  __shared__ int place;
  const int row = blockIdx.x / parts, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const RowAt r = row_at(d, t, row);
  const int step = steps.log[r.s], j0 = (blockIdx.x % parts) * kListKeys;
  if (step == 0 || j0 >= r.tail0) return;
  const int64_t plane = (int64_t)d.L * d.Hkv * d.T;
  const float bound = rows[row].bound;
  float v[kListEach];
#pragma unroll
  for (int u = 0; u < kListEach; ++u) {
    const int j = j0 + u * kListThreads + tid;
    v[u] = j < r.tail0 ? planes[r.base + j] : 0.f;
  }
  for (int p = 1; p < n_planes; ++p) {
#pragma unroll
    for (int u = 0; u < kListEach; ++u) {
      const int j = j0 + u * kListThreads + tid;
      if (j < r.tail0) v[u] += planes[p * plane + r.base + j];
    }
  }
  uint32_t mine = 0;                        // bit u: key u of the thread is listed
  int n = 0;                                // keys the wavefront lists
#pragma unroll
  for (int u = 0; u < kListEach; ++u) {
    const int j = j0 + u * kListThreads + tid;
    const bool listed = j < r.tail0 && ((j >> tile_log) & ((1 << step) - 1)) != 0 && !(v[u] < bound);
    mine |= (listed ? 1u : 0u) << u;
    n += __popcll(__ballot(listed));
  }
  if (lane == 0) wave_tot[wave] = n;
  __syncthreads();
  int at = 0, total = 0;
  for (int w = 0; w < kListThreads / 64; ++w) {
    if (w < wave) at += wave_tot[w];
    total += wave_tot[w];
  }
  if (tid == 0 && total > 0) place = reserve(rows, row, total, item_keys, items, n_items);
  __syncthreads();
  int32_t *out = list + r.base + place;
  for (int u = 0; u < kListEach; ++u) {
    const bool listed = ((mine >> u) & 1u) != 0;
    const uint64_t b = __ballot(listed);
    if (listed) out[at + __popcll(b & ((1ull << lane) - 1ull))] = j0 + u * kListThreads + tid;
    at += __popcll(b);
  }
}
static_assert(kListEach <= 32, "one bit per key");

// The check that pruning found every score that matters: at least c_max pooled scores, counted by first digit, reach the row's
// digit (shared budget: see there).  A row that falls short lists every key outside the sample, one workgroup per row.
__global__ __launch_bounds__(kListThreads) void prune_check_kernel(Dims d, SeqTab t, Steps steps, int tile_log, int item_keys,
                                                                   const uint32_t *__restrict__ hist0, PruneRow *__restrict__ rows,
                                                                   int32_t *__restrict__ list, int2 *__restrict__ items,
                                                                   int32_t *__restrict__ n_items, int c_floor) {
  __shared__ int wave_tot[kListThreads / 64];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const RowAt r = row_at(d, t, row);
  const int step = steps.log[r.s], digit = rows[row].digit;
  if (step == 0 || digit == 0) return;
  static_assert(kListThreads * 4 == 2048, "four counters per thread");
  const uint4 c = reinterpret_cast<const uint4 *>(hist0 + (int64_t)row * 2048)[tid];
  const int b = tid * 4;
  int n = (b >= digit ? c.x : 0) + (b + 1 >= digit ? c.y : 0) + (b + 2 >= digit ? c.z : 0) + (b + 3 >= digit ? c.w : 0);
  for (int o = 32; o > 0; o /= 2) n += __shfl_xor(n, o, 64);
  if (lane == 0) wave_tot[wave] = n;
  __syncthreads();
  n = 0;
  for (int w = 0; w < kListThreads / 64; ++w) n += wave_tot[w];
  const int kept = min(d.c_max, r.m);
  if (c_floor < 0) {
    if (n >= kept) return;
  } else {
    // shared budget: the head's floor, and with the other heads what the layer keeps beyond the floors
    const int floor_ = min(c_floor, kept), layer_digit = rows[row].layer_digit, row0 = row / d.Hkv * d.Hkv;
    int beyond = 0;
    for (int h = wave; h < d.Hkv; h += kListThreads / 64) {
      const uint32_t *hist = hist0 + (int64_t)(row0 + h) * 2048;
      int reach = 0;
      for (int x = lane; x < 2048; x += 64) reach += x >= layer_digit ? (int)hist[x] : 0;
      for (int o = 32; o > 0; o /= 2) reach += __shfl_xor(reach, o, 64);
      beyond += max(reach - floor_, 0);
    }
    __syncthreads();
    if (lane == 0) wave_tot[wave] = beyond;
    __syncthreads();
    beyond = 0;
    for (int w = 0; w < kListThreads / 64; ++w) beyond += wave_tot[w];
    if (n >= floor_ && beyond >= d.Hkv * (kept - floor_)) return;
  }
  const int tiles = r.tail0 >> tile_log, other = tiles - ((tiles + (1 << step) - 1) >> step);
  if (tid == 0) {
    rows[row].failed = 1;
    rows[row].listed = other << tile_log;
    const int n_new = ((other << tile_log) + item_keys - 1) / item_keys, first = atomicAdd(n_items, n_new);
    for (int i = 0; i < n_new; ++i) items[first + i] = make_int2(row, i * item_keys);
  }
  for (int x = tid; x < other << tile_log; x += kListThreads) {
    const int tile = x >> tile_log;
    list[r.base + x] = ((tile + 1 + tile / ((1 << step) - 1)) << tile_log) + (x & ((1 << tile_log) - 1));
  }
}

Steps steps_of(const Plan &pl) {
  Steps s;
  for (int i = 0; i < pl.d.S; ++i) s.log[i] = prune_step(pl.chunk_of[i]);
  return s;
}
int tile_log_of(const Plan &pl) { return __builtin_ctz((unsigned)prune_tile_keys(pl)); }

}  // namespace

hipError_t launch_prune_references(const PruneArgs &A, int tile_keys, hipStream_t st) {
  const int rows = A.d.L * A.d.Hkv * A.g.RS * A.g.RSB;
  hipLaunchKernelGGL(prune_reference_kernel, dim3((rows + kRefThreads - 1) / kRefThreads, A.d.S), dim3(kRefThreads), 0, st, A, tile_keys);
  return hipGetLastError();
}

// Output rows of a pruned call: of prompt tokens one, the merged planes.
struct RowsOf {
  Dims d;
  unsigned n;
  int planes, group_rows;
  explicit RowsOf(const Plan &pl) : d(pl.d), planes(pl.g.RS), group_rows(pl.g.RS * pl.g.RSB) {
    if (pl.prune_keep != 0) {
      group_rows *= d.L * d.Hkv;
      d.L = d.Hkv = planes = 1;
      d.c_max = pl.prune_keep;
    }
    n = (unsigned)((int64_t)d.L * d.S * d.Hkv);
  }
};

hipError_t launch_prune_thresholds(const Plan &pl, const float *planes, const float *row_extra, PruneRow *rows, int32_t *n_items,
                                   hipStream_t st, int32_t c_floor, uint32_t *counts) {
  const RowsOf r(pl);
  hipLaunchKernelGGL(prune_threshold_kernel, dim3(r.n), dim3(kThrThreads), 0, st, r.d, pl.t, steps_of(pl), tile_log_of(pl), r.planes,
                     planes, row_extra, r.group_rows, rows, n_items, c_floor, counts);
  if (counts != nullptr)
    hipLaunchKernelGGL(prune_shared_threshold_kernel, dim3((unsigned)(r.d.L * r.d.S)), dim3(kThrThreads), 0, st, r.d, pl.t, steps_of(pl),
                       tile_log_of(pl), c_floor, r.group_rows, rows, counts);
  return hipGetLastError();
}

hipError_t launch_prune_list(const Plan &pl, const float *planes, PruneRow *rows, int32_t *list, int2 *items, int32_t *n_items,
                             hipStream_t st) {
  const RowsOf r(pl);
  int most = 0;
  for (int s = 0; s < pl.d.S; ++s)
    if (prune_step(pl.chunk_of[s]) != 0) most = std::max(most, pl.t.tail0[s]);
  const int parts = (most + kListKeys - 1) / kListKeys;
  hipLaunchKernelGGL(prune_list_kernel, dim3(r.n * (unsigned)parts), dim3(kListThreads), 0, st, r.d, pl.t, steps_of(pl),
                     tile_log_of(pl), r.planes, parts, pl.item_keys, planes, rows, list, items, n_items);
  return hipGetLastError();
}

hipError_t launch_prune_check(const Plan &pl, const uint32_t *hist0, PruneRow *rows, int32_t *list, int2 *items, int32_t *n_items,
                              hipStream_t st, int32_t c_floor) {
  const RowsOf r(pl);
  hipLaunchKernelGGL(prune_check_kernel, dim3(r.n), dim3(kListThreads), 0, st, r.d, pl.t, steps_of(pl), tile_log_of(pl), pl.item_keys,
                     hist0, rows, list, items, n_items, c_floor);
  return hipGetLastError();
}

}  // namespace speckv
