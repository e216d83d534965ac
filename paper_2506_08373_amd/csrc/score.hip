// Importance scoring: the kernels that may stand between the two sweeps and the host entry that strings the
// sweeps together (Sec. 3.1 Eq. 1; Alg. 1 CrossAttention and reduce steps).  The sweeps themselves
// are in score_sweep.h (compiled in score_rows.hip and score_cols.hip) and score_qs.hip.
#include <algorithm>
#include <map>
#include <mutex>
#include <utility>

#include "score_common.h"

namespace speckv {
namespace {

// Merges the per-chunk (max2, sum) pairs of each row into lse2 = max2 + log2(sum), in the order of merge_pairs.
// A block covers 64 rows.
constexpr int kMergeRows = 64;

// Up to this many chunks a sequence, every workgroup of the column sweep merges the pairs of its own rows instead, and
// converts a caller's normalisers by itself: the kernel is a launch of 3 to 5 us between two sweeps that wait for each other,
// while the pairs (8 bytes per row and chunk, 1 to 2 us for 32 chunks of 512 rows) arrive beside the first key tile.
// Calls with the kernel / without: one layer of 4K keys 48.1 / 45.1 us, 32K (29 chunks) 120.3 / 116.7, 128K (32 chunks)
// 348.6 / 344.2, 4 layers x 60K with a caller's normalisers 267.7 / 262.2, 32 layers x 16K 1113 / 1109.  With more chunks the
// workgroups' reads (the same pairs again for every chunk) outgrow the launch.
constexpr int kMergeInSweep = 40;

// row_extra: of a pruned call, whose first references stand in A.lse (score_prune.hip).
template <int SLICES>
__global__ __launch_bounds__(kMergeRows * SLICES) void lse_combine_kernel(ScoreArgs A, float *row_extra) {
  clear_scratch(A, ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x,
                (int64_t)gridDim.x * gridDim.y * blockDim.x);
  __shared__ float2 partial[SLICES][kMergeRows];
  const Dims &d = A.d;
  const int RSB = A.g.RSB;
  const int blocks_per_unit = RSB / kMergeRows;
  const int unit = blockIdx.x / blocks_per_unit;     // (layer, head, row super-block)
  const int r = (blockIdx.x % blocks_per_unit) * kMergeRows + (threadIdx.x % kMergeRows);
  const int slice = threadIdx.x / kMergeRows;
  const int s = blockIdx.y;
  const int rs = unit % A.g.RS;
  const int lh = unit / A.g.RS;                       // layer * Hkv + head
  const int n_entries = A.t.cc[s + 1] - A.t.cc[s] + 1;
  const float2 *pp = A.part + ((int64_t)unit * A.g.n_chunks) * RSB + r;
  float top = kNegBig, sum = 0.f;
  constexpr int BATCH = kMergeFirst / SLICES;         // entries requested together
  for (int e0 = slice; e0 < n_entries; e0 += BATCH * SLICES) {
    float2 in[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int e = e0 + u * SLICES;
      in[u] = e < n_entries ? pp[(int64_t)(e == 0 ? A.g.n_fast_chunks + s : A.t.cc[s] + e - 1) * RSB] : make_float2(kNegBig, 0.f);
    }
    if (e0 == slice) {
      merge_pairs(top, sum, in);
    } else {
#pragma unroll
      for (int u = 0; u < BATCH; u += kMergeNext) merge_pairs<kMergeNext>(top, sum, in + u);
    }
  }
  if constexpr (SLICES > 1) {
    partial[slice][threadIdx.x % kMergeRows] = make_float2(top, sum);
    __syncthreads();
    if (slice != 0) return;
    float2 in[SLICES - 1];
#pragma unroll
    for (int u = 1; u < SLICES; ++u) in[u - 1] = partial[u][threadIdx.x];
    merge_pairs(top, sum, in);
  }
  const int64_t at = ((int64_t)lh * d.S + s) * ((int64_t)A.g.RS * RSB) + rs * RSB + r;
  const float lse = top + log2f(sum);
  if (row_extra != nullptr) {
    int hh, i;
    row_extra[at] = decode_row(d, A.g, rs, r, &hh, &i) ? A.lse[at] - lse : -INFINITY;
  }
  A.lse[at] = lse;
}

// Converts caller-supplied natural-log normalisers [L][S][R][Hq] into the padded log2 layout
// the column-reduction sweep reads.
__global__ __launch_bounds__(256) void lse_import_kernel(ScoreArgs A) {
  clear_scratch(A, ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x,
                (int64_t)gridDim.x * gridDim.y * blockDim.x);
  const Dims &d = A.d;
  const int RSB = A.g.RSB;
  const int unit = blockIdx.x;            // (layer, head, row super-block)
  const int s = blockIdx.y;
  const int rs = unit % A.g.RS;
  const int lh = unit / A.g.RS;           // layer * Hkv + head
  const int g = lh % d.Hkv, layer = lh / d.Hkv;
  for (int lr = threadIdx.x; lr < RSB; lr += blockDim.x) {
    int hh, i;
    float v = 0.f;
    if (decode_row(d, A.g, rs, lr, &hh, &i))
      v = A.lse_in[(((int64_t)layer * d.S + s) * d.R + i) * d.Hq + g * d.G + hh] * 1.4426950408889634f;
    A.lse[((int64_t)lh * d.S + s) * ((int64_t)A.g.RS * RSB) + rs * RSB + lr] = v;
  }
}

}  // namespace

// Raises a kernel's dynamic LDS limit; the runtime call is made once per (device, kernel, size)
// and remembered, so a fused call does not pay for it on every launch.
hipError_t allow_dynamic_lds(const void *kernel, size_t bytes) {
  static std::mutex mu;
  static std::map<std::pair<int, const void *>, size_t> granted;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  size_t &have = granted[std::make_pair(dev, kernel)];
  if (have >= bytes && have != 0) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) have = bytes;
  return e;
}

int64_t score_fail_words(const Dims &d, const ScoreGeom &g, int64_t n_fast_chunks) {
  return score_chunk_workgroups(d, g, n_fast_chunks) * kFailWaves * kFailWords;
}

bool score_uses_qs(const Plan &pl, int pass) {
  ScoreArgs A;
  A.d = pl.d; A.t = pl.t; A.g = pl.g;
  A.q = nullptr; A.k = nullptr; A.part = nullptr; A.lse = nullptr; A.planes = nullptr; A.lse_in = nullptr; A.chunk_blocks = 0; A.clear = nullptr; A.clear_words = 0; A.fail = nullptr; A.norm_from = kNormMerged; A.share = 0;
  return qs_supported(A, pass);
}

hipError_t launch_lse_combine(const ScoreArgs &A, float *row_extra, hipStream_t st) {
  const dim3 blocks(A.d.L * A.d.Hkv * A.g.RS * (A.g.RSB / kMergeRows), A.d.S);
  if (merge_slices(A.g.MB) == 1) hipLaunchKernelGGL(lse_combine_kernel<1>, blocks, dim3(kMergeRows), 0, st, A, row_extra);
  else hipLaunchKernelGGL(lse_combine_kernel<2>, blocks, dim3(kMergeRows * 2), 0, st, A, row_extra);
  return hipGetLastError();
}

hipError_t launch_score(const Plan &pl, const void *q, const void *k, float2 *part, float *lse,
                        float *planes, hipStream_t st, hipEvent_t *events, const float *lse_in,
                        uint32_t *clear, int64_t clear_words) {
  ScoreArgs A;
  A.d = pl.d; A.t = pl.t; A.g = pl.g;
  A.q = (const char *)q; A.k = (const char *)k;
  A.part = part; A.lse = lse; A.planes = planes; A.lse_in = lse_in; A.chunk_blocks = 0;
  A.clear = clear; A.clear_words = clear != nullptr ? clear_words : 0;
  A.share = A.d.reduce_max == 0 || A.d.head_max != 0;        // a head's own maximum is taken over whole blocks
  A.norm_from = kNormMerged;
  if (!qs_supported(A, 2)) {
    int most = 0;                       // chunks of a sequence
    for (int s = 0; s < A.d.S; ++s) most = std::max(most, A.t.cc[s + 1] - A.t.cc[s]);
    if (lse_in != nullptr) A.norm_from = kNormCaller;
    else if (most <= kMergeInSweep) A.norm_from = kNormPairs;
  }
  A.fail = reinterpret_cast<int32_t *>(part + (int64_t)A.d.L * A.d.Hkv * A.g.RS * A.g.n_chunks * A.g.RSB);
  hipEvent_t *ev = events;
  hipError_t e;
  if (ev && (e = hipEventRecord(ev[0], st)) != hipSuccess) return e;
  if (A.lse_in == nullptr && (e = launch_row_statistics_sweep(A, st)) != hipSuccess) return e;
  if (ev && (e = hipEventRecord(ev[1], st)) != hipSuccess) return e;
  if (A.norm_from != kNormMerged) {
    // nothing: the column sweep makes its normalisers
  } else if (A.lse_in == nullptr) {
    e = launch_lse_combine(A, nullptr, st);
    if (e != hipSuccess) return e;
  } else {
    hipLaunchKernelGGL(lse_import_kernel, dim3(A.d.L * A.d.Hkv * A.g.RS, A.d.S), dim3(256), 0, st, A);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (ev && (e = hipEventRecord(ev[2], st)) != hipSuccess) return e;
  if ((e = launch_column_sweep(A, st)) != hipSuccess) return e;
  if (ev && (e = hipEventRecord(ev[3], st)) != hipSuccess) return e;
  return hipSuccess;
}

}  // namespace speckv
