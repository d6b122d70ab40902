// Softmax statistics and top-K candidate selection over the full vocabulary: one
// workgroup per row (the row code is in sweep.h).
//
// Method / Unigram Proposer, Eq. (ubtree-unigram), q_i = softmax(u_i), and "Candidate
// Sets": C_i = the K tokens of largest q_i, ranked on the logits with ties to the lower
// token id.
#include "sweep.h"
#include "sweep_big.h"
#include "ubt_launch.h"

namespace ubt {
namespace {

// kBig: K > 16 (a tighter first threshold, a larger buffer with a running top K instead
// of the re-scan, and the workgroup-wide selection of sweep_big.h).
template <typename T, int kRows, bool kBig>
__global__ __launch_bounds__(kWave* kWaves, 4) void topk_row_kernel(const T* __restrict__ logits, int gamma,
                                                                    int64_t V, int64_t stride_b, int64_t stride_i,
                                                                    int K, int32_t* __restrict__ cand_ids,
                                                                    float* __restrict__ cand_logit,
                                                                    float* __restrict__ cand_logprob,
                                                                    float* __restrict__ lse) {
  const int64_t row = blockIdx.x;
  const int64_t b = row / gamma, i = row - b * gamma;
  const RowOut out{cand_ids, cand_logit, cand_logprob, lse, false};
  if constexpr (kBig) {
    __shared__ BigRowLds lds;
    sweep_row_big<T, kRows>(lds, logits + b * stride_b + i * stride_i, V, K, row, out);
  } else {
    __shared__ RowLds lds;
    sweep_row<T, kRows, kWaves, false>(lds, logits + b * stride_b + i * stride_i, V, K, row, out);
  }
}

// ---- few rows: each row cut over several workgroups -----------------------------------
//
// One workgroup per row leaves most compute units idle when there are few rows.  A chunk's
// workgroup runs the same sweep on its elements and leaves its maximum, sum of exponentials
// and sorted top K in the workspace; the merge kernel combines them in chunk order.
constexpr int kSplitChunks = 8;
constexpr int kMergeThreads = kSplitChunks * 64;  // one per chunk candidate

struct SplitArgs {
  int tiles;          // of a row; chunk c starts at tile c tiles / kSplitChunks
  int32_t* ids;       // [rows][chunks][K] sorted, ids relative to the chunk
  float* logit;       // [rows][chunks][K]
  float* sum;         // [rows][chunks]
  float* row_max;     // [rows][chunks]
};

template <typename T>
__device__ __forceinline__ int64_t chunk_start(const SplitArgs& p, int c) {
  constexpr int64_t SUB = static_cast<int64_t>(kSubGroups) * kWave * Traits<T>::kPer;
  return static_cast<int64_t>(c) * p.tiles / kSplitChunks * SUB;
}

template <typename T, int kRows, bool kBig>
__global__ __launch_bounds__(kWave* kWaves, 4) void topk_chunk_kernel(const T* __restrict__ logits, int gamma,
                                                                      int64_t V, int64_t stride_b, int64_t stride_i,
                                                                      int K, SplitArgs p) {
  const int64_t rc = blockIdx.x;
  const int64_t row = rc / kSplitChunks;
  const int c = static_cast<int>(rc - row * kSplitChunks);
  const int64_t c0 = chunk_start<T>(p, c);
  const int64_t b = row / gamma, i = row - b * gamma;
  const int64_t len = (c == kSplitChunks - 1 ? V : chunk_start<T>(p, c + 1)) - c0;
  const T* rp = logits + b * stride_b + i * stride_i + c0;
  const RowOut out{p.ids, p.logit, nullptr, p.sum, false, p.row_max};
  if constexpr (kBig) {
    __shared__ BigRowLds lds;
    sweep_row_big<T, kRows>(lds, rp, len, K, rc, out);
  } else {
    __shared__ RowLds lds;
    sweep_row<T, kRows, kWaves, false>(lds, rp, len, K, rc, out);
  }
}

// One workgroup per row: a chunk candidate's rank is its place in its own list plus, for
// every other list, the entries above it (binary search in the sorted list).
template <typename T>
__global__ __launch_bounds__(kMergeThreads) void topk_merge_kernel(SplitArgs p, int K, int32_t* __restrict__ cand_ids,
                                                                   float* __restrict__ cand_logit,
                                                                   float* __restrict__ cand_logprob,
                                                                   float* __restrict__ lse) {
  __shared__ uint64_t ord[kMergeThreads];
  const int t = static_cast<int>(threadIdx.x);
  const int64_t row = blockIdx.x;
  constexpr int C = kSplitChunks;
  const bool on = t < C * K;
  const int c = on ? t / K : 0, e = on ? t - c * K : 0;
  float v = 0.f;
  uint32_t id = 0u;
  uint64_t mine = 0ull;
  if (on) {
    const int64_t o = row * C * K + t;
    id = static_cast<uint32_t>(p.ids[o] + chunk_start<T>(p, c));
    v = p.logit[o];
    mine = cand_order(Traits<T>::key_value(v), id);
  }
  float m = neg_inf(), s = 0.f;
  float cm[kSplitChunks], cs[kSplitChunks];
#pragma unroll
  for (int j = 0; j < kSplitChunks; ++j) {
    cm[j] = p.row_max[row * C + j];
    cs[j] = p.sum[row * C + j];
  }
  if (on) ord[t] = mine;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSplitChunks; ++j) m = fmaxf(m, cm[j]);
#pragma unroll
  for (int j = 0; j < kSplitChunks; ++j)
    if (cm[j] != neg_inf()) s += cs[j] * fast_exp2((cm[j] - m) * kLog2e);
  const float l = m == neg_inf() ? neg_inf() : m + fast_log2(s) * kLn2;
  if (t == 0 && lse) lse[row] = l;
  if (!on) return;
  int lo[kSplitChunks];  // entries of list j known to be above mine
#pragma unroll
  for (int j = 0; j < kSplitChunks; ++j) lo[j] = 0;
  for (int step = 64; step > 0; step >>= 1) {
#pragma unroll
    for (int j = 0; j < kSplitChunks; ++j)
      if (lo[j] + step <= K && ord[j * K + lo[j] + step - 1] > mine) lo[j] += step;
  }
  int rank = e;
#pragma unroll
  for (int j = 0; j < kSplitChunks; ++j) rank += j != c ? lo[j] : 0;
  if (rank < K) {
    const int64_t o = row * K + rank;
    cand_ids[o] = static_cast<int32_t>(id);
    cand_logit[o] = v;
    if (cand_logprob) cand_logprob[o] = v - l;
  }
}

size_t up256(size_t n) { return (n + 255) & ~static_cast<size_t>(255); }

struct SplitPlan {
  int tiles;  // of a row; 0: not cut
  size_t ids, logit, sum, row_max, total;
};

// Rows are cut when there are at most 32 of at least 64 tiles of bf16 (131,072 elements) or 96
// of fp32 (98,304).  A chunk keeps a row's start and selection (about 10 us at K = 64) and the
// merge adds 5 us, so only a long row has enough streaming to share out; with more rows the
// chunks of one compute unit queue up.  bf16, whole / cut: 15 rows of 151,936 14.1 / 12.4 us at
// K = 4, 17.8 / 14.1 at K = 16, 23.4 / 18.3 at K = 64; one row of 129,280 at K = 1 10.1 / 10.2;
// 60 rows 23.2 / 22.3, 240 rows 24.1 / 28.1 (K = 64); 15 rows of 50,000 13.9 / 16.2.  fp32: 15
// rows of 100,000 14.2 / 12.2 us at K = 4, 23.7 / 19.1 at K = 64; of 72,000 11.0 / 11.7 at K = 4.
// The chunks have a row's tiles in equal shares, at least 8 each: a last chunk of one tile has
// too few lanes for a bound on the K-th element (15 rows of 131,100 in chunks of 9 tiles and
// a rest, K = 64: 30.4 us, whole 25.6).
constexpr int kSplitMaxRows = 32, kSplitMinTiles16 = 64, kSplitMinTiles32 = 96;

SplitPlan split_plan(int64_t rows, int64_t V, int K, int dtype) {
  SplitPlan p{};
  const int64_t tile = static_cast<int64_t>(kSubGroups) * kWave * (dtype == 1 ? 8 : 4);
  const int64_t tiles = (V + tile - 1) / tile;
  if (rows > kSplitMaxRows || tiles < (dtype == 1 ? kSplitMinTiles16 : kSplitMinTiles32)) return p;
  p.tiles = static_cast<int>(tiles);
  const size_t n = static_cast<size_t>(rows) * kSplitChunks;
  p.ids = 0;
  p.logit = p.ids + up256(n * K * sizeof(int32_t));
  p.sum = p.logit + up256(n * K * sizeof(float));
  p.row_max = p.sum + up256(n * sizeof(float));
  p.total = p.row_max + up256(n * sizeof(float));
  return p;
}

template <typename T, bool kAligned>
void launch_split(const void* logits, int B, int gamma, int64_t V, int64_t stride_b, int64_t stride_i, int K,
                  int32_t* cand_ids, float* cand_logit, float* cand_logprob, float* lse, const SplitArgs& p,
                  hipStream_t stream) {
  const int64_t rows = static_cast<int64_t>(B) * gamma;
  const dim3 grid(static_cast<unsigned>(rows * kSplitChunks)), block(kWave * kWaves);
  if (K > 16)
    hipLaunchKernelGGL((topk_chunk_kernel<T, kAligned ? kRaggedRows : kAnyRows, true>), grid, block, 0, stream,
                       static_cast<const T*>(logits), gamma, V, stride_b, stride_i, K, p);
  else
    hipLaunchKernelGGL((topk_chunk_kernel<T, kAligned ? kWholeRows : kAnyRows, false>), grid, block, 0, stream,
                       static_cast<const T*>(logits), gamma, V, stride_b, stride_i, K, p);
  const int threads = (kSplitChunks * K + kWave - 1) / kWave * kWave;
  hipLaunchKernelGGL((topk_merge_kernel<T>), dim3(static_cast<unsigned>(rows)), dim3(static_cast<unsigned>(threads)),
                     0, stream, p, K, cand_ids, cand_logit, cand_logprob, lse);
}

template <typename T, bool kAligned>
void launch_typed(const void* logits, int B, int gamma, int64_t V, int64_t stride_b, int64_t stride_i, int K,
                  int32_t* cand_ids, float* cand_logit, float* cand_logprob, float* lse, hipStream_t stream) {
  const int64_t rows = static_cast<int64_t>(B) * gamma;
  if (K > 16)
    hipLaunchKernelGGL((topk_row_kernel<T, kAligned ? kRaggedRows : kAnyRows, true>), dim3(static_cast<unsigned>(rows)),
                       dim3(kWave * kWaves), 0, stream, static_cast<const T*>(logits), gamma, V, stride_b, stride_i, K,
                       cand_ids, cand_logit, cand_logprob, lse);
  else
    hipLaunchKernelGGL((topk_row_kernel<T, kAligned ? kWholeRows : kAnyRows, false>), dim3(static_cast<unsigned>(rows)),
                       dim3(kWave * kWaves), 0, stream, static_cast<const T*>(logits), gamma, V, stride_b, stride_i, K,
                       cand_ids, cand_logit, cand_logprob, lse);
}

}  // namespace

size_t topk_workspace_bytes(int B, int gamma, int64_t V, int K, int dtype) {
  return split_plan(static_cast<int64_t>(B) * gamma, V, K, dtype).total;
}

hipError_t launch_topk(const void* logits, int dtype, bool aligned, int B, int gamma, int64_t V, int64_t stride_b,
                       int64_t stride_i, int K, int32_t* cand_ids, float* cand_logit, float* cand_logprob, float* lse,
                       void* workspace, size_t ws_bytes, hipStream_t stream) {
  // Rows that start on 16 bytes need no mask at their start, and those of whole 16-byte groups none
  // inside a group either (RowIn); past K = 16 the kernel masks the end of any row, up to the
  // longest whose 16-byte groups one descriptor can state.
  const int64_t bytes = V * (dtype == 1 ? 2 : 4);
  aligned = aligned && (K > 16 ? bytes <= (int64_t(1) << 32) - 16 : bytes % 16 == 0);
  if (workspace) {
    const SplitPlan sp = split_plan(static_cast<int64_t>(B) * gamma, V, K, dtype);
    if (sp.tiles != 0 && ws_bytes >= sp.total) {
      char* ws = static_cast<char*>(workspace);
      SplitArgs p{};
      p.tiles = sp.tiles;
      p.ids = reinterpret_cast<int32_t*>(ws + sp.ids);
      p.logit = reinterpret_cast<float*>(ws + sp.logit);
      p.sum = reinterpret_cast<float*>(ws + sp.sum);
      p.row_max = reinterpret_cast<float*>(ws + sp.row_max);
#define UBT_SPLIT(T, AL) \
  launch_split<T, AL>(logits, B, gamma, V, stride_b, stride_i, K, cand_ids, cand_logit, cand_logprob, lse, p, stream)
      if (dtype == 1) {
        if (aligned)
          UBT_SPLIT(uint16_t, true);
        else
          UBT_SPLIT(uint16_t, false);
      } else {
        if (aligned)
          UBT_SPLIT(float, true);
        else
          UBT_SPLIT(float, false);
      }
#undef UBT_SPLIT
      return hipGetLastError();
    }
  }
  if (dtype == 1) {
    if (aligned)
      launch_typed<uint16_t, true>(logits, B, gamma, V, stride_b, stride_i, K, cand_ids, cand_logit, cand_logprob,
                                   lse, stream);
    else
      launch_typed<uint16_t, false>(logits, B, gamma, V, stride_b, stride_i, K, cand_ids, cand_logit, cand_logprob,
                                    lse, stream);
  } else {
    if (aligned)
      launch_typed<float, true>(logits, B, gamma, V, stride_b, stride_i, K, cand_ids, cand_logit, cand_logprob, lse,
                                stream);
    else
      launch_typed<float, false>(logits, B, gamma, V, stride_b, stride_i, K, cand_ids, cand_logit, cand_logprob, lse,
                                 stream);
  }
  return hipGetLastError();
}

}  // namespace ubt
