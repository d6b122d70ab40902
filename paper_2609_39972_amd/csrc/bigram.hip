// Selector scores and normalised transition log-probabilities for every adjacent
// candidate pair.
//
// Background, Eq. (dflash2-selector): delta_i(a,b) = (P(h_i) (.) phi(a))^T psi(b).
// Method / Parallel Computation, Eq. (ubtree-edge-matrix): all pairs of one depth form
// Delta_i = Phi_{i-1} diag(P(h_i)) Psi_i^T, with C_0 = {x_0} (one row at depth 1).
// Method / Depth Calibration, Eq. (ubtree-depth): s_i = alpha_i u_i(b) + lambda_i delta_i.
// Appendix A / Path Scores, Eq. (ubtree-path): log q^bi(b|a) = s_i(a,b) - log sum_v exp s_i(a,v).
// Without the normalisation (normalise = false) the same kernels write s_i itself: the
// edge scores of the unigram-plus-bigram scoring, given the candidates' log-probabilities
// in place of their logits.
//
// bf16 features: the rows of Phi and Psi are gathered straight into MFMA operand
// registers (v_mfma_f32_16x16x32_bf16, 16x16 output tiles).  K <= 16 (one tile) takes one
// wavefront per (sequence, depth).  Larger K takes one wavefront per row of output tiles:
// the waves split the r-contraction between them (wave w takes the 32-wide k-steps
// w, w + KT, ...), so each gathers a fraction of the rows' slots and all of its loads are
// in flight at once; the partial tiles then meet in LDS, each wave sums its own tile row
// over the waves in wave order and runs that row's epilogue (bigram_split_tile).  The
// gate is folded into the predecessor operand: g_k * phi_k(a) is exact in fp32 (two 8-bit
// significands) and is split into hi + lo bf16 parts, so the two MFMAs form every product
// g_k phi_k(a) psi_k(b) exactly and only the fp32 accumulation rounds.  The row
// log-softmax runs on the accumulator tile: a row of the tile lives in one aligned group
// of 16 lanes.  fp32 features use fp32 FMAs on the vector ALUs.
#include "bigram_tile.h"
#include "ubt_launch.h"

namespace ubt {
namespace {

template <bool kNormalise>
__global__ __launch_bounds__(kWave) void bigram_bf16_kernel(const uint16_t* __restrict__ phi,
                                                            const uint16_t* __restrict__ psi,
                                                            const uint16_t* __restrict__ gate, int64_t V, int r,
                                                            const int32_t* __restrict__ anchor,
                                                            const int32_t* __restrict__ cand_ids,
                                                            const float* __restrict__ cand_logit, Scales sc,
                                                            int gamma, int K, float* __restrict__ delta,
                                                            float* __restrict__ logq) {
  const int64_t bi = blockIdx.x;  // b * gamma + i
  const int i = static_cast<int>(bi % gamma);
  const int64_t b = bi / gamma;
  bigram_tile_bf16<1, kNormalise>(phi, psi, gate + bi * r, V, r, i, K, anchor + b, i > 0 ? cand_ids + (bi - 1) * K : cand_ids, cand_ids + bi * K,
                       cand_logit + bi * K, sc.alpha[i], sc.lambda[i], delta ? delta + bi * K * K : nullptr,
                       logq + bi * K * K, nullptr, static_cast<int>(threadIdx.x));
}

template <int KT, bool kNormalise>  // output tiles per side, 16 (KT - 1) < K <= 16 KT; KT waves
__global__ __launch_bounds__(KT * kWave) __attribute__((amdgpu_waves_per_eu(2))) void bigram_bf16_split_kernel(
    const uint16_t* __restrict__ phi, const uint16_t* __restrict__ psi, const uint16_t* __restrict__ gate, int64_t V,
    int r, const int32_t* __restrict__ anchor, const int32_t* __restrict__ cand_ids,
    const float* __restrict__ cand_logit, Scales sc, int gamma, int K, float* __restrict__ delta,
    float* __restrict__ logq) {
  __shared__ f32x4 part[kSplitPartBytes<KT> / sizeof(f32x4)];
  const int lane = static_cast<int>(threadIdx.x) & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int64_t bi = blockIdx.x;  // b * gamma + i
  const int i = static_cast<int>(bi % gamma);
  const int64_t b = bi / gamma;
  bigram_split_tile<KT, kNormalise>(phi, psi, gate + bi * r, V, r, i, K, anchor + b,
                                    i > 0 ? cand_ids + (bi - 1) * K : cand_ids, cand_ids + bi * K, cand_logit + bi * K,
                                    sc.alpha[i], sc.lambda[i], delta ? delta + bi * K * K : nullptr, logq + bi * K * K,
                                    part, w, lane);
}

constexpr int kF32Threads = 256;
constexpr int kF32Chunk = 32;               // features staged at a time
constexpr int kF32Stride = kF32Chunk + 4;   // floats per staged row: 16 consecutive rows hit distinct banks

// fp32 features: one workgroup per (sequence, position).  Latency and LDS bound (2 K^2 r
// flops on 2 K r gathered floats): the candidates' rows come in chunks of 32 features
// (whole cache lines, 32 lanes per row) with the gate folded into the predecessors' rows,
// and each thread forms TM x TM scores from registers.  Every score is one chain of fused
// multiply-adds in feature order, and a row's normaliser sums its candidates in order.
// (One wave reading both rows of a pair from memory took 217 us at B = 100, gamma = 20,
// K = 24, r = 96, this 17 us.)
// TM: scores per thread and side, TM >= K / 16.
template <int TM>
__global__ __launch_bounds__(kF32Threads) void bigram_f32_kernel(
    const float* __restrict__ phi, const float* __restrict__ psi, const float* __restrict__ gate, int64_t V, int r,
    const int32_t* __restrict__ anchor, const int32_t* __restrict__ cand_ids, const float* __restrict__ cand_logit,
    Scales sc, int gamma, int K, float* __restrict__ delta, float* __restrict__ logq, int normalise) {
  constexpr int kMax = 16 * TM;  // most candidates
  __shared__ __align__(16) float s_a[kMax * kF32Stride], s_b[kMax * kF32Stride];
  __shared__ float s_delta[kMax * (kMax + 1)];
  __shared__ float s_u[kMax], s_norm[kMax];
  __shared__ int32_t s_pred[kMax], s_succ[kMax];
  const int tid = static_cast<int>(threadIdx.x);
  const int64_t bi = blockIdx.x;
  const int i = static_cast<int>(bi % gamma);
  const int64_t b = bi / gamma;
  const int n_pred = (i == 0) ? 1 : K;
  const float al = sc.alpha[i], la = sc.lambda[i];
  if (tid < K) {
    s_succ[tid] = static_cast<int32_t>(clamp_id(cand_ids[bi * K + tid], V));
    s_u[tid] = al * cand_logit[bi * K + tid];
    if (tid < n_pred) s_pred[tid] = static_cast<int32_t>(clamp_id(i == 0 ? anchor[b] : cand_ids[(bi - 1) * K + tid], V));
  }
  __syncthreads();
  const float* g = gate + bi * r;
  // Thread (ta, tb) owns the pairs (ta + nT x, tb + nT y).
  const int nT = (K + TM - 1) / TM;
  const int ta = tid / nT, tb = tid - ta * nT;
  const bool work = ta < nT && ta < n_pred;
  const float* pa[TM];
  const float* pb[TM];
#pragma unroll
  for (int x = 0; x < TM; ++x) {  // rows past the end repeat a valid one, never stored
    const int ra = ta + nT * x, rb = tb + nT * x;
    pa[x] = s_a + (work && ra < n_pred ? ra : 0) * kF32Stride;
    pb[x] = s_b + (rb < K ? rb : 0) * kF32Stride;
  }
  float d[TM][TM] = {};
  const int col = tid % kF32Chunk, row0 = tid / kF32Chunk;
  for (int k0 = 0; k0 < r; k0 += kF32Chunk) {
    const int kc = r - k0 < kF32Chunk ? r - k0 : kF32Chunk;  // 16 or 32
    if (col < kc) {
      const float gk = g[k0 + col];
#pragma unroll 4
      for (int e = row0; e < K; e += kF32Threads / kF32Chunk) {
        s_b[e * kF32Stride + col] = psi[static_cast<int64_t>(s_succ[e]) * r + k0 + col];
        if (e < n_pred) s_a[e * kF32Stride + col] = gk * phi[static_cast<int64_t>(s_pred[e]) * r + k0 + col];
      }
    }
    __syncthreads();
    if (work) {
      for (int k = 0; k < kc; k += 4) {
        f32x4 va[TM], vb[TM];
#pragma unroll
        for (int x = 0; x < TM; ++x) {
          va[x] = *reinterpret_cast<const f32x4*>(pa[x] + k);
          vb[x] = *reinterpret_cast<const f32x4*>(pb[x] + k);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int y = 0; y < TM; ++y) d[x][y] = fmaf(va[x][j], vb[y][j], d[x][y]);
      }
    }
    __syncthreads();
  }
  if (work) {
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
      for (int y = 0; y < TM; ++y)
        if (ta + nT * x < n_pred && tb + nT * y < K) s_delta[(ta + nT * x) * (kMax + 1) + tb + nT * y] = d[x][y];
  }
  __syncthreads();
  if (tid < n_pred) {
    float norm = 0.f;
    if (normalise) {
      const float* sd = s_delta + tid * (kMax + 1);
      float m = neg_inf();
      for (int c = 0; c < K; ++c) m = fmaxf(m, fmaf(la, sd[c], s_u[c]));
      float e = 0.f;
      for (int c = 0; c < K; ++c) e += __builtin_amdgcn_exp2f((fmaf(la, sd[c], s_u[c]) - m) * kLog2e);
      norm = m + __builtin_amdgcn_logf(e) * kLn2;
    }
    s_norm[tid] = norm;
  }
  __syncthreads();
  float* dslab = delta ? delta + bi * K * K : nullptr;
  float* qslab = logq + bi * K * K;
  for (int e = tid; e < K * K; e += kF32Threads) {
    const int a = e / K, c = e - a * K;
    const bool live = a < n_pred;  // depth 1: row 0 holds the scores, the others are 0
    const float dv = live ? s_delta[a * (kMax + 1) + c] : 0.f;
    const float s = live ? fmaf(la, dv, s_u[c]) : 0.f;
    if (dslab) dslab[e] = dv;
    qslab[e] = live && normalise ? fminf(s - s_norm[a], 0.f) : s;
  }
}

}  // namespace

hipError_t launch_bigram(const void* phi, const void* psi, const void* gate, int feat_dtype, int64_t V, int r,
                         const int32_t* anchor, const int32_t* cand_ids, const float* cand_logit, const Scales& scales,
                         int B, int gamma, int K, float* delta, float* logq, hipStream_t stream, bool normalise) {
  const dim3 grid(static_cast<unsigned>(static_cast<int64_t>(B) * gamma));
  if (feat_dtype == 1) {
    const uint16_t* p = static_cast<const uint16_t*>(phi);
    const uint16_t* s = static_cast<const uint16_t*>(psi);
    const uint16_t* g = static_cast<const uint16_t*>(gate);
#define UBT_BIGRAM_ARGS p, s, g, V, r, anchor, cand_ids, cand_logit, scales, gamma, K, delta, logq
#define UBT_BIGRAM_K(NORM)                                                                                       \
  do {                                                                                                           \
    if (K <= 16)                                                                                                 \
      hipLaunchKernelGGL((bigram_bf16_kernel<NORM>), grid, dim3(kWave), 0, stream, UBT_BIGRAM_ARGS);             \
    else if (K <= 32)                                                                                            \
      hipLaunchKernelGGL((bigram_bf16_split_kernel<2, NORM>), grid, dim3(2 * kWave), 0, stream, UBT_BIGRAM_ARGS); \
    else                                                                                                         \
      hipLaunchKernelGGL((bigram_bf16_split_kernel<4, NORM>), grid, dim3(4 * kWave), 0, stream, UBT_BIGRAM_ARGS); \
  } while (0)
    if (normalise)
      UBT_BIGRAM_K(true);
    else
      UBT_BIGRAM_K(false);
#undef UBT_BIGRAM_K
#undef UBT_BIGRAM_ARGS
  } else {
#define UBT_BIGRAM_F32(TM)                                                                                            \
  hipLaunchKernelGGL((bigram_f32_kernel<TM>), grid, dim3(kF32Threads), 0, stream, static_cast<const float*>(phi),    \
                     static_cast<const float*>(psi), static_cast<const float*>(gate), V, r, anchor, cand_ids,         \
                     cand_logit, scales, gamma, K, delta, logq, normalise ? 1 : 0)
    if (K <= 16)
      UBT_BIGRAM_F32(1);
    else if (K <= 32)
      UBT_BIGRAM_F32(2);
    else
      UBT_BIGRAM_F32(4);
#undef UBT_BIGRAM_F32
  }
  return hipGetLastError();
}

}  // namespace ubt
