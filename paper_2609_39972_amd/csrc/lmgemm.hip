// The LM-head projection for more rows of h than one MFMA tile: a matrix product whose
// epilogue reduces the softmax statistics, then the candidate sets.
//
// Background, "DFlash & DFlash 2" (u_i = W_lm h_i); Method / Unigram Proposer, Eq.
// (ubtree-unigram) and "Candidate Sets".
//
// A call with M rows does 2 M d V flops on V d weights.  Streaming the head once per 16
// rows (the drafting block of one sequence) reads it M / 16 times; from a few row groups
// on, the weights have to be reused on chip.  Here a workgroup of 8 waves computes a tile
// of 256 vocabulary rows x up to 160 rows of h with v_mfma_f32_16x16x32_bf16, both
// operands staged in LDS by direct loads, so each weight byte is staged once per 160 rows.
//
// The fp32 logits go to the workspace (16-byte stores that overlap the next tile's
// loads; 292 MB at 480 x 151,936, a fraction of the memory time that the product leaves
// idle), and with them the maximum and sum of exp(u - max) of every 64 columns.  The
// select kernel then never reads the row: the K-th largest of the 64-column maxima bounds
// the row's K-th logit from below, so only the columns of about K groups are looked at.
#include "bigram_tile.h"
#include "search.h"
#include "ubt_launch.h"

namespace ubt {
namespace {

constexpr int kGmWaves = 8;
constexpr int kGmThreads = kGmWaves * kWave;
constexpr int kGmBN = 256;             // vocabulary rows per tile
constexpr int kGmBK = 64;              // k per stage: 128-byte rows, whole cache lines
constexpr int kGmRowBytes = kGmBK * 2;
constexpr int kGmBM = 160;             // most rows of h per tile
constexpr int kGmGroup = 64;           // columns per statistics entry (one wave's columns)
constexpr int kGmMaxGroups = 8192;     // statistics entries per row that the select kernel holds in LDS

struct GemmArgs {
  const uint16_t* h;  // [M, d] bf16
  const uint16_t* w;  // [V, d] bf16
  int M, d;
  int64_t V;
  int row_blocks, bm;  // blocks of bm rows of h (bm a multiple of 32, at most kGmBM)
  int fold;            // stages per partial sum
  int ranges, cpr;     // column ranges of cpr columns (a multiple of 16), one per workgroup and row block
  int gpr;             // statistics groups per range: ceil(cpr / 64)
  int64_t ls;          // logits per row
  float* logits;       // [M][ls]
  float2* stats;       // [M][ranges * gpr] (max, sum of exp(u - max)) of up to 64 columns
};

// The 16-byte chunk c of a staged 128-byte row r sits at chunk position c ^ swz(r): the 16
// rows that one MFMA fragment read touches then cover all banks once.
__device__ __forceinline__ int gm_swz(int row) { return (row >> 1) & 7; }

template <int N>
__device__ __forceinline__ void gm_wait_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));  // vmcnt(N), lgkmcnt(0)
  asm volatile("s_barrier" ::: "memory");
}

template <bool B>
struct BoolTag {
  static constexpr bool value = B;
};

// TH: 16-row tiles of h per wave (a block is 32 TH rows); S: stages in LDS; kOnce: nothing
// will read the weights again before they leave the last-level cache.
template <int TH, int S, bool kOnce>
__global__ __launch_bounds__(kGmThreads, 2) void lm_gemm_kernel(GemmArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int kBM = 32 * TH;
  constexpr int kStage = (kGmBN + kBM) * kGmRowBytes;
  constexpr int kWLoads = kGmBN / 8 / kGmWaves;             // 1 KB load instructions per wave and stage
  constexpr int kHInstr = kBM / 8;
  constexpr int kHLoads = (kHInstr + kGmWaves - 1) / kGmWaves;
  static_assert(kWLoads == 4, "the waits below count 1 to 4 weight loads");
  const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int lane = static_cast<int>(threadIdx.x) % kWave;
  const int lr = lane & 15, kg = lane >> 4;
  const int hw = w & 1, vw = w >> 1;  // the wave's half of the block's rows, quarter of the columns
  const int nk = (a.d + kGmBK - 1) / kGmBK;
  const int nk_full = a.d / kGmBK;  // an odd d / 32: the last stage holds 32 of 64 k
  const bool half_tail = nk_full < nk;
  const uint32_t rb = static_cast<uint32_t>(a.d) * 2u;
  // Every workgroup takes one range of columns for one row block, in tiles of 256 (the last
  // one narrower): even ranges keep all compute units busy to the end, where whole tiles
  // dealt out in rounds leave the last round partly empty (594 tiles on 256 units: three
  // rounds for 2.3 rounds of work).  Workgroup g is on XCD g % 8; the row blocks of a
  // range are neighbours on one XCD and share its weights through that XCD's L2.
  const int G = static_cast<int>(gridDim.x);
  const int g = static_cast<int>(blockIdx.x);
  const int at = G % 8 == 0 ? (g % 8) * (G / 8) + g / 8 : g;
  const int range = at / a.row_blocks, mb = at - range * a.row_blocks;
  const int64_t c_lo = static_cast<int64_t>(range) * a.cpr;
  const int width = static_cast<int>(a.V - c_lo < a.cpr ? a.V - c_lo : a.cpr);
  if (range >= a.ranges || width <= 0) return;
  const int nt = (width + kGmBN - 1) / kGmBN;
  const int m0 = mb * a.bm;
  const int mmax = (a.M - m0 < kBM ? a.M - m0 : kBM) - 1;

  // Load lanes: instruction u of a stage fills rows 8 u .. 8 u + 7, 8 lanes per row.
  const int lrow = lane >> 3;
  const int cpos = lane & 7;
  auto issue = [&](int tile, int kt, int slot) {
    // Rows past the range repeat its last one, whole 64-row passes of them are left out.
    const int cmax = min(width - tile * kGmBN, kGmBN) - 1;
    const int nq = cmax / 64 + 1;
    const char* wb = reinterpret_cast<const char*>(a.w) + (c_lo + tile * kGmBN) * static_cast<int64_t>(rb) +
                     kt * kGmRowBytes;
    const char* hb = reinterpret_cast<const char*>(a.h) + static_cast<int64_t>(m0) * rb + kt * kGmRowBytes;
    const bool tail = half_tail && kt == nk - 1;
    unsigned char* st = smem_raw + slot * kStage;
#pragma unroll
    for (int q = 0; q < kWLoads; ++q) {
      if (q >= nq) break;
      const int u = w + q * kGmWaves;
      const int r = 8 * u + lrow;
      int c = cpos ^ gm_swz(r);
      if (tail) c &= 3;  // the second half is never used; its loads stay inside the row
      const uint32_t off = static_cast<uint32_t>(min(r, cmax)) * rb + 16u * static_cast<uint32_t>(c);
      if (kOnce)  // nontemporal
        __builtin_amdgcn_global_load_lds(wb + off, st + u * 1024, 16, 0, 2);
      else
        __builtin_amdgcn_global_load_lds(wb + off, st + u * 1024, 16, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < kHLoads; ++q) {
      // Fewer instructions than waves: the surplus waves repeat one (the same bytes).
      const int u = (w + q * kGmWaves) % kHInstr;
      const int r = 8 * u + lrow;
      int c = cpos ^ gm_swz(r);
      if (tail) c &= 3;
      const uint32_t off = static_cast<uint32_t>(min(r, mmax)) * rb + 16u * static_cast<uint32_t>(c);
      __builtin_amdgcn_global_load_lds(hb + off, st + kGmBN * kGmRowBytes + u * 1024, 16, 0, 0);
    }
  };

  // Fragment reads: row 16 t + lr of a staged operand, chunk 4 s + kg.
  const int sw = gm_swz(lr);
  const int wrow = (vw * 64 + lr) * kGmRowBytes;
  const int hrow = kGmBN * kGmRowBytes + (hw * 16 * TH + lr) * kGmRowBytes;
  f32x4 acc[TH][4], sum[TH][4];
  // One stage.  The matrix cores do not round their running sum to nearest, so a sum carried
  // through all of d drifts (error of 480 rows, d = 4096 against 64 bits 9.8e-7), and fp32
  // adds of many short partial sums each round at the running sum's size (one add per 64
  // products 3.6e-7).  `fold` cuts d into up to 8 partial sums, as the row-group kernels do
  // (2.0e-7 for both).  The two accumulators bound the tile to 160 rows, which leaves room
  // for a third stage: 480 x 4096 x 151,936 takes 705 us, 709 us with 256 rows, two stages
  // and one add per 64 products.
  auto compute = [&](int slot, auto both_tag) {
    constexpr bool both = decltype(both_tag)::value;
    const unsigned char* st0 = smem_raw + slot * kStage + ((kg ^ sw) << 4);
    const unsigned char* st1 = smem_raw + slot * kStage + (((4 + kg) ^ sw) << 4);
    u32x4 fw0[4], fw1[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      fw0[j] = *reinterpret_cast<const u32x4*>(st0 + wrow + j * 16 * kGmRowBytes);
      fw1[j] = *reinterpret_cast<const u32x4*>(st1 + wrow + j * 16 * kGmRowBytes);
    }
    u32x4 fh0 = *reinterpret_cast<const u32x4*>(st0 + hrow);
    u32x4 fh1 = *reinterpret_cast<const u32x4*>(st1 + hrow);
#pragma unroll
    for (int i = 0; i < TH; ++i) {
      // The fragments of row tile i + 1 load while tile i is on the matrix cores; the barrier
      // keeps the compiler from hoisting more loads than there are registers for.
      u32x4 n0 = fh0, n1 = fh1;
      if (i + 1 < TH) {
        n0 = *reinterpret_cast<const u32x4*>(st0 + hrow + (i + 1) * 16 * kGmRowBytes);
        n1 = *reinterpret_cast<const u32x4*>(st1 + hrow + (i + 1) * 16 * kGmRowBytes);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fw0[j]), as_bf16x8(fh0), acc[i][j], 0, 0, 0);
      if (both) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fw1[j]), as_bf16x8(fh1), acc[i][j], 0, 0, 0);
      }
      fh0 = n0;
      fh1 = n1;
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto fold = [&]() {
#pragma unroll
    for (int i = 0; i < TH; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        sum[i][j] += acc[i][j];
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
  };

  // The stages of all of this workgroup's tiles form one sequence; S - 1 of them are in
  // flight.  A step waits for its own stage, passes the barrier (every wave has then
  // finished the stage before it, whose slot the next load refills) and computes.
  int lt = 0, lk = 0;  // the next stage to load
  auto advance = [&]() {
    if (++lk == nk) {
      lk = 0;
      ++lt;
    }
  };
  int slot_l = 0;
#pragma unroll
  for (int s = 0; s < S - 1; ++s) {
    if (lt < nt) {
      issue(lt, lk, slot_l);
      advance();
    }
    slot_l = slot_l + 1 == S ? 0 : slot_l + 1;
  }
  int slot = 0;
  for (int tile = 0; tile < nt; ++tile) {
    const int cols = min(max(width - tile * kGmBN - vw * kGmGroup, 0), kGmGroup);  // of this wave
#pragma unroll
    for (int i = 0; i < TH; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nq = min((width - tile * kGmBN + 63) / 64, kWLoads);  // weight loads per wave and stage
    auto step = [&](int kt) {
      // Wait for this step's stage: all but the loads of the S - 2 stages after it.  Stores
      // of the previous tile's epilogue are younger than the loads in flight, and the
      // stages after a tile's end may have fewer loads: both wait for everything.
      if (S == 2 || kt == 0 || (tile >= nt - 2 && kt + S - 1 > nk))
        gm_wait_barrier<0>();
      else if (nq == 4)
        gm_wait_barrier<(4 + kHLoads) * (S - 2)>();
      else if (nq == 3)
        gm_wait_barrier<(3 + kHLoads) * (S - 2)>();
      else if (nq == 2)
        gm_wait_barrier<(2 + kHLoads) * (S - 2)>();
      else
        gm_wait_barrier<(1 + kHLoads) * (S - 2)>();
      if (lt < nt) {
        issue(lt, lk, slot_l);
        advance();
      }
      slot_l = slot_l + 1 == S ? 0 : slot_l + 1;
    };
    auto next_slot = [&]() { slot = slot + 1 == S ? 0 : slot + 1; };
    if (cols == 0) {  // a wave past the end of the range only loads
      for (int kt = 0; kt < nk; ++kt) {
        step(kt);
        next_slot();
      }
      continue;
    }
    int left = a.fold;
    for (int kt = 0; kt < nk_full; ++kt) {
      step(kt);
      compute(slot, BoolTag<true>{});
      next_slot();
      if (--left == 0) {
        fold();
        left = a.fold;
      }
    }
    if (nk_full < nk) {
      step(nk_full);
      compute(slot, BoolTag<false>{});
      next_slot();
    }
    fold();
    // Epilogue: sum[i][j][e] = u(row m, column c0 + 16 j + 4 kg + e).
    const int64_t c0 = c_lo + tile * kGmBN + vw * kGmGroup;
    const int64_t ss = static_cast<int64_t>(a.ranges) * a.gpr;
    const int64_t group = static_cast<int64_t>(range) * a.gpr + tile * 4 + vw;
    int me = m0;  // opaque, so that the rows' addresses are formed here and not kept in registers
    asm volatile("" : "+s"(me));
#pragma unroll
    for (int i = 0; i < TH; ++i) {
      const int m_in = hw * 16 * TH + 16 * i + lr;
      const int64_t m = me + m_in;
      const bool row = m_in < a.bm && m < a.M;
      float mx = neg_inf();
      if (cols == kGmGroup) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) mx = fmaxf(mx, sum[i][j][e]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            mx = 16 * j + 4 * kg + e < cols ? fmaxf(mx, sum[i][j][e]) : mx;
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      float se = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          t[e] = __builtin_amdgcn_exp2f((sum[i][j][e] - mx) * kLog2e);
          if (cols != kGmGroup) t[e] = 16 * j + 4 * kg + e < cols ? t[e] : 0.f;
        }
        se += (t[0] + t[1]) + (t[2] + t[3]);
      }
      se += __shfl_xor(se, 16);
      se += __shfl_xor(se, 32);
      if (row) {
        float* lp = a.logits + m * a.ls + c0 + 4 * kg;
        // A range ends at a multiple of 16 columns or at the vocabulary's end, past which
        // the row is padded to a multiple of 16.
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (16 * j < cols) *reinterpret_cast<f32x4*>(lp + 16 * j) = sum[i][j];
        if (kg == 0) a.stats[m * ss + group] = make_float2(mx, se);
      }
    }
  }
}

// ---- candidate sets from the logits and the group maxima -------------------------------

constexpr int kSelThreads = 512;
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kSelMax = 2048;  // candidates ranked by counting in LDS; more stream from memory
constexpr int kSelGroups = kGmMaxGroups / kSelThreads;  // groups per thread
constexpr int kSelBatch = 8;   // groups whose logits a wave reads at once

struct SelectArgs {
  const float* logits;  // [M][ls]
  const float2* stats;  // [M][ss], ng of them in use
  int64_t ls, ss, V;
  int ng, gpr, cpr, K;  // group i: columns from (i / gpr) cpr + (i % gpr) 64, inside its range
  int32_t* cand_ids;
  float* cand_logit;
  float* cand_logprob;
  float* lse;
};

__device__ __forceinline__ uint64_t sel_order(uint32_t key, uint32_t id) {
  return (static_cast<uint64_t>(key) << 32) | static_cast<uint32_t>(~id);
}

// The digit of a 256-bin histogram that holds the need-th largest entry (need >= 1, at
// most the entries counted), and what is still needed inside it.  Called by every thread;
// wave 0 works.  misc[0] = digit, misc[1] = rest.
__device__ __forceinline__ void sel_digit(const uint32_t* hist, uint32_t* misc, int need) {
  if (threadIdx.x < kWave) {
    const int lane = static_cast<int>(threadIdx.x);
    const uint32_t c0 = hist[4 * lane], c1 = hist[4 * lane + 1], c2 = hist[4 * lane + 2], c3 = hist[4 * lane + 3];
    const uint32_t own = c0 + c1 + c2 + c3;
    const uint32_t below = wave_prefix_sum(own);  // entries in lanes 0 .. lane
    const uint32_t total = __builtin_amdgcn_readlane(below, 63);
    uint32_t above = total - below;  // entries in the lanes after this one
    const uint32_t nd = static_cast<uint32_t>(need);
    if (above < nd && nd <= above + own) {
      const uint32_t cs[4] = {c0, c1, c2, c3};
#pragma unroll
      for (int b = 3; b >= 0; --b) {
        if (above + cs[b] >= nd) {
          misc[0] = static_cast<uint32_t>(4 * lane + b);
          misc[1] = nd - above;
          break;
        }
        above += cs[b];
      }
    }
  }
}

// One workgroup per row of h; latency bound (about 20 KB of statistics and K groups of 64
// logits per row), so each phase issues all of its loads at once.
//  * LSE from the groups' (max, sum) pairs, each thread summing its groups in order, then
//    the threads in order.
//  * The bound: about the K-th largest of 256 maxima over the groups of a thread pair, by
//    the ballot radix search.  At least K groups have a maximum at or above it, so the
//    row's top K elements do; it lets about K + K / 8 + K^2 / 512 groups through.  Where fewer
//    than K thread pairs hold a group (K = 64: up to 8,192 columns), or past K = 16 so few
//    that the bound is the least of them, the pairs' maxima over the elements they read give a
//    second one: without a bound every element was ranked or selected (d = 2880, 17 rows of
//    1,500 columns: 91.9 us, so 37.4; 480 rows of 4,000: 82.2, so 51.3).
//  * The elements at or above the bound lie in the groups whose maximum is; they are read,
//    collected and ranked by counting.
//  * More than kSelMax of them (long runs of equal logits) take an 8-bit radix selection
//    of the K-th 64-bit order value that re-reads the groups once per digit.
__global__ __launch_bounds__(kSelThreads) void lm_select_kernel(SelectArgs a) {
  __shared__ uint16_t glist[kGmMaxGroups];  // groups at or above the bound
  __shared__ __align__(16) uint64_t cand[kSelMax];
  __shared__ __align__(16) uint32_t best[kSelThreads / 2];  // maxima of the thread pairs, as order keys
  __shared__ uint32_t hist[256];
  __shared__ uint32_t misc[6];
  __shared__ float red[2 * kSelWaves];
  const int tid = static_cast<int>(threadIdx.x);
  const int lane = tid % kWave, w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int64_t m = blockIdx.x;
  const float2* st = a.stats + m * a.ss;
  const float* row = a.logits + m * a.ls;
  const int K = a.K;

  // Statistics.
  float2 p[kSelGroups];
#pragma unroll
  for (int q = 0; q < kSelGroups; ++q) {
    const int i = tid + q * kSelThreads;
    p[q] = i < a.ng ? st[i] : make_float2(neg_inf(), 0.f);
  }
  if (tid < 6) misc[tid] = 0u;
  float mx = neg_inf();
#pragma unroll
  for (int q = 0; q < kSelGroups; ++q) mx = fmaxf(mx, p[q].x);
  {
    const float pm = fmaxf(mx, __shfl_xor(mx, 1));
    if (!(tid & 1)) best[tid >> 1] = pm == neg_inf() ? 0u : f32_key(pm);
  }
  mx = wave_max(mx);
  if (lane == 0) red[w] = mx;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kSelWaves; ++i) mx = fmaxf(mx, red[i]);
  float se = 0.f;
#pragma unroll
  for (int q = 0; q < kSelGroups; ++q)
    if (p[q].x != neg_inf()) se += p[q].y * __builtin_amdgcn_exp2f((p[q].x - mx) * kLog2e);
  se = wave_sum(se);
  if (lane == 0) red[kSelWaves + w] = se;
  // The K-th largest (about) of the entries of `best`, found by every wave for itself; 1 with fewer
  // than K of them.  few: that bound is poor or none.
  bool few;
  auto kth_best = [&]() {
    const uint4 o = reinterpret_cast<const uint4*>(best)[lane];
    const uint32_t key[4] = {o.x, o.y, o.z, o.w};
    uint64_t live[4];
    int have = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      live[r] = ballot(key[r] != 0u);
      have += popc(live[r]);
    }
    few = have < (K > 16 ? K + K / 8 + 1 : K);
    return max(wave_threshold<4>(key, live, K, K + K / 8), 1u);  // key 0: no column
  };
  uint32_t bound = kth_best();
  __syncthreads();
  float tot = red[kSelWaves];
#pragma unroll
  for (int i = 1; i < kSelWaves; ++i) tot += red[kSelWaves + i];
  const float lsum = __builtin_amdgcn_logf(tot) * kLn2;
  if (tid == 0 && a.lse) a.lse[m] = mx + lsum;
#pragma unroll
  for (int q = 0; q < kSelGroups; ++q)
    if (p[q].x != neg_inf() && f32_key(p[q].x) >= bound)
      glist[atomicAdd(&misc[2], 1u)] = static_cast<uint16_t>(tid + q * kSelThreads);
  __syncthreads();
  const int nl = static_cast<int>(misc[2]);

  auto visit = [&](auto&& f) {  // f(order value) of every element at or above the bound
    for (int q0 = w; q0 < nl; q0 += kSelWaves * kSelBatch) {
      float x[kSelBatch];
      int64_t v[kSelBatch];
#pragma unroll
      for (int e = 0; e < kSelBatch; ++e) {
        const int q = q0 + e * kSelWaves;
        x[e] = neg_inf();
        v[e] = -1;
        if (q < nl) {
          const int r = glist[q] / a.gpr, in = (glist[q] - r * a.gpr) * kGmGroup + lane;
          const int64_t c = static_cast<int64_t>(r) * a.cpr + in;
          if (in < a.cpr && c < a.V) {
            x[e] = row[c];
            v[e] = c;
          }
        }
      }
#pragma unroll
      for (int e = 0; e < kSelBatch; ++e) {
        const uint32_t key = f32_key(x[e]);
        if (v[e] >= 0 && key >= bound) f(sel_order(key, static_cast<uint32_t>(v[e])));
      }
    }
  };
  if (few) {
    uint32_t top = 0u;
    visit([&](uint64_t o) { top = max(top, static_cast<uint32_t>(o >> 32)); });
    top = max(top, static_cast<uint32_t>(__shfl_xor(static_cast<int>(top), 1)));
    if (!(tid & 1)) best[tid >> 1] = top;
    __syncthreads();
    bound = max(bound, kth_best());
  }
  visit([&](uint64_t o) {
    const uint32_t at = atomicAdd(&misc[3], 1u);
    if (at < kSelMax) cand[at] = o;
  });
  __syncthreads();
  const int n = static_cast<int>(misc[3]);
  auto emit = [&](uint64_t o, int rank) {
    const float v = f32_key_value(static_cast<uint32_t>(o >> 32));
    const int64_t at = m * K + rank;
    a.cand_ids[at] = static_cast<int32_t>(~static_cast<uint32_t>(o));
    a.cand_logit[at] = v;
    // (u - max) - log sum exp(u - max): the error stays relative to the log-probability.
    if (a.cand_logprob) a.cand_logprob[at] = (v - mx) - lsum;
  };
  int have = n;
  if (n > kSelMax) {
    uint64_t prefix = 0ull;
    int need = K;
    for (int shift = 56; shift >= 0; shift -= 8) {
      if (tid < 256) hist[tid] = 0u;
      __syncthreads();
      const uint64_t hmask = shift == 56 ? 0ull : (~0ull << (shift + 8));
      visit([&](uint64_t o) {
        if (((o ^ prefix) & hmask) == 0ull) atomicAdd(&hist[(o >> shift) & 255u], 1u);
      });
      __syncthreads();
      sel_digit(hist, misc, need);
      __syncthreads();
      prefix |= static_cast<uint64_t>(misc[0]) << shift;
      need = static_cast<int>(misc[1]);
      __syncthreads();
    }
    if (tid == 0) misc[3] = 0u;
    __syncthreads();
    // Order values are distinct, so exactly K are at or above the K-th.
    visit([&](uint64_t o) {
      if (o >= prefix) cand[atomicAdd(&misc[3], 1u)] = o;
    });
    __syncthreads();
    have = K;
  }
  for (int i = tid; i < have; i += kSelThreads) {
    const uint64_t me = cand[i];
    int rank = 0;
    for (int j = 0; j < have; ++j) rank += cand[j] > me ? 1 : 0;
    if (rank < K) emit(me, rank);
  }
}

int gm_cu_count() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  return cus;
}

constexpr int kGmMaxRows = 512;  // rows of h per product (bounds the workspace)

size_t gm_up(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

struct GemmPlan {
  int row_blocks, th, ranges, cpr, gpr;
  int64_t ls;
  size_t stats_bytes, total;
};

// The split of `rows` x V over G workgroups.
GemmPlan gm_plan(int rows, int64_t V, int G) {
  GemmPlan p{};
  p.row_blocks = (rows + kGmBM - 1) / kGmBM;
  p.th = ((rows + p.row_blocks - 1) / p.row_blocks + 31) / 32;
  const int64_t most = G / p.row_blocks > 0 ? G / p.row_blocks : 1;
  p.cpr = static_cast<int>(((V + most - 1) / most + 15) / 16 * 16);
  p.ranges = static_cast<int>((V + p.cpr - 1) / p.cpr);
  p.gpr = (p.cpr + kGmGroup - 1) / kGmGroup;
  p.ls = (V + 15) / 16 * 16;
  p.stats_bytes = gm_up(static_cast<size_t>(rows) * p.ranges * p.gpr * sizeof(float2));
  p.total = p.stats_bytes + static_cast<size_t>(rows) * p.ls * sizeof(float);
  return p;
}

int gm_grid() {
  const int cus = gm_cu_count();
  return cus >= 8 ? cus / 8 * 8 : cus;
}

}  // namespace

size_t lm_gemm_workspace_bytes(int M, int d, int64_t V, int K) {
  // Up to 16 rows fit one tile of the row-group kernels, which read the head once: the one that
  // splits d (512 n, n in {2, .., 8, 10}) streams it as fast (15 rows, d = 2560: 132 us), the other
  // one at less than half the rate (15 rows, d = 2880: 317 us, here 156).
  // Past 16 rows the row groups read the head once each, at a cost in groups * V, while the product's
  // grid is too small below some 10,000 columns to get faster with V.  Where the two meet, in groups * V,
  // K = 8, d = 1024 .. 3072 (us, row groups and product on either side, at d = 2560): two groups
  // 20,000 (V = 8,000: 22.4, 26.8; 14,000: 31.9, 26.8); three 15,000 (4,000: 26.2, 28.4; 6,000: 28.7,
  // 28.8); four 10,000 (1,500: 21.3, 28.3; 4,000: 32.8, 28.5); 8 to 30 15,000 .. 22,000 (30 groups,
  // 300: 27.8, 40.8; 1,000: 54.6, 42.2).  A larger K costs the product's selection 1.5 to 2 times
  // as much there (two groups, K = 64, 10,000: 25.8, 30.9; 14,000: 31.3, 30.6); past d = 3072 the row
  // groups hold fewer waves (d = 4096, 8 groups: 1,500: 44.4, 50.2; 2,500: 68.1, 51.0).
  if (lm_head_split_fits(d)) {
    const int64_t groups = (M + 15) / 16;
    int64_t line = groups == 2 ? 20480 : groups == 3 ? 15360 : groups == 4 ? 10240 : 18432;
    if (K > 16) line += line / 2;
    if (d > 3072) line -= line / 4;
    if (groups == 1 || groups * V < line) return 0;
  }
  if (V > (int64_t(1) << 24)) return 0;
  const GemmPlan p = gm_plan(M < kGmMaxRows ? M : kGmMaxRows, V, gm_grid());
  // The last rows of a longer call: fewer row blocks cut V into more ranges, so at a small V their
  // statistics may take more room than those of 512 rows.
  const GemmPlan q = M > kGmMaxRows ? gm_plan((M - 1) % kGmMaxRows + 1, V, gm_grid()) : p;
  if (static_cast<int64_t>(p.ranges) * p.gpr > kGmMaxGroups || static_cast<int64_t>(q.ranges) * q.gpr > kGmMaxGroups)
    return 0;
  return p.total > q.total ? p.total : q.total;
}

hipError_t launch_lm_gemm_topk(const void* h, const void* w_lm, int M, int d, int64_t V, int K, int32_t* cand_ids,
                               float* cand_logit, float* cand_logprob, float* lse, void* workspace,
                               hipStream_t stream) {
  const int G = gm_grid();
  for (int row0 = 0; row0 < M; row0 += kGmMaxRows) {
    const int rows = M - row0 < kGmMaxRows ? M - row0 : kGmMaxRows;
    const GemmPlan p = gm_plan(rows, V, G);
    GemmArgs a{};
    a.h = static_cast<const uint16_t*>(h) + static_cast<int64_t>(row0) * d;
    a.w = static_cast<const uint16_t*>(w_lm);
    a.M = rows;
    a.d = d;
    a.V = V;
    a.row_blocks = p.row_blocks;
    a.bm = 32 * p.th;
    a.fold = ((d + kGmBK - 1) / kGmBK + 7) / 8;
    a.ranges = p.ranges;
    a.cpr = p.cpr;
    a.gpr = p.gpr;
    a.ls = p.ls;
    a.stats = static_cast<float2*>(workspace);
    a.logits = reinterpret_cast<float*>(static_cast<char*>(workspace) + p.stats_bytes);
    // One row block reads the weights once; past the 256 MB last-level cache the next call
    // finds none of them there either, and nontemporal loads stream faster (M = 32, d =
    // 2560, V = 151,936: 139 against 148 us).  A head that fits stays cached between calls.
    const bool once = p.row_blocks == 1 && static_cast<int64_t>(d) * V * 2 > (int64_t(256) << 20);
#define UBT_GEMM1(THV, SV, ONCE)                                                                       \
  do {                                                                                                 \
    constexpr int smem = SV * (kGmBN + 32 * THV) * kGmRowBytes;                                        \
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&lm_gemm_kernel<THV, SV, ONCE>),           \
                              hipFuncAttributeMaxDynamicSharedMemorySize, smem);                       \
    hipLaunchKernelGGL((lm_gemm_kernel<THV, SV, ONCE>), dim3(static_cast<unsigned>(G)), dim3(kGmThreads), smem, \
                       stream, a);                                                                     \
  } while (0)
#define UBT_GEMM(THV, SV)        \
  do {                           \
    if (once)                    \
      UBT_GEMM1(THV, SV, true);  \
    else                         \
      UBT_GEMM1(THV, SV, false); \
  } while (0)
    switch (p.th) {
      case 1: UBT_GEMM(1, 4); break;
      case 2: UBT_GEMM(2, 4); break;
      case 3: UBT_GEMM(3, 3); break;
      case 4: UBT_GEMM(4, 3); break;
      default: UBT_GEMM(5, 3); break;
    }
#undef UBT_GEMM1
#undef UBT_GEMM
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    SelectArgs s{};
    s.logits = a.logits;
    s.stats = a.stats;
    s.ls = p.ls;
    s.V = V;
    s.ng = (p.ranges - 1) * p.gpr;  // the last range's groups end with the vocabulary
    s.ng += static_cast<int>((V - static_cast<int64_t>(p.ranges - 1) * p.cpr + kGmGroup - 1) / kGmGroup);
    s.ss = static_cast<int64_t>(p.ranges) * p.gpr;
    s.gpr = p.gpr;
    s.cpr = p.cpr;
    s.K = K;
    s.cand_ids = cand_ids + static_cast<int64_t>(row0) * K;
    s.cand_logit = cand_logit + static_cast<int64_t>(row0) * K;
    s.cand_logprob = cand_logprob ? cand_logprob + static_cast<int64_t>(row0) * K : nullptr;
    s.lse = lse ? lse + row0 : nullptr;
    hipLaunchKernelGGL(lm_select_kernel, dim3(static_cast<unsigned>(rows)), dim3(kSelThreads), 0, stream, s);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ubt
