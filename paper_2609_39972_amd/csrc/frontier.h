// One slot of a stored frontier F_d (search.h), in plain C++: the host compiles it as well.
#pragma once

#include <cstdint>

#if defined(__HIP__)
#include <hip/hip_runtime.h>
#define UBT_HD __host__ __device__ __forceinline__
#else
#define UBT_HD inline
#endif

namespace ubt {

struct FrontierSlot {
  uint32_t key;   // score as an order key
  uint32_t info;  // parent's position | candidate rank << 16: the rank is the slab row of its children
};

// Slot r of F_{d-1}, which holds np <= W entries in rank order.  At depth 1 that is the root
// (score key root_key, slab row 0).  Slots past the np-th were never written (with K < W the
// first depths fill fewer than W), and what LDS holds there would index far past the slab:
// they read as the root and are dropped by their rank.
UBT_HD FrontierSlot frontier_slot(const uint32_t* s_key, const uint32_t* s_info, int d, int W, int np, int r,
                                  uint32_t root_key) {
  FrontierSlot f{root_key, 0u};
  if (d > 1 && r < np) {
    f.key = s_key[(d - 2) * W + r];
    f.info = s_info[(d - 2) * W + r];
  }
  return f;
}

}  // namespace ubt
