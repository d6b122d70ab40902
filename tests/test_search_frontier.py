"""The four-wave search's read of the stored frontier, compiled for the host: no slot that was
never written becomes a slab index, whatever LDS held before."""
from __future__ import annotations

import ctypes
import os
import subprocess

import pytest

import paper_2609_39972_amd as ubt

HARNESS = r"""
#include <vector>
#include "frontier.h"
// The largest slab index formed by 64 lanes x 64 parents over all depths, with every slot
// that no depth has stored left at `poison`.
extern "C" int max_slab_index(int gamma, int K, int W, unsigned poison) {
  std::vector<uint32_t> key(gamma * W, poison), info(gamma * W, poison);
  int np = 1, worst = 0;
  for (int d = 1; d <= gamma; ++d) {
    for (int r = 0; r < 64; ++r) {
      const ubt::FrontierSlot f = ubt::frontier_slot(key.data(), info.data(), d, W, np, r, 0x80000000u);
      for (int lane = 0; lane < 64; ++lane) {
        const int at = static_cast<int>(f.info >> 16) * K + (lane < K ? lane : 0);
        worst = at > worst ? at : worst;
      }
    }
    const int w_d = np * K < W ? np * K : W;
    for (int r = 0; r < w_d; ++r) {
      key[(d - 1) * W + r] = 0x80000001u;
      info[(d - 1) * W + r] = static_cast<uint32_t>(r % np) | (static_cast<uint32_t>(r % K) << 16);
    }
    np = w_d;
  }
  return worst;
}
"""


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    d = tmp_path_factory.mktemp("frontier")
    src, so = d / "h.cpp", d / "h.so"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{os.path.join(ubt.PKG, 'csrc')}", str(src),
                    "-o", str(so)], check=True, capture_output=True, text=True)
    f = ctypes.CDLL(str(so)).max_slab_index
    f.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_uint]
    return f


@pytest.mark.parametrize("gamma,K,W", [
    (5, 1, 4), (9, 2, 5), (16, 2, 64), (4, 3, 64), (11, 10, 24), (7, 10, 10), (6, 16, 33), (5, 31, 64), (16, 63, 64),
    (16, 64, 64), (1, 10, 24),
])
def test_every_slab_index_lies_in_the_slab(harness, gamma, K, W):
    for poison in (0, 0x7FFFFFFF, 0xFFFFFFFF):
        assert harness(gamma, K, W, poison) < K * K
