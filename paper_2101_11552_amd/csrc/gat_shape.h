// The lane layout of the fused attention kernels (host code, no HIP).
#pragma once

#include <algorithm>

namespace tfg {
namespace rows {

constexpr int kSlotLanes = 64;  // lanes of a wavefront (kWave)

// Columns per lane, lanes per head, lanes per slot: lane g of a head holds its
// columns min(g * vec, D - vec) .. + vec - 1.
struct GatShape {
  int vec, G, lps;
};

// Four columns per lane where a head has them. For the additive score the lanes
// of a head are rounded up to a multiple of 4 or 2 (more of them then share a
// score) where that leaves the slot as it is; the lanes added repeat the head's
// last columns. A dot product sums its lanes' parts (D a power of two), so its
// lanes hold each column once and are not rounded.
inline GatShape gat_shape(int H, int D, bool dot) {
  GatShape t;
  t.vec = D >= 4 ? 4 : D == 2 ? 2 : 1;
  t.G = (D + t.vec - 1) / t.vec;
  auto lanes = [&](int G) {
    int n = 4;
    while (n < std::min(H * G, kSlotLanes)) n <<= 1;
    return n;
  };
  t.lps = lanes(t.G);
  if (!dot && t.vec == 4 && t.G > 1)
    for (int r : {4, 2}) {
      const int G = (t.G + r - 1) / r * r;
      if (lanes(G) == t.lps && (H * G <= kSlotLanes || G == t.G)) {
        t.G = G;
        break;
      }
    }
  return t;
}

}  // namespace rows
}  // namespace tfg
