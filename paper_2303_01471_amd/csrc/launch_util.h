// Host-side helpers of the pass launchers.
#pragma once

#include <hip/hip_runtime.h>

namespace qhd {

// points of a line per lane
template <int N>
constexpr int pts_per_lane() { return N >= 1024 ? 16 : 8; }

inline int ilog2(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

inline int blocks_for(long long items, int per_block, int cap) {
  long long b = (items + per_block - 1) / per_block;
  if (cap > 0 && b > cap) b = cap;
  return (int)(b < 1 ? 1 : b);
}

// run BODY (a block that returns) with N_ = n as a constant
#define QHD_SWITCH_N(n, BODY)                 \
  switch (n) {                                \
    case 8: { constexpr int N_ = 8; BODY; }     \
    case 16: { constexpr int N_ = 16; BODY; }   \
    case 32: { constexpr int N_ = 32; BODY; }   \
    case 64: { constexpr int N_ = 64; BODY; }   \
    case 128: { constexpr int N_ = 128; BODY; } \
    case 256: { constexpr int N_ = 256; BODY; } \
    case 512: { constexpr int N_ = 512; BODY; } \
    case 1024: { constexpr int N_ = 1024; BODY; } \
    default: return hipErrorInvalidValue;     \
  }

}  // namespace qhd
