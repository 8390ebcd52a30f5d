// Device-side pieces shared by the per-step kernels (step.hip) and the whole-recurrence kernels (recur.hip).
#pragma once
#include "common.h"
#include "kernels.h"

namespace cmt {

// keep-and-rescale factor of element (b, col) of a dropout slice (see DropSpec)
__device__ __forceinline__ float drop_factor(const DropSpec& d, int b, int col) {
  if (!d.on) return 1.f;
  unsigned long long x = d.key0 + (unsigned long long)b * (unsigned long long)d.width + (unsigned long long)col;
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  x ^= x >> 31;
  return (unsigned)(x >> 40) >= d.thresh ? d.scale : 0.f;
}

// the dropout slice of position t of a site whose slices are `step` elements apart
__device__ __forceinline__ DropSpec seq_drop(DropSpec d, unsigned long long step, int t) {
  d.key0 += (unsigned long long)t * step;
  return d;
}

}  // namespace cmt
