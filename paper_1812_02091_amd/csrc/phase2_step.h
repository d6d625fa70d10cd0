// Device helpers shared by the phase-2 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lcemd {

// One transfer step of Eq. (6)-(8) against table entry (z, w).  rem >= +0
// (never -0: rem - rem is +0) and w > 0 (or +inf), so the smaller float is
// the smaller bit pattern: one integer minimum (fminf would first
// canonicalise both operands).  A step with rem = +0 changes nothing
// (r = +0, acc + 0 z = acc for finite z >= 0): so the second entry of a
// table row's first 16-byte pair, which is always written (as (0, 0) when
// the row has one entry), is stepped without testing rem; later pairs count
// only while some mass remains (their entries past the row's sink are never
// written).  For z = +inf, 0 z has no number: a walk that ends at a row's first
// entry has none either where the second is infinitely far.
__device__ __forceinline__ void step(float& rem, float& acc, float z, float w) {
  const float r = __uint_as_float(min(__float_as_uint(rem), __float_as_uint(w)));
  rem -= r;
  acc = fmaf(r, z, acc);
}

__device__ __forceinline__ int64_t uniform64(int64_t x) {
  const int lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  const int hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo);
}

}  // namespace lcemd
