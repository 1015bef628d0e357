// Order of a grid's workgroups over the XCDs (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace infcl {

// Position of workgroup wg of a grid of n in an order in which each of the 8
// XCDs (workgroup wg runs on XCD wg mod 8) has one contiguous range.
__host__ __device__ __forceinline__ uint32_t xcd_slot(uint32_t wg, uint32_t n) {
  const uint32_t x = wg & 7, e = n & 7;
  return x * (n >> 3) + (x < e ? x : e) + (wg >> 3);
}

}  // namespace infcl
