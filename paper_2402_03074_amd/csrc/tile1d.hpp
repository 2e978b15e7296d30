// Helpers of the 1D kernels (their stage operator is tile1d_terms.inc).
#pragma once

#include "hwenou_internal.hpp"

namespace hwenou {

// The boundary rule of bc_index (periodic wrap, transmissive copy, mirror
// image at a reflective wall) as selects, so that the lanes of a tile form
// their source cells without branching on their own indices.
__device__ __forceinline__ int source_cell(int i, int n, int bc_lo, int bc_hi, bool& mirrored) {
  const bool lo = i < 0, out = lo || i >= n;
  const int bc = lo ? bc_lo : bc_hi;
  const int wrap = lo ? i + n : i - n;
  const int mirror = lo ? -1 - i : 2 * n - 1 - i;
  const int edge = lo ? 0 : n - 1;
  mirrored = out && bc == BC_REFLECTIVE;
  const int j = bc == BC_PERIODIC ? wrap : (bc == BC_REFLECTIVE ? mirror : edge);
  return out ? j : i;
}

}  // namespace hwenou
