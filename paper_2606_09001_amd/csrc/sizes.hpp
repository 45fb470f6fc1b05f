// Host arithmetic of launch sizes that can pass 32 bits.  No HIP in here: the
// CPU tests compile it by itself.
#pragma once

#include <algorithm>
#include <cstdint>

namespace amg {

// Workgroups of a grid-stride kernel over `items` work-items.  HIP refuses a
// launch of 2^32 work-items or more in x, and a kernel with 2^sh lanes per
// entry passes that at 2^(32 - sh) entries (64 systems: 67 million); from 2^31
// on the workgroups take several strides.
inline unsigned stride_grid(int64_t items, int block) {
  const int64_t most = ((int64_t)1 << 31) / block;
  return (unsigned)std::min(most, std::max<int64_t>(1, (items + block - 1) / block));
}

// Whether sliced rows (struct Ell) of `steps` steps of 64 entries are kept:
// padding at most doubles the nnz entries (64 per slice always pass: rows
// shorter than a step), and positions fit 32 bits.
inline bool ell_fits(int64_t steps, int64_t nnz, int64_t slices) {
  const int64_t len = 64 * steps;
  return len <= 2 * nnz + 64 * slices && len <= INT32_MAX;
}

}  // namespace amg
