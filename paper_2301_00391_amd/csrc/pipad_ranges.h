// Index arithmetic of lists that may hold up to 2^31 - 1 entries, where a sum past the end of one
// would not fit 32 bits: plain C++, the same on the host and in kernels.
#ifndef PIPAD_RANGES_H_
#define PIPAD_RANGES_H_

#include <cstdint>

namespace pipad {

// A list of nnz entries has `reach` of them from `start` on (0 <= start <= nnz).
constexpr bool reaches(int32_t start, int32_t reach, int32_t nnz) { return nnz - start >= reach; }

// Place of entry `offset` from `start` on, or the list's last one behind the end (0 <= start < nnz).
constexpr int32_t place_in(int32_t start, int32_t offset, int32_t nnz) {
  return start + (offset < nnz - 1 - start ? offset : nnz - 1 - start);
}

}  // namespace pipad

#endif  // PIPAD_RANGES_H_
