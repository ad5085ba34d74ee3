// Host rules of the transposes' launches, plain C++: what a level's grid asks
// of the kernels, apart from the launches so that it can be checked without a
// device.
#pragma once

#include <cstddef>
#include <cstdint>

namespace bm {

// Whether the byte offset of every node (y, x) of an n x n block column from
// the block's first node fits in 32 bits, at element strides sy and sx.
inline bool lane_offsets_fit(int64_t n, int64_t sy, int64_t sx, size_t esize) {
  return uint64_t(n - 1) * (uint64_t(sy) + uint64_t(sx)) * esize < (uint64_t(1) << 32);
}

}  // namespace bm
