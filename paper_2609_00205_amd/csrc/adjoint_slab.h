// How the transposes cut a block level into slabs: plain C++, so that it can
// be checked without a device.
//
// The blocks of a slab leave b^3 contributions each in a scratch array, which
// a second launch sums node by node.  The scratch has a bound that does not
// grow with the grid: at most the Infinity Cache (256 MB), so that the second
// launch finds there what the first wrote, and half of it for 9- and 17-node
// blocks (98 x 1200 x 1200 FP32 1.00 / 0.92 ms a level against 1.04 / 0.95
// with 256 MiB, decomposition / recomposition; 64 x 2048 x 2048 1.67 / 1.58
// against 1.70 / 1.58).  A 33-node block run twice costs more, and a slab of
// few of them does not fill the chip: 256 x 1024 x 1024 FP32 2.58 / 3.04 ms
// with 128 MiB, 2.37 / 2.86 with two layers however large (294 MB), 256 MiB
// (and the slabs' blocks in runs per die) 2.06 / 2.49.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>

namespace bm {

inline size_t slab_bytes(int64_t b) { return size_t(b < 33 ? 128 : 256) << 20; }

// Blocks [lo, hi) along an axis whose nodes a strip sums, and the first block
// it runs (one before lo, for the face they share, where there is one).
struct BlockRange {
  int64_t run, lo, hi;
};

// A level's strips: `cut` blocks along y and x each (the whole axis where
// that fits), every strip marching along z in slabs of `layers` layers of
// blocks.  A layer's contributions stay in the scratch until the next slab
// has summed the plane they share (`ring` layers in all; as many as there are
// where one slab takes them all), so nothing is run twice along z.  Along a
// cut axis the strip after it runs the face's blocks once more.
struct SlabCut {
  int64_t layers, ring;
  int64_t cut[2];       // blocks a strip sums along y, x
  int64_t run[2];       // most blocks it runs: one more where the axis is cut
  int64_t blocks() const { return ring * run[0] * run[1]; }
};

// at most `most` blocks a part, one of them run for the part before
inline void cut_axis(int64_t n, int64_t most, int64_t& cut, int64_t& run) {
  if (most >= n) {
    cut = run = n;
    return;
  }
  const int64_t part = std::max<int64_t>(most - 1, 1), k = (n + part - 1) / part;
  cut = (n + k - 1) / k;
  run = cut + 1;
}

inline SlabCut slab_cut(const int64_t nb[3], int64_t b, size_t esize) {
  const int64_t fit = int64_t(slab_bytes(b) / (size_t(b * b * b) * esize));   // blocks in the scratch
  SlabCut c{};
  // blocks per layer of a strip: two layers have to fit, or the only one
  const int64_t most = fit / (nb[0] > 1 ? 2 : 1);
  if (nb[1] * nb[2] <= most) {
    c.cut[0] = c.run[0] = nb[1];
    c.cut[1] = c.run[1] = nb[2];
  } else {
    // whole rows where nine fit (an eighth of a strip's blocks run twice at
    // most), else strips of about as many rows as columns
    int64_t rows = most / nb[2];
    if (rows < 9) rows = std::max<int64_t>(int64_t(std::sqrt(double(most))), 2);
    cut_axis(nb[1], rows, c.cut[0], c.run[0]);
    cut_axis(nb[2], std::max<int64_t>(most / c.run[0], 2), c.cut[1], c.run[1]);
  }
  const int64_t z = fit / (c.run[0] * c.run[1]);                           // layers in the scratch
  if (z >= nb[0]) {
    c.layers = c.ring = nb[0];
  } else {
    const int64_t part = std::max<int64_t>(z - 1, 1), k = (nb[0] + part - 1) / part;
    c.layers = (nb[0] + k - 1) / k;
    c.ring = c.layers + 1;
  }
  return c;
}

// strip k of an axis of n blocks
inline BlockRange strip(int64_t n, int64_t cut, int64_t k) {
  const int64_t lo = k * cut;
  return {std::max<int64_t>(lo - 1, 0), lo, std::min(n, lo + cut)};
}

}  // namespace bm
