// Grid of a launch of `tiles` workgroups for each of BH (batch, KV head)
// pairs, in plain C++.
#pragma once

#include <stdint.h>

namespace pisa {

struct HeadGrid {
  uint32_t x, y, z;
};

// x: the pair, so that the workgroups started one after another are the pairs'
// same tiles; y and z: the tile, z * grid.y + y, to be skipped from `tiles` on.
// A dimension holds fewer than 2^32 threads and y and z at most 65535
// workgroups: one dimension for the product overflows from 2^24 workgroups of
// 256 threads on (2^29 rows in tiles of 32, inside the ABI's limits).
constexpr uint32_t kHeadGridY = 32768;
constexpr HeadGrid head_grid(int64_t tiles, int32_t BH) {
  const int64_t y = tiles < kHeadGridY ? tiles : kHeadGridY;
  return HeadGrid{static_cast<uint32_t>(BH), static_cast<uint32_t>(y), static_cast<uint32_t>((tiles + y - 1) / y)};
}

}  // namespace pisa
