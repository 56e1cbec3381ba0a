// Walks the grids of two convolutions in one launch as conv_window.hip numbers them: every tile of either has to be
// taken by one workgroup, no more and no less.  Prints the number of pairs walked; exit status 1 with the first
// pair that fails.
#include <algorithm>
#include <cstdio>
#include <utility>
#include <vector>

#include "window_patch.h"

using namespace fupr;

int main() {
  // tiles of a 3 x 3 convolution and of the 1 x 1 convolution beside it (ResNet-18, 1 - 12 images), and all small pairs
  std::vector<std::pair<int, int>> pairs = {{140, 98}, {90, 26}, {66, 16}, {102, 28}, {218, 148}, {147, 189}, {1, 100000}, {99999, 8}};
  for (int a = 1; a <= 150; ++a)
    for (int b = 1; b <= 150; ++b) pairs.emplace_back(a, b);
  for (const auto& pair : pairs) {
    const int blocks = std::max(tiles_per_xcd(pair.first), tiles_per_xcd(pair.second)) * kXcds;
    for (int total : {pair.first, pair.second}) {
      std::vector<int> taken(total, 0);
      for (uint32_t block = 0; block < (uint32_t)blocks; ++block) {
        const int tile = tile_of_workgroup(block, tiles_per_xcd(total), total);
        if (tile >= total) return std::printf("tile %d of %d\n", tile, total), 1;
        if (tile >= 0) ++taken[tile];
      }
      for (int tile = 0; tile < total; ++tile)
        if (taken[tile] != 1)
          return std::printf("%d and %d tiles: tile %d of %d is taken %d times\n", pair.first, pair.second, tile, total, taken[tile]), 1;
    }
  }
  std::printf("%zu\n", pairs.size());
  return 0;
}
