// Which reduces run with tiles of eight segments (csrc/zc_large_tiles.h): the calls that they were measured to be slower for have none.
#include <cstdio>
#include <initializer_list>

#include "../../paper_2502_18554_amd/csrc/zc_large_tiles.h"

struct Call {
  int k;
  uint64_t tiles;
  bool large;
};

int main() {
  int wrong = 0;
  const Call sums[] = {{1, 900, false}, {2, 900, false}, {2, 901, true}, {3, 784, false}, {3, 785, true}, {5, 640, false}, {5, 641, true}, {8, 720, false}, {8, 785, true}, {13, 900, false}, {4, 1500, true}, {5, 1400, false},
                       {7, 1401, true}, {8, 1500, false}, {2, 1537, false}, {2, 1700, false}, {2, 1701, true}, {3, 1700, false}, {3, 1781, true}, {4, 1709, false}, {4, 1851, true},
                       {6, 1709, false}, {6, 2048, true}, {6, 2442, false}, {5, 3072, true}, {5, 3073, false}, {7, 4096, false}, {6, 8192, false}, {4, 8192, true}, {2, 1 << 18, true}};
  const Call extremes[] = {{1, 900, false}, {2, 769, false}, {8, 784, false}, {2, 785, true}, {64, 1024, true}, {2, 1030, false}, {3, 1030, false}, {8, 1099, false}, {2, 1201, true}, {4, 1301, true},
                           {8, 1401, true}, {9, 1500, false}, {2, 1600, true}, {3, 1600, false}, {8, 1600, false}, {3, 1751, true}, {4, 1800, false}, {4, 1851, true}, {8, 1931, true},
                           {8, 2048, true}, {2, 2049, false}, {2, 2401, true}, {3, 2049, false}, {8, 2056, false}, {4, 2056, false}, {5, 4096, false}, {3, 4300, false}, {3, 8192, true}, {4, 8192, false}};
  for (const Call& c : sums)
    if (zc::sum_large_tiles(c.k, c.tiles) != c.large) ++wrong, std::printf("sum of %d, %llu tiles\n", c.k, (unsigned long long)c.tiles);
  for (const Call& c : extremes)
    if (zc::op_large_tiles(c.k, c.tiles) != c.large) ++wrong, std::printf("extreme of %d, %llu tiles\n", c.k, (unsigned long long)c.tiles);

  // n values: tiles as the workspace tells them, the output's room (bytes of values, or of the longest stream) and the shortest operand's bytes
  const uint64_t plenty = uint64_t(1) << 40;
  for (const uint64_t n : {1ull, 8191ull, 8192ull, 8193ull, 4194301ull, 20000003ull, 67108864ull, 2147483648ull}) {
    const uint64_t tiles = (n + 8191) / 8192, blocks = (n + 31) / 32, longest = 32 + 133 * blocks;
    const bool holds = zc::tiles_are_there(4 * n, 11 * blocks, tiles) && zc::tiles_are_there(longest, longest, tiles) && zc::tiles_are_there(plenty, plenty, tiles) &&
                       (tiles < 40 || (!zc::tiles_are_there(longest, plenty, tiles + tiles / 16) && !zc::tiles_are_there(plenty, 11 * blocks, tiles + tiles / 4)));
    if (!holds) ++wrong, std::printf("tiles of %llu values\n", (unsigned long long)n);
  }
  // 4 194 304 values in a workspace for many more; with an output for as many, and 34 bytes a block
  if (zc::tiles_are_there(32 + 133ull * 131072, plenty, 3600) || zc::tiles_are_there(plenty, 34ull * 131072, 3600)) ++wrong, std::printf("larger workspaces\n");
  return wrong != 0;
}
