// Which k-way reduces of indexed streams run with tiles of eight segments, a wave each, instead of four (host code).
//
// Half as many tiles look back sooner (a wave of a Sum of few operands spends a third of its life on that, and the chains are half as long); but what
// is at work at the same time is the same in both forms, so that twice as much of the chip stands idle when the last of them are under way, and with many operands a
// large tile's waves end too far apart.  So which is better depends on how full the last round of workgroups is.
// A compute unit has room for three large workgroups of reduce_kernel where it has for six of the others, 1536 tiles of four on the chip, and for two of reduce_op_kernel where it
// has for four, 1024 tiles; large ones also need as many as there are compute units (512 tiles) to be spread evenly.
#pragma once

#include <cstdint>

namespace zc {

constexpr int kLargeWaves = 8;

// tiles: tiles of four segments.  What tiles of eight change, per cent (power-law fields at 1e-4 of their range | hard data), with us by tiles of four, from both sides of every limit:
//   2 operands   769: 11.7 +3 +19 | 800: 12.5 -3 +13 | 900: 13.1 -6 +9 | 1000: 13.7 -8 +6 | 1030: 17.0 -19 -12 | 1530: 19.1 -20 -17 | 1550: 19.7 +4 +8 | 1650: 21.4 0 +1 | 1720: 22.1 -2 -1 | 2048: 25.8 -8 -12 | 2250: 27.5 -3 -3 | 3090: 33.6 -6 -5 | 8192: 76.4 -4 -4
//   3            769: 13.6 -1 0 | 800: 14.8 -9 -5 | 1000: 16.5 -14 -8 | 1030: 18.5 -11 -6 | 1530: 21.4 -16 -11 | 1750: 25.4 -2 +1 | 1780: 25.7 -3 0 | 2048: 28.8 -6 -8 | 2250: 30.8 -3 -2 | 3200: 39.1 -1 0 | 8192: 85.2 -1 -3
//   4            769: 15.3 -3 +3 | 800: 16.2 -8 -3 | 1000: 18.0 -14 -10 | 1030: 20.1 -4 -2 | 1250: 22.1 -4 0 | 1530: 23.5 -6 -3 | 1800: 29.1 +1 +1 | 1850: 30.0 -1 -2 | 2048: 32.1 -4 -5 | 3090: 42.6 -1 0 | 4800: 60.8 +1 -1 | 8192: 95.4 0 -2
//   5            645: 17.7 -10 -4 | 1020: 21.7 -20 -14 | 1150: 23.4 0 +1 | 1405: 26.5 -6 -1 | 1530: 25.9 -5 -2 | 1800: 32.3 +1 +1 | 1850: 33.0 0 -2 | 2048: 35.3 -3 -5 | 3060: 47.7 -3 -1 | 3090: 48.0 +1 +3 | 3400: 52.1 +1 -1
//   6, 7         6 x 645: 18.8 -9 -2 | 1020: 24.1 -21 -12 | 1030: 23.7 +9 +3 | 1300: 27.7 0 +1 | 1405: 28.9 -2 0 | 1530: 28.3 -2 -2;   7 x 1440: 32.8 -3 0 | 1800: 39.3 -1 0 | 1850: 40.3 -2 -2 | 2048: 42.3 +1 -4 | 2250: 45.3 +2 +3 | 3200: 61.4 +3 +3
//   8 to 12      8 x 720: 21.8 -7 0 | 780: 23.2 -8 -3 | 1020: 28.0 -16 -9;   12 x 645: 25.7 -1 +7 | 720: 27.3 +1 +6 | 780: 30.3 -6 -1 | 1020: 35.0 -12 -3
// (up to 1024 tiles of up to four operands what they are measured against is reduce_few_kernel.)
constexpr bool sum_large_tiles(int k, uint64_t tiles) {
  if (k < 2) return false;
  if (tiles <= 1024) return k <= 12 && tiles > (k == 2 ? 900u : k >= 5 && k <= 7 ? 640u : 784u);
  if (tiles <= 1536) return k <= 4 || (k <= 7 && tiles > 1400);
  if (k <= 3) return tiles > (k == 2 ? 1700u : 1780u);
  return tiles > 1850 && (k == 4 || (k == 5 && tiles <= 3072) || (k <= 7 && tiles <= 2048));
}

// The same of Max and Min:
//   2 operands   769: 14.1 0 +7 | 800: 15.1 -6 -5 | 1020: 15.6 -6 -6 | 1030: 18.8 +10 +9 | 1099: 20.8 +3 +3 | 1220: 22.4 -4 -2 | 1530: 26.3 -17 -15 | 1540: 26.4 -6 0 | 1650: 27.5 -6 +1 | 2046: 31.4 -13 -10 | 2100: 32.1 +1 +2 | 2350: 35.2 0 0 | 2400: 35.9 -1 -1 | 8192: 102 -3 -2
//   3            1250: 25.4 -1 +1 | 1350: 27.5 -8 -6 | 1540: 29.3 +2 +5 | 1750: 31.7 -3 +1 | 1850: 33.1 -6 -2 | 2046: 35.3 -9 -7 | 2100: 36.0 +4 +4 | 2700: 44.1 +1 +2 | 3200: 50.6 +1 +2 | 4300: 64.8 0 +1 | 5140: 75.6 -1 -1 | 8192: 115 -2 -1
//   4            769: 19.1 0 +3 | 800: 20.3 -5 -4 | 1250: 28.1 0 +2 | 1350: 30.3 -6 -4 | 1540: 32.2 +7 +10 | 1750: 35.1 +2 +4 | 1850: 36.9 -3 0 | 2046: 39.0 -6 -5 | 2056: 39.5 +6 +7 | 8192: 129 0 +1
//   8            769: 28.9 -3 +3 | 800: 29.6 -5 -2 | 1020: 30.7 -5 -4 | 1030: 36.0 +12 +15 | 1300: 41.9 -1 +2 | 1410: 43.8 -4 -2 | 1540: 44.9 +13 +15 | 1850: 52.9 0 +2 | 1930: 53.8 -2 0 | 2046: 55.1 -2 -2 | 2056: 57.3 +10 +11 | 8192: 194 +2 +3
//   12, 32       12 x 770: 40.1 -6 -2 | 1020: 40.2 -5 -2 | 1410: 56.1 -1 -1 | 1500: 57.0 -3 -2 | 2000: 72.3 +2 -1;   32 x 770: 85.6 -2 -2 | 1020: 91.8 -4 -2
constexpr bool op_large_tiles(int k, uint64_t tiles) {
  if (k < 2 || tiles <= 784) return false;
  if (tiles <= 1024) return true;
  if (tiles <= 1536) return k <= 8 && tiles > (k == 2 ? 1200u : k <= 4 ? 1300u : 1400u);
  if (tiles <= 2048) return k == 2 || (k <= 8 && tiles > (k == 3 ? 1750u : k == 4 ? 1850u : 1930u));
  return (k == 2 && tiles > 2400) || (k == 3 && tiles > 4400);
}

// Tiles are what the workspace and the operands' bytes allow; with a larger workspace than a call needs they are far fewer, and tiles of eight, of which then not every
// compute unit has one, are up to 20 % slower (Max of 8 x 2^20 values in a workspace for 1000 tiles 15.1 us by tiles of four, 18.2).  So the output must have room for as
// many too, for their values at 4 bytes each, or a stream of them at its longest, which is a little more; and the shortest operand must have twice the bytes that as many blocks
// take at least (a field at 1e-2 of its range has four times as many, sinusoids twice; streams of hardly anything but constant blocks, up to 20 % slower for that, have fewer).  Where all of
// these are larger than the call, which for a field at 1e-4 is up to five times, the loss remains: only the GPU knows better, and kernels that could take
// either tile when they know are 8 to 15 % slower for all calls (more registers spilled; Sum of 4 x 2^26 values 95.3 us, 102.4).
constexpr bool tiles_are_there(uint64_t out_cap, uint64_t least_bytes, uint64_t tiles) {
  constexpr uint64_t kBlocks = 4 * 64;         // of a tile
  return tiles == 0 || (out_cap / (4 * 32 * kBlocks) >= tiles - 1 && least_bytes / (2 * 5 * kBlocks) >= tiles - 1);
}

}  // namespace zc
