// The Sum of zc_reduce.h for calls of few tiles.
//
// Such a call is one tile lifetime: its workgroups all run at the same time, and what bounds it is the string of memory
// round trips and the instructions of a wave, which has its SIMD to itself (one instruction in 4.5 cycles) or shares it with
// one or two others.  reduce_kernel, made for full compute units and 80 registers, takes an operand in some 500 instructions, of which
// the sum itself is a fifth, and 256 blocks per workgroup, so that most SIMDs of the chip have nothing to do.  Here
//  - what a wave has to know to ask for its share of an operand is worked out for all operands at once, in lane s for
//    operand s (LaneOperands), and read from there as scalars;
//  - it asks for up to AREAS operands at once, widths, first codes and payloads, the payloads from memory straight to LDS (an
//    area each, which is what the idle LDS of a part-filled chip is for);
//  - one scan places the blocks of two operands, and the number of planes is chosen once for all operands of a batch, so that
//    adding a block is straight code (add_block);
//  - a segment's operands are divided among PARTS waves, each on a SIMD of its own, whose sums meet in LDS.  The tile is then SEGS
//    segments, SEGS x PARTS = 4 waves a workgroup; there are more of them, closer descriptors (kDescApartFine), and all waves of the
//    workgroup take part in the direct look-back.
// us per call with reduce_kernel, as it was when this was made, and with this (power-law fields at 1e-4 of their range):
//   tiles     1              13             128            245            512            1024
//   2 x    7.1  6.1       8.6  7.4       9.3  8.2       9.5  8.4      10.8  9.9      15.0 13.1
//   4 x    8.6  6.8      10.4  8.0      11.1  9.0      11.3  9.4      12.9 11.5      20.3 17.1
//   8 x   12.1  7.2      14.1  8.6      14.9 10.1      15.4 11.6      17.9 16.0
//  16 x   20.3  7.9      22.3  9.7      24.1 12.6      23.8 15.1      29.3 24.2
//  64 x   70   16.2                     83   23.0      77   36.6     100   71.5
// 4 x 4 194 301 of hard data 14.3 and 11.8, 4 x 1000 of it 10.4 and 8.0.  (reduce_kernel now, in a workspace for more tiles, see few_segments: 128 tiles of 2, 4, 8, 16 and
// 64 operands 8.9 10.6 14.2 21.8 69; 512 tiles 12.4 13.3 17.5 27.4 87; 1024 tiles of 2 and 4 22.5 24.8.)
#pragma once

#include "zc_common.h"
#include "zc_lds_words.h"
#include "zc_place.h"
#include "zc_reduce.h"
#include "zc_scan.h"

namespace zc {

// LDS of one operand's payload of a wave: what load_operand_payload can bring in of the longest segment, and the reads behind its last word.
constexpr u32 kFewArea = kMostStaged + 32;         // words
static_assert(kFewArea % 4 == 0 && kFewArea >= kMostStaged + u32(kSumPlanes) + 8, "16-byte pieces, and the reads behind the last sign word");

// acc += another wave's sum of the same blocks, `theirs` planes of it (in LDS, 64 words a plane); planes [0, top) are valid before and after.
template <int C>
__device__ inline void add_partial(u32 (&acc)[kSumPlanes], const u32* planes, u32 theirs, u32 ext, u32& carry, u32 top) {
  if constexpr (C * kSumChunk < kSumPlanes) {
    if (u32(C * kSumChunk) >= top) return;        // uniform
    u32 x[kSumChunk];
#pragma unroll
    for (int i = 0; i < kSumChunk; ++i) x[i] = ext;
    if (u32(C * kSumChunk) < theirs) {            // uniform
#pragma unroll
      for (int i = 0; i < kSumChunk; ++i) x[i] = planes[64 * (C * kSumChunk + i)];
    }
#pragma unroll
    for (int i = 0; i < kSumChunk; ++i) {
      constexpr int kFirst = C * kSumChunk;
      const u32 cur = acc[kFirst + i];
      acc[kFirst + i] = xor3(cur, x[i], carry);
      carry = majority(cur, x[i], carry);
    }
    add_partial<C + 1>(acc, planes, theirs, ext, carry, top);
  }
}
template <int C>
__device__ inline void store_partial(const u32 (&acc)[kSumPlanes], u32* planes, u32 top) {
  if constexpr (C * kSumChunk < kSumPlanes) {
    if (u32(C * kSumChunk) >= top) return;        // uniform
#pragma unroll
    for (int i = 0; i < kSumChunk; ++i) planes[64 * (C * kSumChunk + i)] = acc[C * kSumChunk + i];
    store_partial<C + 1>(acc, planes, top);
  }
}

// What the waves of a workgroup tell each other.
template <int SEGS, int PARTS>
struct SumParts {
  i64 outlier[PARTS > 1 ? (PARTS - 1) * SEGS * 64 : 1];
  u32 bound[PARTS > 1 ? (PARTS - 1) * SEGS : 1];
  u32 fits[SEGS * PARTS];
};

// The sum so far of a wave's operands.
struct PartialSum {
  u32 acc[kSumPlanes];      // two's complement planes, `top` of them
  u32 top, bound;           // bound on the magnitude; both uniform
  i64 outlier;              // sum of the first codes
};

// acc += a block of at most CAP planes, w of them, whose sign word and planes lie from `mine` on.  All planes are valid (two's complement).
template <int CAP, int TOP>
__device__ __forceinline__ void add_block(u32 (&acc)[TOP], const u32* mine, u32 w) {
  const u32 sgn = w ? mine[0] : 0u;
  const u32 keep = (1u << w) - 1u;                // bit P set iff the block has plane P
  u32 carry = sgn;                                // two's complement of the operand: (mag ^ s) + s
#pragma unroll
  for (int P = 0; P < TOP; ++P) {
    u32 x = sgn;
    if (P < CAP) x = and_xor(mine[1 + P], u32(__builtin_amdgcn_sbfe(i32(keep), u32(P), 1u)), sgn);
    const u32 cur = acc[P];
    acc[P] = xor3(cur, x, carry);
    carry = majority(cur, x, carry);
  }
}

template <int C, int TOP>
__device__ __forceinline__ void add_more(u32 (&acc)[kSumPlanes], const u32 (&more)[TOP], u32& carry, u32 top) {
  if constexpr (C * kSumChunk < kSumPlanes) {
    if (u32(C * kSumChunk) >= top) return;        // uniform
#pragma unroll
    for (int i = 0; i < kSumChunk; ++i) {
      constexpr int kFirst = C * kSumChunk;
      const u32 x = more[kFirst + i < TOP ? kFirst + i : TOP - 1], cur = acc[kFirst + i];
      acc[kFirst + i] = xor3(cur, x, carry);
      carry = majority(cur, x, carry);
    }
    add_more<C + 1>(acc, more, carry, top);
  }
}

// `n` operands (1 .. AREAS) of the wave: first, first + STEP, ...; FIRST: nothing has been added before.
// fits(widths): called when all their widths are there and nothing has been added; false: the sums are not wanted.
template <bool IX, int STEP, int AREAS, typename FitsFn>
__device__ __forceinline__ bool add_batch(const ReduceCall& c, int k, const LaneOperands& o, u32 seg, int first, int n, u32* wl, PartialSum& sum, u32& err, FitsFn fits) {
  static_assert(AREAS == 2 || AREAS == 4, "pairs of sizes below; sums of four blocks of CAP planes take three planes more");
  const int lane = fresh_lane();
  const u32 b = seg * kWaveBlocks + u32(lane);
  u32 width[AREAS], pick[AREAS], bytes[AREAS];
  i32 code[AREAS];
  u32 shape[AREAS];
#pragma unroll
  for (int i = 0; i < AREAS; ++i) {
    const int s = min(first + i * STEP, k - 1);
    width[i] = u32(__builtin_amdgcn_raw_buffer_load_b8(widths_buffer(o, c, s, i < n), int(b), 0, 0));
  }
#pragma unroll
  for (int i = 0; i < AREAS; ++i) {
    const int s = min(first + i * STEP, k - 1);
    code[i] = i32(__builtin_amdgcn_raw_buffer_load_b32(outliers_buffer(o, c, s, i < n), int(4u * b), 0, 0));
  }
  __builtin_amdgcn_sched_barrier(0);
  auto ask = [&] {
#pragma unroll
    for (int i = 0; i < AREAS; ++i) {
      if (i >= n) break;                          // uniform
      ask_payload_to_lds(o, first + i * STEP, bytes[i], wl + i * kFewArea, lane);
    }
    lds_words_line();
  };
#pragma unroll
  for (int i = 0; i < AREAS; ++i) {
    const int s = min(first + i * STEP, k - 1);
    shape[i] = lane_value(o.shape, s);
    bytes[i] = lane_value(o.bytes, s);
  }
  if (IX) ask();
  if (!fits(width)) return false;

  // Where the blocks are: sizes of two operands a word (at most 64 x 256 words each) through one scan.
  const u32 w_max = c.wide_streams ? 31u : 15u;
  u32 total[AREAS];
#pragma unroll
  for (int i = 0; i < AREAS; i += 2) {
    const u32 lo = psize_words(width[i]), hi = psize_words(width[i + 1]);
    const u32 incl = wave_inclusive_sum(lo | hi << 16), all = lane_value(incl, 63);
    total[i] = all & 0xffffu;
    total[i + 1] = all >> 16;
    pick[i] = (incl & 0xffffu) - lo + (shape[i] & 3u);
    pick[i + 1] = (incl >> 16) - hi + (shape[i + 1] & 3u);
  }
  // An indexed stream is checked as it is used: see place_operand.  (Plain streams: cannot happen.)
  u32 bad = 0, tails = 0;
#pragma unroll
  for (int i = 0; i < AREAS; ++i) {
    const int s = min(first + i * STEP, k - 1);
    bool wrong = __any(width[i] > w_max);
    if (IX) {
      wrong |= i < n && total[i] != shape[i] >> 2;
      tails |= u32(o.tails >> s) & 1u;
    } else {
      const u32 room = lane_value(o.room, s), span = (shape[i] & 3u) + total[i];
      wrong |= span > room;
      const u32 pieces = (span + 3u) & ~3u, whole = min(pieces, room & ~3u);
      bytes[i] = wrong ? 0u : 4u * whole;
      tails |= u32(!wrong && (pieces != whole || span > 256u * kStageLoads));
    }
    bad |= u32(wrong) << i;
  }
  if (bad) {                                      // uniform
    if (IX) err |= status_bit(ZC_ERR_FORMAT);
#pragma unroll
    for (int i = 0; i < AREAS; ++i)
      if ((bad >> i) & 1u) width[i] = 0;
  }
  if (!IX) ask();
  wait_all_but<0>();
  if (tails) {                                    // uniform, and rare
#pragma unroll
    for (int i = 0; i < AREAS; ++i) {
      if (i >= n || ((bad >> i) & 1u)) continue;
      fetch_payload_end(o, first + i * STEP, bytes[i], (shape[i] & 3u) + total[i], wl + i * kFewArea, lane);
    }
  }
  wave_lds_sync();

  u32 widest = max(width[0], width[1]);
  if constexpr (AREAS == 4) widest = max(widest, max(width[2], width[3]));
  auto add = [&](auto cap) {
    constexpr int CAP = decltype(cap)::value, TOP = CAP + 4 < kSumPlanes ? CAP + 4 : kSumPlanes;
    u32 acc[TOP];
#pragma unroll
    for (int P = 0; P < TOP; ++P) acc[P] = 0;
#pragma unroll
    for (int i = 0; i < AREAS; ++i) {
      if (i >= n) break;                          // uniform
      add_block<CAP>(acc, wl + i * kFewArea + (width[i] ? pick[i] : 0u), width[i]);
    }
    sum.bound += u32(n) * ((1u << CAP) - 1u);
    if (sum.top == 0) {                           // uniform
      sum.top = TOP;
#pragma unroll
      for (int P = 0; P < TOP; ++P) sum.acc[P] = acc[P];
    } else {
      const u32 new_top = planes_for(sum.bound);
      grow_sum<0>(sum.acc, sum.top, new_top);
      sum.top = new_top;
      u32 carry = 0;
      add_more<0>(sum.acc, acc, carry, new_top);
    }
  };
#pragma unroll
  for (int i = 0; i < AREAS; ++i) sum.outlier += i64(code[i]);
  if (__any(widest > 16)) add(std::integral_constant<int, 24>{});
  else if (__any(widest > 12)) add(std::integral_constant<int, 16>{});
  else if (__any(widest > 8)) add(std::integral_constant<int, 12>{});
  else if (__any(widest > 4)) add(std::integral_constant<int, 8>{});
  else if (__any(widest != 0)) add(std::integral_constant<int, 4>{});
  return true;
}

// Workgroups of kFewThreads threads: 4 = SEGS x PARTS waves.
constexpr int kFewWaves = 4, kFewThreads = 64 * kFewWaves;

// Segments per tile for a Sum of k operands of so many tiles of four; 0: not here.  With four areas a wave, two workgroups fit a compute
// unit: 512 of them run at the same time.  Beyond, with two areas a wave and four workgroups, it is worth it for few operands (640 tiles, 4 operands 17.3 and 13.8;
// 1024 tiles, 8 operands 26.3 and 26.4; 2048 tiles, 2 operands 26.5 and 28.0).  Fewer segments a tile, us:
//   of four, two, one    128 tiles   4 operands 9.5 9.6 11.2 | 5: 11.2 10.1 11.5 | 8: 12.3 10.6 11.8 | 12: 15.7 12.7 12.7 | 16: 18.6 13.9 13.4
//                        245 tiles   4: 9.8 11.0 20.2 | 5: 11.6 11.3 20.5 | 16: 19.4 16.1 25.2 | 64: 60 49 59;   512 tiles   16: 25.6 32.9
// (From 769 tiles on reduce_kernel with large tiles is faster, where a call may have those, see zc_large_tiles.h.)
constexpr u64 kFewTiles = 512, kFewTilesFull = 1024;
__host__ constexpr int few_segments(int k, u64 tiles) {
  if (k < 2) return 0;
  if (k >= 12 && tiles <= kFewTiles / 4) return 1;
  if (k >= 5 && tiles <= kFewTiles / 2) return 2;
  return tiles <= kFewTiles || (k <= 4 && tiles <= kFewTilesFull) ? 4 : 0;
}

template <bool IX, int SEGS, int AREAS, typename... A>
__global__ __launch_bounds__(kFewThreads, AREAS > 2 ? 2 : 4) void reduce_few_kernel(ReduceArgs a, A... answer) {
  __shared__ __attribute__((aligned(16))) u32 lds[kFewWaves * AREAS * kFewArea];
  __shared__ SumParts<SEGS, kFewWaves / SEGS> parts;
  __shared__ u32 sh_wave_total[SEGS];
  __shared__ u64 sh_base[kFewWaves];
  __shared__ PlainSurvey<IX ? 1 : ZC_MAX_K> survey;
  const AnswerAtEnd<ReduceArgs, A...> at_end(a, answer...);

  ReduceCall c;
  constexpr int PARTS = kFewWaves / SEGS;
  static_assert(AREAS * kFewArea >= kWholeStage + kCopyOver, "the output's words lie there too");
  u32 tile = 0, ntiles = 0, none = 0;
  if (!open_reduce<IX, SEGS, false>(a, c, none, false, tile, ntiles, nullptr, &survey)) return;
  tile = uniform(tile);
  const int wave = wave_id() % SEGS, part = PARTS > 1 ? wave_id() / SEGS : 0;
  u32* const wl = lds + wave_id() * AREAS * kFewArea;
  const u32 seg = tile * u32(SEGS) + u32(wave);
  PayloadSink sink = sum_sink(a, c, ntiles, IX);
  sink.direct = looks_direct(ntiles, kDirectTiles, a.coherent != 0, 0);
  if (SEGS < kTileWaves) sink.apart = kDescApartFine;

  // Whether the tile's blocks fit (see fits_common_path): asked where there may be wide blocks, and of the widths of the operands
  // themselves if they are all there.
  auto all_fit = [&](bool mine) {
    if (lane_id() == 0) parts.fits[wave_id()] = mine;
    lds_barrier();
    u32 all = 1;
#pragma unroll
    for (int i = 0; i < kFewWaves; ++i) all &= parts.fits[i];
    return uniform(all) != 0;
  };
  const bool at_once = a.k <= AREAS * PARTS;
  bool common = true;
  if (c.wide_streams && !at_once) common = all_fit(fits_common_path(a, c, seg, IX));

  PartialSum sum;
#pragma unroll
  for (int p = 0; p < kSumPlanes; ++p) sum.acc[p] = 0;
  sum.top = sum.bound = 0;
  sum.outlier = 0;
  u32 err = 0;
  const LaneOperands o = lane_operands<IX>(c);
#pragma nounroll
  for (int s = part; common && s < a.k; s += AREAS * PARTS) {
    const int n = min((a.k - s + PARTS - 1) / PARTS, AREAS);
    common = add_batch<IX, PARTS, AREAS>(c, a.k, o, seg, s, n, wl, sum, err, [&](const u32 (&width)[AREAS]) {
      if (!c.wide_streams || !at_once) return true;
      bool unfit = false;
      u32 reach = 0, words = 0;
#pragma unroll
      for (int i = 0; i < AREAS; ++i) {
        unfit |= i < n && width[i] > width_limit(c, s + i * PARTS);
        reach += (1u << min(width[i], u32(kSumPlanes))) - 1u;
        words = max(words, psize_words(width[i]));
      }
      return all_fit(!__any(unfit || reach >= (1u << (kSumPlanes - 1)) / PARTS) && wave_sum_u32(words) + 3u <= kMostStaged);
    });
  }
  if (c.ends_bad) err |= status_bit(ZC_ERR_FORMAT);
  if (IX && common && err && lane_id() == 0) raise_status(a.ctl, c.tag, err);
  wait_all_but<0>();

  if (!common) {
    if (part == 0) {
      reduce_wide_tile<IX, SEGS>(a, c, sink, tile, ntiles, wl, sh_wave_total, sh_base);
    } else {
      lds_barrier();
      help_look_back(sink, tile, sh_base, wave_id());
    }
    return;
  }

  // ---- the sums of all waves of a segment meet in the first one ----
  if constexpr (PARTS > 1) {
    const int lane = lane_id();
    if (part) {
      store_partial<0>(sum.acc, wl + lane, sum.top);
      parts.outlier[int(threadIdx.x) - SEGS * 64] = sum.outlier;
      if (lane == 0) parts.bound[wave_id() - SEGS] = sum.bound;
    }
    lds_barrier();
    if (part) {
      lds_barrier();
      help_look_back(sink, tile, sh_base, wave_id());
      return;
    }
#pragma unroll
    for (int p = 1; p < PARTS; ++p) {
      const u32 more = uniform(parts.bound[(p - 1) * SEGS + wave]), theirs = planes_for(more);
      sum.outlier += parts.outlier[(p - 1) * SEGS * 64 + int(threadIdx.x)];
      if (more == 0) continue;
      sum.bound += more;
      const u32 new_top = planes_for(sum.bound);
      grow_sum<0>(sum.acc, sum.top, new_top);
      sum.top = new_top;
      const u32* const planes = lds + (p * SEGS + wave) * AREAS * kFewArea + lane;
      u32 carry = 0;
      add_partial<0>(sum.acc, planes, theirs, planes[64 * (theirs - 1)], carry, sum.top);
    }
  }
  u32 sgn, w;
  close_sum(sum.acc, sum.top, sgn, w);
  auto word = [&](auto i) {
    constexpr int I = decltype(i)::value;        // 0: sign, 1 + p: plane p
    if constexpr (I == 0) return sgn;
    else return sum.acc[I - 1];
  };
  const int lane = fresh_lane();
  const u32 b = seg * kWaveBlocks + u32(lane);
  place_sum_staged<kSumPlanes>(a, c, sink, sum.acc, sgn, w, sum.outlier, b < c.h.nb, b, tile, ntiles, word, wl, sh_wave_total, sh_base, wave, lane);
}

}  // namespace zc
