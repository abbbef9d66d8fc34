// k-way Max and Min of compressed operands (the other aggregation functions of Section 3.2, in
// the k-operand form of the local step of Section 3.1.2).  All operands share the quantisation
// step and the quantiser is monotone, so the largest code is the code of the largest value:
// the result is exact on the grid, one error bound away from the true extreme whatever k is.
// Unlike the Sum of zc_reduce.h an extreme is not linear in the deltas: every operand's block
// is decoded to its 32 codes (payload through LDS, bit-matrix transpose, walk along the Lorenzo
// chain), the running extreme is kept per value in registers, and the result is encoded like a
// compressed block (new deltas, width, planes, look-back placement).
//
// What bounds it is arithmetic, and the registers that the running extremes occupy.  So the common
// path never unpacks the codes: the transposes leave a block's deltas as 16 words of two 16-bit
// fields, and chain, extreme and new deltas work on those words with packed 16-bit instructions,
// two values at a time, 16 registers for the extremes of a block.  For that a block's codes are
// taken relative to the lane's base (the first code of its block in the first operand), or to
// their own first code where that is 2^13 or more away from the base: of two blocks that
// far apart the one behind is shifted to the base of the other, and what leaves 16 bits by that has lost
// (meet_far_codes).  Relative to whichever it is the codes have to stay within [0, 2^15) or
// [-2^15, 0), which the sign bits of the fields show: a delta is below 2^15 in magnitude, so a
// chain cannot leave that range and be back in it within one step.  A wave that meets a block with
// a code 16384 or more away from its first (or a code near the limits of the format) goes on from
// that operand with 32 codes of 32 bits per lane (extreme_rest).  A call with an operand that may have blocks wider
// than 15 bits does so from the start, in all its waves (extreme_any).
// Measured, 8 x 2^24 values unless said otherwise, first with codes unpacked throughout (145 registers, three waves
// per SIMD, and a kernel of its own for wide blocks, launched with every call), then now:
//   smooth field, bound 1e-4 of its range                     79.5   55.5 us
//   8 x 2^23 (1024 tiles)                                     36.2   32.9
//   16 x 2^20                                                 29.7   15.2
//   hard data, 4 x 4 194 304                                  28.2   15.5
//   8 x 1000                                                  18.7    7.6
// (before: those ahead of payloads that go straight to LDS and of trimmed loads, see OperandPipe; the last three are tiles of fewer segments now, see few_op_segments).
// 128 registers, four waves per SIMD, and 12 bytes of scratch that only the
// wide blocks' loop and the ends of the others touch.  It pays that the segment number is a scalar and the lane number
// is computed where it is used: with both in registers across the loops these spilled 240 bytes, and every reload waits
// for the loads under way.
#pragma once

#include "zc_bitmatrix.h"
#include "zc_common.h"
#include "zc_decompress.h"
#include "zc_lds_words.h"
#include "zc_place.h"
#include "zc_reduce.h"
#include "zc_scan.h"

namespace zc {

template <int OP>
__device__ inline i32 extreme(i32 a, i32 b) {
  return OP == ZC_OP_MAX ? max(a, b) : min(a, b);
}

// Two 16-bit values per word.
typedef short i16x2_t __attribute__((ext_vector_type(2)));
__device__ inline i16x2_t as_pair(u32 v) { return __builtin_bit_cast(i16x2_t, v); }
__device__ inline u32 as_word(i16x2_t v) { return __builtin_bit_cast(u32, v); }
__device__ inline u32 add_pairs(u32 a, u32 b) { return as_word(as_pair(a) + as_pair(b)); }
__device__ inline u32 sub_pairs(u32 a, u32 b) { return as_word(as_pair(a) - as_pair(b)); }
__device__ inline u32 max_pairs(u32 a, u32 b) { return as_word(__builtin_elementwise_max(as_pair(a), as_pair(b))); }
__device__ inline u32 min_pairs(u32 a, u32 b) { return as_word(__builtin_elementwise_min(as_pair(a), as_pair(b))); }
template <int OP>
__device__ inline u32 extreme_pairs(u32 a, u32 b) {
  return OP == ZC_OP_MAX ? max_pairs(a, b) : min_pairs(a, b);
}

// The extremes of a wave's blocks as the kernel keeps them until the tile's place is known: Lorenzo deltas
// (d0 = 0), as 16 words of paired 16-bit fields (deltas j and j + 16) when the wave's blocks are at most 15 bits
// wide, else one by one; the largest magnitude among a block's deltas; the first code.
struct ExtremeBlock {
  u32 d[32];
  u32 any;
  i32 outlier;
};

// The lane's sign and plane words out of what lies in its wave's staging area from the sign word on: lo[0..15) = planes
// 0..14, lo[15] = sign word (what is not the block's own is dropped: see pick_block_words).
__device__ inline void keep_operand_words(u32 w, const u32 (&t)[16], u32 (&lo)[16]) {
  const u32 sign = t[0];
  const u32 keep = w ? (1u << w) - 1u : 0u;      // bit p: the block has plane p
#pragma unroll
  for (int p = 0; p < 15; ++p) {
    // (the AND spelled out: seen as one, it is compiled into a test and a selection per plane)
    const u32 m = u32(__builtin_amdgcn_sbfe(i32(keep), u32(p), 1u));
    lo[p] = __builtin_amdgcn_bitop3_b32(t[1 + p], m, m, 0xC0);
  }
  lo[15] = w ? sign : 0u;
}

// The deltas of the lane's block, fields as transpose16x16_pairs leaves them (word j: deltas j and j + 16), from the words
// that were read from its wave's staging area, in place.
__device__ inline void operand_delta_pairs(u32 w, u32 (&f)[16]) {
  if (!__any(w > 7)) {                     // byte fields: word j = deltas j, j + 8, j + 16, j + 24
    keep_operand_words(w, f, f);
    u32 r[8];
#pragma unroll
    for (int p = 0; p < 7; ++p) r[p] = f[p];
    r[7] = f[15];
    magnitude_planes_to_twos<8>(r);
    transpose8x8_quads(r);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      f[j] = __builtin_amdgcn_perm(0u, r[j] << 8, 0x09030801u);       // (8, 9: the sign of bytes 1 and 3, eight times)
      f[j + 8] = __builtin_amdgcn_perm(0u, r[j], 0x09030801u);
    }
  } else {
    const u32 sign = f[0];
#pragma unroll
    for (int p = 0; p < 15; ++p) f[p] = f[p + 1];
    f[15] = sign;
    deltas_from_raw_planes16(f, w);
  }
}

// The operands of a call without wide blocks one after the other.  What bounds this loop is how many bytes a wave has on
// their way: with the extremes in registers a SIMD holds four waves, and with one operand's payload (in 16 registers
// more) on its way per wave, 8 x 2^24 values took 65.2 us, half of it arithmetic.  So the payload goes from memory
// straight to LDS, where a wave has two areas: while operand s is decoded, s + 1 and, as soon as the words of s have
// been read from their area, s + 2 are on their way (63.8 us; 16 x 2^20 29.5 -> 25.6; 8 x 1024, a string of round trips,
// 17.6 -> 15.7).
// What a round needs to ask for an operand's share comes from lane s of values worked out for all operands at once (LaneOperands), and an indexed
// stream's payload is asked for by its index alone, with the widths and first codes: 8 x 2^24 values 58.7 -> 56.0, 16 x 1000 23.6 -> 20.9.
// Each round ends with the four loads to LDS of operand s + 2 and has no other memory access behind them, so that
// "all but the newest four" is what a round waits for at its start; none of the round's loads is behind a branch
// (behind the last operand the range of a load is empty).  The words are read by instructions of our own: ordinary reads
// would wait for every load to LDS that is under way, not only for those to their area.
constexpr u32 kOperandArea = 1056;             // words
static_assert(kOperandArea >= 1027 + 16 && kOperandArea % 4 == 0, "an operand's payload, and the reads behind its last word, must fit");
constexpr u32 kExtremeStage = 2 * kOperandArea;
static_assert(kExtremeStage >= u32(kWaveStage) && kExtremeStage >= 64 * 32, "the output is staged in the same place, and a wave's extremes");

__device__ inline u32 lds_address(const u32* p) { return u32(reinterpret_cast<uintptr_t>((const LdsWord*)p)); }
// Words FIRST .. FIRST + 7 of what lies in LDS from byte address `at` on.  Instructions of our own: ordinary reads would wait for every load to LDS that is
// under way, not only for those to their area.
template <int FIRST, int ROOM>
__device__ __forceinline__ void read_lds_words(u32 at, u32 (&t)[ROOM]) {
  static_assert(FIRST + 8 <= ROOM);
  u64 v[4];
  asm volatile(
      "ds_read2_b32 %0, %4 offset0:%5 offset1:%6\n\t"
      "ds_read2_b32 %1, %4 offset0:%7 offset1:%8\n\t"
      "ds_read2_b32 %2, %4 offset0:%9 offset1:%10\n\t"
      "ds_read2_b32 %3, %4 offset0:%11 offset1:%12\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
      : "v"(at), "n"(FIRST), "n"(FIRST + 1), "n"(FIRST + 2), "n"(FIRST + 3), "n"(FIRST + 4), "n"(FIRST + 5), "n"(FIRST + 6), "n"(FIRST + 7)
      : "memory");
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    t[FIRST + 2 * i] = u32(v[i]);
    t[FIRST + 2 * i + 1] = u32(v[i] >> 32);
  }
}

// What a wave knows about an operand's blocks once their widths are there.
struct PipeOperand {
  u32 w, pick;              // the lane's block: its width, and where its sign word lies in the operand's area
  u32 bytes, span;          // uniform: what is asked for, and the words that the segment takes
  bool tail;                // uniform: the one leaves out some of the other
};

// PARTS: the wave's operands are `share.count` of the call's, PARTS apart (s counts those).
template <bool IX, int PARTS>
struct OperandPipe {
  LaneOperands o;
  PipeOperand cur, next, ahead;            // operands s (whose words have been read), s + 1 and s + 2
  i32 first, first_next, first_ahead;      // the first code of the lane's block in them
  // The width of the lane's block: in operands s, s + 1 and s + 2 (indexed streams, whose segments are found without it), or in s + 3
  u32 width, width_next, width_ahead;

  // Which of the call's operands is the wave's s-th (behind the last one: the last one).
  __device__ __forceinline__ static int which(const ReduceShare& share, int s) { return share.first + PARTS * min(s, share.count - 1); }

  // What to ask for of operand s (nothing behind the last one); of a plain stream its widths have to be there.
  __device__ __forceinline__ void open_ahead(PipeOperand& p, const ReduceShare& share, int s, u32 blocks_width, u32& err) {
    const int of = which(share, s);
    if (IX) {
      p.bytes = lane_value(o.bytes, of);
    } else {
      place(p, of, blocks_width, err);
      const u32 room = lane_value(o.room, of), pieces = (p.span + 3u) & ~3u, whole = min(pieces, room & ~3u);
      p.bytes = 4u * whole;
      p.tail = pieces != whole || p.span > 256u * kStageLoads;
    }
    if (s >= share.count) p.bytes = 0;
  }
  // See place_operand (s: one of the call's operands).
  __device__ __forceinline__ void place(PipeOperand& p, int s, u32 blocks_width, u32& err) {
    const u32 words = psize_words(blocks_width), incl = wave_inclusive_sum(words), total = lane_value(incl, 63);     // (at most 64 x 256)
    const u32 shape = lane_value(o.shape, s);
    p.span = (shape & 3u) + total;
    p.pick = (shape & 3u) + incl - words;
    p.w = blocks_width;
    if (IX) p.tail = ((o.tails >> s) & 1u) != 0;
    if (__any(blocks_width > 15) || (IX ? total != shape >> 2 : p.span > lane_value(o.room, s))) {      // uniform
      if (IX) err |= status_bit(ZC_ERR_FORMAT);
      p.w = p.span = 0;
      p.tail = false;
    }
  }

  __device__ __forceinline__ void open(const ReduceCall& c, const ReduceShare& share, u32* wl, u32& err) {
    const int lane = fresh_lane();
    const u32 b = share.seg * kWaveBlocks + u32(lane);
    o = lane_operands<IX>(c);
    width = load_width(c, share, 0, b);
    width_next = load_width(c, share, 1, b);
    if (!IX) width_ahead = load_width(c, share, 2, b);
    first = load_first(c, share, 0, b);
    first_next = load_first(c, share, 1, b);
    lds_words_line();
    open_ahead(cur, share, 0, width, err);
    ask_payload_to_lds(o, which(share, 0), cur.bytes, wl, lane);
    lds_words_line();
    u32 bad = 0;
    open_ahead(next, share, 1, width_next, bad);
    ask_payload_to_lds(o, which(share, 1), next.bytes, wl + kOperandArea, lane);
    lds_words_line();
  }
  __device__ __forceinline__ u32 load_width(const ReduceCall& c, const ReduceShare& share, int s, u32 b) const {
    return u32(__builtin_amdgcn_raw_buffer_load_b8(widths_buffer(o, c, which(share, s), true), int(b), 0, 0));
  }
  __device__ __forceinline__ i32 load_first(const ReduceCall& c, const ReduceShare& share, int s, u32 b) const {
    return i32(__builtin_amdgcn_raw_buffer_load_b32(outliers_buffer(o, c, which(share, s), true), int(4u * b), 0, 0));
  }
  // The words of operand s from its lanes' sign words on, and operand s + 2 on its way.  Operands in turn from 0 on.
  __device__ __forceinline__ void take(const ReduceCall& c, const ReduceShare& share, int s, u32* wl, u32 (&t)[16], u32& err) {
    u32* const area = wl + (s & 1 ? kOperandArea : 0u);
    const int lane = fresh_lane();
    if (s) {
      cur = next;
      first = first_next;
      next = ahead;
      first_next = first_ahead;
      if (IX) {
        width = width_next;
        width_next = width_ahead;
      }
    }
    lds_words_line();
    wait_all_but<kStageLoads>();
    if (IX) place(cur, which(share, s), width, err);
    if (cur.tail) {                            // uniform, and rare
      fetch_payload_end(o, which(share, s), cur.bytes, cur.span, area, lane);
      wave_lds_sync();
    }
    const u32 at = lds_address(area) + 4u * (cur.w ? cur.pick : 0u);
    read_lds_words<0>(at, t);
    read_lds_words<8>(at, t);
    // operand s + 2, in the place of operand s
    open_ahead(ahead, share, s + 2, width_ahead, err);
    const u32 b = share.seg * kWaveBlocks + u32(lane);
    first_ahead = load_first(c, share, s + 2, b);
    width_ahead = load_width(c, share, s + (IX ? 2 : 3), b);
    lds_words_line();
    ask_payload_to_lds(o, which(share, s + 2), ahead.bytes, area, lane);
    lds_words_line();
  }
  // Behind the last operand: what is still on its way (empty ranges, which leave zeros) has landed.
  __device__ __forceinline__ void close() { wait_all_but<0>(); }
};

// The common path keeps codes as 16-bit code - base + bias, where base is the first code of one of the operands'
// blocks and the codes must lie within kCodeReach of it: in [0, 2^15) for Max, in [-2^15, 0) for Min.
constexpr i32 kCodeReach = 1 << 14;
template <int OP>
constexpr i32 kCodeBias = OP == ZC_OP_MAX ? kCodeReach : -kCodeReach;
// A block whose first code is within kNearFirst of the base is taken relative to the base, one that lies farther away
// relative to its own first code (see meet_far_codes).
constexpr i32 kNearFirst = 1 << 13;
constexpr i32 kFirstLimit = i32(kMaxCode) - 2 * kCodeReach;

// Brings the extremes acc and an operand's codes f to one base, where f's is `ahead` of acc's (positive: towards the
// extreme): whichever lies behind is shifted to the base of the other.  A distance of more than 2^15 - 1 counts as
// that: what is shifted then ends at or behind the limit that the other's codes do not pass, so the other's codes win,
// as they should.  No sum overflows: acc and f have the same sign throughout (see kCodeReach), and a shift goes
// against it.
template <int OP>
__device__ inline void meet_far_codes(u32 (&acc)[16], u32 (&f)[16], i32 ahead) {
  const i32 shift = max(-0x7fff, min(ahead, 0x7fff));
  const i32 toward = OP == ZC_OP_MAX ? shift : -shift;
  const u32 acc_by = ahead > 0 ? u32(-toward) & 0xffffu : 0u, f_by = ahead > 0 ? 0u : u32(toward) & 0xffffu;
  const u32 acc_pair = acc_by | (acc_by << 16), f_pair = f_by | (f_by << 16);
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    acc[j] = add_pairs(acc[j], acc_pair);
    f[j] = add_pairs(f[j], f_pair);
  }
}

// The common path: the extremes of as many operands as it can take (returned, uniform).  If that is not all, the next
// one is decoded: f = its codes modulo 2^16, `from` what the first of them starts from.
template <bool IX, int OP, int PARTS>
__device__ __forceinline__ int extreme_packed(const ReduceCall& c, const ReduceShare& share, u32* wl,
                                              OperandPipe<IX, PARTS>& pipe, u32 (&acc)[16], u32 (&f)[16], u32& from, i32& base, u32& err) {
  base = pipe.first;
  // (every code is within reach of some operand's first code, that of its base, and so inside the format's limits: no
  // check of the result is needed)
  bool outside = u32(base) + u32(kFirstLimit) > u32(2 * kFirstLimit);
#pragma unroll
  for (int j = 0; j < 16; ++j) acc[j] = OP == ZC_OP_MAX ? 0u : 0xffffffffu;
  // The loop has one exit, told in a scalar that the compiler cannot see through, and one place where acc changes: with
  // an exit from its middle the two exits are merged and acc is copied in every round (8 x 2^24 values 64.9 -> 64.4 us,
  // 64 x 100 003, a chain of round trips, 115 -> 111.5).
  int s = 0;
  u32 going = 1;
#pragma nounroll
  while (going) {
    pipe.take(c, share, s, wl, f, err);
    const u32 apart = u32(pipe.first) - u32(base);
    const bool far = apart + u32(kNearFirst) >= u32(2 * kNearFirst);
    const u32 start = ((far ? 0u : apart) + u32(kCodeBias<OP>)) & 0xffffu;
    // f, word j: the deltas, and then the codes, j and j + 16
    if (!__any(pipe.cur.w != 0)) {                  // nothing but constant blocks: every code is the block's first
      const u32 both = start | (start << 16);
#pragma unroll
      for (int j = 0; j < 16; ++j) f[j] = both;
    } else {
      operand_delta_pairs(pipe.cur.w, f);
      // both halves of the block at once, the second one from zero; then it gets what the first one ends with
      f[0] = add_pairs(f[0], start);
#pragma unroll
      for (int j = 1; j < 16; ++j) f[j] = add_pairs(f[j], f[j - 1]);
      const u32 half = f[15] << 16;
      u32 seen = OP == ZC_OP_MAX ? 0u : ~0u;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        f[j] += half;                          // (the low field of `half` is zero: no carry between the fields)
        seen = OP == ZC_OP_MAX ? seen | f[j] : seen & f[j];
      }
      outside |= ((OP == ZC_OP_MAX ? seen : ~seen) & 0x80008000u) != 0;
    }
    bool stop = false;
    if (__any(outside || far)) {               // (one vote, one branch: in a small call these are time, too)
      outside |= far && u32(pipe.first) + u32(kFirstLimit) > u32(2 * kFirstLimit);
      stop = __any(outside);
      if (!stop) {
        const i32 ahead = far ? i32(OP == ZC_OP_MAX ? apart : 0u - apart) : 0;
        meet_far_codes<OP>(acc, f, ahead);
        if (ahead > 0) base = pipe.first;
      }
    }
    from = start;
    if (!stop) {
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[j] = extreme_pairs<OP>(acc[j], f[j]);
      ++s;
    }
    going = uniform(!stop && s < share.count ? 1u : 0u);
  }
  return s;
}

// The new deltas of packed extremes, in pairs; those of the second half's first value cross the halves.
template <int OP>
__device__ __forceinline__ void close_packed(const u32 (&acc)[16], i32 base, ExtremeBlock& out) {
  u32 top = 0, bottom = 0;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const u32 before = j ? acc[j - 1] : acc[15] << 16;
    out.d[j] = j ? sub_pairs(acc[j], before) : sub_pairs(acc[j], before) & 0xffff0000u;
    top = max_pairs(top, out.d[j]);
    bottom = min_pairs(bottom, out.d[j]);
  }
  const i32 hi = max(i32(top) >> 16, i32(top << 16) >> 16), lo = min(i32(bottom) >> 16, i32(bottom << 16) >> 16);
  out.any = u32(max(hi, -lo));
  out.outlier = base + (i32(acc[0] << 16) >> 16) - kCodeBias<OP>;
}

// A segment whose payload is more than stage_to_lds brings in (all its blocks are wide then) comes in two parts,
// the blocks of lanes 0..31 and those of lanes 32..63.
static_assert(kMostStaged >= 3 + 32 * 32 && kMostStaged + 32 <= kExtremeStage, "half a segment of widest blocks, and the reads behind its last word, must fit the wave's area");

__device__ inline u32 operand_parts(const OperandPlace& p) { return p.span > kMostStaged ? 2u : 1u; }     // uniform

__device__ inline OperandPlace operand_part(const OperandPlace& p, u32 part, int lane) {
  if (operand_parts(p) == 1) return p;
  const u32 split = lane_value(p.pick, 32);                // where lane 32's words start
  const u32 begin = part ? split & ~3u : 0u;
  OperandPlace q = p;
  q.src0 = p.src0 + begin;
  q.room = p.room - begin;
  q.span = (part ? p.span : split) - begin;
  const bool mine = u32(lane >> 5) == part;
  q.w = mine ? p.w : 0u;
  q.pick = mine ? p.pick - begin : 0u;
  return q;
}

// The new deltas of extremes held in 32 bits.
__device__ __forceinline__ void close_any(i32 (&acc)[32], bool active, ExtremeBlock& out, u32& err) {
  // range of the codes (operands of a valid stream are inside it, so is their extreme)
  i32 hi = acc[0], lo = acc[0];
#pragma unroll
  for (int j = 1; j < 32; ++j) {
    hi = max(hi, acc[j]);
    lo = min(lo, acc[j]);
  }
  const bool out_of_range = active && (i64(hi) > kMaxCode || i64(lo) < -kMaxCode);
  if (out_of_range) err |= status_bit(ZC_ERR_RANGE);
  out.outlier = acc[0];
  // codes -> Lorenzo deltas, last first
  i32 top = 0, bottom = 0;
#pragma unroll
  for (int j = 31; j >= 1; --j) {
    acc[j] = i32(u32(acc[j]) - u32(acc[j - 1]));
    top = max(top, acc[j]);
    bottom = min(bottom, acc[j]);
  }
  acc[0] = 0;
  out.any = out_of_range ? 0u : max(u32(top), u32(-bottom));
  if (__any(active && out.any > 0x7fffu)) {
#pragma unroll
    for (int j = 0; j < 32; ++j) out.d[j] = u32(acc[j]);
  } else {
#pragma unroll
    for (int j = 0; j < 16; ++j) out.d[j] = field16_pair(acc[j], acc[j + 16]);
  }
}

// The operands from s on, none of them with wide blocks, in 32 bits.  f: the deltas of operand s.
template <bool IX, int OP, int PARTS>
__device__ __forceinline__ void extreme_rest(const ReduceCall& c, const ReduceShare& share, u32* wl,
                                             OperandPipe<IX, PARTS>& pipe, i32 (&acc)[32], u32 (&f)[16], int s, u32& err) {
#pragma nounroll
  for (;;) {
    u32 code = u32(pipe.first);
#pragma unroll
    for (int j = 0; j < 32; ++j) {
      code += u32(__builtin_amdgcn_sbfe(i32(f[j & 15]), u32(16 * (j >> 4)), 16u));
      acc[j] = extreme<OP>(acc[j], i32(code));
    }
    if (++s >= share.count) return;
    pipe.take(c, share, s, wl, f, err);
    operand_delta_pairs(pipe.cur.w, f);
  }
}

// Operands without wide blocks.  True: they are in `out` (the common path has taken them all), false: in acc.
template <bool IX, int OP, int PARTS>
__device__ __forceinline__ bool extreme_narrow(const ReduceCall& c, const ReduceShare& share, u32* wl,
                                               ExtremeBlock& out, i32 (&acc)[32], u32& err) {
  OperandPipe<IX, PARTS> pipe;
  pipe.open(c, share, wl, err);
  u32 pairs[16], f[16], from = 0;
  i32 base;
  const int s = extreme_packed<IX, OP, PARTS>(c, share, wl, pipe, pairs, f, from, base, err);
  if (s == share.count) {
    pipe.close();
    if constexpr (PARTS == 1) {
      close_packed<OP>(pairs, base, out);
      return true;
    }
#pragma unroll
    for (int j = 0; j < 32; ++j) acc[j] = base + i32(i16x2_t(as_pair(pairs[j & 15]))[j >> 4]) - kCodeBias<OP>;
    return false;
  }
  // its deltas again
  from |= f[15] << 16;
#pragma unroll
  for (int j = 15; j >= 1; --j) f[j] = sub_pairs(f[j], f[j - 1]);
  f[0] = sub_pairs(f[0], from);
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    const i32 code = base + i32(i16x2_t(as_pair(pairs[j & 15]))[j >> 4]) - kCodeBias<OP>;
    acc[j] = s ? code : OP == ZC_OP_MAX ? i32(0x80000000u) : i32(0x7fffffff);
  }
  extreme_rest<IX, OP, PARTS>(c, share, wl, pipe, acc, f, s, err);
  pipe.close();
  return false;
}

// Any codes and widths.
template <bool IX, int OP, int PARTS>
__device__ __forceinline__ void extreme_any(const ReduceArgs& a, const ReduceCall& c, const ReduceShare& share, u32* wl,
                                            i32 (&acc)[32], u32& err) {
#pragma unroll
  for (int j = 0; j < 32; ++j) acc[j] = OP == ZC_OP_MAX ? i32(0x80000000u) : i32(0x7fffffff);
  const LaneOperands o = lane_operands<IX>(c, 3 + 64 * 32);
  u32 width = u32(__builtin_amdgcn_raw_buffer_load_b8(widths_buffer(o, c, share.first, true), int(share.seg * kWaveBlocks + u32(fresh_lane())), 0, 0));
#pragma nounroll
  for (int s = share.first; s < a.k; s += PARTS) {
    const int lane = fresh_lane();
    const u32 b = share.seg * kWaveBlocks + u32(lane);
    const u32* const payload = lane_share(o, s);
    OperandPlace cur;
    {
      const u32 words = psize_words(width), incl = wave_inclusive_sum(words), total = lane_value(incl, 63);     // (at most 64 x 256)
      const u32 shape = lane_value(o.shape, s);
      cur.src0 = 0;
      cur.room = lane_value(o.room, s);
      cur.span = (shape & 3u) + total;
      cur.pick = (shape & 3u) + incl - words;
      cur.w = width;
      if (__any(width > width_limit(c, s)) || (IX ? total != shape >> 2 : cur.span > cur.room)) {      // uniform; see place_operand
        if (IX) err |= status_bit(ZC_ERR_FORMAT);
        cur.w = cur.span = 0;
      }
    }
    u32 code = u32(__builtin_amdgcn_raw_buffer_load_b32(outliers_buffer(o, c, s, true), int(4u * b), 0, 0));
    if (!__any(cur.w > 15)) {
      const OperandStage stage = load_operand_payload(payload, cur, lane);
      if (s + PARTS < a.k) width = u32(__builtin_amdgcn_raw_buffer_load_b8(widths_buffer(o, c, s + PARTS, true), int(b), 0, 0));
      stage_to_lds(stage, cur, payload, wl, lane);
      wave_lds_sync();
      u32 f[16];
      const u32* const mine = wl + (cur.w ? cur.pick : 0u);
#pragma unroll
      for (int p = 0; p < 15; ++p) f[p] = mine[1 + p];
      f[15] = mine[0];
      wave_lds_sync();
      deltas_from_raw_planes16(f, cur.w);
#pragma unroll
      for (int j = 0; j < 32; ++j) {
        code += u32(__builtin_amdgcn_sbfe(i32(f[j & 15]), u32(16 * (j >> 4)), 16u));
        acc[j] = extreme<OP>(acc[j], i32(code));
      }
    } else {
      if (s + PARTS < a.k) width = u32(__builtin_amdgcn_raw_buffer_load_b8(widths_buffer(o, c, s + PARTS, true), int(b), 0, 0));
      u32 lo[16], hi[16];                       // planes 0..15; planes 16..30 and the sign word
#pragma unroll
      for (int p = 0; p < 16; ++p) lo[p] = hi[p] = 0;
#pragma nounroll
      for (u32 part = 0; part < operand_parts(cur); ++part) {
        const OperandPlace here = operand_part(cur, part, lane);
        stage_to_lds(load_operand_payload(payload, here, lane), here, payload, wl, lane);
        wave_lds_sync();
        const u32* const mine = wl + (here.w ? here.pick : 0u);
        const u32 keep = (1u << here.w) - 1u;  // bit p: the block has plane p
#pragma unroll
        for (int p = 0; p < 16; ++p) lo[p] |= mine[1 + p] & u32(__builtin_amdgcn_sbfe(i32(keep), u32(p), 1u));
#pragma unroll
        for (int p = 0; p < 15; ++p) hi[p] |= mine[17 + p] & u32(__builtin_amdgcn_sbfe(i32(keep), u32(16 + p), 1u));
        hi[15] |= here.w ? mine[0] : 0u;
        wave_lds_sync();
      }
      transpose16x16_pairs(lo);
      transpose16x16_pairs(hi);
#pragma unroll
      for (int j = 0; j < 32; ++j) {
        const u32 f = j < 16 ? (lo[j & 15] & 0xffffu) | (hi[j & 15] << 16) : (lo[j & 15] >> 16) | (hi[j & 15] & 0xffff0000u);
        code += u32(delta_from_field<32>(f));
        acc[j] = extreme<OP>(acc[j], i32(code));
      }
    }
  }
}

// Segments per tile for k operands of so many tiles of four: with fewer, their operands are divided among more waves, and there are more
// workgroups, of which four fit a compute unit.  us per call, tiles of four, two and one (Max of power-law fields at 1e-4 of their range | of hard data):
//            1 tile             49                  128                 245                 384             512
//    2 x   7.8  7.1           9.1  8.4            9.5  9.2           10.0 10.7           11.2 12.1       11.6 14.0
//    4 x   9.4  8.0  7.3     11.1  9.4  9.0      11.5 10.0 10.6      11.8 11.9 13.2      14.1 14.2       14.5 16.2
//    8 x  13.5  9.8  8.1     15.4 11.4 10.0      15.8 12.0 12.2      16.1 15.2 15.6      19.7 18.0 26.4  20.2 20.9 30.9
//   16 x  21.8 13.7 10.3     23.9 15.6 12.0      25.2 16.5 15.2      24.1 20.2 20.4      31.7 25.2 32.5  31.9 30.1 39.1
//    8 x  18.8 12.7 10.1     17.8 12.5 10.5      18.3 13.4 12.1      18.5 15.6 16.3      22.2 18.9 26.4  22.6 22.2 31.0
__host__ constexpr int few_op_segments(int k, u64 tiles) {
  if (k < 2) return 4;
  if (tiles <= 128) return k >= (tiles <= 64 ? 4 : 8) ? 1 : 2;
  return (tiles <= 256 ? k >= 8 : tiles <= 512 && k >= 12) ? 2 : 4;
}

// SEGS: segments of a tile (eight: see zc_large_tiles.h).  Their operands are divided among PARTS = 4 / SEGS waves each (one from four segments on), whose extremes meet in LDS: see zc_reduce_few.h.
template <bool IX, int OP, int SEGS = kTileWaves, typename... A>
__global__ __launch_bounds__(SEGS > kTileWaves ? 64 * SEGS : kTileThreads, 4) void reduce_op_kernel(ReduceArgs a, A... answer) {
  constexpr int WAVES = SEGS > kTileWaves ? SEGS : kTileWaves;
  __shared__ __attribute__((aligned(16))) u32 lds[WAVES * kExtremeStage];
  __shared__ u32 sh_tile;
  __shared__ u32 sh_wave_total[SEGS];
  __shared__ u64 sh_base[WAVES];
  __shared__ PlainSurvey<IX ? 1 : ZC_MAX_K> survey;
  const AnswerAtEnd<ReduceArgs, A...> at_end(a, answer...);

  ReduceCall c;
  constexpr int PARTS = WAVES / SEGS;
  u32 width0 = 0, tile = 0, ntiles = 0;
  if (!open_reduce<IX, SEGS, PARTS == 1>(a, c, width0, false, tile, ntiles, &sh_tile, &survey)) return;
  const ParsedHeader& h = c.h;
  const int wave = wave_id() % SEGS, part = PARTS > 1 ? wave_id() / SEGS : 0;
  u32* const wl = lds + wave_id() * kExtremeStage;
  const u32 seg = uniform(tile * u32(SEGS) + u32(wave));
  const ReduceShare share{seg, part, (a.k - part + PARTS - 1) / PARTS};
  u32 err = 0;
  if (c.ends_bad) err |= status_bit(ZC_ERR_FORMAT);

  ExtremeBlock eb;
  i32 codes[32];
  bool closed = false;
  if (c.wide_streams) extreme_any<IX, OP, PARTS>(a, c, share, wl, codes, err);
  else closed = extreme_narrow<IX, OP, PARTS>(c, share, wl, eb, codes, err);
  PayloadSink sink{a.out, a.out_cap, h.nb, a.ctl, a.desc, IX, a.coherent != 0, looks_direct(ntiles, kDirectTiles, a.coherent != 0, 0u), 0u, c.tag};
  if constexpr (PARTS > 1) {
    sink.apart = kDescApartFine;
    if (part) {
      u32* const mine = wl + fresh_lane();
#pragma unroll
      for (int j = 0; j < 32; ++j) mine[64 * j] = u32(codes[j]);
      if (err) raise_status(a.ctl, c.tag, err);
    }
    lds_barrier();
    if (part) {
      lds_barrier();
      help_look_back(sink, tile, sh_base, wave_id());
      return;
    }
#pragma unroll
    for (int p = 1; p < PARTS; ++p) {
      const u32* const theirs = lds + (p * SEGS + wave) * kExtremeStage + fresh_lane();
#pragma unroll
      for (int j = 0; j < 32; ++j) codes[j] = extreme<OP>(codes[j], i32(theirs[64 * j]));
    }
  }
  if (!closed) close_any(codes, share.seg * kWaveBlocks + u32(fresh_lane()) < h.nb, eb, err);

  const int lane = fresh_lane();
  const u32 b = seg * kWaveBlocks + u32(lane);
  const bool active = b < h.nb;
  Placement pl;
  pl.w = (active && eb.any) ? 32u - u32(__builtin_clz(eb.any)) : 0u;
  pl.wmax = wave_max_u32(pl.w);
  const u32 words = psize_words(pl.w);
  const u32 incl = wave_inclusive_sum(words);
  pl.wave_total = lane_value(incl, 63);
  pl.half0_total = lane_value(incl, 31);
  pl.off_in_wave = incl - words;
  if (lane == 0) sh_wave_total[wave] = pl.wave_total | (IX && pl.wmax > 15 ? kWaveWideMark : 0u);
  lds_barrier();
  sum_wave_totals(sh_wave_total, wave, IX, pl);
  if (threadIdx.x == 0) publish_tile_size(sink, tile, pl.tile_total, pl.tile_wide);
  if (err) raise_status(a.ctl, c.tag, err);
  const bool narrow = pl.wmax <= 15;         // uniform
  const TileBase tb = resolve_tile_base(sink, pl, tile, sh_base, wave, lane, [&] {
    if (!narrow) return;
    u32 pw[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) pw[j] = eb.d[j];
    planes16_from_fields(pw);
    stage_wave_words<16>([&](auto i) {
      constexpr int I = decltype(i)::value;          // 0: sign, 1 + p: plane p
      if constexpr (I == 0) return pw[15];
      else return pw[I - 1];
    }, pl, wl);
  });
  if (lane == 0) write_index_entry(sink, seg, tb.words + pl.wave_off);
  if (narrow) {
    copy_staged_wave<16, true>(sink, pl, tb.words, wl, lane);
  } else {
    i32 d[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) d[j] = i32(eb.d[j]);
    u32 plo[16], phi[16];
    planes_from_deltas32(d, plo, phi);
    copy_wave_out<32, true>(sink, [&](auto i) {
      constexpr int I = decltype(i)::value;
      if constexpr (I == 0) return phi[15];
      else if constexpr (I <= 16) return plo[I - 1];
      else return phi[I - 17];
    }, pl, tb.words, wl, lane);
  }
  store_tables<kAccessOnce>(sink, b, pl.w, eb.outlier);     // (at the very end: a store under way is waited for by every poll of the look-back)
  finish_stream<SEGS>(sink, pl, tile, ntiles, tb);
}

}  // namespace zc
