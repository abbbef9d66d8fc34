// Fused local step of the compressed Allreduce (Section 3.1.2: per round "decompress, reduce,
// recompress"; Sum aggregation of Section 3.2), for k operands at once.
//
// All operands share the quantisation step, and both the Lorenzo delta and the sum are
// linear, so the sum of the operands' deltas is the delta of the summed codes: nothing has to
// be dequantised, and no prefix sum is needed.  More than that, the deltas never have to leave
// their bit-plane form.  One lane owns one block; a plane word holds one bit of each of the
// block's 32 deltas, so a ripple-carry adder written with bitwise operations on plane words
// adds 32 deltas at once: a handful of operations per plane per operand for the whole block.
// The sum is kept in two's complement planes, converted back to sign + magnitude planes at
// the end, and its highest non-zero plane gives the new code length.  Output placement is
// the same ticketed look-back scan as in compression.
//
// A tile takes one of two paths.  On the common one a wave brings its payload of one operand into
// LDS with 16-byte loads, and the loads of the next operand fly while the current one is added;
// the summed planes go to LDS in one pass and leave as coalesced stores.  Operand payloads are
// read, and the output stream is written, with the non-temporal hint (see load_once).  Its
// accumulator and its staging take all blocks of at most 15 bits, and most segments that have a
// wider one (fits_common_path).  The other path (reduce_wide_tile) takes any widths with per-lane
// loads, a few planes at a time.  Whether any operand has a wide block anywhere is known when a
// workgroup starts (from the width tables of plain streams, from the version words of indexed
// ones); only in such a call do the waves look where.
// IX = the streams are indexed (see index_bytes): operands bring the positions of their
// segments along, which every wave checks against the widths it reads, and the output gets
// its own index as it is placed.
#pragma once

#include "zc_common.h"
#include "zc_large_tiles.h"
#include "zc_place.h"
#include "zc_report.h"
#include "zc_scan.h"

namespace zc {

struct ReduceArgs {
  StreamRef in[ZC_MAX_K];
  int k;
  StreamIndex index;
  u32 self;          // plain streams: the kernel sums the width tables itself (see judge_plain_streams)
  u8* out;
  u64 out_cap;
  Control* ctl;
  u64* desc;
  u32 ticketed;      // tiles handed out by tickets instead of by workgroup id
  u32 coherent;      // the look-back reads the tile's own chain with device-coherent loads too
  u64 nonce;         // drawn by the host per call, goes into the call's tag (see launch_tag)
  // A reduce done in parts (zc_reduce_compressed_part): this launch takes the tiles
  // [first_tile, end_tile) of the output, end_tile = 0 meaning all of them; a later part
  // (adopt) belongs to the call whose tag the first part left in the control block.
  u32 first_tile, end_tile, adopt;
  // The n that the call takes: of a reduce done in parts the one that the parts were laid out for; else any that has a descriptor in the
  // workspace for each of its tiles.
  u64 n_least, n_most;
};

// What a workgroup knows about the call once the headers are judged.
struct ReduceCall {
  ParsedHeader h;    // header of operand 0 (all operands have its n and bound)
  u64 tag;           // the call's tag
  u64 ltag;          // this launch's tag (tile tickets)
  u64 nsum;          // sum of the operands' nsum
  u64 wide_streams;  // bit s: operand s may have blocks wider than 15 bits
  u32 part_end;      // a reduce done in parts: one past the last tile of this part; else 0
  u32 places, ends;  // lane s: payload word offset of the wave's segment in operand s (0 if there is no such segment), and where it ends (indexed streams)
  u64 base, bytes;   // lane s: where operand s is, and its buffer's size
  bool ends_bad;     // indexed streams: the wave holds an end of the index, which some operand contradicts
  u32 nb, widths, firsts, payload;      // blocks of every stream, and where its width bytes, first codes and payload begin (all below 2^29)
};

// Header fields and table padding of the output stream; one thread.
__device__ inline void write_reduce_header(const ReduceArgs& a, const ReduceCall& c, u32 ntiles, bool ix) {
  const ParsedHeader& h = c.h;
  const u64 tend = tables_end(h.nb, ix);
  if (c.nsum > 0xffffffffull) raise_status(a.ctl, c.tag, status_bit(ZC_ERR_RANGE));
  if (a.out_cap >= tend) write_stream_header(a.out, h.n, h.nb, h.eb_bits, u32(c.nsum), ix, ntiles == 0);
  else raise_status(a.ctl, c.tag, status_bit(ZC_ERR_CAPACITY));
  if (ntiles == 0) a.ctl->result = tend;
}

// Exact range check of one block's summed codes, for lanes whose cheap bound did not settle
// it: rebuild every delta from the magnitude planes and walk the Lorenzo chain in 64 bits.
template <int NP>
__device__ inline bool block_out_of_range(const u32 (&mag)[NP], u32 sign, i64 outlier) {
  i64 q = outlier;
  bool bad = q > kMaxCode || q < -kMaxCode;
  for (int j = 1; j < 32; ++j) {
    i64 m = 0;
#pragma unroll
    for (int p = 0; p < NP; ++p) m |= i64((mag[p] >> j) & 1u) << p;
    q += ((sign >> j) & 1u) ? -m : m;
    bad |= q > kMaxCode || q < -kMaxCode;
  }
  return bad;
}

// Whether the tiles of a Sum look back directly (see kDirectTiles, with the measurements).
__device__ inline bool sum_looks_direct(const ReduceArgs& a, u32 ntiles) {
  return looks_direct(ntiles, a.k <= 3 ? kDirectTiles : kDirectTiles / 2, a.coherent != 0, a.end_tile);
}

__device__ inline PayloadSink sum_sink(const ReduceArgs& a, const ReduceCall& c, u32 ntiles, bool ix) {
  return {a.out, a.out_cap, c.h.nb, a.ctl, a.desc, ix, a.coherent != 0, sum_looks_direct(a, ntiles), c.part_end, c.tag};
}

// Range screen and placement of a summed block inside its wave and tile, then the shared
// back half.  mag[0..NP) = magnitude planes, sign = sign word, w = highest non-zero plane + 1;
// `word(i)` hands out the sign word (i = 0) and plane i - 1, for at most NW words.
// SEGS: segments of a tile; LOOK: waves that look back.
template <int NW, int NP, int SEGS, int LOOK, typename WordFn>
__device__ inline void place_sum(const ReduceArgs& a, const ReduceCall& c, const PayloadSink& sink, const u32 (&mag)[NP], u32 sign, u32 w,
                                 i64 outlier, bool active, u32 b, u32 tile, u32 ntiles, WordFn word, u32* wl,
                                 u32 (&sh_wave_total)[SEGS], u64 (&sh_base)[LOOK], int wave, int lane) {
  const ParsedHeader& h = c.h;
  const bool ix = sink.ix;
  const u64 tend = tables_end(h.nb, ix);
  if (!active) w = 0;
  u32 err = 0;
  if (active) {
    const i64 ao = outlier < 0 ? -outlier : outlier;
    const i64 reach = ao + 31 * ((i64(1) << w) - 1);
    if (reach > kMaxCode || w > 31) {
      if (w > 31 || block_out_of_range(mag, sign, outlier)) {
        err |= status_bit(ZC_ERR_RANGE);
        w = 0;
      }
    }
  }
  Placement pl;
  pl.w = w;
  pl.wmax = wave_max_u32(w);
  const u32 words = psize_words(w);
  const u32 incl = wave_inclusive_sum(words);
  pl.wave_total = lane_value(incl, 63);
  pl.half0_total = lane_value(incl, 31);
  pl.off_in_wave = incl - words;
  if (lane == 0) sh_wave_total[wave] = pl.wave_total | (ix && pl.wmax > 15 ? kWaveWideMark : 0u);
  if (active && a.out_cap >= tend) {
    a.out[widths_begin(h.nb, ix) + b] = u8(w);
    reinterpret_cast<i32*>(a.out + outliers_begin(h.nb, ix))[b] = i32(outlier);
  }
  lds_barrier();                // the wave totals; the stores above stay in flight
  sum_wave_totals(sh_wave_total, wave, ix, pl);
  if (threadIdx.x == 0) publish_tile_size(sink, tile, pl.tile_total, pl.tile_wide);
  if (err) raise_status(a.ctl, c.tag, err);
  finish_tile<NW, SEGS>(sink, word, pl, tile, ntiles, wl, sh_base, wave, lane);
}

// The same for a wave whose whole payload fits its staging area (kWholeStage words per wave):
// the plane words go to LDS in one pass before the wait for the tile's base offset, so the
// registers that hold them are free from then on, and the copy-out is a plain LDS-to-memory
// copy of the wave's words.
constexpr int kWholeStage = 64 * 24;

template <int NW, int NP, int SEGS, int LOOK, typename WordFn>
__device__ inline void place_sum_staged(const ReduceArgs& a, const ReduceCall& c, const PayloadSink& sink, const u32 (&mag)[NP], u32 sign, u32 w,
                                        i64 outlier, bool active, u32 b, u32 tile, u32 ntiles, WordFn word, u32* wl,
                                        u32 (&sh_wave_total)[SEGS], u64 (&sh_base)[LOOK], int wave, int lane) {
  const bool ix = sink.ix;
  static_assert(64 * NW <= kWholeStage, "a wave of widest blocks must fit the staging area");
  const ParsedHeader& h = c.h;
  const u64 tend = tables_end(h.nb, ix);
  if (!active) w = 0;
  u32 err = 0;
  if (active) {
    const i64 ao = outlier < 0 ? -outlier : outlier;
    const i64 reach = ao + 31 * ((i64(1) << w) - 1);
    if (reach > kMaxCode || w > 31) {
      if (w > 31 || block_out_of_range(mag, sign, outlier)) {
        err |= status_bit(ZC_ERR_RANGE);
        w = 0;
      }
    }
  }
  Placement pl;
  pl.w = w;
  pl.wmax = wave_max_u32(w);
  const u32 words = psize_words(w);
  const u32 incl = wave_inclusive_sum(words);
  pl.wave_total = lane_value(incl, 63);
  pl.half0_total = lane_value(incl, 31);
  pl.off_in_wave = incl - words;
  if (lane == 0) sh_wave_total[wave] = pl.wave_total | (ix && pl.wmax > 15 ? kWaveWideMark : 0u);
  // (width and outlier go to their tables at the very end: a store that is under way is waited for by
  // every poll of the look-back)
  stage_wave_words<NW>(word, pl, wl);
  lds_barrier();                // the wave totals (and the words above); the stores stay in flight
  sum_wave_totals(sh_wave_total, wave, ix, pl);
  if (threadIdx.x == 0) publish_tile_size(sink, tile, pl.tile_total, pl.tile_wide);
  if (err) raise_status(a.ctl, c.tag, err);
  const TileBase tb = resolve_tile_base(sink, pl, tile, sh_base, wave, lane);
  const u64 cap_words = a.out_cap > tend ? (a.out_cap - tend) / 4 : 0;
  const u64 d0 = tb.words + pl.wave_off;
  if (lane == 0) write_index_entry(sink, tile * u32(SEGS) + u32(wave), d0);
  u32* const dst = reinterpret_cast<u32*>(a.out + tend) + d0;
  const u64 room = cap_words > d0 ? cap_words - d0 : 0;
  const u32 limit = u64(pl.wave_total) < room ? pl.wave_total : u32(room);
  copy_staged_words<NW + 1, true>(wl, dst, limit, lane);
  wave_lds_sync();
  store_tables<kAccessOnce>(sink, b, w, i32(outlier));     // (the whole output stream is written with the non-temporal hint, see store_once)
  finish_stream<SEGS>(sink, pl, tile, ntiles, tb);
}

// ---------------------------------------------------------------------------------------
// The common path.
// ---------------------------------------------------------------------------------------

// The accumulator: 24 two's complement planes hold the sum of up to 64 deltas below 2^16 in
// magnitude.  Planes [0, top) are valid, top a multiple of 4 and wave-uniform; plane top - 1
// is a copy of the sign plane.
constexpr int kSumPlanes = 24;
static_assert(64 * kSumPlanes <= kWholeStage && kWholeStage >= kWaveStage, "staging area of reduce_kernel");   // (planes 0..22 and the sign: 24 words)
constexpr int kSumChunk = 4;

// What a wave needs to know about one operand's share.
struct OperandPlace {
  u32 w;            // this lane's block width (0 if the block must be skipped)
  u32 pick;         // LDS word index of this lane's sign word
  u32 wcap;         // uniform: 0 (nothing to add), 4, 8, 12, 16 or 24: at least the widest block of a wave on the common path
  u32 span;         // uniform: words the wave stages, from the aligned start
  u32 src0;         // uniform: payload word index of the aligned start
  u32 room;         // uniform: words from src0 to the end of the caller's buffer
};

// (A wave's loads of its share of an operand are buffer loads, see bytes_from.  With conditions and addresses per lane an
// operand took 420 instructions: Sum of 8 x 2^26 values 161.6 us, then 157.0; of 8 x 1024, when those still came here, 15.8, then 13.9.)
// The first code of the lane's block (b; 0 if there is no such block).
__device__ inline i32 load_operand_outlier(const u8* base, const ReduceCall& c, u32 b) {
  return i32(__builtin_amdgcn_raw_buffer_load_b32(bytes_from(base + c.firsts, 4u * c.nb), int(4u * b), 0, 0));
}

// The width of the lane's block (0 if there is no such block).
__device__ inline u32 load_operand_width(const u8* base, const ReduceCall& c, u32 b) {
  return u32(__builtin_amdgcn_raw_buffer_load_b8(bytes_from(base + c.widths, c.nb), int(b), 0, 0));
}

// Words between the start of the payload and the end of the caller's buffer, of a stream whose header is in order (saturated:
// a stream's payload has at most 2^31 words).  The payload is fenced in by that, which a validated stream does
// not exceed (a 16-byte load may run up to 12 bytes past the stream's own end, inside the
// buffer; nothing reads those words).
__device__ inline u32 payload_room(u64 bytes, const ReduceCall& c) {
  const u64 room = (bytes - c.payload) >> 2;
  return u32(room >> 32) ? 0xffffffffu : u32(room);
}

// Words of an operand's payload that load_operand_payload and stage_to_lds can bring in.
constexpr int kStageLoads = 4;
constexpr u32 kMostStaged = 256u * kStageLoads + 64u;

// Lane s: words of operand s from the 16-byte boundary at or below the wave's segment on: up to the end of the caller's buffer, and of an indexed stream (IX),
// which says so by itself, up to the segment's end, so that its payload can be asked for before its widths are there.
// (An index that says what cannot be, of at most `most` words and three, has nothing asked for, and kNoWords for the widths to contradict.)
constexpr u32 kNoWords = 0x3fffffffu;     // more than any widths add up to
struct LaneSegments {
  u32 room, span;
};
template <bool IX>
__device__ inline LaneSegments lane_segments(const ReduceCall& c, u32 most = kMostStaged) {
  const u32 mis = c.places & 3u, room = payload_room(c.bytes, c), words = c.ends - c.places;
  LaneSegments l;
  l.room = c.places <= room ? room - (c.places - mis) : 0u;         // (the start is inside on a validated stream)
  l.span = 0;
  if (IX) {
    const bool inside = mis <= l.room && words <= l.room - mis && words <= most - 3u;
    l.span = inside ? mis + words : kNoWords;
    if (!inside) l.room = 0;
  }
  return l;
}

// Where operand s has the wave's segment; of a plain stream only the start is known.  Everything here is the same in every lane.
// (Out of lanes, where the words of all operands have been worked out at once: with that done for each operand as it came, Sum of 64 x 2^20 values by ticket
// 77.4 us, now 69.4, of 16 x 2^20 in a workspace for more 24.0 and 22.1, of 8 x 2^26 149.6 and 146.9.)
__device__ inline OperandPlace open_operand(int s, const ReduceCall& c, const LaneSegments& l) {
  OperandPlace p;
  p.src0 = lane_value(c.places, s) & ~3u;
  p.room = lane_value(l.room, s);
  p.span = lane_value(l.span, s);
  p.w = p.pick = p.wcap = 0;
  return p;
}

// ... and once the lane's block width is there.
// `err`: an indexed stream is checked as it is used: the widths of the segment must add up to
// what the index says, and no block may be wider than w_max (15 where the stream promised narrow
// blocks, or where the caller has seen that there is no other).
__device__ inline void place_operand(OperandPlace& p, int s, u32 width, const ReduceCall& c, bool ix, u32& err, u32 w_max = 15) {
  const u32 words = psize_words(width);
  const u32 incl = wave_inclusive_sum(words);
  const u32 mis = lane_value(c.places, s) & 3u;
  const u32 span = mis + lane_value(incl, 63);           // (at most 3 + 64 x 256)
  // true on a validated stream (plain ones: cannot happen here; keeps every LDS access in range)
  const bool inside = !__any(width > w_max) && (ix ? span == p.span : span <= p.room);
  if (ix && !inside) err |= status_bit(ZC_ERR_FORMAT);
  p.span = inside ? span : 0u;                 // <= 3 + 64 * (1 + w_max)
  p.pick = mis + (incl - words);
  p.w = inside ? width : 0u;
  p.wcap = w_max > 15 && __any(p.w > 15) ? 24u : __any(p.w > 12) ? 16u : __any(p.w > 8) ? 12u : __any(p.w > 4) ? 8u : __any(p.w != 0) ? 4u : 0u;
}

// The operand's payload for this wave: 16 bytes per lane and load, all in flight together.
// The copy starts at the 16-byte boundary at or below the segment (the payload area itself is
// 16-byte aligned) and keeps that misalignment in LDS.  Four loads cover 1024 words; a wave
// whose 64 blocks are all 15 bits wide can need up to three more words, which stage_to_lds
// fetches on the spot.
struct OperandStage {
  uint4 v[kStageLoads];
};

__device__ inline OperandStage load_operand_payload(const u32* payload, const OperandPlace& p, int lane) {
  OperandStage st;
  // whole 16-byte pieces only: the last words of the caller's buffer are left to stage_to_lds (see load_wave_stage)
  const u32 whole = min((p.span + 3u) & ~3u, p.room & ~3u);
  const __amdgpu_buffer_rsrc_t share = bytes_from(reinterpret_cast<const u8*>(payload + p.src0), 4u * whole);
#pragma unroll
  for (int i = 0; i < kStageLoads; ++i) {
    const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(share, 16 * lane + 1024 * i, 0, kAccessOnce);
    st.v[i] = make_uint4(t.x, t.y, t.z, t.w);
  }
  return st;
}

__device__ inline void stage_to_lds(const OperandStage& st, const OperandPlace& p, const u32* payload, u32* wl, int lane) {
#pragma unroll
  for (int i = 0; i < kStageLoads; ++i) {
    if (256u * u32(i) < p.span) *reinterpret_cast<uint4*>(wl + 4u * u32(lane) + 256u * u32(i)) = st.v[i];      // uniform
  }
  if (p.span > 256u * kStageLoads || ((p.span + 3u) & ~3u) > p.room) {      // uniform, and rare: more than four loads, or the buffer ends inside a 16-byte piece
    asm volatile("");                            // (keeps the branch: merged with the condition below, all of this runs every time)
    const u32 whole = min(min((p.span + 3u) & ~3u, p.room & ~3u), 256u * kStageLoads);
    const u32 idx = whole + u32(lane);
    if (idx < min(p.span, p.room)) wl[idx] = payload[p.src0 + idx];
  }
}

// Three-input bitwise functions, one v_bitop3_b32 each.  The table is the function evaluated
// on a = 0xF0, b = 0xCC, c = 0xAA.
__device__ inline u32 xor3(u32 a, u32 b, u32 c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }
__device__ inline u32 majority(u32 a, u32 b, u32 c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8); }
__device__ inline u32 and_xor(u32 a, u32 b, u32 c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x6A); }   // (a & b) ^ c

// acc += operand, planes [4C, 4C + 4).  DATA: the operand has magnitude planes here, read
// from LDS (`mine` points at the lane's sign word) and masked by the block's own width (bit P
// of `keep` is set iff the block has plane P); otherwise the operand only contributes its
// sign extension.  Four instructions per plane: mask, operand bit, sum, carry.
template <int C, bool DATA>
__device__ inline void add_chunk(u32 (&acc)[kSumPlanes], const u32* mine, u32 keep, u32 sgn, u32& carry) {
#pragma unroll
  for (int i = 0; i < kSumChunk; ++i) {
    constexpr int kFirst = C * kSumChunk;
    const int P = kFirst + i;
    u32 x = sgn;                                  // two's complement of the operand: (mag ^ s) + s
    if (DATA) {
      const u32 m = u32(__builtin_amdgcn_sbfe(i32(keep), u32(P), 1u));   // all ones iff the block has plane P
      x = and_xor(mine[1 + P], m, sgn);
    }
    const u32 cur = acc[P];                       // full adder
    acc[P] = xor3(cur, x, carry);
    carry = majority(cur, x, carry);
  }
}

template <int C>
__device__ inline void add_operand_chunks(u32 (&acc)[kSumPlanes], const u32* mine, u32 keep, u32 sgn, u32& carry,
                                          u32 wcap, u32 top) {
  if constexpr (C * kSumChunk < kSumPlanes) {
    if (u32(C * kSumChunk) >= top) return;        // uniform
    if (u32(C * kSumChunk) < wcap) add_chunk<C, true>(acc, mine, keep, sgn, carry);
    else add_chunk<C, false>(acc, mine, keep, sgn, carry);
    add_operand_chunks<C + 1>(acc, mine, keep, sgn, carry, wcap, top);
  }
}

// Extends the valid planes from `top` to `new_top` with copies of the sign plane.
template <int C>
__device__ inline void grow_sum(u32 (&acc)[kSumPlanes], u32 top, u32 new_top) {
  if constexpr (C * kSumChunk < kSumPlanes) {
    if (u32(C * kSumChunk) >= new_top) return;    // uniform
    if (u32(C * kSumChunk) >= top) {
      u32 e = 0;
      if constexpr (C > 0) e = acc[C * kSumChunk - 1];
#pragma unroll
      for (int i = 0; i < kSumChunk; ++i) acc[C * kSumChunk + i] = e;
    }
    grow_sum<C + 1>(acc, top, new_top);
  }
}

// Planes that hold sums of a magnitude of at most `bound`, as many chunks as it takes.
__device__ inline u32 planes_for(u32 bound) {
  const u32 top = bound ? (32u - u32(__builtin_clz(bound)) + 1u + 3u) & ~3u : 0u;
  return top > u32(kSumPlanes) ? u32(kSumPlanes) : top;
}

// Two's complement planes -> magnitude planes (in place), given the sign plane; tracks the width.
template <int C>
__device__ inline void sum_to_magnitude(u32 (&acc)[kSumPlanes], u32 sgn, u32& carry, u32& width, u32 top) {
  if constexpr (C * kSumChunk < kSumPlanes) {
    if (u32(C * kSumChunk) >= top) {
#pragma unroll
      for (int i = 0; i < kSumChunk; ++i) acc[C * kSumChunk + i] = 0;
    } else {
#pragma unroll
      for (int i = 0; i < kSumChunk; ++i) {
        constexpr int kFirst = C * kSumChunk;
        const int P = kFirst + i;
        const u32 t = acc[P] ^ sgn;
        const u32 m = t ^ carry;
        carry = t & carry;
        acc[P] = m;
        width = m ? u32(P + 1) : width;
      }
    }
    sum_to_magnitude<C + 1>(acc, sgn, carry, width, top);
  }
}

template <int C>
__device__ inline u32 sign_plane(const u32 (&acc)[kSumPlanes], u32 top) {
  if constexpr ((C + 1) * kSumChunk > kSumPlanes) {
    return 0u;
  } else {
    if (top == u32((C + 1) * kSumChunk)) return acc[(C + 1) * kSumChunk - 1];
    return sign_plane<C + 1>(acc, top);
  }
}

// What a wave knows about its share of a tile.
struct ReduceShare {
  u32 seg;                  // the segment (a stream has at most 2^26 blocks, so byte offsets into tables fit 32 bits)
  int first = 0, count = 0; // Max and Min, whose waves may share a segment's operands (see reduce_op_kernel): the wave's first one, and how many
};

// The widest block that stream s may have: 31, but 15 if it promised narrow blocks.
__device__ inline u32 width_limit(const ReduceCall& c, int s) { return (c.wide_streams >> s) & 1u ? 31u : 15u; }

static_assert(kMostStaged + kSumPlanes <= u32(kWholeStage), "payload staging, and the reads behind its last word, must fit the wave's area");

// Whether the wave's blocks fit the common path: the sums its accumulator, every operand's payload the staging.
// Without blocks wider than 15 bits they always do, and usually with some (a segment that has one is mostly
// narrow blocks all the same: one or two spikes among 2048 values).  Only calls whose headers announce wide
// blocks ask; the operands' width bytes are asked for together, which costs one round trip.
__device__ inline bool fits_common_path(const ReduceArgs& a, const ReduceCall& c, u32 seg, bool ix) {
  const ParsedHeader& h = c.h;
  const u32 b = seg * kWaveBlocks + u32(fresh_lane());
  const u32 at = u32(widths_begin(h.nb, ix)) + b;
  bool unfit = false;
  u32 reach = 0, words = 0;                    // bound on the sum of the lane's block (saturates by 2^23 a term); its largest payload
  if (b < h.nb) {
#pragma unroll 8
    for (int s = 0; s < a.k; ++s) {
      const u32 w = u32(*at_bytes(a.in[s].base, at));
      unfit |= w > width_limit(c, s);          // (malformed: the other path says so)
      reach += (1u << (w < u32(kSumPlanes) ? w : u32(kSumPlanes))) - 1u;      // k <= 64 terms of at most 2^24
      words = max(words, psize_words(w));
    }
  }
  // (64 x the largest possible width byte fits 32 bits; the sum over the lanes of the largest is at least any operand's)
  return !__any(unfit || reach >= 1u << (kSumPlanes - 1)) && wave_sum_u32(words) + 3u <= kMostStaged;
}

// The sum of a wave's blocks as planes: acc = two's complement, `top` of them, outlier = sum of the first codes.
// `width0`: the widths of operand 0 if the workgroup asked for them early (`early`).
template <bool IX>
__device__ __forceinline__ void sum_operands(const ReduceArgs& a, const ReduceCall& c, const ReduceShare& share, u32 width0,
                                             bool early, u32* wl, u32 (&acc)[kSumPlanes], u32& top, i64& outlier, u32& err) {
  const u32 w_max = c.wide_streams ? 31u : 15u;
  const u32 seg = share.seg;
  const LaneSegments segments = lane_segments<IX>(c);
  // What travels together: an operand's payload and first codes, and of an indexed one, whose segment is found without them,
  // the widths; a plain one's widths a step ahead of the others.
  OperandPlace next;
  OperandStage stage;
  i32 outlier_next;
  u32 width_next = 0;
  // Where operands s, s + 1 and s + 2 are, asked for a step before it is needed (a scalar load on the spot is waited for,
  // with all LDS reads under way, three times an operand: Sum of 8 x 1024 values, when those still came here, 12.4 us, then 12.0).
  StreamRef at0 = a.in[0], at1 = a.in[min(1, a.k - 1)], at2 = a.in[min(2, a.k - 1)];
  {
    const int lane = fresh_lane();
    const u32 b = seg * kWaveBlocks + u32(lane);
    next = open_operand(0, c, segments);
    if (IX) {
      width_next = load_operand_width(at0.base, c, b);
    } else {
      u32 width = early ? width0 : load_operand_width(at0.base, c, b);
      if (b >= c.nb) width = 0;
      place_operand(next, 0, width, c, IX, err, w_max);
      if (a.k > 1) width_next = load_operand_width(at1.base, c, b);
    }
    stage = load_operand_payload(reinterpret_cast<const u32*>(at0.base + c.payload), next, lane);
    outlier_next = load_operand_outlier(at0.base, c, b);
  }
  // the ends of every operand's index, by the waves that hold them
  if (c.ends_bad) err |= status_bit(ZC_ERR_FORMAT);

  // ---- add the k operands' blocks in plane form; loads run ahead of the adds ----
#pragma unroll
  for (int p = 0; p < kSumPlanes; ++p) acc[p] = 0;
  top = 0;
  u32 bound = 0;          // wave-uniform bound on |sum of deltas| so far (the true sums are below 2^23: see fits_common_path)
  outlier = 0;
  for (int s = 0; s < a.k; ++s) {
    const int lane = fresh_lane();
    const u32 b = seg * kWaveBlocks + u32(lane);
    OperandPlace cur = next;
    const u32 width = width_next;
    const StreamRef here = at0, ahead1 = at1, ahead2 = at2;
    at0 = at1;
    at1 = at2;
    at2 = a.in[min(s + 3, a.k - 1)];
    stage_to_lds(stage, cur, reinterpret_cast<const u32*>(here.base + c.payload), wl, lane);
    wave_lds_sync();
    outlier += i64(outlier_next);
    if (IX) place_operand(cur, s, width, c, IX, err, w_max);
    if (s + 1 < a.k) {
      next = open_operand(s + 1, c, segments);
      if (IX) {
        width_next = load_operand_width(ahead1.base, c, b);
      } else {
        place_operand(next, s + 1, width, c, IX, err, w_max);
        if (s + 2 < a.k) width_next = load_operand_width(ahead2.base, c, b);
      }
      stage = load_operand_payload(reinterpret_cast<const u32*>(ahead1.base + c.payload), next, lane);
      outlier_next = load_operand_outlier(ahead1.base, c, b);
    }
    if (cur.wcap) {
      bound += (1u << cur.wcap) - 1u;
      const u32 new_top = planes_for(bound);
      grow_sum<0>(acc, top, new_top);
      top = new_top;
      const u32* mine = wl + cur.pick;
      const u32 sgn = cur.w ? mine[0] : 0u;
      u32 carry = sgn;
      const u32 keep = (1u << cur.w) - 1u;      // bit P set iff the block has plane P
      add_operand_chunks<0>(acc, mine, keep, sgn, carry, cur.wcap, top);
    }
    wave_lds_sync();
  }
}

// Back to sign + magnitude planes; new code length.
__device__ __forceinline__ void close_sum(u32 (&acc)[kSumPlanes], u32 top, u32& sgn, u32& w) {
  sgn = sign_plane<0>(acc, top);
  u32 carry = sgn;
  w = 0;
  sum_to_magnitude<0>(acc, sgn, carry, w, top);
}

// ---------------------------------------------------------------------------------------
// Any widths.
// ---------------------------------------------------------------------------------------
constexpr int kAccPlanes = 38;   // |sum of 64 deltas| < 2^37: 37 magnitude bits + sign
constexpr int kWideChunk = 2;    // operand planes fetched at a time

// acc (two's complement, `top` planes valid, `ext` = its sign plane) += operand given as sign
// word s and the magnitude planes at src[1 ...] (w of them; zero above), kWideChunk planes at
// a time: their loads are in flight together, then they are added.  Planes [0, new_top) are
// valid afterwards.  top and new_top are wave-uniform.
template <int P0>
__device__ inline void ripple_add(u32 (&acc)[kAccPlanes], const u32* src, u32 w, u32 s, u32 carry, u32 ext, u32 top,
                                  u32 new_top, u32& ext_out) {
  if constexpr (P0 < kAccPlanes) {
    if (u32(P0) >= new_top) return;             // uniform
    u32 x[kWideChunk];
#pragma unroll
    for (int i = 0; i < kWideChunk; ++i) {
      const int P = P0 + i;
      x[i] = (P < 31 && u32(P) < w) ? src[1 + P] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kWideChunk; ++i) {
      const int P = P0 + i;
      if (P < kAccPlanes && u32(P) < new_top) {
        const u32 cur = u32(P) < top ? acc[P] : ext;
        const u32 xx = s ^ x[i];                // two's complement of the operand: (mag ^ s) + s
        const u32 t = cur ^ xx;
        const u32 sum = t ^ carry;
        carry = (t & carry) | (~t & cur);       // majority(cur, xx, carry)
        acc[P] = sum;
        ext_out = sum;
      }
    }
    ripple_add<P0 + kWideChunk>(acc, src, w, s, carry, ext, top, new_top, ext_out);
  }
}

// Two's complement planes -> magnitude planes; returns the code length.
template <int P>
__device__ inline void magnitude_planes(u32 (&acc)[kAccPlanes], u32 s, u32 carry, u32 top, u32& width) {
  if constexpr (P < kAccPlanes) {
    if (u32(P) >= top) return;
    const u32 t = acc[P] ^ s;
    const u32 m = t ^ carry;
    acc[P] = m;
    if (m) width = P + 1;
    magnitude_planes<P + 1>(acc, s, t & carry, top, width);
  }
}

// One wave per segment of the tile; wl: its LDS.
template <bool IX, int SEGS, int LOOK>
__device__ inline void reduce_wide_tile(const ReduceArgs& a, const ReduceCall& c, const PayloadSink& sink, u32 tile, u32 ntiles, u32* wl,
                                        u32 (&sh_wave_total)[SEGS], u64 (&sh_base)[LOOK]) {
  const ParsedHeader& h = c.h;
  const u64 tend = tables_end(h.nb, IX);
  const int lane = fresh_lane();
  const int wave = wave_id();
  const u32 seg = tile * u32(SEGS) + u32(wave);            // a stream has at most 2^26 blocks
  const bool seg_live = seg < num_segments(h.nb);
  const u32 b = seg * kWaveBlocks + u32(lane);
  const bool active = b < h.nb;
  if (c.ends_bad && lane == 0) raise_status(a.ctl, c.tag, status_bit(ZC_ERR_FORMAT));

  u32 acc[kAccPlanes];
#pragma unroll
  for (int p = 0; p < kAccPlanes; ++p) acc[p] = 0;
  u32 ext = 0, top = 0;
  u64 bound = 0;          // wave-uniform bound on |sum of deltas| so far
  i64 outlier = 0;
#pragma nounroll
  for (int s = 0; s < a.k; ++s) {
    const u8* base = a.in[s].base;
    const u64 total_s = reinterpret_cast<const u64*>(base)[3];
    const u64 pw64 = total_s >= tend ? (total_s - tend) / 4 : 0;
    const u32 pw = pw64 > 0xffffffffull ? 0xffffffffu : u32(pw64);   // payload words (a stream has at most 2^31)
    u32 w = active ? u32(*at_bytes(base, u32(widths_begin(h.nb, IX)) + b)) : 0u;
    const bool bad_w = w > 31;                    // plain streams: cannot happen on a validated stream
    if (bad_w) w = 0;
    const u32 words = psize_words(w);
    const u32 incl = wave_inclusive_sum(words);
    const u32 seg_off = lane_value(c.places, s);
    bool fits = seg_live;
    if (IX) {                                     // the stream's own index must agree with the widths
      const bool narrow_promised = (reinterpret_cast<const u32*>(base)[1] & 1u) == 0;
      if (lane_value(c.ends, s) - seg_off != lane_value(incl, 63) || __any(bad_w) || (narrow_promised && __any(w > 15))) {
        if (lane == 0) raise_status(a.ctl, c.tag, status_bit(ZC_ERR_FORMAT));
        fits = false;
      }
    }
    // (cannot fail on a validated stream) the segment lies inside the payload
    if (!fits || seg_off > pw || lane_value(incl, 63) > pw - seg_off) w = 0;
    const u32 wmax = wave_max_u32(w);
    if (active) outlier += i64(*reinterpret_cast<const i32*>(at_bytes(base, u32(outliers_begin(h.nb, IX)) + 4u * b)));
    if (wmax == 0) continue;
    const u32* src = reinterpret_cast<const u32*>(base + tend) + seg_off + (incl - words);
    const u32 sgn = w ? src[0] : 0u;
    bound += (u64(1) << wmax) - 1;
    u32 new_top = 64u - u32(__builtin_clzll(bound)) + 1u;
    if (new_top > u32(kAccPlanes)) new_top = kAccPlanes;
    u32 ext_out = ext;
    ripple_add<0>(acc, src, w, sgn, sgn, ext, top, new_top, ext_out);
    ext = ext_out;
    top = new_top;
  }

  u32 w = 0;
  magnitude_planes<0>(acc, ext, ext, top, w);
  auto word = [&](auto i) {
    constexpr int I = decltype(i)::value;        // 0: sign, 1 + p: plane p
    if constexpr (I == 0) return ext;
    else return acc[I - 1];
  };
  place_sum<32>(a, c, sink, acc, ext, w, outlier, active, b, tile, ntiles, word, wl, sh_wave_total, sh_base, wave, lane);
}

// One tile on the common path.
template <bool IX, int WAVES>
__device__ inline void reduce_common_tile(const ReduceArgs& a, const ReduceCall& c, u32 tile, u32 ntiles, u32 width0, bool early, u32* lds,
                                          u32 (&sh_wave_total)[WAVES], u64 (&sh_base)[WAVES]) {
  const int wave = wave_id();
  u32* const wl = lds + wave * kWholeStage;
  const u32 seg = tile * u32(WAVES) + u32(wave);
  const ReduceShare share{seg};
  u32 acc[kSumPlanes], top, sgn, w, err = 0;
  i64 outlier;
  sum_operands<IX>(a, c, share, width0, early, wl, acc, top, outlier, err);
  close_sum(acc, top, sgn, w);
  auto word = [&](auto i) {
    constexpr int I = decltype(i)::value;        // 0: sign, 1 + p: plane p
    if constexpr (I == 0) return sgn;
    else return acc[I - 1];
  };
  const int lane = fresh_lane();
  const u32 b = seg * kWaveBlocks + u32(lane);
  if (IX && err && lane == 0) raise_status(a.ctl, c.tag, err);
  place_sum_staged<kSumPlanes>(a, c, sum_sink(a, c, ntiles, IX), acc, sgn, w, outlier, b < c.h.nb, b, tile, ntiles, word, wl, sh_wave_total, sh_base, wave,
                               lane);
}

// What every workgroup of a reduce kernel does first: the call's verdict, tag and header, and its tile.
// Returns false when the workgroup has nothing (more) to do.  The headers, and the width tables of plain streams, are
// judged here, by every workgroup alike.
// The segments' places in all operands are found here too.  `width0`, `early`: see sum_operands.
// SEGS: segments of a tile, wave i of the workgroup on segment i % SEGS of its tile; TICKETS: tiles may be handed out by tickets.
template <bool IX, int SEGS = kTileWaves, bool TICKETS = true>
__device__ inline bool open_reduce(const ReduceArgs& a, ReduceCall& c, u32& width0, bool early, u32& tile, u32& ntiles,
                                   u32* sh_tile, PlainSurvey<IX ? 1 : ZC_MAX_K>* survey) {
  const StreamRef any = lane_stream(a.in);   // (before the other arguments are there)
  __builtin_amdgcn_sched_barrier(0);
  // (with tickets the ticket is asked for first of all: its round trip runs beside the headers')
  u64 asked = 0;
  if (TICKETS && a.ticketed && threadIdx.x == 0) asked = ask_ticket(ticket_counter(a.ctl, ticket_shard()));
  const int wave = wave_id();
  tile = a.first_tile + blockIdx.x;          // tiles in the order in which workgroups start
  u32 seg = tile * u32(SEGS) + u32(wave % SEGS);     // < 2^22: the host launches at most 2^18 tiles of four
  SurveyLoads ask{};
  if (!IX) ask = ask_plain_streams<ZC_MAX_K, true>(a.in, a.k, a.index, a.self != 0, seg, wave);
  if (early) {
    const u32 b = seg * kWaveBlocks + u32(fresh_lane());
    const StreamRef first = a.in[0];
    width0 = u64(kHeaderBytes) + b < first.bytes ? u32(*at_bytes(first.base, kHeaderBytes + b)) : 0u;
  }
  LaneStream in = ask_headers<IX>(any, a.k, seg);
  // (the tag, some 100 dependent scalar instructions, while the loads are on their way)
  c.ltag = launch_tag(a.nonce, a.ctl);
  asm volatile("" : "+s"(c.ltag));
  StreamsVerdict v = judge_headers<IX>(in, a.k, true);
  // (a later part of a reduce done in parts belongs to the call its first part opened)
  c.tag = call_tag(a.ctl, c.ltag, a.adopt != 0);
  c.places = 0;
  if (!IX) c.places = judge_plain_streams<IX ? 1 : ZC_MAX_K, true>(a.in, a.k, a.index, a.self != 0, seg / kTileWaves, wave, ask, v, *survey, int(seg % kTileWaves));
  c.base = in.base;
  c.bytes = in.bytes;
  c.h = v.h0;
  c.nb = u32(c.h.nb);
  c.widths = u32(widths_begin(c.h.nb, IX));
  c.firsts = u32(outliers_begin(c.h.nb, IX));
  c.payload = u32(tables_end(c.h.nb, IX));
  c.nsum = v.nsum;
  c.wide_streams = v.wide;
  if (v.err) {
    // (a workspace too small for some stream is told ahead of what else is wrong, as judge_plain_streams does)
    if (IX && !a.n_least && __any(v.mine.ok && v.mine.n > a.n_most)) v.err |= status_bit(ZC_ERR_ARG);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      if (!a.adopt) a.ctl->result = 0;
      raise_status(a.ctl, c.tag, v.err);
    }
    return false;
  }
  if (c.h.n < a.n_least || c.h.n > a.n_most) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      if (!a.adopt) a.ctl->result = 0;
      raise_status(a.ctl, c.tag, status_bit(a.n_least ? ZC_ERR_MISMATCH : ZC_ERR_ARG));
    }
    return false;
  }
  ntiles = (u32(num_segments(c.h.nb)) + u32(SEGS) - 1) / u32(SEGS);
  const u32 end_tile = a.end_tile && a.end_tile < ntiles ? a.end_tile : ntiles;
  c.part_end = a.end_tile ? end_tile : 0u;
  if (blockIdx.x == 0 && threadIdx.x == 0 && a.first_tile == 0) write_reduce_header(a, c, ntiles, IX);
  if (ntiles == 0) {                         // streams without blocks: their one index entry must say so
    if (IX && blockIdx.x == 0 && wave == 0 && !index_ends_consistent(a.in, a.k, c.h, 0) && lane_id() == 0)
      raise_status(a.ctl, c.tag, status_bit(ZC_ERR_FORMAT));
    return false;
  }
  if (a.first_tile >= end_tile) return false;
  if (TICKETS && a.ticketed) {                          // ... or handed out by tickets, see take_tile
    if (threadIdx.x == 0) {
      const u32 t = take_tile(a.ctl, c.ltag, end_tile - a.first_tile, ticket_shard(), asked);
      *sh_tile = t == kNoTile ? kNoTile : a.first_tile + t;
    }
    __syncthreads();
    tile = uniform(*sh_tile);
    seg = tile * u32(SEGS) + u32(wave % SEGS);
    if (!IX && tile < end_tile) {            // (the verdict stands: once more, for the place of this tile)
      ask = ask_plain_streams<ZC_MAX_K, true>(a.in, a.k, a.index, a.self != 0, seg, wave);
      c.places = judge_plain_streams<IX ? 1 : ZC_MAX_K, true>(a.in, a.k, a.index, a.self != 0, seg / kTileWaves, wave, ask, v, *survey, int(seg % kTileWaves));
    }
    if (IX) in = ask_headers<IX>(any, a.k, tile < end_tile ? seg : 0u);
  }
  const u32 nseg = u32(num_segments(c.h.nb));
  const bool live = seg < nseg;
  if (IX) {
    const int lane = lane_id();
    c.places = live ? in.begin : 0u;
    c.ends = live ? in.end : 0u;
    // the ends of every operand's index, by the waves that hold them (see index_ends_ok)
    c.ends_bad = __any(lane < a.k && ((seg == 0 && c.places != 0) || (seg + 1 == nseg && u64(c.payload) + 4 * u64(c.ends) != v.mine.total)));
  } else {
    if (!live) c.places = 0;
    c.ends = 0;
    c.ends_bad = false;
  }
  return tile < end_tile;
}

// One launch per call, whatever the widths (many plain streams: behind the one of zc_scan.h; plain ones with a workgroup less
// per compute unit, so that reduce_wide_tile, which has its segments' places to add up there, spills less: nothing
// but wide blocks, 4 x 4 194 301 values, 47 us with six and 41 with five; narrow ones, 8 x 2^24, 61.4 and 61.7.
// The kernel of its own that plain streams with wide blocks had before was a launch of 3 us on every call.)
// 80 registers and 32 bytes of scratch (plain streams: 96 and 44), which the common path's operand loop does not touch.
// WAVES: segments of a tile, a wave each: see zc_large_tiles.h.
template <bool IX, int WAVES = kTileWaves, typename... A>
__global__ __launch_bounds__(64 * WAVES, IX ? 6 : 5) void reduce_kernel(ReduceArgs a, A... answer) {
  __shared__ __attribute__((aligned(16))) u32 lds[WAVES * kWholeStage + kCopyOver];   // also holds an operand's payload
  __shared__ u32 sh_tile;
  __shared__ u32 sh_wave_total[WAVES];
  __shared__ u64 sh_base[WAVES];
  __shared__ PlainSurvey<IX ? 1 : ZC_MAX_K> survey;
  const AnswerAtEnd<ReduceArgs, A...> at_end(a, answer...);

  ReduceCall c;
  u32 width0 = 0;
  // A workgroup that takes the tile of its own number asks for the first operand's widths
  // together with the headers, before it knows them: one memory
  // round trip instead of two.  The loads are fenced in by sizes the host passed.  (Not for
  // indexed streams: where their width bytes are is only known with the header.  But where their segments are is, see
  // ask_headers, and with that the widths and the payload are asked for together.)
  const bool early = !a.ticketed && !IX;
  u32 tile = 0, ntiles = 0;
  if (!open_reduce<IX, WAVES>(a, c, width0, early, tile, ntiles, &sh_tile, &survey)) return;
  // The segment number stays a scalar: in a vector register, with all the addresses that follow from it, it made the
  // kernel spill in the operand loops.  (8 x 2^24 smooth values of plain streams 53.6 us, then 52.9; of nothing but wide blocks, 4 x 4 194 301, which go
  // to zc_reduce_few.h now, 43.7 and 41.0.)
  tile = uniform(tile);
  // A tile leaves the common path only if one of its waves has to.  (A call with a block wider than 15 bits in
  // some operand used to send every tile through reduce_wide_tile: 8 x 2^24 values of hard data 84 us, now 50;
  // 4 x 4 194 301, two tiles per compute unit, 24.2 -> 18.1.  Calls without wide blocks, 8 x 2^26: 159.5 and
  // 158.8; with the mixed case as a function of its own, or as a second instance of the common path, they lost 2 and
  // 4 % to another register allocation.)
  bool common = true;
  if (c.wide_streams) {                // (the same in every wave)
    const bool fits = fits_common_path(a, c, tile * u32(WAVES) + u32(wave_id()), IX);
    if (lane_id() == 0) sh_wave_total[wave_id()] = fits;
    lds_barrier();
    u32 all = 1;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) all &= sh_wave_total[i];
    common = uniform(all) != 0;
    lds_barrier();                     // the words are used again
  }
  if (common) reduce_common_tile<IX, WAVES>(a, c, tile, ntiles, width0, early, lds, sh_wave_total, sh_base);
  else reduce_wide_tile<IX>(a, c, sum_sink(a, c, ntiles, IX), tile, ntiles, lds + wave_id() * kWholeStage, sh_wave_total, sh_base);
}

}  // namespace zc
