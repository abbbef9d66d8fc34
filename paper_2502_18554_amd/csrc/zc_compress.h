// fZ-light compression kernel (Section 3.3): quantise, per-block Lorenzo delta, code length,
// sign + plane packing, single-pass placement of the variable-size blocks.
//
// Work split.  A tile is 512 blocks (16384 values, 64 KiB of input) handled by a workgroup of
// 8 waves (256 and 4 where that shortens the call, see packs_small_tiles).  Each wave loads 2048 consecutive values with 16-byte loads,
// quantises them where they land, and transposes the integer codes through LDS so that one
// lane owns one block.  Deltas (kept as 16 words of paired 16-bit fields), width and the
// bit-matrix transpose that yields the plane words are then in-lane; the packed words wait
// in registers for the tile's base offset from the look-back scan and leave through LDS as
// coalesced stores.
#pragma once

#include "zc_bitmatrix.h"
#include "zc_common.h"
#include "zc_place.h"
#include "zc_report.h"

namespace zc {

// A scan tile of the compression kernel: the blocks of one workgroup, one descriptor of the
// look-back scan.  Every tile pays the latency of that scan once, so compression uses tiles
// twice the size of the other kernels' tiles (512 blocks, 64 KiB of input); 1024 blocks
// measured slower, because a compute unit then holds a single workgroup.
constexpr int kPackWaves = 8;
constexpr int kPackThreads = kPackWaves * 64;
constexpr int kPackBlocks = kPackWaves * kWaveBlocks;
constexpr int kPackValues = kPackBlocks * kBlockValues;
__host__ __device__ inline u64 num_pack_tiles(u64 nb) { return (nb + kPackBlocks - 1) / kPackBlocks; }

struct CompressArgs {
  const float* in;
  u64 n, nb;
  double inv;        // 1 / step, divided on the host
  double step;       // abs_eb * 63 / 32
  double eb;         // abs_eb as binary64
  float screen;      // 2^17 * abs_eb: |x| at or below it needs no per-value checks
  u32 eb_bits;
  u8* out;           // stream base
  u64 out_cap;       // bytes
  Control* ctl;
  u64* desc;
  u32 ticketed;      // tiles handed out by tickets instead of by workgroup id
  u32 coherent;      // the look-back reads the tile's own chain with device-coherent loads too
  u32 ix;            // write an indexed stream (see index_bytes)
  u32 part_end;      // zc_compress_part: one past the last tile of this call; else 0
  u32 adopt;         // this launch continues a call (a later part): its tag is in the control block
  u64 nonce;         // drawn by the host per call, goes into the tag (see launch_tag)
  Answer answer;
};

// What a workgroup's first loads need comes ahead of the other arguments, one by one: such arguments are in scalar registers when a wave starts (the compiler is told so,
// see build.py), and others are asked for and waited for.  (The compression of 2^22 values of a field 7.41 us, then 6.94; 2^24: 19.2 18.7; 512^3: 116.9 116.0; the
// decompression of 2^23 8.0, then 7.9.  Not for the ring round, which needs nine registers for them: 2^22 values 9.26 and 9.09, but 2^24 25.1 and 26.0.)
struct CompressInput {
  const float* in;
  u64 n;
};
constexpr int kCompressArgsAt = 24;          // bytes of arguments in front of CompressArgs (checked behind the kernel)

// Round-to-nearest-even of r for |r| < 2^31 as the low word of r + 1.5 * 2^52.
__device__ inline i32 rint_small(double r) {
  double t = __dadd_rn(r, 6755399441055744.0);
  return i32(__double2loint(t));
}

// The largest magnitude of three (the first is not negative), NaN if there is one.  (One instruction, which takes magnitudes
// by itself; integer maxima of the bit patterns need a signed and an unsigned one.)
__device__ inline float most_of(float so_far, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(so_far, __builtin_fabsf(b)), __builtin_fabsf(c));
}

// Codes of one value that failed the cheap screen: the defining arithmetic, with its checks.
__device__ inline i32 quantize_checked(float x, const CompressArgs& a, u32& err) {
  if (!(__builtin_fabsf(x) <= 3.4028234663852886e38f)) {   // NaN or Inf
    err |= status_bit(ZC_ERR_NONFINITE);
    return 0;
  }
  double t = __builtin_rint(__dmul_rn(double(x), a.inv));
  if (__builtin_fabs(t) > double(kMaxCode)) {
    err |= status_bit(ZC_ERR_RANGE);
    return 0;
  }
  i32 q = i32(t);
  float xr = float(__dmul_rn(double(q), a.step));
  if (!(__builtin_fabs(double(x) - double(xr)) <= a.eb)) err |= status_bit(ZC_ERR_BOUND);
  return q;
}

// Inside |x| <= 2^17 eb the code is below 2^17 and the bound cannot fail (the guard of 1/64
// of eb exceeds the binary32 rounding of the reconstruction there), so the checks are skipped.
__device__ inline bool needs_checks(float x, const CompressArgs& a) { return !(__builtin_fabsf(x) <= a.screen); }

__device__ inline i32 quantize_fast(float x, const CompressArgs& a) {
  return rint_small(__dmul_rn(double(x), a.inv));
}

__device__ inline i32 quantize_value(float x, const CompressArgs& a, u32& err) {
  if (__builtin_expect(needs_checks(x, a), 0)) return quantize_checked(x, a, err);
  return quantize_fast(x, a);
}

// FRESH: checked values are taken in a way that the compiler does not recognise.  Or the 32 compares of a wave's checked
// values are made ahead of the branch, for every wave, and their results, 64 scalar registers, push others out into
// vector registers.
template <bool FRESH>
__device__ inline int4 quantize4(const float4& x, const CompressArgs& a, bool checked, u32& err) {
  int4 q;
  if (__builtin_expect(checked, 0)) {
    float4 y = x;
    if (FRESH) asm volatile("" : "+v"(y.x), "+v"(y.y), "+v"(y.z), "+v"(y.w));
    q.x = quantize_value(y.x, a, err);
    q.y = quantize_value(y.y, a, err);
    q.z = quantize_value(y.z, a, err);
    q.w = quantize_value(y.w, a, err);
  } else {
    q.x = quantize_fast(x.x, a);
    q.y = quantize_fast(x.y, a);
    q.z = quantize_fast(x.z, a);
    q.w = quantize_fast(x.w, a);
  }
  return q;
}

// Values of a wave's share of a tile (from value v0 on) that exist: 2048 but for the wave at the end of the
// input and those behind it.
constexpr u32 kWaveValues = u32(kWaveBlocks) * kBlockValues;
__device__ inline u32 share_values(u64 n, u64 v0) {
  const u64 left = n > v0 ? n - v0 : 0;
  return left < kWaveValues ? u32(left) : kWaveValues;
}

// Raw input of one wave's share of a tile: 8 x 16 bytes per lane, every load in flight at once.  They are
// buffer loads whose range is the share's whole 16-byte pieces, so the ragged end of an input needs no branch
// and no launch of its own: what lies beyond reads as zero without an access.  (The one to three values of an
// incomplete last piece: see block_codes.)  The range check covers the vector offset and the instruction's own; a
// scalar offset is not part of it, so there is none: the second four loads have a vector offset of their own.
__device__ inline void load_raw(const float* in, u64 wblock0, int lane, u32 have, float4 (&x)[8]) {
  const __amdgpu_buffer_rsrc_t share =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(in + wblock0 * kBlockValues), 0, int(4u * (have & ~3u)), kRawBuffer);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(share, 16 * lane + 1024 * i, 0, kAccessOnce);
    x[i] = make_float4(__uint_as_float(t.x), __uint_as_float(t.y), __uint_as_float(t.z), __uint_as_float(t.w));
  }
  // Nothing moves across this line: left to itself the compiler puts the first use of the first value,
  // and the wait for it, in front of the last four loads, which then go out a round trip late.
  __builtin_amdgcn_sched_barrier(0);
}

// Quantise the wave's values where they landed and transpose the codes through LDS so that one
// lane owns one block: q[j] = code j of the lane's block.  have: see share_values.
// (quantize4 for fresh values in both halves with tiles by ticket, in the second half without: 38 and 54 scalar registers
// pushed out.  In both halves without tickets it needs fewer, but then has 20 bytes of scratch set aside, which
// zc_compress_noalloc is not to need; in none it needs twice as many.  2^26 values by ticket 80.7 us with none, 80.0 with one,
// 78.1 with both; without tickets 66.8, 65.6, 65.2.)
template <bool TICKETS>
__device__ __forceinline__ void block_codes(const CompressArgs& a, const float4 (&x)[8], u64 wblock0, u32 have, int lane, u32* wl,
                                   i32 (&q)[32], u32& err) {
  // Some value of this wave outside the screened domain: the checked arithmetic for all of it.
  // (By maxima 16 instructions; by comparisons 64, and their results take scalar registers: 512^3 values 118.0 us, then 116.9.)
  float most = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) most = most_of(most_of(most, x[i].x, x[i].y), x[i].z, x[i].w);
  const bool outside = needs_checks(most, a);
  const bool checked = __any(outside);

  // Loads 0..3 hold blocks 0..31, loads 4..7 blocks 32..63.  Either half goes through LDS as 32 rows
  // of 32 codes, and every lane takes half a row: lane l and lane l + 32 the first and the second 16
  // codes of block l (then of block 32 + l).  That keeps 16 registers per half and lane instead of 32 in
  // half the lanes; one swap of the upper 32 lanes of a register with the lower 32 of another per pair
  // of codes then gives every lane the 32 codes of its own block.
  i32 h0[16], h1[16];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int4* const at = reinterpret_cast<int4*>(wl + (8 * i + (lane >> 3)) * kStageRow + 4 * (lane & 7));
      *at = half || TICKETS ? quantize4<true>(x[4 * half + i], a, checked, err) : quantize4<false>(x[4 * half + i], a, checked, err);
    }
    wave_lds_sync();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int4 r = *reinterpret_cast<const int4*>(wl + (lane & 31) * kStageRow + 16 * (lane >> 5) + 4 * t);
      i32* const h = half ? h1 : h0;
      h[4 * t + 0] = r.x; h[4 * t + 1] = r.y; h[4 * t + 2] = r.z; h[4 * t + 3] = r.w;
    }
    wave_lds_sync();
  }
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    // -> {lanes 0..31 of h0 | lanes 0..31 of h1}, {lanes 32..63 of h0 | lanes 32..63 of h1}
    const auto r = __builtin_amdgcn_permlane32_swap(u32(h0[j]), u32(h1[j]), false, false);
    q[j] = i32(r[0]);
    q[16 + j] = i32(r[1]);
  }
  if (have < kWaveValues) {
    // uniform: the end of the input.  The values behind the last whole 16-byte piece first ...
    const u32 whole = have & ~3u;
    const float* const tail = a.in + wblock0 * kBlockValues + whole;
#pragma nounroll
    for (u32 t = 0; t < have - whole; ++t) {
      const i32 code = quantize_value(tail[t], a, err);
      const u32 at = whole + t;
#pragma unroll
      for (int j = 0; j < 32; ++j) q[j] = at == u32(kBlockValues) * u32(lane) + u32(j) ? code : q[j];
    }
    // ... then the last block repeats its last code up to 32 values
    const u32 first = u32(kBlockValues) * u32(lane);
    const u32 cnt = have > first ? have - first : 0u;
#pragma unroll
    for (int j = 1; j < 32; ++j) q[j] = u32(j) < cnt ? q[j] : q[j - 1];
  }
}

// The block as the kernel keeps it: the Lorenzo deltas (d0 = 0) as two's complement fields of
// 16 bits, two per word (exact for widths up to 15), their largest magnitude, which gives the
// width, and the first code (the outlier).
struct BlockFields {
  u32 f[16];
  u32 any;
  i32 outlier;
};

template <bool TICKETS>
__device__ inline void block_fields(const CompressArgs& a, const float4 (&x)[8], u64 wblock0, u32 have, int lane, u32* wl,
                                    BlockFields& bf, u32& err) {
  i32 q[32];
  block_codes<TICKETS>(a, x, wblock0, have, lane, wl, q, err);
  bf.outlier = q[0];
  i32 top = 0, bottom = 0;              // largest and smallest delta (d0 = 0 is one of them)
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const i32 lo = j ? q[j] - q[j - 1] : 0;
    const i32 hi = q[j + 16] - q[j + 15];
    top = max(top, max(lo, hi));
    bottom = min(bottom, min(lo, hi));
    bf.f[j] = field16_pair(lo, hi);
    // (pins the field here: left to itself the compiler keeps all 32 deltas alive instead and
    //  builds the fields where they are used, after the barrier)
    asm volatile("" : "+v"(bf.f[j]));
  }
  const u32 any = max(u32(top), u32(-bottom));   // largest magnitude: its bit length is the width
  bf.any = any;
}

// Sign and plane words of two blocks (a and b, which may be the same), one per half of the wave, as ballots of their deltas: lane j of a half holds delta j.  w, at:
// widths of the blocks, and where their words go, `to` + at, which has room for `room` words.
__device__ __forceinline__ void store_block_ballots(i32 nd, u32 w_a, u32 w_b, u32 at_a, u32 at_b, u32* to, u64 room, u32 lane) {
  const u32 half = lane >> 5, j = lane & 31u;
  const u32 nmag = u32(nd < 0 ? -nd : nd);
  const u32 w = half ? w_b : w_a, dst = half ? at_b : at_a;
  const u64 sign = __ballot(nd < 0);
  if (j == 0 && w && dst < room) to[dst] = half ? u32(sign >> 32) : u32(sign);
  const u32 top = w_a > w_b ? w_a : w_b;
#pragma nounroll
  for (u32 p = 0; p < top; ++p) {
    const u64 plane = __ballot(((nmag >> p) & 1u) != 0);
    if (j == 0 && p < w && dst + 1 + p < room) to[dst + 1 + p] = half ? u32(plane >> 32) : u32(plane);
  }
}

// The value of `v` in lane `src` (any lane, chosen per lane).
__device__ inline u32 from_lane(u32 v, u32 src) { return u32(__builtin_amdgcn_ds_bpermute(int((src & 63u) << 2), int(v))); }

// Blocks wider than 15 bits of a wave up to which they are staged one by one (see stage_wide_blocks): two of them a step, and every step waits for its values, where a wave
// that goes over all its values again (store_wide_wave) loads them once.  A tile of four waves has its look-back to fill with that, one step; where eight waves share a SIMD
// and the values are in flight for other waves, three steps still pay.  us, every wave with so many blocks of 16 bits among narrow ones: all staged | none | by this rule
//            1                   2                   3                   4                   6                   8                    32
//   2^20     6.9   7.9   7.0     6.9   8.1   7.0     8.4   8.1   7.9     8.4   8.1   7.9     9.8   8.1   7.9    11.2   8.1   8.0    27.8   8.5   8.3
//   2^23    11.6  16.7  11.6    11.5  16.7  11.6    13.5  16.8  13.4    13.6  16.8  13.5    15.6  16.8  15.3    17.4  16.9  15.6    40.0  17.6  16.5
//   2^26    62.7 100.8  62.7    63.3 100.6  62.9    71.5 100.7  71.1    71.9 101.2  71.5    81.3 101.6  81.0    91.5 101.5 100.4     222   107   106
// (one wave in ten with such blocks, 2^26: 58.2 69.1 58.0 | 57.9 69.7 57.9 | 61.2 70.0 60.8 | 61.1 70.1 61.2 | 66.0 69.7 65.3 | 71.1 69.9 67.8 | 138 71 69)
template <int WAVES>
constexpr int kStagedWide = WAVES == kPackWaves ? 6 : 2;

// A block wider than 15 bits: the 16-bit fields are of no use then, and 32 deltas of 32 bits do not fit the registers beside
// everything else.  Its values are fetched and quantised again, and its words staged beside those of the wave's other blocks while the look-back is under way: 32 lanes a
// block, two blocks a step.  There are few of them as a rule: of the hard-data configuration one block in 3000, one wave in 50, one tile in 6.
// (The whole wave used to go over its values again, behind the look-back, see store_wide_wave, and its tile stayed that much longer.  us for 2^28 such values 228.6, now
// 208.0; 2^26: 64.0 58.2; 20 000 003: 25.5 22.3; 2^23: 13.4 11.4; 2^20: 7.4 6.4.  Data without wide blocks: level.)
__device__ __forceinline__ void stage_wide_blocks(const Placement& pl, u64 wblock0, u64 wide, u32* wl) {
  CompressArgs a;
  {
    const CompressArgs& again = kernel_args_again<CompressArgs, kCompressArgsAt>();
    a.in = again.in;
    a.n = again.n;
    a.inv = again.inv;
    a.step = again.step;
    a.eb = again.eb;
    a.screen = again.screen;
  }
  const u32 lane = u32(fresh_lane()), half = lane >> 5, j = lane & 31u;
#pragma nounroll
  while (wide) {
    const u32 blk_a = u32(__builtin_ctzll(wide));
    wide &= wide - 1;
    const u32 blk_b = wide ? u32(__builtin_ctzll(wide)) : blk_a;       // (an odd one out is done twice)
    wide &= wide - 1;
    const u64 v0 = (wblock0 + (half ? blk_b : blk_a)) * kBlockValues;
    const u64 left = a.n > v0 ? a.n - v0 : 0;
    const u32 cnt = left < 32 ? u32(left) : 32u;         // values of this block that exist
    u32 ignored = 0;                                     // errors were raised on the first pass
    i32 q = 0;
    if (j < cnt) q = quantize_value(a.in[v0 + j], a, ignored);
    const i32 last = i32(from_lane(u32(q), 32u * half + (cnt ? cnt - 1u : 0u)));
    if (j >= cnt) q = last;                              // the last block repeats its last code
    const i32 before = i32(from_lane(u32(q), lane + 63u));             // lane - 1 (lane 0 gets lane 63: unused)
    store_block_ballots(j ? q - before : 0, lane_value(pl.w, int(blk_a)), lane_value(pl.w, int(blk_b)), lane_value(pl.off_in_wave, int(blk_a)),
                        lane_value(pl.off_in_wave, int(blk_b)), wl, kWaveStage, lane);
  }
}

// A wave with more wide blocks than that, or with more words than its staging area is made for.  Once the wave's place is known it fetches and quantises all its values
// again, turns them into sign and plane words and stores those.  Only that wave does, and no tile waits for it.
// (2^28 hard values, compressed and decompressed, when a tile with a wide block stored all its blocks by ballots: 674 us, then 455.)
template <bool TICKETS>
__device__ __forceinline__ void store_wide_wave(const CompressArgs& a, const PayloadSink& sink, const Placement& pl, u64 base,
                                                u64 wblock0, u32 have, int lane, u32* wl) {
  asm volatile("" : "+v"(lane));               // (or the compiler keeps what it has loaded and quantised before, in scratch)
  i32 q[32];
  {
    float4 x[8];
    u32 ignored = 0;                           // errors were raised on the first pass
    load_raw(a.in, wblock0, lane, have, x);
    block_codes<TICKETS>(a, x, wblock0, have, lane, wl, q, ignored);
  }
#pragma unroll
  for (int j = 31; j >= 1; --j) q[j] -= q[j - 1];
  q[0] = 0;
  u32 lo[16], hi[16];
  planes_from_deltas32(q, lo, hi);
  copy_wave_out<32, false>(sink, [&](auto i) {
    constexpr int I = decltype(i)::value;      // 0: sign, 1 + p: plane p
    if constexpr (I == 0) return hi[15];
    else if constexpr (I <= 16) return lo[I - 1];
    else return hi[I - 17];
  }, pl, base, wl, lane);
}

// One workgroup per tile: tile = first_tile + workgroup id, or (TICKETS) + a ticket (see
// take_tile), over [first_tile, end_tile).  There is no set-up launch: tile 0 writes the header,
// and nothing in the workspace needs clearing (see launch_tag).  A workgroup that knows its tile
// from its id asks for its values before anything else, so that the scalar work that opens a call
// (tag, table positions: some 150 dependent instructions) runs while they are on their way: 512^3 field
// 122.4 -> 121.7 us when that was done, 116.4 now.  The ragged end is a tile like any other (see
// load_raw); as a launch of its own behind the full tiles it cost 7 us per call on any input that is not
// a multiple of 16384 values (20 000 003 values, compress and decompress: 59.0 us, now 51.9).
// WAVES: kPackWaves, or kTileWaves where that shortens the call (packs_small_tiles): with few tiles two waves of a workgroup of eight
// share a SIMD, which one alone keeps busy, while other compute units have nothing to do, and between one and one and a half workgroups of eight per compute unit
// three of four waves share it more evenly.  There it is the instructions that count, so these kernels also
// copy out by ranges and stage narrow blocks without conditions (stage_words_downward).  us, tiles of eight waves and of four:
//   sinusoids at 1e-4   1000 values 5.6 5.1 | 2^20: 6.6 5.4 | 2 000 003: 7.0 6.3 | 3 000 000: 7.1 6.8 | 5 000 000: 9.4 8.2 | 6 500 000: 9.5 9.7
//   a field at 1e-4     1000 values 6.0 5.3 | 2^20: 6.8 5.8 | 2 000 003: 7.2 6.5 | 3 400 000: 7.6 7.8 | 5 000 000: 10.3 9.0 | 6 500 000: 10.5 10.7
//   hard data           1000 values 5.7 4.6 | 2^20: 8.8 7.4 | 2 000 003: 9.1 7.7 | 3 000 000: 9.2 9.0 | 5 000 000: 11.7 10.2 | 8 000 000: 13.2 12.9
// With ZC_CHAINS_COHERENT, whose look-back takes longer the more tiles there are, only the former: a field at 1e-4, 2 090 000 values 10.0 9.7 | 4 300 000: 12.0 12.4 |
// 6 200 000: 13.7 14.4; hard data 11.9 11.2 | 13.8 14.1 | 15.7 16.2.
__host__ inline bool packs_small_tiles(const CompressArgs& a) {
  const u64 tiles = num_tiles(a.nb);
  return !a.ticketed && (tiles <= 256 || (tiles > 512 && tiles <= 768 && !a.coherent));
}

template <bool TICKETS, int WAVES>
__device__ __forceinline__ void compress_tile(const CompressInput& first, const CompressArgs& a, u32 first_tile, u32 end_tile, u32 (&lds)[WAVES * kWaveStage], u32& sh_tile,
                                             u32 (&sh_wave_total)[WAVES], u64 (&sh_base)[WAVES]) {
  constexpr int kBlocks = WAVES * kWaveBlocks;
  constexpr bool FEW = WAVES != kPackWaves;
  const int lane = lane_id();
  const int wave = wave_id();
  u32 tile = first_tile + blockIdx.x;        // tiles in the order in which workgroups start
  u32 have = 0;
  float4 x[8];
  if (!TICKETS) {
    const u64 wblock0 = u64(tile) * kBlocks + u64(wave) * kWaveBlocks;
    have = share_values(first.n, wblock0 * kBlockValues);
    load_raw(first.in, wblock0, lane, have, x);
  }
  const u32 ntiles = (u32(a.nb) + kBlocks - 1) / kBlocks;
  u32* const wl = lds + wave * kWaveStage;
  const bool tables_fit = a.out_cap >= tables_end(a.nb, a.ix);
  u32 err = 0;

  const u64 ltag = launch_tag(a.nonce, a.ctl);
  const u64 tag = call_tag(a.ctl, ltag, a.adopt != 0);
  if (TICKETS) {                             // ... or handed out by tickets, see take_tile
    if (threadIdx.x == 0) {
      const u32 t = take_tile(a.ctl, ltag, end_tile - first_tile, ticket_shard());
      sh_tile = t == kNoTile ? kNoTile : first_tile + t;
    }
    __syncthreads();
    tile = uniform(sh_tile);
  }
  if (tile >= end_tile) return;
  // the first tile also writes the fixed header fields and the padding of the tables
  if (tile == 0 && threadIdx.x == 0) {
    if (tables_fit) write_stream_header(a.out, a.n, a.nb, a.eb_bits, 1u, a.ix != 0, false);
    else raise_status(a.ctl, tag, status_bit(ZC_ERR_CAPACITY));
  }
  {
    const u64 wblock0 = u64(tile) * kBlocks + u64(wave) * kWaveBlocks;
    const bool active = u32(wblock0) + u32(lane) < u32(a.nb);      // (a stream has at most 2^26 blocks)
    if (TICKETS) {
      have = share_values(a.n, wblock0 * kBlockValues);
      load_raw(a.in, wblock0, lane, have, x);
    }

    BlockFields bf;
    block_fields<TICKETS>(a, x, wblock0, have, lane, wl, bf, err);
    Placement pl;
    pl.w = (active && bf.any) ? 32u - u32(__builtin_clz(bf.any)) : 0u;
    pl.wmax = wave_max_u32(pl.w);
    // (the width and the outlier go to their tables at the very end: a store that is under way is
    // waited for by the barrier below, and by every poll of the look-back)

    // ---- place the block inside the wave and the wave inside the tile ----
    const u32 words = psize_words(pl.w);
    const u32 incl = wave_inclusive_sum(words);
    pl.wave_total = lane_value(incl, 63);
    pl.half0_total = lane_value(incl, 31);
    pl.off_in_wave = incl - words;
    if (lane == 0) sh_wave_total[wave] = pl.wave_total | (a.ix && pl.wmax > 15 ? kWaveWideMark : 0u);
    lds_barrier();     // wave totals visible
    sum_wave_totals(sh_wave_total, wave, a.ix != 0, pl);
    // publish the tile's size as early as possible: the tiles after this one wait for it
    const PayloadSink sink{a.out, a.out_cap, a.nb, a.ctl, a.desc, a.ix != 0, a.coherent != 0, looks_direct(ntiles, kDirectTiles, a.coherent != 0, a.part_end), a.part_end, tag};
    if (threadIdx.x == 0) publish_tile_size(sink, tile, pl.tile_total, pl.tile_wide);

    // ---- fields -> sign + plane words, then the back half ----
    // uniform (always, without wide blocks)
    const bool staged = pl.wmax <= 15 || (pl.wave_total <= 64u * 16u && __builtin_popcountll(__ballot(pl.w > 15)) <= kStagedWide<WAVES>);
    const TileBase tb = resolve_tile_base(sink, pl, tile, sh_base, wave, lane, [&] {
      if (!staged) return;
      constexpr u32 kAside = 64 * 16 + 16;
      static_assert(kAside + 16 <= u32(kWaveStage));
      u32 pw[16];          // pw[0] = sign, pw[1 + p] = plane p
      if (pl.wmax <= 7) {
        u32 r[8];
        planes8_from_fields16(bf.f, r);
        pw[0] = r[7];
#pragma unroll
        for (int p = 0; p < 7; ++p) pw[1 + p] = r[p];
        if constexpr (FEW) {
          stage_words_downward<8>([&](auto i) { return pw[decltype(i)::value]; }, pl.w, pl.off_in_wave, wl, kAside);
          return;
        }
#pragma unroll
        for (int p = 8; p < 16; ++p) pw[p] = 0;
      } else {
        planes16_from_fields(bf.f);
        pw[0] = bf.f[15];
#pragma unroll
        for (int p = 0; p < 15; ++p) pw[1 + p] = bf.f[p];
      }
      // (what a lane writes for a wide block, 16 words, is overwritten by the block's own, which other lanes write)
      stage_wave_words<16>([&](auto i) { return pw[decltype(i)::value]; }, pl, wl);
      if (pl.wmax > 15) {                        // uniform
        wave_lds_sync();
        stage_wide_blocks(pl, wblock0, __ballot(pl.w > 15), wl);
      }
    });
    if (lane == 0) write_index_entry(sink, tile * u32(WAVES) + u32(wave), tb.words + pl.wave_off);
    if (staged) copy_staged_wave<16, FEW>(sink, pl, tb.words, wl, lane);
    else store_wide_wave<TICKETS>(a, sink, pl, tb.words, wblock0, have, lane, wl);
    finish_stream<WAVES>(sink, pl, tile, ntiles, tb);
    if (active && tables_fit) {                // (not store_tables: see copy_staged_words)
      const u64 b = wblock0 + u64(lane);
      a.out[widths_begin(a.nb, a.ix) + b] = u8(pl.w);
      reinterpret_cast<i32*>(a.out + outliers_begin(a.nb, a.ix))[b] = bf.outlier;
    }
  }
  if (err) raise_status(a.ctl, tag, err);
}

template <bool TICKETS, int WAVES = kPackWaves>
__global__ __launch_bounds__(64 * WAVES, WAVES == kPackWaves ? 8 : 4) void compress_kernel(const float* in, u64 n, u32 first_tile, u32 end_tile, CompressArgs a) {
  __shared__ __attribute__((aligned(16))) u32 lds[WAVES * kWaveStage];
  __shared__ u32 sh_tile;
  __shared__ u32 sh_wave_total[WAVES];
  __shared__ u64 sh_base[WAVES];
  compress_tile<TICKETS, WAVES>({in, n}, a, first_tile, end_tile, lds, sh_tile, sh_wave_total, sh_base);
  give_answer(a.answer, a.ctl);
}
static_assert(kernel_args_at<CompressArgs>(decltype(&compress_kernel<false>){}) == kCompressArgsAt);

// The stream of no values: a header (and the one closing entry of an indexed stream's index).
struct EmptyStreamArgs {
  Control* ctl;
  u8* out;
  u64 out_cap;
  u32 eb_bits;
  u32 ix;
  u64 nonce;
};

__global__ void empty_stream_kernel(EmptyStreamArgs a) {
  const u64 tag = call_tag(a.ctl, launch_tag(a.nonce, a.ctl), false);
  if (threadIdx.x != 0) return;
  const u64 tend = tables_end(0, a.ix != 0);
  a.ctl->result = tend;
  if (a.out_cap >= tend) write_stream_header(a.out, 0, 0, a.eb_bits, 1u, a.ix != 0, true);
  else raise_status(a.ctl, tag, status_bit(ZC_ERR_CAPACITY));
}

}  // namespace zc
