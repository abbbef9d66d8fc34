// Block positions of an existing stream: header validation and the exclusive prefix sum of
// the block sizes implied by its width table (Section 3.3 stores one code length per block;
// a block's position is the sum of the sizes before it), kept per segment of 64 blocks, the
// share of one wave.  An indexed stream (Section 3.5.2) brings these positions along: the main kernels judge the headers
// (judge_headers) and every wave of a consumer checks that its own segment's entries
// agree with its width bytes and with the ends of the index, which together is the whole index.
//
// stream_index_kernel records the offset of every segment inside its index span and the size of
// every span, with what it has seen in the width bytes; the main kernels add up the spans and judge header and widths (judge_plain_streams).  No workgroup
// waits for, or counts, another, and nothing needs to be cleared beforehand.  Streams of few blocks go without it.
#pragma once

#include "zc_common.h"

namespace zc {

struct StreamRef {
  const u8* base;
  u64 bytes;
};

struct ParsedHeader {
  u64 n, nb, total;
  u32 eb_bits, nsum;
  bool ok;
  bool wide;        // an indexed stream that may hold blocks wider than 15 bits
};

// Field checks that need nothing but the 32 header bytes and the buffer size.
__device__ inline ParsedHeader parse_header_words(const u32 (&w)[8], u64 bytes, bool ix) {
  ParsedHeader h;
  h.ok = false;
  h.wide = false;
  h.nb = 0;
  h.n = u64(w[2]) | (u64(w[3]) << 32);
  h.eb_bits = w[4];
  h.nsum = w[5];
  h.total = u64(w[6]) | (u64(w[7]) << 32);
  if (bytes < kHeaderBytes) return h;
  if (w[0] != kMagic || (ix ? (w[1] | 1u) != (kVersionIndexed | 1u) : w[1] != kVersionPlain)) return h;
  h.wide = ix && (w[1] & 1u) != 0;
  if (h.n > ZC_MAX_N) return h;
  // abs_eb must be a finite binary32 >= 2^-96: sign 0, biased exponent in [31, 254]
  const u32 e = h.eb_bits >> 23;
  if (e < 31 || e > 254) return h;
  if (h.nsum < 1) return h;
  h.nb = num_blocks(h.n);
  if (h.total > bytes || h.total < tables_end(h.nb, ix)) return h;
  h.ok = true;
  return h;
}

__device__ inline ParsedHeader parse_header(const StreamRef& s, bool ix) {
  u32 w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (s.bytes >= kHeaderBytes) {
    const u32* src = reinterpret_cast<const u32*>(s.base);
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = src[i];
  }
  return parse_header_words(w, s.bytes, ix);
}

// The same for a main kernel's first instructions: the header is asked for with vector loads
// (see opaque_zero), so that it travels together with whatever else the kernel can ask for before it knows the header.  The stream must have
// at least kHeaderBytes bytes (the host checks that before it launches anything).
struct HeaderWords {
  uint4 lo, hi;
};

__device__ inline HeaderWords load_header_words(const u8* base, u32 zero) {
  HeaderWords hw;
  hw.lo = *reinterpret_cast<const uint4*>(at_bytes(base, zero));
  hw.hi = *reinterpret_cast<const uint4*>(at_bytes(base, zero + 16u));
  return hw;
}

__device__ inline ParsedHeader parse_header(const HeaderWords& hw, u64 bytes, bool ix) {
  const u32 w[8] = {uniform(hw.lo.x), uniform(hw.lo.y), uniform(hw.lo.z), uniform(hw.lo.w),
                    uniform(hw.hi.x), uniform(hw.hi.y), uniform(hw.hi.z), uniform(hw.hi.w)};
  return parse_header_words(w, bytes, ix);
}

struct ScanArgs {
  StreamRef streams[ZC_MAX_K];
  int k;
  StreamIndex index;
};

// An entry of the list of spans: its payload words (less than 2^24), and whether it has a width byte above 31 and one
// above 15.
constexpr u32 kSpanSize = (1u << 30) - 1u;
constexpr u32 kSpanBadWidth = 1u << 30;
constexpr u32 kSpanWide = 1u << 31;

// Whether the caller's workspace has room for the index of this stream.
__device__ inline bool stream_fits(const ParsedHeader& h, const StreamIndex& ix) {
  return num_tiles(h.nb) <= ix.tiles_cap && num_spans(h.nb) <= ix.spans_cap;
}

// Payload word offset of segment `seg` of an indexed stream, from its own index.  `zero`: 0, or opaque_zero() to have a
// vector load whatever the compiler knows about seg.
__device__ inline u32 load_segment_offset(const u8* base, u32 seg, u32 zero = 0) {
  return *reinterpret_cast<const u32*>(at_bytes(base, kHeaderBytes + 4u * seg + zero));
}

// The entry after a segment's own in the index of an indexed stream: where the segment ends.
__device__ inline u32 load_segment_end(const u8* base, u32 seg, u32 zero = 0) {
  return *reinterpret_cast<const u32*>(at_bytes(base, kHeaderBytes + 4u + 4u * seg + zero));
}

// 16 width bytes from block b0 on of a table of nb, without those behind nb.
__device__ inline uint4 clip_widths16(const uint4& v, u32 b0, u32 nb) {
  const u32 live = nb > b0 ? nb - b0 : 0u;
  u32 x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) x[j] &= live >= 4u * j + 4 ? 0xFFFFFFFFu : (live > 4u * j ? (1u << (8 * (live - 4u * j))) - 1u : 0u);
  return make_uint4(x[0], x[1], x[2], x[3]);
}

// Payload words of 16 blocks: the sum of (1 + w) over the non-zero bytes (`seen`: OR of the width bytes).  A masked sum of differences
// leaves out the bytes that are zero: from 32 it is 32 for every other one, less the sum of the bytes.  (With a byte above 31 the result is
// wrong; it makes the stream malformed, whatever it is.)
__device__ inline u32 psize_words16(const uint4& v, u32& seen) {
  const u32 x[4] = {v.x, v.y, v.z, v.w};
  u32 sum = 0, rest = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    seen |= x[j];
    sum = __builtin_amdgcn_sad_u8(x[j], 0u, sum);
    rest = __builtin_amdgcn_msad_u8(0x20202020u, x[j], rest);
  }
  return sum + ((sum + rest) >> 5);
}
constexpr u32 kBadWidths = 0xE0E0E0E0u;                // bits of a width byte above 31 ...
constexpr u32 kWideWidths = 0xF0F0F0F0u;               // ... and above 15

// A workgroup covers one index span of one stream.  Each thread takes 16 blocks of a group of 4096 (one 16-byte load of
// the width table), four threads make a segment; a scan over the workgroup gives every segment its offset inside the
// group, the groups' totals the rest, and the span its size.
__global__ __launch_bounds__(256) void stream_index_kernel(ScanArgs a) {
  __shared__ u32 sh_wave[kIndexGroups][4];
  __shared__ u32 sh_flags;
  const int s = blockIdx.y;
  const StreamRef st = a.streams[s];
  const ParsedHeader h = parse_header(st, false);
  if (!h.ok || !stream_fits(h, a.index)) return;        // judge_plain_streams reports both
  const u64 group0 = u64(blockIdx.x) * kIndexGroups;
  if (u64(blockIdx.x) >= num_spans(h.nb)) return;

  const int lane = lane_id();
  const int wave = int(threadIdx.x) >> 6;
  if (threadIdx.x == 0) sh_flags = 0;
  const u8* widths = st.base + kHeaderBytes;
  // all loads first: the table is padded to a multiple of 16 bytes, so a 16-byte load that
  // starts below nb stays inside it; bytes of blocks that do not exist are masked off
  uint4 v[kIndexGroups];
#pragma unroll
  for (int i = 0; i < kIndexGroups; ++i) {
    const u64 b0 = (group0 + u64(i)) * kIndexGroupBlocks + u64(threadIdx.x) * 16;
    v[i] = make_uint4(0, 0, 0, 0);
    if (b0 < h.nb) v[i] = *reinterpret_cast<const uint4*>(widths + b0);
  }
  u32 sum[kIndexGroups], incl[kIndexGroups];
  u32 seen = 0;
#pragma unroll
  for (int i = 0; i < kIndexGroups; ++i) {
    const u64 b0 = (group0 + u64(i)) * kIndexGroupBlocks + u64(threadIdx.x) * 16;
    if (b0 + 16 > h.nb) v[i] = clip_widths16(v[i], u32(b0), u32(h.nb));
    sum[i] = psize_words16(v[i], seen);
    incl[i] = wave_inclusive_sum(sum[i]);
    if (lane == 63) sh_wave[i][wave] = incl[i];
  }
  const bool bad = (seen & kBadWidths) != 0, wide = (seen & kWideWidths) != 0;
  __syncthreads();                                       // sh_flags cleared, wave sums visible
  if (bad || wide) atomicOr(&sh_flags, (bad ? kSpanBadWidth : 0u) | (wide ? kSpanWide : 0u));
  u32* seg_off = a.index.seg_off + u64(s) * 4 * a.index.tiles_cap;
  const u64 nsegs = num_segments(h.nb);
  u32 span_before = 0;                                   // payload words of the span's groups so far
#pragma unroll
  for (int i = 0; i < kIndexGroups; ++i) {
    u32 before = 0, all = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const u32 t = sh_wave[i][j];
      if (j < wave) before += t;
      all += t;
    }
    const u64 seg = (group0 + u64(i)) * kIndexGroupSegs + (threadIdx.x >> 2);
    if ((threadIdx.x & 3) == 0 && seg < nsegs) seg_off[seg] = span_before + before + incl[i] - sum[i];
    span_before += all;
  }
  __syncthreads();                                       // every thread's flags are in
  if (threadIdx.x == 0) a.index.spans[u64(s) * a.index.spans_cap + blockIdx.x] = span_before | sh_flags;
}

// ---------------------------------------------------------------------------------------
// The main kernels read the headers of all input streams themselves, every workgroup, and come to the same verdict.
// Indexed streams need no launch ahead of them: every wave checks the part
// of the index it uses (the entries of its segment against its width bytes; the wave of the
// first segment that entry 0 is 0, the wave of the last that the closing entry accounts for
// total_bytes), which together is the whole index.
// ---------------------------------------------------------------------------------------

// Verdict on the k <= 64 input streams of a call, from their headers alone.  Lane s of the
// calling wave reads (ask_headers) and judges the header of stream s, so that all headers are in flight at
// once; every wave of every workgroup comes to the same verdict.
struct StreamsVerdict {
  ParsedHeader h0;      // header of stream 0 (uniform)
  u32 err;              // status bits: FORMAT, MISMATCH (uniform)
  u64 nsum;             // sum of the nsum fields of the valid streams
  u64 sum_n;            // sum of their n fields
  u64 wide;             // bit s: stream s may hold blocks wider than 15 bits (uniform; plain streams: see judge_plain_streams)
  ParsedHeader mine;    // lane s: header of stream s
};

// What a wave asks for before it knows anything about the streams: in lane s stream s itself (the arguments have room for ZC_MAX_K
// of them, so that this does not wait for k, which is in the arguments too), then its header and, of an indexed one, where the wave's
// segment lies in its payload, as its own index says: the entries sit right behind the header, whatever n is.  Lanes from k on ask for
// stream 0 once more, and for entries outside the caller's buffer comes the header: no load is behind a branch, and nothing that is asked
// for later may go ahead of them.
__device__ inline StreamRef lane_stream(const StreamRef* streams) { return streams[lane_id()]; }
struct LaneStream {
  uint4 lo, hi;         // the header
  u64 base, bytes;      // (at least kHeaderBytes: the host has checked)
  u32 begin, end;       // the segment's two entries
};
template <bool IX>
__device__ inline LaneStream ask_headers(const StreamRef& any, int k, u32 seg) {      // any = lane_stream(streams)
  const int lane = lane_id();
  const uint64_t base = reinterpret_cast<uint64_t>(any.base);
  const u64 base0 = u64(lane_value(u32(base), 0)) | (u64(lane_value(u32(base >> 32), 0)) << 32);
  const u64 bytes0 = u64(lane_value(u32(any.bytes), 0)) | (u64(lane_value(u32(any.bytes >> 32), 0)) << 32);
  const u64 from = lane < k ? base : base0;
  LaneStream l;
  l.base = from;
  l.bytes = lane < k ? any.bytes : bytes0;
  // (said to be global memory, see ask_plain_streams)
  typedef const __attribute__((address_space(1))) u32x4_t Global;
  const u32x4_t lo = reinterpret_cast<Global*>(from)[0], hi = reinterpret_cast<Global*>(from)[1];
  l.lo = make_uint4(lo.x, lo.y, lo.z, lo.w);
  l.hi = make_uint4(hi.x, hi.y, hi.z, hi.w);
  l.begin = l.end = 0;
  if (IX) {
    typedef const __attribute__((address_space(1))) u32 GlobalWord;
    const u64 at = u64(kHeaderBytes) + 4 * u64(seg);
    GlobalWord* const p = reinterpret_cast<GlobalWord*>(from + (at + 8 <= l.bytes ? at : 0));
    l.begin = p[0];
    l.end = p[1];
  }
  __builtin_amdgcn_sched_barrier(0);
  return l;
}

// The headers alone, where they are judged.  (The decompression of several streams asks for its own stream's header and segment
// first: with these headers ahead of that 8 x 2^26 values took 469 us, behind it 457.)
__device__ inline LaneStream read_headers(const StreamRef* streams, int k) {
  LaneStream l{};
  const int lane = lane_id();
  if (lane < k) {
    l.bytes = streams[lane].bytes;
    const uint4* src = reinterpret_cast<const uint4*>(streams[lane].base);
    l.lo = src[0];
    l.hi = src[1];
  }
  return l;
}

template <bool IX>
__device__ inline StreamsVerdict judge_headers(const LaneStream& asked, int k, bool check_match) {
  const int lane = lane_id();
  const bool mine = lane < k;
  const u64 bytes = asked.bytes;
  const u32 w[8] = {asked.lo.x, asked.lo.y, asked.lo.z, asked.lo.w, asked.hi.x, asked.hi.y, asked.hi.z, asked.hi.w};
  ParsedHeader h = parse_header_words(w, bytes, IX);
  h.ok = mine && h.ok;
  if (!mine) h.nb = 0;
  StreamsVerdict v;
  v.mine = h;
  v.h0.n = u64(lane_value(u32(h.n), 0)) | (u64(lane_value(u32(h.n >> 32), 0)) << 32);
  v.h0.nb = num_blocks(v.h0.n);
  v.h0.total = u64(lane_value(u32(h.total), 0)) | (u64(lane_value(u32(h.total >> 32), 0)) << 32);
  v.h0.eb_bits = lane_value(h.eb_bits, 0);
  v.h0.nsum = lane_value(h.nsum, 0);
  v.h0.ok = lane_value(u32(h.ok), 0) != 0;
  v.h0.wide = lane_value(u32(h.wide), 0) != 0;
  if (!v.h0.ok) v.h0.nb = 0;
  v.err = 0;
  if (__any(mine && !h.ok)) v.err |= status_bit(ZC_ERR_FORMAT);
  if (check_match && v.h0.ok && __any(mine && h.ok && (h.n != v.h0.n || h.eb_bits != v.h0.eb_bits)))
    v.err |= status_bit(ZC_ERR_MISMATCH);
  v.wide = __ballot(mine && h.ok && h.wide);
  // (in every workgroup: behind a branch for the first one, the Sum of 8 x 1000 values of plain streams took 13.4 us, without 13.1)
  const u32 ns = mine && h.ok ? h.nsum : 0u;
  v.nsum = u64(wave_sum_u32(ns & 0xffffu)) + (u64(wave_sum_u32(ns >> 16)) << 16);
  const u64 nn = mine && h.ok ? h.n : 0;              // <= 2^31
  v.sum_n = u64(wave_sum_u32(u32(nn) & 0xffffu)) + (u64(wave_sum_u32(u32(nn >> 16))) << 16);
  return v;
}

// The checks on the two ends of the index that fall to the wave that holds segment `seg`:
// seg_off and seg_end are its two entries.  (A stream without blocks has a single entry, which
// nobody uses: see index_ends_consistent.)
__device__ inline bool index_ends_ok(const ParsedHeader& h, u32 seg, u32 seg_off, u32 seg_end) {
  const u64 nseg = num_segments(h.nb);
  if (seg == 0 && seg_off != 0) return false;
  if (u64(seg) + 1 == nseg && tables_end(h.nb, true) + 4 * u64(seg_end) != h.total) return false;
  return true;
}

// The same for a kernel with k <= 64 input streams of the same n (headers judged already):
// called by the wave that holds segment `seg`, it does something only for the first and the
// last segment (and for a stream without blocks, whose one entry must be 0): lane s looks at
// stream s.  Uniform result.
__device__ inline bool index_ends_consistent(const StreamRef* streams, int k, const ParsedHeader& h, u32 seg) {
  const u64 nseg = num_segments(h.nb);
  const bool first = seg == 0;
  const bool last = nseg == 0 || u64(seg) + 1 == nseg;
  if (!first && !last) return true;                    // uniform
  const int lane = lane_id();
  bool bad = false;
  if (lane < k) {
    const u8* base = streams[lane].base;
    const u32* index = reinterpret_cast<const u32*>(base + kHeaderBytes);
    if (first && index[0] != 0) bad = true;
    if (last) {
      const u64 total = reinterpret_cast<const u64*>(base)[3];
      if (tables_end(h.nb, true) + 4 * u64(index[nseg]) != total) bad = true;
    }
  }
  return !__any(bad);
}

// ---------------------------------------------------------------------------------------
// Plain streams store no positions, so their width tables have to be summed, whole: the sums say where a segment is,
// whether every width is in order and whether total_bytes is.  Streams of few blocks are summed by every workgroup of the
// main kernel for itself (`self`), with the table asked for together with the header; for others stream_index_kernel
// runs ahead and a workgroup only adds up the sizes of the spans.  Either way all workgroups come to the same verdict before
// anything is written.  What this saves is launches (a dependent one costs 3 to 4 us, however little it does): with two
// ahead of the main kernel decompress took 10.4 us for a few thousand values (now 5.1) and 63.6 for 2^26 (61.5), a ring
// round of 40 000 values 13.4 (7.7), the Sum of 8 x 2^20 23.8 (20.0), a round trip of 20 000 003 values 53.5 (50.3).
// ---------------------------------------------------------------------------------------

// What the waves of a workgroup tell each other about up to K streams, four words each: unit s * parts + p is part p of
// stream s (see survey_parts).
template <int K>
struct PlainSurvey {
  u32 before[4 * K];        // payload words before the workgroup's tile (self) or its span
  u32 total[4 * K];         // payload words
  u32 seen[4 * K];          // OR of the width bytes (of the spans' flags)
  u32 in_tile[4 * K];       // self: per segment of the tile, payload words of the tile before it
};

// Tiles of all k streams of a call together up to which every workgroup sums their tables itself: the work grows with the
// square of the tiles, the launch it saves does not.  What bounds it is round trips to the L2, so several loads of a table are under way at once (with two of them
// decompress took 6.0 us for 2^20 values, now 5.6, and 7.6 for 2 000 003, now 6.75; a ring round 8.4, 8.0 and 10.2, 9.2; Max of 2 x 2^20 11.2, 10.3; 12 buffers of
// 200 000 11.2, 9.9).  us per call, with the launch ahead and without (power-law fields, 1e-3):
//   decompress   1 tile 9.2 4.6 | 245: 9.2 6.8 | 367: 9.4 8.4 | 512: 9.7 9.4 | 611: 10.3 11.7;   ring round   367: 12.7 11.6 | 512: 13.1 12.8
//   4 buffers    264: 10.3 7.3 | 392: 10.4 9.4 | 512: 10.5 10.2 | 588: 11.7 12.8;   16 buffers   400: 12.3 11.3 | 464: 13.9 11.8
//   32 buffers   416: 15.7 13.7 | 512: 15.1 12.8;   64 buffers   448: 19.1 17.8 | 512: 17.7 17.4
// The tables are summed one stream after the other, and what a launch ahead leaves to do is done for many at once in the
// reduces (see below), so that there the launch pays earlier with many streams:
//   Max of 2     368: 12.7 11.7 | 490: 12.8 12.9;   Sum of 4   392: 12.4 11.2 | 512: 12.5 11.9 | 588: 12.8 12.6;   of 8   392: 13.3 12.2 | 512: 13.3 12.7
//   Sum of 12    300: 14.0 12.4 | 396: 13.8 13.9;   of 16   256: 13.4 12.0 | 352: 13.6 13.5;   of 24   192: 14.7 14.4;   of 32   32: 16.0 16.9
// Where tiles are handed out by tickets a workgroup does it twice in a call that writes (the verdict ahead of its ticket, the place behind it), and it pays less far; with the
// launch ahead and without:
//   ring round   320: 18.8 16.3 | 340: 22.2 23.0 | 400: 16.0 17.2 | 512: 16.1 18.8; hard data   320: 22.5 19.9 | 340: 23.4 24.1 | 512: 20.5 22.8
//   Sum of 4     340: 22.6 21.0 | 480: 23.3 22.7;   Max of 8   320: 24.2 21.7 | 400: 22.9 23.1 | 480: 22.7 24.0;   Sum of 16   256: 29.5 27.5 | 288: 26.0 28.7 | 320: 26.4 29.0
__host__ constexpr u64 self_tiles(int k, bool reduce, bool tickets) {
  if (!reduce) return tickets ? 320 : 512;
  if (tickets && k > 4) return k <= 12 ? 320 : k <= 16 ? 256 : k <= 24 ? 192 : 0;
  return k <= 8 ? 480 : k <= 16 ? 320 : k <= 24 ? 192 : 0;
}

// The host does not know the tiles, only what the output or the workspace has room for and the bytes, which are at most
// kMostTables times what the tables of so many tiles need (133 bytes a block where its tables take 5).  With more bytes than
// the largest such streams have there may be tables that take every workgroup long to read, if only to find that the call fails.
constexpr u64 kMostTables = 27;

// How the lists of spans of a call of several streams are added up: by whole waves, one stream after the other, or in rows (ROWS)
// of 16 lanes, a stream each, four a wave at once.  The reduces have rows throughout, and with four streams or fewer every wave
// adds all of them up for itself, without a barrier; the decompression of many from 17 streams on, with fewer it runs into
// itself where every tile does nothing but read and write.  us per call, by waves and in rows:
//   Sum of 2 x 2 000 003 13.6 13.2, 2 x 2^26 81.5 80.2 | 5 x 2^26 106.6 104.3 | 16 x 2^24 62.9 59.5 | 64 x 2^20 70.7 65.8
//   17 buffers of 2^20 21.8 21.4 | 32 x 2^20 37.8 30.8 | 64 x 2^20 89.2 57.7;   12 x 2^24 141 152
// (A kernel of one workgroup that added them up for all before the main kernel started took 78.2 for the Sum of 2 x 2^26, but
// 104.2 for that of 5, 19.2 for 2 x 2 000 003 and 74.8 for the 64 buffers.)
constexpr int kManyByWave = 16;
// The first stream of the lane's row.
__device__ inline u32 row_stream(int k, int wave) { return (k <= 4 ? 0u : 4u * u32(wave)) + (u32(lane_id()) >> 4); }

// Waves that share a stream's table.
__device__ inline u32 survey_parts(int k, bool self) { return !self ? 1u : k == 1 ? 4u : k == 2 ? 2u : 1u; }

// Two loads of a width table by one wave, 1024 blocks each, `stride` blocks apart.  Fenced in by the caller's buffer (the
// table is padded to 16 bytes, so a piece of it never reaches beyond): what the header rules out is dropped later.
constexpr int kSurveyLoads = 2;
typedef u32 u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
struct SurveyLoads {
  uint4 v[kSurveyLoads];
};
// The rest of a table of nb blocks, once nb is known, BATCH loads under way at once.
template <int BATCH>
__device__ inline void load_widths(const StreamRef& in, u32 nb, u32 b0, u32 stride, uint4 (&v)[BATCH]) {
  const __amdgpu_buffer_rsrc_t table = bytes_from(in.base + kHeaderBytes, u32(pad16(nb)));
#pragma unroll
  for (int i = 0; i < BATCH; ++i) {
    const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(table, int(b0 + u32(i) * stride + 16u * u32(lane_id())), 0, 0);
    v[i] = make_uint4(t.x, t.y, t.z, t.w);
  }
}

// Asked for before the headers are known.  self: the wave's first part of a table.  Else: [0] the first spans of stream
// `wave` (of the only one: every wave; in rows: of the rows' streams, four a lane), [1] in lane s where the wave's segment lies in its span of stream s (of
// both the first word only, but in rows; the workspace ends 64 bytes behind the last table, see workspace_bytes).  Two loads either way and
// none behind a branch, so that a kernel that has asked for more behind them can wait for these alone; what must not be
// read is replaced by the first stream's header.
template <int K, bool ROWS>
__device__ __forceinline__ SurveyLoads ask_plain_streams(const StreamRef* streams, int k, const StreamIndex& index, bool self, u32 seg,
                                                         int wave) {
  const u32 parts = survey_parts(k, self);
  const u32 lane = u32(lane_id());
  const int s = K == 1 ? 0 : min(int(u32(wave) / parts), k - 1);
  const u8* const safe = streams[0].base;
  const u8* at[kSurveyLoads];
  if (self) {
#pragma unroll
    for (int i = 0; i < kSurveyLoads; ++i) {
      const u64 t = u64(kHeaderBytes) + 1024u * (u32(wave) % parts) + u32(i) * 1024u * parts + 16u * lane;
      at[i] = t + 16 <= streams[s].bytes ? streams[s].base + t : safe;
    }
  } else {
    const u32 of = ROWS ? row_stream(k, wave) : u32(s), i = ROWS ? 4u * (lane & 15u) : lane;
    const bool list = (ROWS ? int(of) < k : k == 1 || wave < k) && i < index.spans_cap, place = int(lane) < k && seg < 4 * index.tiles_cap;
    at[0] = list ? reinterpret_cast<const u8*>(index.spans + u64(of) * index.spans_cap + i) : safe;
    at[1] = place ? reinterpret_cast<const u8*>(index.seg_off + (K == 1 ? 0 : u64(lane) * 4 * index.tiles_cap) + seg) : safe;
  }
  SurveyLoads l;
#pragma unroll
  for (int i = 0; i < kSurveyLoads; ++i) {
    // (said to be global memory: the compiler no longer sees that through the choice above, and a load that may go to LDS
    // as well makes every wait a wait for all)
    typedef const __attribute__((address_space(1))) u32x4_a4 Global;
    const u32x4_a4 v = *reinterpret_cast<Global*>(reinterpret_cast<uintptr_t>(at[i]));
    l.v[i] = make_uint4(v.x, v.y, v.z, v.w);
  }
  return l;
}

// The spans of stream s (asked: the first 64 are in `ask`), one per lane and round: the lane's share of the payload words of
// those before the tile's own span (`before`) and of all, and OR of their flags.
__device__ inline void sum_spans(const StreamIndex& index, u32 s, u32 nb, u32 tile, bool asked, const SurveyLoads& ask, u32& before,
                                 u32& total, u32& seen) {
  const u32 nspans = u32(num_spans(nb)), span = tile / (kSpanSegs / kTileWaves);
  const u32 lane = u32(lane_id());
#pragma nounroll
  for (u32 i0 = 0; i0 < nspans; i0 += 64) {
    const u32 i = i0 + lane;
    const bool have = asked && i0 == 0;
    const u32 entry = i < nspans ? (have ? ask.v[0].x : index.spans[u64(s) * index.spans_cap + i]) : 0u;
    seen |= entry;
    total += entry & kSpanSize;
    before += i < span ? entry & kSpanSize : 0u;
  }
}

// Sum over the 16 lanes of a row, in all of them.
__device__ inline u32 row_sum(u32 v) {
  v += dpp_mov<kDppQuadSwap1>(v);
  v += dpp_mov<kDppQuadSwap2>(v);
  v += dpp_mov<kDppRowHalfMirror>(v);
  v += dpp_mov<kDppRowMirror>(v);
  return v;
}

// The spans of the stream `s` of the lane's row (nspans of them, 64 at a time, four a lane): payload words of those before the
// tile's own, of all, and OR of their flags, in every lane of the row.  first: entries 4 at ... 4 at + 3 (at: the lane's
// place in its row).
struct RowOfSpans {
  u32 before, total, seen;
};
__device__ inline uint4 load_spans(const StreamIndex& index, u32 s, u32 nspans, u32 i) {
  const u32x4_a4 v = *reinterpret_cast<const u32x4_a4*>(index.spans + (i < nspans ? u64(s) * index.spans_cap + i : 0));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ inline RowOfSpans sum_row_of_spans(const StreamIndex& index, u32 s, u32 nspans, u32 tile, const uint4& first) {
  const u32 lane = u32(lane_id());
  const u32 span = tile / (kSpanSegs / kTileWaves);
  uint4 e = first;
  u32 before = 0, total = 0, seen = 0;
  u32 i = 4u * (lane & 15u);
#pragma nounroll
  for (;;) {
    const u32 x[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
    for (u32 j = 0; j < 4; ++j) {
      const u32 entry = i + j < nspans ? x[j] : 0u;
      seen |= entry;
      total += entry & kSpanSize;
      before += i + j < span ? entry & kSpanSize : 0u;
    }
    i += 64;
    if (!__any(i < nspans)) break;
    e = load_spans(index, s, nspans, i);
  }
  const u64 bad = __ballot((seen & kSpanBadWidth) != 0), wide = __ballot((seen & kSpanWide) != 0);
  const u32 row = lane & 48u;
  return {row_sum(before), row_sum(total), (u32(bad >> row) & 0xffffu ? kSpanBadWidth : 0u) | (u32(wide >> row) & 0xffffu ? kSpanWide : 0u)};
}

// Lane r holds what is in row r (r < 4), and the other way round.
__device__ inline u32 rows_to_lanes(u32 v) {
  const u32 a = lane_value(v, 0), b = lane_value(v, 16), c = lane_value(v, 32), d = lane_value(v, 48);
  const int lane = lane_id();
  return lane == 0 ? a : lane == 1 ? b : lane == 2 ? c : d;
}
__device__ inline u32 lanes_to_rows(u32 v) {
  const u32 a = lane_value(v, 0), b = lane_value(v, 1), c = lane_value(v, 2), d = lane_value(v, 3);
  const int row = lane_id() >> 4;
  return row == 0 ? a : row == 1 ? b : row == 2 ? c : d;
}

// The lists of spans of a call in rows, for `sh`: four streams a wave and round.  blocks: lane s: of stream s (none from stream k on).
template <int K>
__device__ inline void sum_spans_by_rows(const StreamIndex& index, int k, u32 blocks, u32 tile, int wave, const SurveyLoads& ask, PlainSurvey<K>& sh) {
  const u32 lane = u32(lane_id());
  uint4 next = ask.v[0];
  u32 s = row_stream(k, wave);
  u32 nspans = (u32(__builtin_amdgcn_ds_bpermute(int(4u * s), int(blocks))) + kSpanBlocks - 1) / kSpanBlocks;
#pragma nounroll
  for (u32 s0 = 4u * u32(wave); s0 < u32(k); s0 += 4u * kTileWaves) {
    const uint4 first = next;
    const u32 here = s, spans_here = nspans;
    s = (s + 4u * kTileWaves) & 63u;           // (asked for ahead of time; beyond the last stream nothing comes of it)
    nspans = (u32(__builtin_amdgcn_ds_bpermute(int(4u * s), int(blocks))) + kSpanBlocks - 1) / kSpanBlocks;
    next = load_spans(index, s, nspans, 4u * (lane & 15u));
    const RowOfSpans r = sum_row_of_spans(index, here, spans_here, tile, first);
    if ((lane & 15u) == 0 && here < u32(k)) {
      sh.before[here] = r.before;
      sh.total[here] = r.total;
      sh.seen[here] = r.seen;
    }
  }
}

// Called by all waves of a workgroup of kTileWaves waves; at most one barrier.  `v`: the verdict on the headers, completed here (err,
// wide).  Returns, in lane s, the payload word offset of the wave's segment, kTileWaves * tile + in_tile, in stream s.
template <int K, bool ROWS>
__device__ __forceinline__ u32 judge_plain_streams(const StreamRef* streams, int k, const StreamIndex& index, bool self, u32 tile, int wave,
                                          const SurveyLoads& ask, StreamsVerdict& v, PlainSurvey<K>& sh, int in_tile = wave_id() % kTileWaves) {
  const int lane = lane_id();
  const u32 parts = survey_parts(k, self);
  const bool mine = lane < k;
  const bool fits = v.mine.ok && stream_fits(v.mine, index);
  u32 off = 0, total = 0, seen = 0;            // lane s: of stream s
  if (K == 1 && !self) {
    // every wave for itself: no wave has to wait for another
    sum_spans(index, 0, fits ? u32(v.mine.nb) : 0u, tile, true, ask, off, total, seen);
    off = wave_sum_u32(off) + ask.v[1].x;
    total = wave_sum_u32(total);
    seen = (__any((seen & kSpanBadWidth) != 0) ? kSpanBadWidth : 0u) | (__any((seen & kSpanWide) != 0) ? kSpanWide : 0u);
  } else if (ROWS && !self && k <= 4) {
    // and so with four streams, a row each
    const u32 nspans = (lanes_to_rows(fits ? u32(v.mine.nb) : 0u) + kSpanBlocks - 1) / kSpanBlocks;
    const RowOfSpans r = sum_row_of_spans(index, row_stream(k, wave), nspans, tile, ask.v[0]);
    off = rows_to_lanes(r.before) + ask.v[1].x;
    total = rows_to_lanes(r.total);
    seen = rows_to_lanes(r.seen);
  } else {
    const bool rows = ROWS && !self;
    if (rows) sum_spans_by_rows(index, k, fits ? u32(v.mine.nb) : 0u, tile, wave, ask, sh);
#pragma nounroll
    for (u32 u = u32(wave); !rows && u < u32(k) * parts; u += kTileWaves) {
      const u32 s = u / parts, p = u % parts;
      const u32 nb = lane_value(u32(fits), int(s)) ? lane_value(u32(v.mine.nb), int(s)) : 0u;
      u32 before = 0, total = 0, seen = 0;
      if (self) {
        const u32 first = tile * kTileBlocks, step = 1024u * parts;
        // the blocks from c0 + 16 * lane on
        auto count = [&](uint4 x, u32 c0) {
          if (c0 + 1024u > nb) x = clip_widths16(x, c0 + 16u * u32(lane), nb);      // uniform
          const u32 sum = psize_words16(x, seen);
          total += sum;
          if (c0 < first) before += c0 + 16u * u32(lane) < first ? sum : 0u;      // uniform
          if (first - c0 < 1024u) {                        // uniform: the tile is one row of 16 lanes here
            u32 incl = sum;
            incl += dpp_row_shr_or_zero<1>(incl);
            incl += dpp_row_shr_or_zero<2>(incl);
            incl += dpp_row_shr_or_zero<4>(incl);
            incl += dpp_row_shr_or_zero<8>(incl);
            if (u32(lane) >> 4 == (first - c0) >> 8 && (lane & 3) == 0) sh.in_tile[4 * s + ((u32(lane) >> 2) & 3u)] = incl - sum;
          }
        };
        u32 b0 = 1024u * p;
        constexpr int kBatch = K == 1 ? 8 : 4;             // (many streams have small tables)
        if (u == u32(wave)) {                              // uniform
#pragma unroll
          for (int i = 0; i < kSurveyLoads; ++i, b0 += step)
            if (b0 < nb) count(ask.v[i], b0);              // uniform
        }
#pragma nounroll
        for (; b0 < nb; b0 += step * kBatch) {
          uint4 x[kBatch];
          load_widths(streams[s], nb, b0, step, x);
#pragma unroll
          for (int i = 0; i < kBatch; ++i)
            if (b0 + step * u32(i) < nb) count(x[i], b0 + step * u32(i));      // uniform
        }
      } else {
        sum_spans(index, s, nb, tile, u == u32(wave), ask, before, total, seen);
      }
      before = wave_sum_u32(before);
      total = wave_sum_u32(total);
      if (self) seen = ((seen & kBadWidths) ? kSpanBadWidth : 0u) | ((seen & kWideWidths) ? kSpanWide : 0u);
      const bool bad = __any((seen & kSpanBadWidth) != 0), wide = __any((seen & kSpanWide) != 0);
      if (lane == 0) {
        sh.before[u] = before;
        sh.total[u] = total;
        sh.seen[u] = (bad ? kSpanBadWidth : 0u) | (wide ? kSpanWide : 0u);
      }
    }
    lds_barrier();
    if (mine) {
#pragma nounroll
      for (u32 p = 0; p < parts; ++p) {
        off += sh.before[u32(lane) * parts + p];
        total += sh.total[u32(lane) * parts + p];
        seen |= sh.seen[u32(lane) * parts + p];
      }
      off += self ? sh.in_tile[4 * lane + in_tile] : ask.v[1].x;
    }
  }
  if (__any(mine && v.mine.ok && !fits)) v.err |= status_bit(ZC_ERR_ARG);
  if (__any(mine && fits && ((seen & kSpanBadWidth) != 0 || tables_end(v.mine.nb, false) + 4 * u64(total) != v.mine.total)))
    v.err |= status_bit(ZC_ERR_FORMAT);
  v.wide = __any(mine && fits && (seen & kSpanWide) != 0) ? ~u64(0) : 0;
  return off;
}

}  // namespace zc
