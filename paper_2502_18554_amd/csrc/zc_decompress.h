// fZ-light decompression kernel: the inverse of the stages of Section 3.3.
//
// Same geometry as compression: a tile is 256 blocks, one lane owns one block, and there is no
// dependency between workgroups: a wave's payload offset comes from the stream index
// (computed by zc_scan.h for a plain stream, carried by an indexed one), and a scan of the
// block sizes places each lane inside the wave.  The wave's
// payload is contiguous, so it is copied into LDS with coalesced loads (each byte leaves the
// L2 once) and every lane then picks its sign and plane words there.  A bit-matrix transpose
// turns them back into deltas; the Lorenzo chain from the block's outlier and the
// dequantisation follow in registers; the floats go back through LDS, in two halves of 32
// blocks, so that they leave as 16-byte coalesced stores.
#pragma once

#include "zc_bitmatrix.h"
#include "zc_common.h"
#include "zc_report.h"
#include "zc_scan.h"

namespace zc {

struct DecompressArgs {
  StreamRef in;
  float* out;
  u64 out_cap_elems;
  StreamIndex index;
  Control* ctl;
  u64 first_value;   // decompress_range_kernel only: the part [first_value, first_value + count) of the
  u64 count;         // stream, first_value a multiple of the values of a segment
  u64 nonce;         // drawn by the host per call, goes into the call's tag (see launch_tag)
};

// The sign and plane words of the lane's block (width w, 0 for a block that does not exist) out
// of a stream's payload.  seg_off = payload word offset of the wave's segment.  The wave's
// payload goes through its LDS staging area `wl` (kWaveStage words); a wave with a block wider
// than 15 bits fetches per lane instead.  Returns the widest block of the wave.  Widths up to
// 15: lo[0..15) = planes 0..14, lo[15] = sign word.  Wider: lo[0..16) = planes 0..15,
// hi[0..15) = planes 16..30, hi[15] = sign word.  `wl` is free again on return.
// Indexed stream (ix): seg_words = the segment's size by the stream's own index.  The staged
// copy is asked for on that figure, before the widths are looked at, so it travels together
// with the loads of the tables; a segment whose widths add up to another figure, a width above
// 31, or one above 15 in a stream that promised none (!may_be_wide) make the stream malformed
// (`err`), and nothing of the segment's payload is used.
constexpr int kWaveStageLoads = 4;
struct WaveStage {
  uint4 v[kWaveStageLoads];
};

// The copy starts at the 16-byte boundary at or below the segment (the payload area itself is
// 16-byte aligned) and keeps that misalignment in LDS, so it moves 16 bytes per lane and
// instruction, all loads in flight together.  span = words to bring in, <= 1027.
// Four loads cover 1024 words; only whole 16-byte pieces are asked for here: the up to three
// words beyond (a wave whose 64 blocks are all 15 bits wide, off the 16-byte grid) and the
// last words of a stream that do not fill a piece are fetched by store_wave_stage.  The loads
// are written without any branch: a lane with nothing to fetch is outside the buffer's range.  (With a branch around a
// load and a zero on its other side, or with the stream's last words fetched into single components of the same
// registers, the compiler copied a component after every 16-byte load and waited for the load to do so: the
// loads went out one round trip after the other.)
__device__ inline u32 whole_pieces(u64 payload_words, u64 src0, u32 span) {
  const u64 room = payload_words > src0 ? (payload_words - src0) & ~u64(3) : 0;
  const u32 wanted = min((span + 3u) & ~3u, 256u * kWaveStageLoads);
  return room < wanted ? u32(room) : wanted;
}
__device__ inline WaveStage load_wave_stage(const u32* payload, u64 payload_words, u64 src0, u32 span, int lane) {
  WaveStage st;
  const __amdgpu_buffer_rsrc_t share = bytes_from(payload + src0, 4u * whole_pieces(payload_words, src0, span));
#pragma unroll
  for (int i = 0; i < kWaveStageLoads; ++i) {
    const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(share, 16 * lane + 1024 * i, 0, 0);
    st.v[i] = make_uint4(t.x, t.y, t.z, t.w);
  }
  return st;
}

__device__ inline void store_wave_stage(const WaveStage& st, const u32* payload, u64 payload_words, u64 src0, u32 span,
                                        u32* wl, int lane) {
#pragma unroll
  for (int i = 0; i < kWaveStageLoads; ++i)
    if (256u * u32(i) < span) *reinterpret_cast<uint4*>(wl + 4u * u32(lane) + 256u * u32(i)) = st.v[i];      // uniform
  const u32 whole = whole_pieces(payload_words, src0, span);
  if (whole < span) {                                  // uniform, and rare: at most three words, or the end of the stream
    asm volatile("");                                  // (keeps the branch: merged with the condition below, all of this runs every time)
    const u32 idx = whole + u32(lane);
    if (idx < span && src0 + idx < payload_words) wl[idx] = payload[src0 + idx];
  }
}

// What a wave knows about its segment's payload once the widths are scanned.
struct WavePayload {
  u32 w;            // this lane's block width (0 if the block must be skipped)
  u32 off_in_wave;  // payload word offset of this lane's block inside the segment
  u32 wmax;         // the widest block of the wave (uniform)
  bool inside;      // the segment lies inside the payload and agrees with the index (uniform)
  bool staged;      // its payload is in the staging area: always if no block is wider than 15 bits (uniform)
};

// First half of wave_block_words: scan of the widths, the checks, and the staged copy of the
// segment's payload into `wl` if it has at most 64 x 16 words (with no block wider than 15 bits it has not more).
// stage_wide: the caller uses the copy of a segment that has wider blocks, too; if not, such a segment of a plain stream,
// whose widths are known ahead of the copy, is not copied.
__device__ inline WavePayload stage_wave_payload(const u32* payload, u64 payload_words, u32 w, u64 seg_off, u32* wl, int lane,
                                                 bool ix, u32 seg_words, bool may_be_wide, u32& err, bool stage_wide) {
  const u32 mis = u32(seg_off) & 3u;
  const u64 src0 = seg_off - mis;                      // in words, multiple of 4
  WaveStage st;
  u32 span = 0;
  if (ix) {
    // at most 64 * 16 words when no block is wider than 15 bits
    if (seg_words <= 64u * 16u && seg_off + seg_words <= payload_words) span = mis + seg_words;
    st = load_wave_stage(payload, payload_words, src0, span, lane);
    store_wave_stage(st, payload, payload_words, src0, span, wl, lane);   // at once: the registers are free for what follows
  }
  bool unfit = false;
  if (ix) {
    unfit = __any(w > (may_be_wide ? 31u : 15u));
    if (unfit) w = 0;
  }
  WavePayload wp;
  const u32 words = psize_words(w);
  const u32 incl = wave_inclusive_sum(words);
  wp.off_in_wave = incl - words;
  const u32 wave_total = lane_value(incl, 63);
  wp.wmax = wave_max_u32(w);
  wp.w = w;
  // a validated stream keeps every segment inside the payload; refuse to read outside anyway
  wp.inside = seg_off + wave_total <= payload_words;
  if (ix && (unfit || wave_total != seg_words)) {
    err |= status_bit(ZC_ERR_FORMAT);
    wp.inside = false;
  }
  wp.staged = wp.inside && wave_total <= 64u * 16u && (stage_wide || wp.wmax <= 15);
  if (wp.staged && !ix) {
    span = mis + wave_total;
    st = load_wave_stage(payload, payload_words, src0, span, lane);
    store_wave_stage(st, payload, payload_words, src0, span, wl, lane);
  }
  return wp;
}

// Second half, widths up to 15: every lane picks its block's words out of the staged copy.
// lo[0..15) = planes 0..14, lo[15] = sign word.  `wl` is free again on return.
// All sixteen reads are issued at once and without conditions (the words behind a block's own
// belong to the next blocks, or are whatever the staging area held: they are dropped
// afterwards; the area is large enough for 15 words behind any staged word).  A loop that
// stops at the wave's widest block costs far more than the reads it saves: it is compiled as
// a loop, with a wait after every read.
// In two parts: the words as they come, and without what is not the block's own (`w`: its width, 0 if it has no payload).
__device__ inline u32 own_width(const WavePayload& wp) { return wp.inside ? wp.w : 0u; }
__device__ inline void pick_raw_words(const WavePayload& wp, u64 seg_off, const u32* wl, u32 (&lo)[16]) {
  static_assert(kWaveStage >= 1027 + 16, "reads behind the last staged word stay inside the staging area");
  wave_lds_sync();
  const u32* mine = wl + (own_width(wp) ? (u32(seg_off) & 3u) + wp.off_in_wave : 0u);
  lo[15] = mine[0];
#pragma unroll
  for (int p = 0; p < 15; ++p) lo[p] = mine[1 + p];
  wave_lds_sync();
}
template <int PLANES>
__device__ inline void keep_block_words(u32 w, u32 (&lo)[16]) {
  const u32 keep = (1u << w) - 1u;                     // bit p: the block has plane p
  lo[15] = w ? lo[15] : 0u;
#pragma unroll
  for (int p = 0; p < PLANES; ++p) {
    // (the AND spelled out: seen as one, it is compiled into a test and a selection per plane)
    const u32 m = u32(__builtin_amdgcn_sbfe(i32(keep), u32(p), 1u));
    lo[p] = __builtin_amdgcn_bitop3_b32(lo[p], m, m, 0xC0);
  }
}
__device__ inline void pick_block_words(const WavePayload& wp, u64 seg_off, const u32* wl, u32 (&lo)[16]) {
  pick_raw_words(wp, seg_off, wl, lo);
  keep_block_words<15>(own_width(wp), lo);
}

__device__ inline u32 wave_block_words(const u32* payload, u64 payload_words, u32 w, u64 seg_off, u32* wl, int lane,
                                       u32 (&lo)[16], u32 (&hi)[16], bool ix, u32 seg_words, bool may_be_wide,
                                       u32& err) {
  const WavePayload wp = stage_wave_payload(payload, payload_words, w, seg_off, wl, lane, ix, seg_words, may_be_wide, err, false);
  if (wp.wmax <= 15) {
    pick_block_words(wp, seg_off, wl, lo);
  } else {
    // a block wider than 15 bits (stream of an input outside the guaranteed domain): each lane
    // fetches its words straight from global memory
#pragma unroll
    for (int p = 0; p < 16; ++p) lo[p] = 0;
#pragma unroll
    for (int p = 0; p < 16; ++p) hi[p] = 0;
    if (wp.w && wp.inside) {
      const u32* mine = payload + seg_off + wp.off_in_wave;
      hi[15] = mine[0];
#pragma unroll
      for (int p = 0; p < 16; ++p)
        if (u32(p) < wp.w) lo[p] = mine[1 + p];
#pragma unroll
      for (int p = 0; p < 15; ++p)
        if (u32(16 + p) < wp.w) hi[p] = mine[17 + p];
    }
  }
  return wp.wmax;
}

// ... and from those words the block's Lorenzo deltas (bit-matrix transposes back).
__device__ inline void deltas_from_block_words(u32 wmax, u32 (&lo)[16], u32 (&hi)[16], i32 (&d)[32]) {
  if (wmax <= 7) {
    u32 r[8];
#pragma unroll
    for (int p = 0; p < 7; ++p) r[p] = lo[p];
    r[7] = lo[15];
    deltas_from_planes8(r, d);
  } else if (wmax <= 15) {
    deltas_from_planes16(lo, d);
  } else {
    deltas_from_planes32(lo, hi, d);
  }
}

// One tile (blockIdx.x) of stream `s` into `out`.
// The header is judged here, by every workgroup alike (see judge_headers, judge_plain_streams, index_ends_ok).
// `IX`: the stream is indexed; its width bytes sit behind the index, whose size only the header tells, so they
// are asked for together with the outlier and the payload.  SELF: a plain stream whose width table the kernel sums itself
// (a template parameter: as an argument it cost the streams that have an index 2 %).  K: room for that many streams in the survey of plain ones (ROWS: see
// kManyByWave); `streams`, `k`: all streams of the call.
// `average`: the values are divided by the stream's nsum (the Average aggregation of Section
// 3.2 on a stream of sums): x' = float((double(q) * s) * r), r = 1.0 / nsum.
// first_value, count: only the values [first_value, first_value + count) of the stream, cut off
// at its end, are produced, into out_values[0 ...] (a chunk handled on its own, Section 3.5.2);
// first_value is a multiple of the 2048 values of a segment.  The whole stream: 0 and ~0.
template <bool IX, bool SELF, int K, bool ROWS = false>
__device__ __forceinline__ void decompress_tile(const StreamRef* streams, int k, int s, float* out_values, u64 out_cap_elems,
                                       const StreamIndex& index, Control* ctl, u64 nonce, u32* lds, PlainSurvey<K>* survey,
                                       bool average = false, u64 first_value = 0, u64 count = ~u64(0)) {
  const StreamRef in = streams[s];
  const DecompressArgs a{in, out_values, out_cap_elems, index, ctl, first_value, count, nonce};
  constexpr bool many = K > 1;

  // Everything that can be asked for before the header is known goes out at once: the header, the segment's position and
  // the width bytes.  The loads are fenced in by sizes the host passed; what the header then rules out is dropped.
  const int lane = lane_id();
  const int wave = wave_id();
  const u32 tile = u32(first_value / kTileValues) + blockIdx.x;
  const u32 seg = tile * kTileWaves + u32(wave);       // < 2^22: the host launches at most 2^18 tiles
  const u32 wblock0 = seg * kWaveBlocks;
  const u32 b = wblock0 + u32(lane);                   // a stream has at most 2^26 blocks
  const u32 zero = opaque_zero();
  const bool first_group = blockIdx.x == 0 && blockIdx.y == 0;
  SurveyLoads ask{};
  if (!IX) ask = ask_plain_streams<K, ROWS>(streams, k, a.index, SELF, seg, wave);
  const HeaderWords hw = load_header_words(a.in.base, zero);
  u32 seg_begin = 0, seg_end = 0, w = 0;
  if (IX) {
    if (u64(kHeaderBytes) + 4 * u64(seg) + 8 <= a.in.bytes) {
      seg_begin = load_segment_offset(a.in.base, seg, zero);
      seg_end = load_segment_end(a.in.base, seg, zero);
    }
  } else {
    if (u64(kHeaderBytes) + b < a.in.bytes) w = u32(*at_bytes(a.in.base, kHeaderBytes + b));
  }

  // (the tag, some 100 dependent scalar instructions, while the loads are on their way)
  u64 ltag = launch_tag(a.nonce, a.ctl);
  asm volatile("" : "+s"(ltag));
  StreamsVerdict v;
  if constexpr (many) v = judge_headers<IX>(read_headers(streams, k), k, false);      // any malformed stream stops the whole call
  const ParsedHeader h = parse_header(hw, a.in.bytes, IX);
  if constexpr (!many) {
    v.mine = h;
    v.err = h.ok ? 0u : status_bit(ZC_ERR_FORMAT);
  }
  const u64 tag = call_tag(a.ctl, ltag, false);
  if (!IX) {
    const u32 off = judge_plain_streams<K, ROWS>(streams, k, a.index, SELF, tile, wave, ask, v, *survey);
    seg_begin = lane_value(off, s);
  }
  if (v.err) {
    if (first_group && threadIdx.x == 0) {
      a.ctl->result = 0;
      raise_status(a.ctl, tag, v.err);
    }
    return;
  }
  // a stream without blocks: nobody looks at its index, which is one closing entry of 0
  if (IX && h.nb == 0 && blockIdx.x == 0 && threadIdx.x == 0 &&
      (h.total != tables_end(0, true) || *reinterpret_cast<const u32*>(a.in.base + kHeaderBytes) != 0))
    raise_status(a.ctl, tag, status_bit(ZC_ERR_FORMAT));
  if (first_value > h.n) {                            // the part lies beyond the stream
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      a.ctl->result = 0;
      raise_status(a.ctl, tag, status_bit(ZC_ERR_ARG));
    }
    return;
  }
  const u64 end_value = count < h.n - first_value ? first_value + count : h.n;     // one past the last value wanted
  const u64 wanted = end_value - first_value;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) a.ctl->result = many ? v.sum_n : wanted;
  if (wanted > a.out_cap_elems) {
    if (blockIdx.x == 0 && threadIdx.x == 0) raise_status(a.ctl, tag, status_bit(ZC_ERR_CAPACITY));
    return;
  }

  u32* const wl = lds + wave * kWaveStage;
  // (no barrier below: waves are independent)
  if (seg >= num_segments(h.nb) || u64(seg) * (kWaveBlocks * kBlockValues) >= end_value || u64(seg) * (kWaveBlocks * kBlockValues) < first_value) return;
  const bool active = b < h.nb;
  if (IX) w = u32(__builtin_amdgcn_raw_buffer_load_b8(bytes_from(a.in.base + widths_begin(h.nb, true), u32(h.nb)), int(b), 0, 0));
  if (!active) w = 0;

  const u32* payload = reinterpret_cast<const u32*>(a.in.base + tables_end(h.nb, IX));
  const u64 payload_words = (h.total - tables_end(h.nb, IX)) / 4;

  u32 cur = __builtin_amdgcn_raw_buffer_load_b32(bytes_from(a.in.base + outliers_begin(h.nb, IX), 4u * u32(h.nb)), int(4u * b), 0, 0);
  const u64 seg_off = u64(uniform(seg_begin));
  i32 d[32];
  {
    u32 lo[16], hi[16];
    u32 err = 0;
    const u32 wmax = wave_block_words(payload, payload_words, w, seg_off, wl, lane, lo, hi, IX,
                                      uniform(seg_end) - u32(seg_off), h.wide, err);
    if (IX && !index_ends_ok(h, seg, u32(seg_off), uniform(seg_end))) err |= status_bit(ZC_ERR_FORMAT);
    if (err && lane == 0) raise_status(a.ctl, tag, err);
    deltas_from_block_words(wmax, lo, hi, d);
  }

  // ---- Lorenzo chain from the outlier, dequantise ----
  const double step = double(__uint_as_float(h.eb_bits)) * 63.0 / 32.0;
  const double r = average ? __ddiv_rn(1.0, double(h.nsum)) : 1.0;
  float x[32];
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    cur += u32(d[j]);
    const double v = __dmul_rn(double(i32(cur)), step);
    x[j] = float(average ? __dmul_rn(v, r) : v);
  }

  // ---- transpose through LDS (two halves of 32 blocks), 16-byte coalesced stores ----
  const u64 v0 = u64(wblock0) * kBlockValues;
  float* const out = a.out + (v0 - first_value);
  const u64 left = end_value - v0;
  const u32 have = left < u32(kWaveBlocks * kBlockValues) ? u32(left) : u32(kWaveBlocks * kBlockValues);     // values of the wave
  const u32 whole = have & ~3u;
  const __amdgpu_buffer_rsrc_t to = bytes_from(out, 4u * whole);      // (whole 16-byte pieces)
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    if ((lane >> 5) == hh) {
#pragma unroll
      for (int t = 0; t < 8; ++t)
        *reinterpret_cast<float4*>(wl + (lane & 31) * kStageRow + 4 * t) =
            make_float4(x[4 * t], x[4 * t + 1], x[4 * t + 2], x[4 * t + 3]);
    }
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x4_t v = *reinterpret_cast<const u32x4_t*>(wl + (8 * i + (lane >> 3)) * kStageRow + 4 * (lane & 7));
      __builtin_amdgcn_raw_buffer_store_b128(v, to, 16 * lane + 4096 * hh + 1024 * i, 0, kAccessOnce);
    }
    if (have != whole && int(whole >> 10) == hh) {     // uniform: the values behind the last piece
      const u32 at = whole + u32(lane);
      if (at < have) reinterpret_cast<u32*>(out)[at] = wl[((at & 1023u) >> 5) * kStageRow + (at & 31u)];
    }
    wave_lds_sync();
  }
}

template <bool IX, bool SELF, bool AVERAGE, typename... A>
__global__ __launch_bounds__(kTileThreads, 5) void decompress_kernel(const u8* base, u64 bytes, DecompressArgs a, A... answer) {
  __shared__ __attribute__((aligned(16))) u32 lds[kTileWaves * kWaveStage];
  __shared__ PlainSurvey<1> survey;
  const AnswerAtEnd<DecompressArgs, A...> at_end(a, answer...);
  const StreamRef in{base, bytes};           // (what the first loads need, see CompressInput)
  decompress_tile<IX, SELF, 1>(&in, 1, 0, a.out, a.out_cap_elems, a.index, a.ctl, a.nonce, lds, &survey, AVERAGE);
}

// A part of a stream (see decompress_tile).
template <bool IX, bool SELF>
__global__ __launch_bounds__(kTileThreads, 5) void decompress_range_kernel(DecompressArgs a) {
  __shared__ __attribute__((aligned(16))) u32 lds[kTileWaves * kWaveStage];
  __shared__ PlainSurvey<1> survey;
  decompress_tile<IX, SELF, 1>(&a.in, 1, 0, a.out, a.out_cap_elems, a.index, a.ctl, a.nonce, lds, &survey, false,
                         a.first_value, a.count);
}

// k streams in one launch (the tail of the compressed Allgather, Section 3.5.1: every rank
// decompresses all the chunks it has received): blockIdx.y = stream, blockIdx.x = tile.
struct DecompressManyArgs {
  StreamRef in[ZC_MAX_K];
  float* out[ZC_MAX_K];
  u64 out_cap_elems[ZC_MAX_K];
  int k;
  StreamIndex index;
  Control* ctl;
  u64 nonce;
};

template <bool IX, bool SELF, bool ROWS, typename... A>
__global__ __launch_bounds__(kTileThreads, 5) void decompress_many_kernel(DecompressManyArgs a, A... answer) {
  __shared__ __attribute__((aligned(16))) u32 lds[kTileWaves * kWaveStage];
  __shared__ PlainSurvey<ZC_MAX_K> survey;
  const AnswerAtEnd<DecompressManyArgs, A...> at_end(a, answer...);
  const int s = blockIdx.y;
  decompress_tile<IX, SELF, ZC_MAX_K, ROWS>(a.in, a.k, s, a.out[s], a.out_cap_elems[s], a.index, a.ctl, a.nonce, lds, &survey);
}

}  // namespace zc
