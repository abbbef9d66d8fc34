// Payloads of compressed operands on their way from memory straight to LDS, shared by the
// reduce kernels that keep several operands under way at once.
#pragma once

#include <utility>

#include "zc_common.h"
#include "zc_reduce.h"

namespace zc {

typedef __attribute__((address_space(3))) u32 LdsWord;

// Nothing moves across this line.
__device__ __forceinline__ void lds_words_line() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// What a wave needs to ask for its share of any operand, in lane s of operand s, worked out for all of them at once.
struct LaneOperands {
  u32 widths_lo, widths_hi;      // address of the width table
  u32 share_lo, share_hi;        // address of the 16-byte boundary at or below the segment's payload
  u32 room;                      // words from there to the end of the caller's buffer
  u32 shape;                     // words between the boundary and the segment's first word (2 bits), and above them, indexed streams, the segment's words
  u32 bytes;                     // indexed streams: whole 16-byte pieces to bring
  u64 tails;                     // indexed streams, bit s: there is more to bring (see fetch_payload_end)
};

// most: words of the longest segment, and three.
template <bool IX>
__device__ __forceinline__ LaneOperands lane_operands(const ReduceCall& c, u32 most = kMostStaged) {
  LaneOperands o;
  const u64 widths = c.base + c.widths;
  o.widths_lo = u32(widths);
  o.widths_hi = u32(widths >> 32);
  const u32 mis = c.places & 3u, src0 = c.places - mis, room = payload_room(c.bytes, c);
  const u64 share = c.base + c.payload + 4 * u64(src0);
  o.share_lo = u32(share);
  o.share_hi = u32(share >> 32);
  o.room = c.places <= room ? room - src0 : 0u;
  const u32 words = c.ends - c.places;
  const bool inside = IX && mis <= o.room && words <= o.room - mis && words <= most - 3u;
  o.shape = mis | (inside ? words : kNoWords) << 2;
  const u32 pieces = inside ? (mis + words + 3u) & ~3u : 0u, whole = min(pieces, o.room & ~3u);
  o.bytes = 4u * whole;
  o.tails = __ballot(inside && (pieces != whole || mis + words > 256u * kStageLoads));
  return o;
}

__device__ __forceinline__ const u32* lane_share(const LaneOperands& o, int s) {
  return reinterpret_cast<const u32*>(u64(lane_value(o.share_lo, s)) | (u64(lane_value(o.share_hi, s)) << 32));
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t lane_buffer(u32 lo, u32 hi, int s, u32 behind, u32 bytes) {
  const u64 at = (u64(lane_value(lo, s)) | (u64(lane_value(hi, s)) << 32)) + behind;
  return bytes_from(reinterpret_cast<const void*>(at), bytes);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t widths_buffer(const LaneOperands& o, const ReduceCall& c, int s, bool there) {
  return lane_buffer(o.widths_lo, o.widths_hi, s, 0u, there ? c.nb : 0u);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t outliers_buffer(const LaneOperands& o, const ReduceCall& c, int s, bool there) {
  return lane_buffer(o.widths_lo, o.widths_hi, s, c.firsts - c.widths, there ? 4u * c.nb : 0u);
}

// The payload of operand s for this wave (`bytes` of it, in whole 16-byte pieces) into `area`, by kStageLoads loads, which write 1024 words of it.
__device__ __forceinline__ void ask_payload_to_lds(const LaneOperands& o, int s, u32 bytes, u32* area, int lane) {
  const __amdgpu_buffer_rsrc_t share = lane_buffer(o.share_lo, o.share_hi, s, 0u, bytes);
#pragma unroll
  for (int i = 0; i < kStageLoads; ++i)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(share, (LdsWord*)(area + 256 * i), 16, 16 * lane + 1024 * i, 0, 0, kAccessOnce);
}

// What those loads have left out of `span` words, once they have landed: words from 1024 on, or the end of a buffer that ends inside a 16-byte piece.
__device__ __forceinline__ void fetch_payload_end(const LaneOperands& o, int s, u32 bytes, u32 span, u32* area, int lane) {
  const u32 from = min(bytes / 4u, 256u * kStageLoads) + u32(lane);
  if (from < min(span, lane_value(o.room, s)))
    area[from] = lane_share(o, s)[from];
}

// All vector memory accesses of the wave but the newest N are done.
template <int N>
__device__ __forceinline__ void wait_all_but() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

}  // namespace zc
