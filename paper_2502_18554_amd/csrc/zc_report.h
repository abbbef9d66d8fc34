// How a synchronous call gets its few result words (status, tag, size) back to the host.
//
// What bounds it: nothing but latency.  A copy to ordinary host memory goes through the runtime's staging
// buffer and is followed by a wait for the stream: 22 us from launch to answer for a kernel that does nothing,
// 15 us with pinned memory, 11 us for that kernel and the wait alone.  Here a kernel of one wave, ordered
// behind the call's kernels on their stream, reads the words and stores them, and then a number that only
// this request has, into pinned host memory that the calling thread polls: 9 us.  (A compress and a
// decompress call of 5120 values, each waited for: 57.3 us, now 27.9.)
#pragma once

#include <hip/hip_runtime.h>

#include "zc_common.h"
#include "zc_report_slots.h"

namespace zc {

// N: room for that many words (4, or all: the arguments travel with every launch).
template <int N>
struct ReportArgs {
  const u64* from[N];
  u32 count;
  ReportSlot* to;
  u64 seq;
};

template <int N>
__global__ __launch_bounds__(128) void report_kernel(ReportArgs<N> a) {
  static_assert(N <= 128, "a thread per word");
  if (threadIdx.x < a.count)
    __hip_atomic_store(&a.to->words[threadIdx.x], *a.from[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(&a.to->seq, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <int N>
inline bool launch_report(ReportSlot* slot, u64 seq, const u64* const* from, u32 count, hipStream_t stream) {
  ReportArgs<N> a;
  for (u32 i = 0; i < count; ++i) a.from[i] = from[i];
  a.count = count;
  a.to = slot;
  a.seq = seq;
  hipLaunchKernelGGL(report_kernel<N>, dim3(1), dim3(N <= 64 ? 64 : 128), 0, stream, a);
  return hipGetLastError() == hipSuccess;
}

// The words at from[0 .. count) as they are when everything enqueued on `stream` so far has run.  `make`: the slots may be
// pinned now.
inline bool report_words(ReportSlots& slots, const u64* const* from, u32 count, u64* to, bool make, hipStream_t stream) {
  return report_words(slots, from, count, to, make, stream, [&](ReportSlot* slot, u64 seq) {
    return count <= 4 ? launch_report<4>(slot, seq, from, count, stream) : launch_report<kReportWords>(slot, seq, from, count, stream);
  });
}

}  // namespace zc
