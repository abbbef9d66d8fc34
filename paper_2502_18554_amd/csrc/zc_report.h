// How a synchronous call gets its few result words (status, tag, size) back to the host.
//
// What bounds it: nothing but latency.  A copy to ordinary host memory goes through the runtime's staging
// buffer and is followed by a wait for the stream: 22 us from launch to answer for a kernel that does nothing,
// 15 us with pinned memory, 11 us for that kernel and the wait alone.  Here a kernel of one wave, ordered
// behind the call's kernels on their stream, reads the words and stores them, and then a number that only
// this request has, into pinned host memory that the calling thread polls: 9 us.  (A compress and a
// decompress call of 5120 values, each waited for: 58.7 -> 33.9 us.)
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <mutex>

#include "zc_common.h"

namespace zc {

constexpr int kReportWords = 4 + ZC_MAX_K;      // status, tag and size of a call (or the four quality sums), and k values of n

// A request's place in pinned memory.
struct ReportSlot {
  u64 seq;                     // the request whose words these are
  u64 words[kReportWords];
};

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

// The slots: a fixed number of them, taken for the length of one request and given back, so that threads and
// streams never share one.  Pinned when the first is asked for, and until the process ends.
class ReportSlots {
 public:
  // Null when all are taken or there is no pinned memory (`make`: pin it now if that has not been done yet).
  ReportSlot* take(bool make) {
    std::lock_guard<std::mutex> g(mu_);
    if (!slots_) {
      if (!make || refused_) return nullptr;
      void* p = nullptr;
      if (hipHostMalloc(&p, sizeof(ReportSlot) * kSlots, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
        (void)hipGetLastError();
        refused_ = true;
        return nullptr;
      }
      slots_ = static_cast<ReportSlot*>(p);
      for (int i = 0; i < kSlots; ++i) slots_[i].seq = 0;
    }
    for (int i = 0; i < kSlots; ++i) {
      if (taken_ & (u64(1) << i)) continue;
      taken_ |= u64(1) << i;
      return slots_ + i;
    }
    return nullptr;
  }
  void give_back(ReportSlot* s) {
    std::lock_guard<std::mutex> g(mu_);
    taken_ &= ~(u64(1) << (s - slots_));
  }
  u64 next_seq() { return seq_.fetch_add(1, std::memory_order_relaxed) + 1; }

 private:
  static constexpr int kSlots = 32;
  std::mutex mu_;
  ReportSlot* slots_ = nullptr;
  u64 taken_ = 0;
  bool refused_ = false;
  std::atomic<u64> seq_{0};
};

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

// The words at from[0 .. count) as they are when everything enqueued on `stream` so far has run.  `make`: see take.
inline bool report_words(ReportSlots& slots, const u64* const* from, u32 count, u64* to, bool make, hipStream_t stream) {
  ReportSlot* const slot = slots.take(make);
  if (!slot) {
    for (u32 i = 0, run; i < count; i += run) {
      for (run = 1; i + run < count && from[i + run] == from[i] + run;) ++run;
      if (hipMemcpyAsync(to + i, from[i], run * sizeof(u64), hipMemcpyDeviceToHost, stream) != hipSuccess) return false;
    }
    return hipStreamSynchronize(stream) == hipSuccess;
  }
  const u64 seq = slots.next_seq();
  bool there = false;
  if (count <= 4 ? launch_report<4>(slot, seq, from, count, stream) : launch_report<kReportWords>(slot, seq, from, count, stream)) {
    // Polled for the length of a large call, then left to the runtime, which also knows
    // when no answer can come (a failed kernel, a stream that is being captured).
    const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(500);
    auto answered = [&] { return __atomic_load_n(&slot->seq, __ATOMIC_ACQUIRE) == seq; };
    for (u32 polls = 1; !(there = answered()); ++polls) {
      __builtin_ia32_pause();
      if ((polls & 63u) == 0 && std::chrono::steady_clock::now() > until) break;
    }
    if (!there) there = hipStreamSynchronize(stream) == hipSuccess && answered();
    if (there)
      for (u32 i = 0; i < count; ++i) to[i] = __atomic_load_n(&slot->words[i], __ATOMIC_RELAXED);
  }
  // (a request without an answer keeps its slot: what was enqueued may still write there)
  if (there) slots.give_back(slot);
  return there;
}

}  // namespace zc
