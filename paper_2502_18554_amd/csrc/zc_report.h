// How a synchronous call gets its few result words (status and size, or a handful of sums) back to the host.
//
// What bounds it: nothing but latency.  A copy to ordinary host memory goes through the runtime's staging
// buffer and is followed by a wait for the stream: 22 us from launch to answer for a kernel that does nothing,
// 15 us with pinned memory, 11 us for that kernel and the wait alone.  Here a kernel of one wave, ordered
// behind the call's kernels on their stream, reads the words and stores them into pinned host memory that the calling thread polls: 9 us with a number behind
// them that says they are there, which the kernel can store only when they have arrived (0.8 us later), and 8.5 with that said by a bit of every word.  (A compress and a
// decompress call of 5120 values, each waited for: 57.3 us, then 27.9; 23.1 when one workgroup answered for itself, see below, now 22.9.
// A waited ring round of 262 177 values 17.2, now 16.4.)
#pragma once

#include <hip/hip_runtime.h>

#include "zc_common.h"
#include "zc_report_slots.h"
#include "zc_scan.h"

namespace zc {

// Without that kernel, for a call of one workgroup: it stores the words itself when it is done (a compress and a decompress
// call of 5120 values, each waited for, 25.9 us with two launches of the kernel above, 23.4 without).  What it has written has to be
// where the next reader finds it by then, whatever stream that runs on, so it is released to the system first, as the end of a kernel
// does.  With more workgroups each of them would have to do so, and they take turns at it: 33 of them and a count of those that are
// done 19.0 us where the kernel above takes 16.5, 512 of them 88.
struct Answer {
  ReportSlot* to;           // null: nobody waits, or by a kernel of its own
};

// A call's answer as its words go over: status (bits count only under the tag of the last call) and size, and then values of n.
__device__ __forceinline__ u64 answer_word(const Control* ctl, u32 i) {
  const u64 w = __hip_atomic_load(i ? &ctl->result : &ctl->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const u64 tag = __hip_atomic_load(&ctl->call_tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return i ? w : (w >> 32) == (tag >> 32) ? u64(u32(w)) : 0ull;
}
__device__ __forceinline__ void store_answer_word(ReportSlot* to, u32 i, u64 w) {
  __hip_atomic_store(&to->words[i], w | kAnswered, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// N: room for that many values of n (1, or all: the arguments travel with every launch).
template <int N>
struct CallReportArgs {
  const Control* ctl;
  ReportSlot* to;
  u32 count;
  const u64* more[N];
};
template <int N>
__global__ __launch_bounds__(128) void call_report_kernel(CallReportArgs<N> a) {
  static_assert(N + 2 <= 128, "a thread per word");
  if (threadIdx.x < 2) store_answer_word(a.to, threadIdx.x, answer_word(a.ctl, threadIdx.x));
  else if (threadIdx.x < 2 + a.count) store_answer_word(a.to, threadIdx.x, *a.more[threadIdx.x - 2]);
}

template <int N>
inline bool launch_call_report(ReportSlot* slot, const Control* ctl, const u64* const* more, u32 count, hipStream_t stream) {
  CallReportArgs<N> a;
  a.ctl = ctl;
  a.to = slot;
  a.count = count;
  for (u32 i = 0; i < count; ++i) a.more[i] = more[i];
  hipLaunchKernelGGL(call_report_kernel<N>, dim3(1), dim3(N + 2 <= 64 ? 64 : 128), 0, stream, a);
  return hipGetLastError() == hipSuccess;
}

// Words of any value, the four sums of zc_quality: a number behind them says that they are there.
constexpr int kSumWords = 4;
struct ReportArgs {
  const u64* from[kSumWords];
  u32 count;
  ReportSlot* to;
  u64 seq;
};
__global__ __launch_bounds__(64) void report_kernel(ReportArgs a) {
  if (threadIdx.x < a.count)
    __hip_atomic_store(&a.to->words[threadIdx.x], *a.from[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  // (what the call has written was released at its kernel's end, and these words go past the caches: all that is missing is that they have
  // arrived before the number goes out.  A fence and a releasing store in this place made an answer 0.6 us later by itself.)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(&a.to->seq, a.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The words at from[0 .. count), at most kSumWords, as they are when everything enqueued on `stream` so far has run.  `make`: the slots may be
// pinned now.
inline bool report_words(ReportSlots& slots, const u64* const* from, u32 count, u64* to, bool make, hipStream_t stream) {
  return report_words(slots, from, count, to, make, stream, [&](ReportSlot* slot, u64 seq) {
    ReportArgs a;
    for (u32 i = 0; i < count; ++i) a.from[i] = from[i];
    a.count = count;
    a.to = slot;
    a.seq = seq;
    hipLaunchKernelGGL(report_kernel, dim3(1), dim3(64), 0, stream, a);
    return hipGetLastError() == hipSuccess;
  });
}

// The end of a main kernel, called by all its threads.
// heads, k: the streams whose n (the second word of a header) follow the call's own words.
__device__ __forceinline__ void give_answer(const Answer& an, const Control* ctl, const StreamRef* heads = nullptr, int k = 0) {
  if (!an.to) return;       // uniform
  // Every wave waits for its own stores and atomics first: a barrier orders LDS, and whether the compiler puts a wait for memory in front
  // of it differs from kernel to kernel; the words read below, and the output that the caller may read next, need it.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (wave_id() != 0) return;
  const int lane = lane_id();
  const u64 own = answer_word(ctl, lane == 0 ? 0u : 1u);
  const u64 n = lane < k ? reinterpret_cast<const u64*>(heads[lane].base)[1] : 0ull;
  __threadfence_system();
  if (lane < 2) store_answer_word(an.to, u32(lane), own);
  if (lane < k) store_answer_word(an.to, u32(2 + lane), n);
}

// The same for a kernel that has an instance for the calls that it answers, with an argument more (A = Answer), and one for all others (no A), in which this
// is nothing: what ends the kernel, wherever it returns.  With one instance, whose arguments said whether somebody
// waits, a Sum of one buffer of 2^20 values took 8.3 us, now 8.1, of 16 of them 12.9 and 12.6, a ring round of 2^24 values by ticket 40.1 and
// 38.3, and a decompression of 2^24 values 14.9 and 14.8.  (One instance for all calls have the compression, which takes 2 % longer on 3 to 4 million values with
// two, and the decompression of plain streams that are indexed ahead, which is level.  A compression and decompression of 20 000 003 values, plain, takes 46.9 us;
// with eight bytes more in Answer 47.5.)
template <typename Args, typename... A>
struct AnswerAtEnd {
  __device__ __forceinline__ AnswerAtEnd(const Args&) {}
};
template <typename Args>
struct AnswerAtEnd<Args, Answer> {
  const Args& a;
  const Answer& answer;
  __device__ __forceinline__ AnswerAtEnd(const Args& args, const Answer& an) : a(args), answer(an) {}
  __device__ __forceinline__ ~AnswerAtEnd() {
    if constexpr (requires { a.out_cap_elems[0]; }) give_answer(answer, a.ctl, a.in, a.k);      // (streams decompressed by one call)
    else give_answer(answer, a.ctl);
  }
};

}  // namespace zc
