// The host side of zc_report.h: the places in pinned memory through which a synchronous call gets its result
// words, and the wait for them.
#pragma once

#include <hip/hip_runtime_api.h>

#include <atomic>
#include <chrono>
#include <cstdint>
#include <mutex>

#include "../../include/zc.h"

namespace zc {

constexpr int kReportWords = 4 + ZC_MAX_K;      // most words that a request is for: status, tag and size of a call, and k values of n

// A request's place in pinned memory.
struct ReportSlot {
  uint64_t seq;                     // the request whose words these are
  uint64_t words[kReportWords];
};

// The slots: a fixed number of them, taken for the length of one request and given back, so that threads and
// streams never share one.  Pinned when the first is asked for, and until the process ends.  Where that is refused (no
// memory to be had at the moment, another thread capturing a graph in the mode that forbids allocations to all) the
// request goes without and a later one asks again.
class ReportSlots {
 public:
  // Null when all are taken or there is no pinned memory (`make`: pin it now if that has not been done yet).
  ReportSlot* take(bool make) {
    std::lock_guard<std::mutex> g(mu_);
    if (!slots_) {
      if (!make) return nullptr;
      void* p = nullptr;
      if (hipHostMalloc(&p, sizeof(ReportSlot) * kSlots, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
      }
      slots_ = static_cast<ReportSlot*>(p);
      for (int i = 0; i < kSlots; ++i) slots_[i].seq = 0;
    }
    for (int i = 0; i < kSlots; ++i) {
      if (taken_ & (uint64_t(1) << i)) continue;
      taken_ |= uint64_t(1) << i;
      return slots_ + i;
    }
    return nullptr;
  }
  void give_back(ReportSlot* s) {
    std::lock_guard<std::mutex> g(mu_);
    taken_ &= ~(uint64_t(1) << (s - slots_));
  }
  uint64_t next_seq() { return seq_.fetch_add(1, std::memory_order_relaxed) + 1; }

 private:
  static constexpr int kSlots = 32;
  std::mutex mu_;
  ReportSlot* slots_ = nullptr;
  uint64_t taken_ = 0;
  std::atomic<uint64_t> seq_{0};
};

// Whether `stream` can be told to be running what is enqueued on it (not while it is being captured).
inline bool stream_runs(hipStream_t stream) {
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  const bool known = hipStreamIsCapturing(stream, &capture) == hipSuccess;
  if (!known) (void)hipGetLastError();
  return known && capture == hipStreamCaptureStatusNone;
}

// A call's answer: every word of it says by its highest bit that it is there (none of them needs that bit: a status, a size, and n of streams whose headers were all
// accepted, for with a malformed one among them a call answers FORMAT and no n is handed on), so that nothing has to be waited for between them and a last word.  The caller clears the slot's words before it is asked for, and has them all before it is
// given back.
constexpr uint64_t kAnswered = uint64_t(1) << 63;

inline void clear_answer(ReportSlot* slot, uint32_t count) {
  for (uint32_t i = 0; i < count; ++i) __atomic_store_n(&slot->words[i], uint64_t(0), __ATOMIC_RELAXED);
  __atomic_thread_fence(__ATOMIC_RELEASE);
}

// Waits for the `count` words of an answer, which something enqueued on `stream` stores in `slot`, and gives the slot back.
inline bool await_answer(ReportSlots& slots, ReportSlot* slot, uint32_t count, uint64_t* to, hipStream_t stream) {
  const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(500);      // (see await_words)
  uint32_t have = 0;
  auto answered = [&] {
    while (have < count && (__atomic_load_n(&slot->words[have], __ATOMIC_ACQUIRE) & kAnswered) != 0) ++have;
    return have == count;
  };
  bool there = false;
  for (uint32_t polls = 1; !(there = answered()); ++polls) {
    __builtin_ia32_pause();
    if ((polls & 63u) == 0 && std::chrono::steady_clock::now() > until) break;
  }
  if (!there) there = hipStreamSynchronize(stream) == hipSuccess && answered();
  if (!there) return false;      // (with its slot: what was enqueued may still write there, if the GPU comes to it)
  for (uint32_t i = 0; i < count; ++i) to[i] = __atomic_load_n(&slot->words[i], __ATOMIC_RELAXED) & ~kAnswered;
  slots.give_back(slot);
  return true;
}

// Waits for the answer to request `seq`, which something enqueued on `stream` stores in `slot`, and gives the slot back.
inline bool await_words(ReportSlots& slots, ReportSlot* slot, uint64_t seq, uint32_t count, uint64_t* to, hipStream_t stream) {
  // Polled for the length of a large call, then left to the runtime, which also knows when no answer can come.
  const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(500);
  auto answered = [&] { return __atomic_load_n(&slot->seq, __ATOMIC_ACQUIRE) == seq; };
  bool there = false;
  for (uint32_t polls = 1; !(there = answered()); ++polls) {
    __builtin_ia32_pause();
    if ((polls & 63u) == 0 && std::chrono::steady_clock::now() > until) break;
  }
  if (!there) there = hipStreamSynchronize(stream) == hipSuccess && answered();
  if (!there) return false;      // (with its slot: what was enqueued may still write there, if the GPU comes to it)
  for (uint32_t i = 0; i < count; ++i) to[i] = __atomic_load_n(&slot->words[i], __ATOMIC_RELAXED);
  slots.give_back(slot);
  return true;
}

// The words at from[0 .. count) as they are when everything enqueued on `stream` so far has run, by copies.
inline bool copy_words(const uint64_t* const* from, uint32_t count, uint64_t* to, hipStream_t stream) {
  // A stream that is being captured runs nothing, so there is no answer to wait for: the wait for the stream says so (and
  // ends the capture, as it does in any synchronous call).
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  const bool known = hipStreamIsCapturing(stream, &capture) == hipSuccess;
  if (!known) (void)hipGetLastError();
  if (known && capture != hipStreamCaptureStatusNone) {
    (void)hipStreamSynchronize(stream);
    return false;
  }
  for (uint32_t i = 0, run; i < count; i += run) {
    for (run = 1; i + run < count && from[i + run] == from[i] + run;) ++run;
    if (hipMemcpyAsync(to + i, from[i], run * sizeof(uint64_t), hipMemcpyDeviceToHost, stream) != hipSuccess) return false;
  }
  return hipStreamSynchronize(stream) == hipSuccess;
}

// A call's answer when everything enqueued on `stream` so far has run: its status and size, and then the `count` words at `more`, by something that stores them in a slot,
// or, where there is none, by copies.  own: the call's status, tag and size.  `make`: see take.
// launch(slot): enqueues on `stream` what stores the words in the slot; false: nothing was enqueued.
template <typename LaunchFn>
inline bool fetch_answer(ReportSlots& slots, const uint64_t* const (&own)[3], const uint64_t* const* more, uint32_t count, uint64_t* to, bool make,
                         hipStream_t stream, LaunchFn launch) {
  if (ReportSlot* const slot = stream_runs(stream) ? slots.take(make) : nullptr) {
    clear_answer(slot, 2 + count);
    // (An error of an earlier call still to be told could not be told from a failed launch: then the slot would be given back that is still written to.)
    if (hipGetLastError() != hipSuccess || !launch(slot)) {
      slots.give_back(slot);
      return false;
    }
    return await_answer(slots, slot, 2 + count, to, stream);
  }
  // no slot, or the stream is being captured, which copy_words knows how to say
  const uint64_t* from[kReportWords] = {own[0], own[1], own[2]};
  uint64_t words[kReportWords];
  for (uint32_t i = 0; i < count; ++i) from[3 + i] = more[i];
  if (!copy_words(from, 3 + count, words, stream)) return false;
  to[0] = (words[0] >> 32) == (words[1] >> 32) ? uint64_t(uint32_t(words[0])) : 0u;      // status bits count only under the tag of the last call
  for (uint32_t i = 0; i < 1 + count; ++i) to[1 + i] = words[2 + i];
  return true;
}

// Words by something that stores them in a slot, if there is one, or by copies.  `make`: see take.
// launch(slot, seq): enqueues on `stream` what stores the words, and then seq, in the slot; false: nothing was enqueued.
template <typename LaunchFn>
inline bool report_words(ReportSlots& slots, const uint64_t* const* from, uint32_t count, uint64_t* to, bool make, hipStream_t stream,
                         LaunchFn launch) {
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  const bool known = hipStreamIsCapturing(stream, &capture) == hipSuccess;
  if (!known) (void)hipGetLastError();
  ReportSlot* const slot = known && capture == hipStreamCaptureStatusNone ? slots.take(make) : nullptr;
  if (!slot) return copy_words(from, count, to, stream);
  const uint64_t seq = slots.next_seq();
  if (!launch(slot, seq)) {
    slots.give_back(slot);
    return false;
  }
  return await_words(slots, slot, seq, count, to, stream);
}

}  // namespace zc
