// The host side of a synchronous call's answer (csrc/zc_report_slots.h) with the runtime's calls replaced: each
// check below prints its name before it runs and the program ends with 1 at the first that does not hold.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../../paper_2502_18554_amd/csrc/zc_report_slots.h"

static int pins_to_refuse = 0, pins = 0, copies = 0, syncs = 0;
static hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
static hipError_t capture_query = hipSuccess, pending = hipSuccess, sync_result = hipSuccess;
static void (*at_sync)() = nullptr;       // what the GPU does while the host waits for the stream
extern "C" {
hipError_t hipHostMalloc(void** p, size_t size, unsigned int) {
  ++pins;
  if (pins_to_refuse > 0) return --pins_to_refuse, hipErrorOutOfMemory;
  *p = std::calloc(1, size);
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = pending;
  return pending = hipSuccess, e;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  ++syncs;
  if (at_sync) at_sync();
  if (sync_result != hipSuccess) return sync_result;
  return capturing == hipStreamCaptureStatusNone ? hipSuccess : hipErrorStreamCaptureUnsupported;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { return *s = capturing, capture_query; }
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t) {
  ++copies;
  std::memcpy(to, from, n);
  return hipSuccess;
}
}

#define CHECK(c) do { if (!(c)) { std::printf("does not hold (line %d): %s\n", __LINE__, #c); return 1; } } while (0)

int main() {
  const uint64_t words[5] = {11, 22, 33, 44, 55};
  const uint64_t* from[5] = {words, words + 1, words + 2, words + 4, words + 3};
  uint64_t to[5];
  int launches = 0;
  auto runs = [&](zc::ReportSlot* s, uint64_t seq) {
    ++launches;
    for (int i = 0; i < 5; ++i) s->words[i] = *from[i];
    return __atomic_store_n(&s->seq, seq, __ATOMIC_RELEASE), true;
  };
  auto fails = [&](zc::ReportSlot*, uint64_t) { return ++launches, false; };
  // the next request is answered through a slot, and with the right words
  auto answered = [&](zc::ReportSlots& slots) {
    std::memset(to, 0, sizeof(to));
    const int before = launches, copies_before = copies;
    const bool ok = zc::report_words(slots, from, 5, to, true, nullptr, runs);
    return ok && launches == before + 1 && copies == copies_before && to[0] == 11 && to[1] == 22 && to[2] == 33 && to[3] == 55 && to[4] == 44;
  };

  std::printf("a launch that fails gives its slot back\n");
  {
    zc::ReportSlots slots;
    for (int i = 0; i < 100; ++i) CHECK(!zc::report_words(slots, from, 5, to, true, nullptr, fails));
    CHECK(answered(slots));
  }
  std::printf("a stream that is being captured gets no request, and costs no slot\n");
  {
    zc::ReportSlots slots;
    for (const hipStreamCaptureStatus s : {hipStreamCaptureStatusActive, hipStreamCaptureStatusInvalidated}) {
      capturing = s;
      const int before = launches, syncs_before = syncs;
      for (int i = 0; i < 100; ++i) CHECK(!zc::report_words(slots, from, 5, to, true, nullptr, runs));
      CHECK(launches == before && syncs == syncs_before + 100);
    }
    capturing = hipStreamCaptureStatusNone;
    CHECK(answered(slots));
  }
  std::printf("a stream whose state is not told goes by copies\n");
  {
    zc::ReportSlots slots;
    capture_query = hipErrorStreamCaptureImplicit;
    const int before = launches;
    std::memset(to, 0, sizeof(to));
    CHECK(zc::report_words(slots, from, 5, to, true, nullptr, runs) && launches == before && to[2] == 33 && to[3] == 55);
    capture_query = hipSuccess;
    CHECK(answered(slots));
  }
  std::printf("more requests at a time than slots go by copies\n");
  {
    zc::ReportSlots slots;
    zc::ReportSlot* held[32];
    for (auto& s : held) CHECK((s = slots.take(true)) != nullptr);
    const int before = launches;
    CHECK(zc::report_words(slots, from, 5, to, true, nullptr, runs) && launches == before && to[4] == 44);
    slots.give_back(held[7]);
    CHECK(answered(slots));
  }
  std::printf("pinned memory that was refused is asked for again\n");
  {
    zc::ReportSlots slots;
    pins_to_refuse = 3;
    const int before = launches;
    for (int i = 0; i < 3; ++i) {
      std::memset(to, 0, sizeof(to));
      CHECK(zc::report_words(slots, from, 5, to, true, nullptr, runs) && to[0] == 11 && to[3] == 55);
    }
    CHECK(launches == before && pins_to_refuse == 0);
    CHECK(answered(slots));
  }
  std::printf("a caller who rules out allocations gets none\n");
  {
    zc::ReportSlots slots;
    const int before = pins;
    CHECK(zc::report_words(slots, from, 5, to, false, nullptr, runs) && pins == before && to[0] == 11);
    CHECK(answered(slots));
    CHECK(zc::report_words(slots, from, 5, to, false, nullptr, runs) && pins == before + 1);
  }

  // The answers of codec calls: status bits under the call's tag, the size, and n of the streams.
  const uint64_t status = (uint64_t(7) << 32) | 6, tag = uint64_t(7) << 32, other_tag = uint64_t(8) << 32, size = 4711, ns[3] = {1, 0, uint64_t(1) << 31};
  const uint64_t* const own[3] = {&status, &tag, &size};
  const uint64_t* const more[3] = {ns, ns + 1, ns + 2};
  const uint64_t want[5] = {6, 4711, 1, 0, uint64_t(1) << 31};
  auto store = [](zc::ReportSlot* s, int i, uint64_t w) { __atomic_store_n(&s->words[i], w | zc::kAnswered, __ATOMIC_RELEASE); };
  auto right = [&](int count) { return std::memcmp(to, want, sizeof(uint64_t) * count) == 0; };
  auto answers = [&](zc::ReportSlot* s) {
    ++launches;
    for (int i : {3, 0, 4, 2, 1}) store(s, i, want[i]);      // in any order
    return true;
  };
  auto no_answer = [&](zc::ReportSlot*) { return ++launches, false; };
  // the next call is answered through a slot, and with the right words
  auto told = [&](zc::ReportSlots& slots) {
    std::memset(to, 0xff, sizeof(to));
    const int before = launches, copies_before = copies;
    return zc::fetch_answer(slots, own, more, 3, to, true, nullptr, answers) && launches == before + 1 && copies == copies_before && right(5);
  };

  std::printf("an answer has none of the marks its words come with\n");
  {
    zc::ReportSlots slots;
    CHECK(told(slots));
    CHECK(told(slots));       // (through the same place, which still holds the marked words of the answer before)
  }
  std::printf("an answer is waited for to its last word, whichever that is\n");
  {
    zc::ReportSlots slots;
    for (int late = 0; late < 5; ++late) {
      CHECK(told(slots));     // (whose words are still there)
      static zc::ReportSlot* slot;
      static int which;
      static uint64_t word;
      which = late, word = want[late];
      const int syncs_before = syncs;
      at_sync = [] { __atomic_store_n(&slot->words[which], word | zc::kAnswered, __ATOMIC_RELEASE); };
      std::memset(to, 0xff, sizeof(to));
      CHECK(zc::fetch_answer(slots, own, more, 3, to, true, nullptr, [&](zc::ReportSlot* s) {
        slot = s;
        for (int i = 0; i < 5; ++i)
          if (i != late) store(s, i, want[i]);
        return true;
      }));
      at_sync = nullptr;
      CHECK(syncs == syncs_before + 1 && right(5));
    }
  }
  std::printf("an answer that does not come is no answer, and its place is not given to another\n");
  {
    zc::ReportSlots slots;
    zc::ReportSlot* lost = nullptr;
    auto all_but_the_size = [&](zc::ReportSlot* s) {
      lost = s;
      for (int i : {0, 2, 3, 4}) store(s, i, want[i]);
      return true;
    };
    CHECK(!zc::fetch_answer(slots, own, more, 3, to, true, nullptr, all_but_the_size));
    zc::ReportSlot* held[32] = {};
    int got = 0;
    while (got < 32 && (held[got] = slots.take(true)) != nullptr) CHECK(held[got++] != lost);
    CHECK(got == 31);
  }
  std::printf("a stream that fails has no answer\n");
  {
    zc::ReportSlots slots;
    sync_result = hipErrorUnknown;
    CHECK(!zc::fetch_answer(slots, own, more, 3, to, true, nullptr, [](zc::ReportSlot*) { return true; }));
    sync_result = hipSuccess;
    CHECK(told(slots));
  }
  std::printf("an answer's launch that fails gives its place back\n");
  {
    zc::ReportSlots slots;
    for (int i = 0; i < 100; ++i) CHECK(!zc::fetch_answer(slots, own, more, 3, to, true, nullptr, no_answer));
    CHECK(told(slots));
  }
  std::printf("an error still to be told is told ahead of a launch, and costs no place\n");
  {
    zc::ReportSlots slots;
    const int before = launches;
    for (int i = 0; i < 100; ++i) {
      pending = hipErrorInvalidValue;
      CHECK(!zc::fetch_answer(slots, own, more, 3, to, true, nullptr, answers) && pending == hipSuccess);
    }
    CHECK(launches == before && told(slots));
  }
  std::printf("an answer by copies, which is no launch, does not mind such an error\n");
  {
    zc::ReportSlots slots;
    for (int i = 0; i < 32; ++i) CHECK(slots.take(true) != nullptr);
    const int before = launches;
    for (const hipError_t e : {hipSuccess, hipErrorInvalidValue}) {
      pending = e;
      std::memset(to, 0xff, sizeof(to));
      CHECK(zc::fetch_answer(slots, own, more, 3, to, true, nullptr, answers) && launches == before && right(5));
    }
    pending = hipSuccess;
    const uint64_t* const of_another[3] = {&status, &other_tag, &size};      // status bits of an earlier call
    CHECK(zc::fetch_answer(slots, of_another, more, 3, to, true, nullptr, answers) && to[0] == 0 && to[1] == 4711);
  }
  std::printf("a call on a stream that is being captured has no answer, and costs no place\n");
  {
    zc::ReportSlots slots;
    capturing = hipStreamCaptureStatusActive;
    const int before = launches;
    for (int i = 0; i < 100; ++i) CHECK(!zc::fetch_answer(slots, own, more, 3, to, true, nullptr, answers));
    capturing = hipStreamCaptureStatusNone;
    CHECK(launches == before && told(slots));
  }
  std::printf("a caller who rules out allocations gets an answer by copies\n");
  {
    zc::ReportSlots slots;
    const int before = launches, pins_before = pins;
    std::memset(to, 0xff, sizeof(to));
    CHECK(zc::fetch_answer(slots, own, nullptr, 0, to, false, nullptr, answers) && launches == before && pins == pins_before && right(2));
  }
  std::printf("ok\n");
  return 0;
}
