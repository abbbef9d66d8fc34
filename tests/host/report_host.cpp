// The host side of a synchronous call's answer (csrc/zc_report_slots.h) with the runtime's calls replaced: each
// check below prints its name before it runs and the program ends with 1 at the first that does not hold.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../../paper_2502_18554_amd/csrc/zc_report_slots.h"

static int pins_to_refuse = 0, pins = 0, copies = 0, syncs = 0;
static hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
static hipError_t capture_query = hipSuccess;
extern "C" {
hipError_t hipHostMalloc(void** p, size_t size, unsigned int) {
  ++pins;
  if (pins_to_refuse > 0) return --pins_to_refuse, hipErrorOutOfMemory;
  *p = std::calloc(1, size);
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) {
  ++syncs;
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
  std::printf("ok\n");
  return 0;
}
