// Who gets the library's scratch (shared_scratch.h), on a made-up HIP runtime: devices, streams and events are
// numbers, and the events are done when this file says so.  api.hip is compiled for the host alone and linked
// against the functions below instead of the runtime.
#include <atomic>
#include <cstdio>
#include <set>
#include <thread>

#include "../../paper_2301_08984_amd/csrc/shared_scratch.h"

static thread_local int t_device = 0;
static std::atomic<bool> g_capturing{false}, g_done{true};
static std::atomic<int> g_waits{0}, g_records{0};
static char g_symbols[8][4][64];  // device x symbol
static std::set<const void*> g_names;

extern "C" {
hipError_t hipGetDevice(int* d) { *d = t_device; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "made up"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* name) {
  g_names.insert(name);
  *p = g_symbols[t_device][std::distance(g_names.begin(), g_names.find(name))];
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)(intptr_t)(100 + t_device); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return g_done ? hipSuccess : hipErrorNotReady; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { ++g_waits; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { ++g_records; return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
}

static int failed = 0;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); failed = 1; } } while (0)

int main() {
  const hipStream_t s1 = (hipStream_t)1, s2 = (hipStream_t)2;
  {
    ssa::SharedUse a;
    CHECK(a.take(s1) != nullptr && a.counters() != nullptr);
    // held: another call on this GPU does without, one on another GPU has a buffer of its own
    std::thread([&] {
      ssa::SharedUse same;
      CHECK(same.take(s1) == nullptr && same.counters() == nullptr);
      t_device = 1;
      ssa::SharedUse other;
      CHECK(other.take(s2) != nullptr && other.counters() != nullptr);
    }).join();
  }
  CHECK(g_records == 2);
  // given back: the same stream takes it again (ordered after the last call), another one once that is done
  g_done = false;
  { ssa::SharedUse a; CHECK(a.take(s1) != nullptr); }
  CHECK(g_waits == 1);
  { ssa::SharedUse a; CHECK(a.take(s2) == nullptr); }
  g_done = true;
  { ssa::SharedUse a; CHECK(a.take(s2) != nullptr); }
  {  // halves: a user each, and none for a call that wants both
    ssa::SharedUse a, b, c;
    char* first = a.take(s1, ssa::SHARED_FIRST);
    CHECK(first != nullptr && a.counters() == nullptr);
    std::thread([&] {
      CHECK(c.take(s2) == nullptr && c.take(s2, ssa::SHARED_FIRST) == nullptr);
      CHECK(b.take(s2, ssa::SHARED_SECOND) == first + ssa::SHARED_HALF && b.counters() != nullptr);
    }).join();
  }
  g_done = false;  // a half that another stream's call used last keeps the other one free, and one's own stream has it
  { ssa::SharedUse a; CHECK(a.take(s1) == nullptr); }
  { ssa::SharedUse a; CHECK(a.take(s1, ssa::SHARED_FIRST) != nullptr); }
  { ssa::SharedUse a; CHECK(a.take(s2, ssa::SHARED_FIRST) == nullptr && a.take(s2, ssa::SHARED_SECOND) != nullptr); }
  g_done = true;
  { ssa::SharedUse a; CHECK(a.take(s1) != nullptr); }
  g_done = false;
  { ssa::SharedUse a; CHECK(a.take(s2, ssa::SHARED_SECOND) == nullptr); }
  g_done = true;
  g_capturing = true;
  { ssa::SharedUse a; CHECK(a.take(s2) == nullptr); }
  g_capturing = false;
  t_device = 63 + 1;  // more devices than the library counts
  { ssa::SharedUse a; CHECK(a.take(s1) == nullptr); }
  if (!failed) std::printf("all checks passed\n");
  return failed;
}
