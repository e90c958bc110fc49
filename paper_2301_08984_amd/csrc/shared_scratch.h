// Device scratch that the library itself holds, one buffer per GPU, for calls that are faster with
// more scratch than their caller hands over (defined in api.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>

namespace ssa {

constexpr size_t SHARED_BYTES = 64u << 20;
constexpr int SHARED_COUNTERS = 512;  // zero whenever no kernel that uses them is running

struct Shared {
  std::mutex mu;
  void* ptr = nullptr;
  unsigned* counters = nullptr;
  hipEvent_t done = nullptr;     // end of the last call that used the buffer
  hipStream_t stream = nullptr;  // its stream
  bool used = false, broken = false;
};

// One stream uses the buffer at a time.  A call takes it if it is on the stream of the last call that had
// it (stream order keeps them apart) or if that call's work has finished; any other call, and any call
// that is being captured into a graph (a replay is ordered after nothing that the host can see), does
// without.  Nothing ever waits for the buffer.  The lock, one per GPU, is held from the moment the buffer is
// taken until the call's launches are enqueued: threads that drive different GPUs do not meet.
class SharedUse {
 public:
  // the buffer, or NULL if this call has to do without it
  void* take(hipStream_t stream);
  unsigned* counters() const { return s_ ? s_->counters : nullptr; }
  SharedUse() = default;
  SharedUse(const SharedUse&) = delete;
  ~SharedUse();

 private:
  std::unique_lock<std::mutex> lock_;
  Shared* s_ = nullptr;
  hipStream_t st_ = nullptr;
};

}  // namespace ssa
