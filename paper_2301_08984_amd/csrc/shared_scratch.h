// Device scratch that the library itself holds, one buffer per GPU, for calls that are faster with
// more scratch than their caller hands over (defined in api.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>

namespace ssa {

constexpr size_t SHARED_BYTES = 64u << 20, SHARED_HALF = SHARED_BYTES / 2;
constexpr int SHARED_COUNTERS = 512;  // of the second half; zero whenever no kernel that uses them is running

// Two halves with a user each, so that a call that needs one leaves the other: forwards of pair and window attention, whose copy
// of the bias goes into the first, do not keep split contractions or the chunks of a small share on another stream from
// running together.  (A whole buffer for one user: beside a forward of 512 windows of 12 x 12 x 8 heads on another stream the backward of 18 rows x
// 8 heads x 472, k = 16, was done after 796 us instead of 156, that of 12 heads x 2048, k = 4, after 289 instead of 183.)
enum SharedPart { SHARED_FIRST = 1, SHARED_SECOND = 2, SHARED_BOTH = 3 };

struct Shared {
  std::mutex init;
  char* ptr = nullptr;
  unsigned* counters = nullptr;
  hipEvent_t done[4] = {};  // end of the last call that used the halves [parts]
  bool broken = false;
  struct Half {
    std::mutex mu;
    int last = 0;                  // which of `done` the last call recorded
    hipStream_t stream = nullptr;  // its stream
  } half[2];
};

// One stream uses a half at a time.  A call takes it if it is on the stream of the last call that had
// it (stream order keeps them apart) or if that call's work has finished; any other call, and any call
// that is being captured into a graph (a replay is ordered after nothing that the host can see), does
// without.  Nothing ever waits for the buffer.  The lock, one per GPU and half, is held from the moment the half is
// taken until the call's launches are enqueued: threads that drive different GPUs do not meet.
class SharedUse {
 public:
  // the buffer from the first of `parts` on, or NULL if this call has to do without; once per object, again only after a NULL
  char* take(hipStream_t stream, int parts = SHARED_BOTH);
  unsigned* counters() const { return parts_ & SHARED_SECOND ? s_->counters : nullptr; }
  SharedUse() = default;
  SharedUse(const SharedUse&) = delete;
  ~SharedUse();

 private:
  std::unique_lock<std::mutex> lock_[2];
  Shared* s_ = nullptr;
  int parts_ = 0;
  hipStream_t st_ = nullptr;
};

}  // namespace ssa
