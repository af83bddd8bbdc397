// Stream capture that ends on every way out of its scope.
#pragma once
#include <hip/hip_runtime.h>

namespace zr {

// Records what is enqueued on a stream from begin() to end().  The stream lives
// longer than the call that captures on it, so an exception between the two must
// not leave it capturing (every later begin() on it would fail): the destructor
// then ends the capture and drops what was recorded.
class StreamCapture {
 public:
  StreamCapture() = default;
  ~StreamCapture() {
    hipGraph_t g = nullptr;
    (void)end(&g);
    if (g) (void)hipGraphDestroy(g);
  }
  StreamCapture(const StreamCapture&) = delete;
  StreamCapture& operator=(const StreamCapture&) = delete;
  hipError_t begin(hipStream_t s) {
    const hipError_t e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
    s_ = s;
    on_ = e == hipSuccess;
    return e;
  }
  // The recorded graph, the caller's from here on; hipSuccess and null outside a capture.
  hipError_t end(hipGraph_t* g) {
    *g = nullptr;
    if (!on_) return hipSuccess;
    on_ = false;
    return hipStreamEndCapture(s_, g);
  }

 private:
  hipStream_t s_ = nullptr;
  bool on_ = false;
};

}  // namespace zr
