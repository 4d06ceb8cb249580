// Error handling shared by the host-side sources.
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>
#include <shared_mutex>
#include <stdexcept>
#include <string>

namespace ftcc {

struct HipError : std::runtime_error {
  using std::runtime_error::runtime_error;
};

#define FTCC_HIP(expr)                                                                              \
  do {                                                                                              \
    hipError_t _e = (expr);                                                                         \
    if (_e != hipSuccess)                                                                           \
      throw ::ftcc::HipError(std::string(#expr) + ": " + hipGetErrorString(_e) + " at " + __FILE__ + \
                             ":" + std::to_string(__LINE__));                                       \
  } while (0)

// An operation on the legacy stream fails while any thread captures a stream, and spoils the
// capture.  Contexts on several threads take turns: captures one at a time (a unique
// lock), legacy-stream operations in between (FTCC_LEGACY, shared).
inline std::shared_mutex& capture_mutex() {
  static std::shared_mutex m;
  return m;
}

#define FTCC_LEGACY(expr)                                            \
  do {                                                               \
    std::shared_lock<std::shared_mutex> _l(::ftcc::capture_mutex()); \
    FTCC_HIP(expr);                                                  \
  } while (0)

}  // namespace ftcc
