// Internal helpers shared by the library's translation units (error reporting, launch checks,
// workspace carving). Nothing here is exported.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>

#include "../../include/hgnn.h"

namespace hgnn {

int32_t set_error(int32_t code, const char* fmt, ...);

#define HGNN_REQUIRE(cond, code, ...)                         \
  do {                                                        \
    if (!(cond)) return ::hgnn::set_error((code), __VA_ARGS__); \
  } while (0)

#define HGNN_HIP(expr)                                                                      \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess)                                                                   \
      return ::hgnn::set_error(HGNN_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

#define HGNN_LAUNCH_CHECK(name)                                                             \
  do {                                                                                      \
    hipError_t e_ = hipGetLastError();                                                      \
    if (e_ != hipSuccess)                                                                   \
      return ::hgnn::set_error(HGNN_ERR_HIP, "launch of %s failed: %s", name,               \
                               hipGetErrorString(e_));                                      \
  } while (0)

#define HGNN_TRY(expr)            \
  do {                            \
    int32_t s_ = (expr);          \
    if (s_ != HGNN_OK) return s_; \
  } while (0)

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// What a device kernel hands to a waiting host call: one slot of pinned host memory, written by the kernel that has the
// result, so there is no copy behind it. The call waits for the stream all the same: it is documented to leave with
// every output written and every input read.
struct HostMail {
  long long value;
  int status;
  unsigned posted;
};
__device__ inline void post_mail(HostMail* m, long long value, int status) {
  m->value = value;
  m->status = status;
  __threadfence_system();
  __hip_atomic_store(&m->posted, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A slot taken from a process-wide list of MAIL_SLOTS for the duration of one call and given back at its end (defined in
// prof.hip; a call that finds all of them taken by others that are waiting is refused). Once a kernel
// has been handed the slot, it goes back only when the stream has drained, also where the call ends with an error in
// between: a post that comes late would otherwise land in the slot of another call.
class MailSlot {
 public:
  MailSlot() = default;
  ~MailSlot();
  MailSlot(const MailSlot&) = delete;
  MailSlot& operator=(const MailSlot&) = delete;
  int32_t take(hipStream_t st);   // st: the stream of the kernel that posts (not one under capture: it cannot be waited for)
  HostMail* dev() {
    lent_ = true;
    return m_;
  }
  hipError_t wait();   // until the stream has drained; an error if it fails, or drains with nothing posted
  long long value() const { return m_->value; }
  int status() const { return m_->status; }

 private:
  HostMail* m_ = nullptr;
  hipStream_t st_ = nullptr;
  bool lent_ = false;   // a kernel that was given the slot may still be to run
};

// Carves aligned sub-buffers out of a caller workspace; `used()` is what a size query reports.
struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* p) : base(static_cast<char*>(p)) {}
  template <typename T>
  T* take(size_t count) {
    T* r = reinterpret_cast<T*>(base ? base + off : nullptr);
    off += align_up(count * sizeof(T));
    return r;
  }
  size_t used() const { return off; }
};

inline bool valid_H(int H) { return H == 64 || H == 128 || H == 256; }

// compute units of the current device (asked once)
inline int num_cus() {
  static int n = 0;
  if (n == 0) {
    hipDeviceProp_t prop;
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
      n = prop.multiProcessorCount;
    if (n <= 0) n = 256;
  }
  return n;
}

// device-wide exclusive prefix sum of n int32 values; out has n+1 entries (out[n] = total).
// scratch must hold scan_scratch_ints(n) ints.
size_t scan_scratch_ints(int64_t n);
int32_t exclusive_scan_i32(hipStream_t st, const int32_t* in, int32_t* out, int64_t n, int32_t* scratch);

}  // namespace hgnn
