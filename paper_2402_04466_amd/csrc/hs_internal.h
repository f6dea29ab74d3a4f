// Internal declarations shared by the host-side translation units of libhs.
#pragma once

#include <stdint.h>
#include <stdio.h>
#include <time.h>

#include <algorithm>
#include <chrono>

#include <exception>
#include <new>

#include "hs.h"

namespace hs {

// printf-style; stores the message returned by hs_last_error() for the calling thread.
void set_error(const char* fmt, ...) __attribute__((format(printf, 1, 2)));

// XCDs (dies with an L2 of their own, 32 CUs each) of a device with that many CUs.
int xcd_count(int device_cus);

// Admission predicate of the spatial partitions (paper Section IV-A, "Admission Control"):
// HS_E_OVERSUBSCRIBED for an empty mask, a CU the device does not have or a CU claimed by
// another application; HS_E_INVAL for bad arguments or a mask without a CU on every XCD.
hs_status admission_check(const uint32_t* claimed, const uint32_t* req_a, const uint32_t* req_b,
                          int n_words, int device_cus);

inline uint64_t now_ns() {
  timespec ts;
  clock_gettime(CLOCK_MONOTONIC, &ts);
  return (uint64_t)ts.tv_sec * 1000000000ull + (uint64_t)ts.tv_nsec;
}
// A deadline on that clock, which is the steady_clock's, and as its time point.  Neither a time-out nor
// a deadline beyond the clock's range (UINT64_MAX: wait for good) wraps around.
inline uint64_t deadline_after(uint64_t timeout_ns) {
  return now_ns() + std::min<uint64_t>(timeout_ns, (uint64_t)INT64_MAX / 2);
}
inline std::chrono::steady_clock::time_point clock_time(uint64_t t_ns) {
  return std::chrono::steady_clock::time_point(std::chrono::nanoseconds((int64_t)t_ns));
}

// An error text that can be kept where no memory is to be had.
struct Message {
  char text[512] = "";
  bool empty() const { return text[0] == 0; }
  void set(const char* a, const char* b = "", const char* c = "") { snprintf(text, sizeof(text), "%s%s%s", a, b, c); }
};

// No C++ exception may cross the C boundary: calls that allocate host memory or start threads
// run inside this guard.
template <class F>
hs_status guarded(const char* fn, F&& body) {
  try {
    return body();
  } catch (const std::bad_alloc&) {
    set_error("%s: out of host memory", fn);
    return HS_E_NOMEM;
  } catch (const std::exception& e) {
    set_error("%s: %s", fn, e.what());
    return HS_E_DEVICE;
  }
}

}  // namespace hs

// What the per-stream front (hs_mux) must know of the application it drives.
int hs_internal_app_batch(const hs_app* app);      // streams per submit
int hs_internal_app_grouped(const hs_app* app);    // 1 while a member of a group
// The calling thread's current device (-1: unknown), which every call here may change.
int hs_internal_current_device();
void hs_internal_use_device(int device);

