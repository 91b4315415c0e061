"""The server's dispatcher while a batch is out, on the CPU: the program's own HIP
functions run nothing and report each batch finished three milliseconds after it
was recorded."""
from tests._native import run_host

PROGRAM = r"""
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <thread>
#include "internal.h"

using Clock = std::chrono::steady_clock;
static std::atomic<int> yields{0}, early_polls{0}, polls{0};
static Clock::time_point recorded;
static std::atomic<bool> out{false};

extern "C" {
int sched_yield() { ++yields; return 0; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 163840;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { recorded = Clock::now(); out = true; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) {
  const auto age = Clock::now() - recorded;
  ++polls;
  if (age < std::chrono::microseconds(500)) ++early_polls;
  return age < std::chrono::milliseconds(3) ? hipErrorNotReady : hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = dim3(1); *b = dim3(1); *m = 0; *s = nullptr;
  return hipSuccess;
}
}

int main() {
  aiwc_rf_forest f;
  f.n_cols = 4;
  f.params.push_back({5, 2, 1, 1, 1});
  f.first_task.push_back(0);
  f.n_train.push_back(100);
  uint32_t ok = 0;
  f.status_host = &ok;
  f.waited = true;
  aiwc_rf_server* s = nullptr;
  if (aiwc_rf_server_create(&f, 0, 1 << 16, 64, 1, &s) != 0) { std::printf("create: %s\n", aiwc_rf_last_error()); return 1; }
  uint8_t codes[4] = {1, 2, 3, 4};
  double y = 0.0;
  int64_t ticket = -1;
  int rc = 0;
  for (int i = 0; i < 3 && rc == 0; ++i) {
    rc = aiwc_rf_server_submit(s, codes, 1, &y, &ticket);
    if (rc == 0) rc = aiwc_rf_server_drain(s);
  }
  int64_t rows = 0;
  aiwc_rf_server_stats(s, &rows, nullptr, nullptr, nullptr);
  const int y_n = yields, p = polls, e = early_polls;
  aiwc_rf_server_free(s);
  std::printf("%d %d %d %d %d\n", rc, (int)rows, y_n, e, p);
}
"""


def test_dispatcher_sleeps_between_polls(tmp_path):
    rc, rows, yields, early, polls = map(int, run_host(tmp_path, PROGRAM).split())
    assert (rc, rows) == (0, 3)
    # never gives its CPU away, and looks often while a batch may finish any moment:
    # 3 x 100 looks at most in the first half millisecond, fewer on a busy machine
    assert yields == 0 and early >= 3
    # 3 x (100 + 125) sleeps of 5 and 20 us at most, and no busy loop
    assert polls <= 3 * (100 + 125) + 30
