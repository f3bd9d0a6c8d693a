// The staging ring of tide_api.hip under threads, on the CPU: the host half of that file, linked
// with the HIP calls it makes and the kernel launches replaced by the functions below.
//
// A thread stages a small call and is held inside its kernel's launch while another makes more
// calls than the ring has slots.  The slot that the first has filled is read by no kernel yet, so
// with a waiting limit of 0 a call that takes the slot's turn would fail.  Then a launch that
// fails: nothing will read its slot, and the calls after it must not wait for it.
// Prints "ok", or what went wrong.
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <unistd.h>

#include <atomic>
#include <thread>

#include "kernels.h"
#include "tide.h"

static std::atomic<bool> hold{false}, held{false}, others_done{false}, fail_launch{false};

// ---- HIP, as far as tide_api.hip calls it ------------------------------------------------
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, uint3*, uint3*, dim3*, dim3*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipErrorUnknown; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorUnknown; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipErrorUnknown; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipErrorUnknown; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = hipStreamCaptureStatusNone;
  return hipSuccess;
}
}

// ---- launches: the append "kernel" sets its workgroups' flags -----------------------------
namespace tide {
int append_groups(int32_t num_kv_heads) { return (num_kv_heads + 3) / 4; }
int append_waves() { return 4; }
int decode_waves(int32_t) { return 4; }
hipError_t launch_extend(const ExtendArgs&, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_decode(const DecodeArgs&, int, bool, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_decode_stream(const StreamArgs&, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_kv_append(const AppendArgs& a, hipStream_t) {
  if (fail_launch.exchange(false)) return hipErrorUnknown;
  if (hold.exchange(false)) {
    held = true;
    for (int ms = 0; ms < 500 && !others_done; ++ms) usleep(1000);
  }
  if (!a.reads.done) return hipErrorUnknown;  // every call here is small enough to read in place
  for (int i = 0; i < a.num_items * append_groups(a.num_kv_heads); ++i) a.reads.done[i] = a.reads.seq;
  return hipSuccess;
}
}  // namespace tide

static int append() {
  static uint64_t mem[64];
  const int32_t prefix[1] = {0}, extend[1] = {1};
  const tide_dims dims = {4, 4, 64, 16, 0.125f};
  return tide_kv_append(mem, mem, mem, mem, 64, reinterpret_cast<const int32_t*>(mem), 64, 1, prefix,
                        extend, &dims, mem, 1 << 20, nullptr);
}

int main() {
  setenv("TIDE_STAGING_WAIT_US", "0", 1);
  unsetenv("TIDE_DEBUG_CHECKS");
  int bad = 0;
  hold = true;
  std::thread first([&] { bad += append() != TIDE_OK; });
  while (!held) usleep(100);
  for (int i = 0; i < 40 && !bad; ++i)
    if (append() != TIDE_OK) {
      printf("call %d beside a held launch failed\n", i);
      ++bad;
    }
  others_done = true;
  first.join();
  fail_launch = true;
  if (append() != TIDE_ERR_HIP) printf("a failed launch was not reported\n"), ++bad;
  for (int i = 0; i < 40 && !bad; ++i)
    if (append() != TIDE_OK) {
      printf("call %d after a failed launch failed\n", i);
      ++bad;
    }
  tide_shutdown();
  if (!bad) printf("ok\n");
  return bad != 0;
}
