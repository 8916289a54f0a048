// Host check of csrc/host_slot.h against stand-ins for the HIP calls that it
// makes: when slots are given back, waited for and run out.
#include <stdio.h>
#include <stdlib.h>

#include "host_slot.h"

static int n_sync = 0, n_copy = 0, n_stage = 0;
static hipError_t sync_result = hipSuccess, stage_result = hipSuccess;
static uint64_t device_words[8] = {11, 12, 13, 14, 15, 16, 17, 18};

extern "C" {
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned int) { *d = h; return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++n_sync; return sync_result; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  ++n_copy;
  memcpy(d, s, n);
  return hipSuccess;
}
}
namespace awsrc {
hipError_t launch_stage_words(const uint64_t*, int, uint64_t*, const uint64_t* src, int n, uint64_t* out, hipStream_t) {
  ++n_stage;
  memcpy(out, src, 8 * (size_t)n);
  return stage_result;
}
}  // namespace awsrc

#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
  using awsrc::HostSlot;
  uint64_t got[8], dev = 0;
  uint64_t* first = nullptr;
  {  // a whole call: one wait, none when the slot is given back
    HostSlot s;
    first = s.device_or(&dev, nullptr);
    CHECK(first != &dev);
    first[0] = 7;
    CHECK(s.read(got, 8, &dev, nullptr) == hipSuccess && got[0] == 7);
  }
  CHECK(n_sync == 1 && n_copy == 0);
  {  // the slot is free again; never lent, nothing to wait for
    HostSlot s;
    (void)s.holds(8);
  }
  CHECK(n_sync == 1);
  {  // fetch through the slot, and past its size
    HostSlot s;
    CHECK(s.fetch(got, device_words, sizeof got, nullptr) == hipSuccess && got[7] == 18 && n_stage == 1);
    static char big[2 * HostSlot::kBytes], out[2 * HostSlot::kBytes];
    CHECK(s.fetch(out, big, sizeof big, nullptr) == hipSuccess && n_copy == 1);
  }
  CHECK(n_sync == 3);
  {  // the call ends after a launch that writes the slot, before its wait
    HostSlot s;
    CHECK(s.device_or(&dev, nullptr) == first);
  }
  CHECK(n_sync == 4);
  {
    HostSlot s;
    CHECK(s.flag(nullptr) == reinterpret_cast<unsigned long long*>(first) && !s.flag_set());
  }
  CHECK(n_sync == 5);
  stage_result = hipErrorInvalidValue;  // reported by a launch that ran
  {
    HostSlot s;
    CHECK(s.fetch(got, device_words, 8, nullptr) == hipErrorInvalidValue);
  }
  CHECK(n_sync == 6);
  stage_result = hipSuccess;
  sync_result = hipErrorInvalidValue;  // cannot wait: the slot is not used again
  {
    HostSlot s;
    CHECK(s.device_or(&dev, nullptr) == first);
  }
  sync_result = hipSuccess;
  {
    HostSlot s;
    CHECK(s.device_or(&dev, nullptr) != first);
  }
  // 63 slots are left; one more call finds none and copies
  {
    HostSlot all[63];
    uint64_t* seen[63];
    for (int i = 0; i < 63; ++i) {
      seen[i] = all[i].device_or(&dev, nullptr);
      CHECK(seen[i] != &dev && seen[i] != first);
      for (int k = 0; k < i; ++k) CHECK(seen[k] != seen[i]);
    }
    HostSlot none;
    const int copies = n_copy;
    CHECK(!none.holds(8) && none.flag(nullptr) == nullptr && none.device_or(&dev, nullptr) == &dev);
    dev = 9;
    CHECK(none.read(got, 8, &dev, nullptr) == hipSuccess && got[0] == 9 && n_copy == copies + 1);
    CHECK(none.fetch(got, device_words, 8, nullptr) == hipSuccess && got[0] == 11 && n_copy == copies + 2);
  }
  printf("ok\n");
  return 0;
}
