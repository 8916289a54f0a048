// Pinned host memory of one call's results (host code).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <mutex>

namespace awsrc {

// awsrc_internal.h: words from device memory to where the host reads them
hipError_t launch_stage_words(const uint64_t* tab, int n_tab, uint64_t* to, const uint64_t* src, int n_out,
                              uint64_t* out, hipStream_t st);

// A small piece of pinned host memory that kernels write results of a call to,
// so that the host reads them after one stream synchronization (a copy into
// pageable memory costs 11 us more).  64 slots of 4 KiB in one block, allocated
// on first use and kept until the process ends; a slot is taken for the length
// of a call and given back, and a call that finds none free (more than 64 in
// flight, or no pinned memory) reads through a copy instead.  A call that ends
// between a launch that writes its slot and the wait for the stream (an error
// of a launch may be one of earlier work) waits before it gives the slot back,
// or keeps it if it cannot wait.
class HostSlot {
 public:
  static constexpr size_t kBytes = 4096;
  HostSlot() {
    std::lock_guard<std::mutex> lock(mu());
    Block& b = block();
    if (!b.tried) {
      b.tried = true;
      hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;  // another thread may be capturing
      const bool swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
      void* h = nullptr;
      if (hipHostMalloc(&h, 64 * kBytes, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess) {
        b.host = static_cast<char*>(h);
      } else {
        (void)hipGetLastError();
      }
      if (swapped) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    if (b.host && ~b.used) {
      at_ = __builtin_ctzll(~b.used);
      b.used |= 1ull << at_;
      host_ = b.host + (size_t)at_ * kBytes;
      void* d = nullptr;
      if (hipHostGetDevicePointer(&d, host_, 0) == hipSuccess) dev_ = d;
      else (void)hipGetLastError();
    }
  }
  ~HostSlot() {
    if (at_ < 0) return;
    if (busy_ && hipStreamSynchronize(stream_) != hipSuccess) {
      (void)hipGetLastError();
      return;
    }
    std::lock_guard<std::mutex> lock(mu());
    block().used &= ~(1ull << at_);
  }
  HostSlot(const HostSlot&) = delete;
  HostSlot& operator=(const HostSlot&) = delete;
  // where a kernel of stream s writes the results: the slot, or `device` when there is none
  uint64_t* device_or(uint64_t* device, hipStream_t s) {
    if (!dev_) return device;
    lend(s);
    return static_cast<uint64_t*>(dev_);
  }
  // n host bytes (a multiple of 8) of device memory, waiting for the stream
  hipError_t fetch(void* dst, const void* device, size_t n, hipStream_t s) {
    if (!dev_ || n > kBytes) {
      const hipError_t e = hipMemcpyAsync(dst, device, n, hipMemcpyDeviceToHost, s);
      return e != hipSuccess ? e : wait(s);
    }
    lend(s);
    const hipError_t e = launch_stage_words(nullptr, 0, nullptr, static_cast<const uint64_t*>(device), (int)(n / 8),
                                            static_cast<uint64_t*>(dev_), s);
    return e != hipSuccess ? e : read(dst, n, device, s);
  }
  // a word of the slot that kernels of stream s may set, cleared; null when there is no slot
  unsigned long long* flag(hipStream_t s) {
    if (!dev_) return nullptr;
    lend(s);
    *reinterpret_cast<volatile uint64_t*>(host_) = 0;
    return static_cast<unsigned long long*>(dev_);
  }
  bool holds(size_t n) const { return dev_ && n <= kBytes; }
  bool flag_set() const { return *reinterpret_cast<volatile uint64_t*>(host_) != 0; }
  // waits for the stream: no kernel of this call writes the slot any more
  hipError_t wait(hipStream_t s) {
    const hipError_t e = hipStreamSynchronize(s);
    if (e == hipSuccess) busy_ = false;
    return e;
  }
  // waits for the stream and fetches n bytes of results
  hipError_t read(void* dst, size_t n, const void* device, hipStream_t s) {
    if (!dev_) {
      const hipError_t e = hipMemcpyAsync(dst, device, n, hipMemcpyDeviceToHost, s);
      if (e != hipSuccess) return e;
    }
    const hipError_t e = wait(s);
    if (e == hipSuccess && dev_) memcpy(dst, host_, n);
    return e;
  }

 private:
  struct Block {
    char* host = nullptr;
    uint64_t used = 0;
    bool tried = false;
  };
  static std::mutex& mu() { static std::mutex m; return m; }
  static Block& block() { static Block b; return b; }
  // the slot's device pointer goes to a kernel of stream s
  void lend(hipStream_t s) {
    busy_ = true;
    stream_ = s;
  }
  int at_ = -1;
  char* host_ = nullptr;
  void* dev_ = nullptr;
  bool busy_ = false;
  hipStream_t stream_ = nullptr;
};

}  // namespace awsrc
