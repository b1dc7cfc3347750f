// Size helpers and per-thread error text of the C ABI.
#include <string.h>

#include <atomic>
#include <chrono>

#include "kp_common.h"

namespace kp {
static std::atomic<uint32_t> g_rec_cost{0};
uint32_t rec_cost() { return g_rec_cost.load(std::memory_order_relaxed); }

char* last_error_buf() {
  static thread_local char buf[kLastErrorLen] = {0};
  return buf;
}

// ---- the header of a trace, read back ---------------------------------------------------------------
static_assert(sizeof(kp_trace_hdr) == 64, "header words");
constexpr int kHdrWords = 16;

// Copies the header to host memory and then says which call it belongs to.
static __global__ void kp_header_to_host(const uint32_t* hdr, uint32_t* slot, uint32_t call) {
  if (threadIdx.x < kHdrWords) slot[threadIdx.x] = hdr[threadIdx.x];
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(slot + kHdrWords, call, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Host memory that a kernel can write: one small allocation per thread that reads headers back, given back when the thread
// ends.  A thread has one read under way at a time, whatever the stream.
struct HeaderSlot {
  uint32_t* words = nullptr;
  uint32_t calls = 0;
  bool usable = true;
  bool ready() {
    if (words || !usable) return usable;
    // (an allocation is allowed here also while another thread captures a graph)
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess) {
      usable = hipHostMalloc(reinterpret_cast<void**>(&words), 4 * (kHdrWords + 1), hipHostMallocPortable | hipHostMallocMapped) == hipSuccess;
      (void)hipThreadExchangeStreamCaptureMode(&mode);
      if (usable) words[kHdrWords] = 0u;
    } else {
      usable = false;
    }
    if (!usable) { words = nullptr; (void)hipGetLastError(); }
    return usable;
  }
  ~HeaderSlot() { if (words) (void)hipHostFree(words); }
};

// The copying engine's way into pageable memory takes 20 us, into pinned memory 12; a kernel that writes the header to
// where the host looks for it 7.  That way is for device memory of the current device and streams that run: a pointer of
// any other kind is the runtime's to judge, and a stream under capture would not run the kernel.
static bool goes_by_kernel(const void* raw, hipStream_t s) {
  hipPointerAttribute_t at;
  int dev = 0;
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (((uintptr_t)raw & 15u) || hipStreamIsCapturing(s, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone ||
      hipGetDevice(&dev) != hipSuccess || hipPointerGetAttributes(&at, raw) != hipSuccess ||
      hipMemGetAddressRange(&base, &size, const_cast<void*>(raw)) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  const size_t before = (size_t)((uintptr_t)raw - (uintptr_t)base);
  return at.type == hipMemoryTypeDevice && at.device == dev && before <= size && size - before >= sizeof(kp_trace_hdr);
}

kp_status read_header(const void* raw, kp_trace_hdr* hdr, hipStream_t s) {
  static thread_local HeaderSlot slot;
  if (!goes_by_kernel(raw, s) || !slot.ready()) {
    KP_HIP_TRY(hipMemcpyAsync(hdr, raw, sizeof *hdr, hipMemcpyDeviceToHost, s));
    KP_HIP_TRY(hipStreamSynchronize(s));
    return KP_OK;
  }
  const uint32_t call = ++slot.calls;
  hipLaunchKernelGGL(kp_header_to_host, dim3(1), dim3(64), 0, s, static_cast<const uint32_t*>(raw), slot.words, call);
  KP_HIP_TRY(hipGetLastError());
  auto arrived = [&]() { return __atomic_load_n(slot.words + kHdrWords, __ATOMIC_ACQUIRE) == call; };
  const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(200);
  while (!arrived() && std::chrono::steady_clock::now() < until) {}
  if (!arrived()) {  // there is other work ahead of it, or something went wrong
    const hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess || !arrived()) {
      slot.words = nullptr;  // (the kernel may still write to it: never given back)
      slot.usable = false;
      return fail(KP_ERR_HIP, "reading the trace header back failed: %s", hipGetErrorString(e));
    }
  }
  memcpy(hdr, slot.words, sizeof *hdr);
  return KP_OK;
}
}  // namespace kp

extern "C" const char* kp_last_error(void) { return kp::last_error_buf(); }

extern "C" size_t kp_trace_bytes(int n_wg, int waves_per_wg, int cap_per_wg) {
  if (n_wg < 0 || waves_per_wg < 1 || waves_per_wg > KP_MAX_WAVES || cap_per_wg < 0) return 0;
  if (cap_per_wg % waves_per_wg) return 0;
  return sizeof(kp_trace_hdr) + sizeof(kp_wg_hdr) * (size_t)n_wg + (size_t)8 * n_wg * (size_t)cap_per_wg;
}

extern "C" size_t kp_stats_bytes(int n_wg, int waves_per_wg, int n_regions) {
  if (n_wg < 0 || waves_per_wg < 1 || waves_per_wg > KP_MAX_WAVES || n_regions < 1) return 0;
  const size_t R = (size_t)n_regions;
  return sizeof(kp_stats_hdr) + 8 * (KP_HIST_BINS * R + 5 * R + 2 * R * R) +
         sizeof(kp_wave_region_stat) * (size_t)n_wg * waves_per_wg * R;
}

extern "C" void kp_set_rec_cost(uint32_t ticks) { kp::g_rec_cost.store(ticks, std::memory_order_relaxed); }
extern "C" uint32_t kp_get_rec_cost(void) { return kp::rec_cost(); }
