// Size helpers and per-thread error text of the C ABI.
#include <string.h>

#include <atomic>
#include <chrono>
#include <mutex>

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

// Host memory that a kernel can write: 32 places of 128 bytes, one for each header on its way, whatever its thread and
// stream.  One allocation for the process, made by the first call that needs it; it lasts as long as the library does (no
// call of the runtime stands at the end of a thread or of the process, where it could wait for kernels or break another
// thread's capture).  A device reset takes the allocation back under the library: its number, which the runtime gives to no
// other one, says whether it is still there.  With all places taken the header is copied.
class HeaderPlaces {
 public:
  static constexpr uint32_t kPlaces = 32, kWords = 32;
  // A place and the number of the call that it is for, or nullptr.
  uint32_t* take(uint32_t* call) {
    std::lock_guard<std::mutex> hold(lock_);
    if (!ready()) return nullptr;
    for (uint32_t i = 0; i < kPlaces; ++i) {
      if ((taken_ >> i) & 1u) continue;
      taken_ |= 1u << i;
      *call = ++calls_;
      words_[kWords * i + kHdrWords] = ~*call;
      return words_ + kWords * i;
    }
    return nullptr;
  }
  void give_back(const uint32_t* place) {
    std::lock_guard<std::mutex> hold(lock_);
    if (place >= words_ && place < words_ + kPlaces * kWords) taken_ &= ~(1u << ((uint32_t)(place - words_) / kWords));
  }

 private:
  static bool number_of(void* p, uint64_t* id) {
    const bool known = hipPointerGetAttribute(id, HIP_POINTER_ATTRIBUTE_BUFFER_ID, reinterpret_cast<hipDeviceptr_t>(p)) == hipSuccess;
    if (!known) (void)hipGetLastError();
    return known;
  }
  bool ready() {
    uint64_t id = 0;
    if (words_ && number_of(words_, &id) && id == id_) return true;
    words_ = nullptr; taken_ = 0u;
    // (an allocation is allowed here also while another thread captures a graph)
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) { (void)hipGetLastError(); return false; }
    void* p = nullptr;
    if (hipHostMalloc(&p, 4 * kPlaces * kWords, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
      (void)hipGetLastError();
    } else if (!number_of(p, &id_)) {
      (void)hipHostFree(p);
    } else {
      words_ = static_cast<uint32_t*>(p);
    }
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    return words_ != nullptr;
  }
  std::mutex lock_;
  uint32_t* words_ = nullptr;
  uint64_t id_ = 0;
  uint32_t taken_ = 0, calls_ = 0;
};
static HeaderPlaces g_places;

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
  uint32_t call = 0;
  uint32_t* const place = goes_by_kernel(raw, s) ? g_places.take(&call) : nullptr;
  if (!place) {
    KP_HIP_TRY(hipMemcpyAsync(hdr, raw, sizeof *hdr, hipMemcpyDeviceToHost, s));
    KP_HIP_TRY(hipStreamSynchronize(s));
    return KP_OK;
  }
  hipLaunchKernelGGL(kp_header_to_host, dim3(1), dim3(64), 0, s, static_cast<const uint32_t*>(raw), place, call);
  const hipError_t launched = hipGetLastError();
  if (launched != hipSuccess) {  // (nobody writes to the place)
    g_places.give_back(place);
    return fail(KP_ERR_HIP, "launching the read of the trace header failed: %s", hipGetErrorString(launched));
  }
  auto arrived = [&]() { return __atomic_load_n(place + kHdrWords, __ATOMIC_ACQUIRE) == call; };
  const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(200);
  while (!arrived() && std::chrono::steady_clock::now() < until) {}
  if (!arrived()) {  // there is other work ahead of it, or something went wrong
    const hipError_t e = hipStreamSynchronize(s);
    // (a place that the kernel may still write to is not given back)
    if (e != hipSuccess) return fail(KP_ERR_HIP, "reading the trace header back failed: %s", hipGetErrorString(e));
    if (!arrived()) return fail(KP_ERR_HIP, "reading the trace header back failed: its kernel did not run");
  }
  memcpy(hdr, place, sizeof *hdr);
  g_places.give_back(place);
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
