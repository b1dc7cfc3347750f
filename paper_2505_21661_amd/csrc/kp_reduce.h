// What the two statistics decoders (the LDS-resident one and the one for wide geometries) share: the
// layout of the statistics block and the hand-over between them.
#pragma once
#include "kp_common.h"
#include "kp_wave.h"

namespace kp_reduce {

// positions inside kp_stats_hdr, in u64 words
enum { H_SLOTS_VALID = 0, H_PAIRS, H_ORPHAN_START, H_ORPHAN_END, H_INVALID, H_DROPPED, H_DISORDER,
       H_SPAN_OVF, H_NONMONO, H_OVERLAP_WGS, H_STATUS, H_NWG, H_WAVES, H_NREG, H_CAP, H_RSVD };

struct StatsLayout {  // offsets in u64 words
  size_t hist, cnt, sum, min, max, U, O, F, per, total;
};
__host__ __device__ inline StatsLayout stats_layout(uint32_t n_wg, uint32_t W, uint32_t R) {
  StatsLayout l;
  l.hist = 16;
  l.cnt = l.hist + (size_t)64 * R;
  l.sum = l.cnt + R; l.min = l.sum + R; l.max = l.min + R; l.U = l.max + R;
  l.O = l.U + R;
  l.F = l.O + (size_t)R * R;
  l.per = l.F + (size_t)R * R;
  l.total = l.per + (size_t)2 * n_wg * W * R;
  return l;
}

// Recorded workgroups as they would be on a device of 256 CUs, the one that the choice of a decoder was measured on: with how many
// of them a form pays is a question of how many there are per CU.
inline kp_status wgs_of_256_cus(uint32_t n_wg, uint32_t* n) {
  static thread_local int known = -1, cus = 0;
  int dev = 0;
  KP_HIP_TRY(hipGetDevice(&dev));
  if (known != dev) {
    KP_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    if (cus < 1) return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "device %d reports %d compute units", dev, cus);
    known = dev;
  }
  const uint64_t scaled = ((uint64_t)n_wg * 256u + (uint32_t)cus - 1u) / (uint32_t)cus;
  *n = scaled < 0xFFFFFFFFull ? (uint32_t)scaled : 0xFFFFFFFFu;
  return KP_OK;
}

using namespace kp_wave;

// Batcher's odd-even merge sort of N registers: a fixed network (63 exchanges for 16 words, 384 for 48),
// every index known at compile time.
template <int N, typename T>
__device__ __forceinline__ void network_sort(T (&key)[N]) {
#pragma unroll
  for (int pp = 1; pp < N; pp <<= 1) {
#pragma unroll
    for (int k = pp; k >= 1; k >>= 1) {
#pragma unroll
      for (int j = k % pp; j + k < N; j += 2 * k) {
#pragma unroll
        for (int i = 0; i < (k < N - j - k ? k : N - j - k); ++i) {
          if ((i + j) / (2 * pp) == (i + j + k) / (2 * pp)) {
            const T x = key[i + j], y = key[i + j + k];
            key[i + j] = x < y ? x : y;
            key[i + j + k] = x < y ? y : x;
          }
        }
      }
    }
  }
}

// Ascending order of N (a power of two) registers that first rise and then fall, or the reverse.
template <int N, typename T>
__device__ __forceinline__ void bitonic_merge(T (&v)[N]) {
#pragma unroll
  for (int k = N / 2; k >= 1; k >>= 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if ((i & k) == 0) {
        const T x = v[i], y = v[i + k];
        v[i] = x < y ? x : y;
        v[i + k] = x < y ? y : x;
      }
    }
  }
}

// The main kernel of the decoder for geometries the LDS-resident one does not take (more than 32
// regions, more than 16384 record slots per workgroup).  Between the init kernel and the one that derives the
// figures, on the same stream; accumulates into the block exactly as the LDS-resident kernel does (histogram, sums,
// extrema and header counts by atomics, the region-pair sums in the upper triangle of the F area).  The header has
// been validated by the caller.  wide_supported: KP_ERR_UNSUPPORTED_SHAPE when one workgroup's records
// exceed what the kernel can mark in LDS.
kp_status wide_supported(const kp_trace_hdr& h);
kp_status launch_wide(const uint32_t* wg_hdrs, const void* records, uint64_t* out, const kp_trace_hdr& h,
                      hipStream_t s);

}  // namespace kp_reduce
