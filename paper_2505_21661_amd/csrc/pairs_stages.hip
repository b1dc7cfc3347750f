// Per-iteration stage table from the timeline rows (kp_pairs_stages).
//
// The paper's critical-path analysis and overlap models (Sec. 3.3 "Critical-path Analysis",
// Sec. 5.2 / Table 4) take the latency of every stage in every loop iteration.  A stage that the
// waves of a workgroup run together lasts as long as its slowest wave, so the rows {start, dur,
// iter, region} that kp_trace_pairs wrote for the waves of a workgroup are folded into one entry
// per (workgroup, region, iteration): {max dur, min start, max (start + dur), rows folded}.
//
// A streaming kernel: persistent decoder workgroups, one recorded workgroup at a time, its table in LDS.  The rows
// come with 16-byte loads, four per lane and step, two steps in flight, which do not end with a recorded workgroup: the
// first rows of the next are on their way while the table is written (16-byte stores) and reset.
// What bounds it: HBM.  2^25 rows of 4096 workgroups of 8 waves, 16 regions x 64 iterations (0.53 GB, and 67 MB of
// table): 189 us with every wait a wait for all loads (branches around the folds, buffers handed on), every recorded
// workgroup starting with nothing on its way and 4096 adds to one word of the header at the end, 12 ns each; 93 us
// (6.4 TB/s of rows and table) now.
#include <math.h>

#include "kp_common.h"
#include "kp_wave.h"

namespace {

using kp_wave::scan_src;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kBlock = 512;
constexpr uint32_t kWavesHw = kBlock / 64;
constexpr int kDepth = 2;  // steps that a hardware wave has on their way
constexpr uint32_t kMaxTableBytes = 64 * 1024;

struct StagesParams {
  const uint32_t* count;  // rows per (workgroup, wave)
  const u32x4* rows;      // cap_wave / 2 row slots per (workgroup, wave)
  unsigned long long* hdr;  // n_rows, n_clipped, n_bad_region, 0
  u32x4* table;           // [n_wg][R][max_iter]
  uint32_t n_wg, W, R, half, max_iter, stride;
};

__global__ void kp_stages_init(unsigned long long* hdr) {
  if (threadIdx.x < 4) hdr[threadIdx.x] = 0ull;
}

__device__ inline uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// A step is PER rows per lane.
template <int PER>
__global__ __launch_bounds__(kBlock) void kp_stages_main(StagesParams p) {
  constexpr uint32_t kRows = 64u * PER;
  extern __shared__ __align__(16) unsigned char smem[];
  // entry (r, it) at word r * stride + it of four arrays
  const uint32_t stride = p.stride, words = p.R * stride, array = words + 64u;  // (64: a place for every lane without a row)
  uint32_t* longest = reinterpret_cast<uint32_t*>(smem);
  uint32_t* first = longest + array;
  uint32_t* last = first + array;
  uint32_t* folded = last + array;
  unsigned long long* counts = reinterpret_cast<unsigned long long*>(folded + array);  // rows, clipped, of no region
  const uint32_t tid = threadIdx.x, lane = tid & 63u, hw = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t W = p.W, R = p.R, MI = p.max_iter;

  auto reset = [&](uint32_t at) { longest[at] = 0u; first[at] = 0xFFFFFFFFu; last[at] = 0u; folded[at] = 0u; };
  uint32_t n_rows = 0, n_clipped = 0, n_bad = 0;
  // Folds a row if it is one.  Without branches: loads that a branch lies behind would all be waited for at its end.
  auto fold = [&](const u32x4& row, bool is_row) __attribute__((always_inline)) {
    const uint32_t start = row.x, dur = row.y, it = row.z, region = row.w;
    const bool known = is_row && region < R, kept = known && it < MI;
    n_bad += is_row && !known ? 1u : 0u;
    n_clipped += known && !kept ? 1u : 0u;
    n_rows += kept ? 1u : 0u;
    const uint32_t at = kept ? region * stride + it : words + lane;
    atomicMax(&longest[at], dur);
    atomicMin(&first[at], start);
    atomicMax(&last[at], start + dur);
    atomicAdd(&folded[at], 1u);
  };

  // Turn i of this decoder workgroup takes recorded workgroup wg_of(i).  Decoder workgroups are dealt round-robin to the
  // eight XCDs; each XCD takes a run of consecutive recorded workgroups (all of them in turn: 8 % slower at 4096 workgroups of 8 x 1024 rows).
  const uint32_t xcd = blockIdx.x & 7u, many = p.n_wg & 7u, rest = gridDim.x & 7u;
  const uint32_t mine = (p.n_wg >> 3) + (xcd < many ? 1u : 0u), apart = (gridDim.x >> 3) + (xcd < rest ? 1u : 0u);
  const uint32_t from = xcd * (p.n_wg >> 3) + (xcd < many ? xcd : many) + (blockIdx.x >> 3);
  const uint32_t turns = (mine - (blockIdx.x >> 3) + apart - 1u) / apart;
  auto wg_of = [&](uint32_t i) { return from + i * apart; };
  // A turn's steps: the blocks of kRows rows that hold any are its units, numbered as they lie in memory; hardware wave h
  // takes units h, h + 8, ...  Every hardware wave makes the same number of steps, some of the last ones without rows.
  // (Wave after wave instead, eight streams 16 KiB apart: 12 % slower.  Units by the rings' capacity, whatever they hold:
  // 4096 workgroups of 8 x 1024 row slots, all of them empty, 55 us where this takes 21, 51 rows in each 59 / 31, one full
  // wave of eight 58 / 29, all of them full the same.)
  //
  // The step requested next: turn and step; lane w: rows of recorded wave w in that turn, units of the waves below it, and of
  // those and itself.  `ahead`: rows in the turn behind it, on their way since this one was opened.
  uint32_t at_turn = 0, at_step = 0, at_steps, held, below, upto;
  const uint32_t* ahead_at = p.count + (size_t)wg_of(0) * W + (lane < W ? lane : W - 1u);
  auto counts_behind = [&](uint32_t t) __attribute__((always_inline)) -> uint32_t {  // of turn t + 1, behind those of turn t (the last turn's again)
    ahead_at += t + 1u < turns ? (size_t)apart * W : (size_t)0;
    return *ahead_at;
  };
  auto open_turn = [&](uint32_t rows) __attribute__((always_inline)) {
    held = at_turn < turns && lane < W ? (rows < p.half ? rows : p.half) : 0u;  // a count beyond the wave's slots cannot be honoured
    const uint32_t units = (held + kRows - 1u) / kRows;
    upto = units;
    upto += scan_src<0>(upto); upto += scan_src<1>(upto); upto += scan_src<2>(upto); upto += scan_src<3>(upto);  // (16 waves at most)
    below = upto - units;
    at_steps = ((uint32_t)__builtin_amdgcn_readlane((int)upto, 15) + kWavesHw - 1u) / kWavesHw;
    at_step = 0;
  };
  const uint32_t rows_of_first = *ahead_at;
  uint32_t ahead = counts_behind(0);
  open_turn(rows_of_first);
  // Requests it; gives the number of its rows.  Always PER loads, or the waits for the steps behind it would be for all of
  // its own as well: a lane without a row reads the step's last one, a step without rows the first one there is.
  auto request = [&](u32x4 (&r)[PER], uint32_t& turn_of) __attribute__((always_inline)) -> uint32_t {
    auto next_turn = [&]() __attribute__((always_inline)) {
      ++at_turn;
      open_turn(ahead);
      ahead = counts_behind(at_turn);
    };
    if (__builtin_expect(at_step == at_steps && at_turn < turns, 0)) {
      next_turn();
      // (a loop of its own: in the turn opened first the counts are waited for alone, not with the rows behind them)
      while (__builtin_expect(at_steps == 0u && at_turn < turns, 0)) next_turn();
    }
    const uint32_t q = hw + kWavesHw * at_step;
    const uint32_t w = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(upto <= q) & 0xFFFFull);  // (16 past the last unit)
    const uint32_t begin = (q - (uint32_t)__builtin_amdgcn_readlane((int)below, (int)w)) * kRows;
    const uint32_t rows_of_w = (uint32_t)__builtin_amdgcn_readlane((int)held, (int)w);
    uint32_t n = rows_of_w > begin ? rows_of_w - begin : 0u;
    n = n < kRows ? n : kRows;
    const u32x4* rows = p.rows + (n ? ((size_t)wg_of(at_turn) * W + w) * p.half + begin : (size_t)0);
    const uint32_t top = n ? n - 1u : 0u;
#pragma unroll
    for (uint32_t u = 0; u < PER; ++u) {
      const uint32_t j = lane + 64u * u;
      r[u] = __builtin_nontemporal_load(rows + (j < top ? j : top));
    }
    turn_of = at_turn;
    ++at_step;
    return n;
  };
  u32x4 buf[kDepth][PER];
  uint32_t n_of[kDepth], turn_of[kDepth];
#pragma unroll
  for (int d = 0; d < kDepth; ++d) n_of[d] = request(buf[d], turn_of[d]);
  // (behind the first requests: a short call is the latencies of its start)
  for (uint32_t i = tid; i < words; i += kBlock) reset(i);
  if (tid < 3u) counts[tid] = 0ull;
  __syncthreads();
  uint32_t turn = 0;
  // Tables of the turns up to `end` to HBM, and reset for the next one.
  auto write_tables = [&](uint32_t end) __attribute__((always_inline)) {
    for (; turn < end; ++turn) {
      __syncthreads();
      u32x4* dst = p.table + (size_t)wg_of(turn) * R * MI;
      for (uint32_t i = tid; i < R * MI; i += kBlock) {
        const uint32_t r = i / MI, it = i - r * MI;
        const uint32_t at = r * stride + it;
        dst[i] = u32x4{longest[at], first[at], last[at], folded[at]};
        reset(at);
      }
      __syncthreads();
    }
  };
  while (turn_of[0] < turns) {  // (no exit inside: loads that one lies behind would all be waited for)
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
      write_tables(turn_of[d]);
      if (n_of[d] != 0u) {  // (of the last steps: 3000 workgroups of 1 x 256 rows 20.3 / 18.4 us)
#pragma unroll
        for (uint32_t u = 0; u < PER; ++u)
          fold(buf[d][u], lane + 64u * u < n_of[d]);
      }
      n_of[d] = request(buf[d], turn_of[d]);
    }
  }
  write_tables(turns);

  n_rows = wave_sum(n_rows); n_clipped = wave_sum(n_clipped); n_bad = wave_sum(n_bad);
  // One add per count and decoder workgroup: they queue up at the header, 12 ns each (one per hardware wave, with
  // two decoder workgroups per CU: 1000 recorded ones of 4 x 512 rows 57 us where this takes 13).
  if (lane == 0) {
    atomicAdd(&counts[0], (unsigned long long)n_rows);
    atomicAdd(&counts[1], (unsigned long long)n_clipped);
    atomicAdd(&counts[2], (unsigned long long)n_bad);
  }
  __syncthreads();
  if (tid < 3u && counts[tid]) atomicAdd(&p.hdr[tid], counts[tid]);
}

// Entries that the regions' rows of the table lie apart.  Regions that follow one another put an iteration of each of
// them into neighbouring lanes: 64 lanes hold 64 / R iterations of R regions, which this many words apart fall into
// different banks.  Where that would take more than 72 KiB, an odd number does.
constexpr uint32_t kBanks = 64;
inline uint32_t region_stride(uint32_t R, uint32_t max_iter) {
  const uint32_t apart = R < kBanks ? (kBanks + R - 1u) / R : 1u;
  const uint32_t stride = max_iter + ((apart - max_iter) & (kBanks - 1u));
  return 16u * R * stride <= 72u * 1024u ? stride : max_iter | 1u;
}

struct LaunchCache { int dev = -1; uint32_t lds = 0; uint32_t per_cu = 0, cus = 0; };

template <int PER>
kp_status launch(const StagesParams& p, hipStream_t s) {
  const uint32_t lds = 16u * (p.R * p.stride + 64u + 2u);  // (table, places for lanes without a row, counts)
  static thread_local LaunchCache cache;
  int dev = 0;
  KP_HIP_TRY(hipGetDevice(&dev));
  if (cache.dev != dev || cache.lds != lds) {
    KP_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kp_stages_main<PER>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    int per_cu = 0, cus = 0;
    KP_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kp_stages_main<PER>, kBlock, lds));
    if (per_cu < 1) return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "stage kernel does not fit one CU (LDS %u B)", lds);
    KP_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    cache.dev = dev; cache.lds = lds; cache.per_cu = (uint32_t)per_cu; cache.cus = (uint32_t)cus;
  }
  // Decoder workgroups: one per CU streams as fast as the memory gives rows (one / two / three per CU, us: 4096 workgroups of
  // 8 x 1024 rows 93 / 94 / 96, 1500 of 5 x 256 13.0 / 15.2 / 16.3).  The turns of small workgroups are steps between
  // barriers, 0.6 us each, which several take side by side, and each of them queues up at the header for 12 ns: the sum
  // is least at the root of 50 times their number.  (1 / 2 / 3 / 4 per CU, us: 60000 of 4 x 32 141 / 90 / 81 / 77, 8000 of 2 x 128
  // 27.1 / 20.8 / 21.2 / 22.3, 3276 of 5 x 32 13.1 / 14.1 / 16.0 / 18.2.)
  uint32_t per_cu = PER == 1 ? 4u : 1u;
  per_cu = per_cu < cache.per_cu ? per_cu : cache.per_cu;
  uint32_t grid = per_cu * cache.cus;
  const uint32_t least = (uint32_t)sqrt(50.0 * p.n_wg), few = least > cache.cus ? least : cache.cus;
  grid = grid < few ? grid : few;
  grid = grid < p.n_wg ? grid : p.n_wg;
  hipLaunchKernelGGL(kp_stages_main<PER>, dim3(grid), dim3(kBlock), lds, s, p);
  KP_HIP_TRY(hipGetLastError());
  return KP_OK;
}

}  // namespace

extern "C" size_t kp_stages_bytes(int n_wg, int n_regions, int max_iter) {
  if (n_wg < 0 || n_regions < 1 || n_regions > 128 || max_iter < 1) return 0;
  return 32 + sizeof(kp_stage_row) * (size_t)n_wg * (size_t)n_regions * (size_t)max_iter;
}

extern "C" kp_status kp_pairs_stages(const void* pairs, int n_wg, int waves_per_wg, int cap_per_wg, int n_regions,
                                     int max_iter, void* out_stages, void* stream) {
  kp::clear_error();
  if (!pairs || !out_stages) return kp::fail(KP_ERR_INVALID_ARG, "NULL argument");
  if (n_wg < 0 || waves_per_wg < 1 || waves_per_wg > KP_MAX_WAVES || cap_per_wg < 2 * waves_per_wg ||
      cap_per_wg % waves_per_wg || n_regions < 1 || n_regions > 128 || max_iter < 1)
    return kp::fail(KP_ERR_INVALID_ARG, "n_wg=%d waves=%d cap=%d regions=%d max_iter=%d", n_wg, waves_per_wg,
                    cap_per_wg, n_regions, max_iter);
  if (((uintptr_t)pairs & 15u) || ((uintptr_t)out_stages & 15u))
    return kp::fail(KP_ERR_INVALID_ARG, "pairs and out_stages must be 16-byte aligned");
  if ((uint64_t)n_regions * ((uint64_t)max_iter + 1u) * 16u > kMaxTableBytes)
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "a table of %d regions x %d iterations exceeds %u bytes of LDS",
                    n_regions, max_iter, kMaxTableBytes);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const uint8_t* in = static_cast<const uint8_t*>(pairs);
  uint8_t* out = static_cast<uint8_t*>(out_stages);
  const size_t n_seg = (size_t)n_wg * waves_per_wg;
  StagesParams p;
  p.count = reinterpret_cast<const uint32_t*>(in);
  p.rows = reinterpret_cast<const u32x4*>(in + ((n_seg + 3) / 4) * 16);
  p.hdr = reinterpret_cast<unsigned long long*>(out);
  p.table = reinterpret_cast<u32x4*>(out + 32);
  p.n_wg = (uint32_t)n_wg; p.W = (uint32_t)waves_per_wg; p.R = (uint32_t)n_regions;
  p.half = (uint32_t)(cap_per_wg / waves_per_wg) / 2u; p.max_iter = (uint32_t)max_iter;
  p.stride = region_stride(p.R, p.max_iter);

  hipLaunchKernelGGL(kp_stages_init, dim3(1), dim3(64), 0, s, p.hdr);
  KP_HIP_TRY(hipGetLastError());
  if (n_wg == 0) return KP_OK;

  // Waves of up to 128 rows: one row per lane and step.  1 / 2 / 4 rows, us, each with its best number of decoder workgroups:
  // 16000 workgroups of 2 x 16 rows 27 / 31 / 40, 9000 of 16 x 64 30 / 34 / 44, 8000 of 2 x 128 20.8 / 22.3 / 26.5, 2000 of
  // 8 x 128 13.7 / 13.8 / 13.9; 1500 of 5 x 256 14.9 / 14.2 / 13.0, 4096 of 8 x 1024 99 / 95 / 93.
  return p.half <= 128u ? launch<1>(p, s) : launch<4>(p, s);
}
