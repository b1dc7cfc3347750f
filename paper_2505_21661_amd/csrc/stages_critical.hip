// Critical path over the stage table (kp_stages_critical).
//
// The paper reads the critical path of a kernel whose warp groups work on different stages off the
// timeline: a chain of stages each of which could only start when the one before it had finished
// (Sec. 3.3 "Critical-path Analysis"; Sec. 5.2, where a load turns out to be held up by a barrier of another
// warp group), and takes the sum of the latencies along it as the kernel's latency (Table 4, WS model).
// Here the chain is taken per recorded workgroup from its stage table: stages ordered by (max_end,
// index); the path ends in the last one; the stage before X is the latest stage of that order, earlier
// than X, that had ended by the time X started.
//
// One decoder workgroup per recorded workgroup at a time (persistent, grid stride), everything in LDS; the
// table entries of the next recorded workgroup are requested before this one's are worked on:
//   1  the stages become 64-bit keys max_end << 32 | index and are sorted by a counting sort: P cells of
//      equal length over [first end, last end], one LDS atomic with return per stage, a prefix sum over the
//      cells, and inside a cell (one stage on average) the rank by comparison.  A table whose fullest cell
//      holds more than kMaxCell stages is merged in a bitonic network instead;
//   2  every stage finds the stage before it -- the stages that ended by its start are a prefix of the
//      order -- by a search of the cell its start lies in, which gives a forest of "waited for" links;
//   3  the path is the list that starts at the last stage: it is marked by pointer doubling (in round k
//      every marked stage marks the stage 2^k links on and every link is replaced by two), log2(n)
//      rounds instead of a walk of up to n steps;
//   4  marked stages add their latency to their region's totals, and the gaps to the stage before them
//      to the workgroup's bubbles.
// Bound by LDS round trips between barriers.  8192 workgroups of 16 regions x 64 iterations one after the other: 223 us
// with the network alone, every stage searching all ends twice; 154 us with the cells; 138 us with the sums over a wave
// by data-parallel primitives instead of LDS exchanges and without them in waves that hold no stage of the path.
#include <math.h>

#include "kp_common.h"
#include "kp_wave.h"

namespace {

using namespace kp_wave;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kBlock = 256;
constexpr uint32_t kMaxEntries = 4096;
constexpr uint32_t kNone = 0xFFFFFFFFu;
// Ranking inside a cell reads all keys of the cell for each of them; the network reads and writes every key
// 34 times for 16 runs of 64 (55 times without runs), so that a cell of some 64 stages costs the same.
constexpr uint32_t kMaxCell = 32;

struct CriticalParams {
  const u32x4* table;          // [n_wg][R * I] of {max_dur, min_start, max_end, n_waves}
  unsigned long long* hdr;     // 8 words
  unsigned long long* region;  // [R][2]
  u32x4* rows;                 // [n_wg][2]
  uint32_t n_wg, R, I, N, P;
};

__global__ void kp_critical_init(unsigned long long* out, uint32_t n_wg, uint32_t R, uint32_t I) {
  for (uint32_t i = threadIdx.x; i < 8 + 2 * R; i += blockDim.x) out[i] = i == 0 ? n_wg : (i == 1 ? R : (i == 2 ? I : 0ull));
}

// The sum over the wave of values below 2^36.
__device__ __forceinline__ unsigned long long wave_total36(unsigned long long v) {
  return ((unsigned long long)wave_total((uint32_t)(v >> 16)) << 16) + wave_total((uint32_t)v & 0xFFFFu);
}

// LDS: key[P] u64 | start[P] | lat[P] | jump[2][P] (the first one: cells, until the links are known) | mark[P]
// bytes | totals.  PER entries per thread: P = 256 * PER, or P <= 256 and PER = 1.
template <int PER>
__global__ __launch_bounds__(kBlock, PER <= 4 ? 6 : 1) void kp_critical_main(CriticalParams p) {
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t P = p.P, N = p.N, R = p.R, I = p.I;
  unsigned long long* key = reinterpret_cast<unsigned long long*>(smem);
  uint32_t* start = reinterpret_cast<uint32_t*>(smem + 8 * (size_t)P);
  uint32_t* lat = start + P;
  uint32_t* cells = lat + P;
  uint32_t* jump1 = cells + P;
  uint8_t* mark = reinterpret_cast<uint8_t*>(jump1 + P);
  unsigned long long* reg_tot = reinterpret_cast<unsigned long long*>(smem + 25 * (size_t)P);  // [R][2], 8-byte aligned: P >= 64
  unsigned long long* wg_tot = reg_tot + 2 * R;   // stages, latency, bubbles
  // [0] start of the first stage of the path, [1] first end, [2] last end, [3] a cell is too full, [4] a region's keys are
  // out of order, [8..11] stages in the cells of each hardware wave, [12..15] stages of each hardware wave
  uint32_t* wg_small = reinterpret_cast<uint32_t*>(wg_tot + 3);
  unsigned long long* all_tot = reinterpret_cast<unsigned long long*>(wg_small + 16);  // paths, stages, latency, bubbles

  const uint32_t tid = threadIdx.x, lane = tid & 63u, hw = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  for (uint32_t i = tid; i < 2 * R; i += kBlock) reg_tot[i] = 0ull;
  if (tid < 4) all_tot[tid] = 0ull;

  u32x4 entry[PER];
  auto fetch = [&](uint32_t wg) {
    const u32x4* tab = p.table + (size_t)wg * N;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const uint32_t i = tid + kBlock * u;
      entry[u] = i < N ? tab[i] : u32x4{0u, 0u, 0u, 0u};
    }
  };
  fetch(blockIdx.x);

  for (uint32_t wg = blockIdx.x; wg < p.n_wg; wg += gridDim.x) {
    if (tid < 3) wg_tot[tid] = 0ull;
    if (tid < 8) wg_small[tid] = tid < 2u ? 0xFFFFFFFFu : 0u;
    uint32_t end[PER];
    uint32_t live = 0;  // bit u: entry u is a stage
    uint32_t first_end = 0xFFFFFFFFu, last_end = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const uint32_t i = tid + kBlock * u;
      end[u] = entry[u].z;
      if (entry[u].w != 0u) {
        live |= 1u << u;
        first_end = end[u] < first_end ? end[u] : first_end;
        last_end = end[u] > last_end ? end[u] : last_end;
      }
      if (i < P) { start[i] = entry[u].y; lat[i] = entry[u].x; cells[i] = 0u; mark[i] = 0; }
    }
    if (wg + gridDim.x < p.n_wg) fetch(wg + gridDim.x);
    first_end = wave_least(first_end);
    last_end = ~wave_least(~last_end);
    __syncthreads();
    if (lane == 0 && first_end <= last_end) {  // the wave has a stage
      atomicMin(&wg_small[1], first_end);
      atomicMax(&wg_small[2], last_end);
    }
    __syncthreads();
    // ---- 1: order ---------------------------------------------------------------------------------
    // (a clock's cell never falls as the clock rises: rounding, product and conversion are monotonic)
    first_end = wg_small[1];
    last_end = wg_small[2];
    const float per_tick = (float)P / ((float)(last_end - first_end) + 1.0f);
    auto cell_of = [&](uint32_t t) {
      const uint32_t c = (uint32_t)((float)(t - first_end) * per_tick);
      return c < P ? c : P - 1u;
    };
    auto key_of = [&](int u) { return ((unsigned long long)end[u] << 32) | (tid + kBlock * u); };
    uint32_t at[PER];  // arrival number in the cell, then the place in the order
    bool full = false;
    uint32_t n_wave = 0;  // stages of the hardware wave
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      at[u] = 0;
      const bool is = (live >> u & 1u) != 0u;
      const uint64_t here = __builtin_amdgcn_ballot_w64(is);
      if (here == 0ull) continue;  // (uniform)
      n_wave += (uint32_t)__popcll(here);
      const uint32_t c = cell_of(end[u]), some = (uint32_t)__builtin_amdgcn_readlane((int)c, (int)__builtin_ctzll(here));
      // (a cell that these stages alone fill: their atomics on one word would be done one after the other)
      full = full || __popcll(__builtin_amdgcn_ballot_w64(is && c == some)) > (int)kMaxCell;
      if (is && !full) { at[u] = atomicAdd(&cells[c], 1u); full = at[u] >= kMaxCell; }
      full = __builtin_amdgcn_ballot_w64(full) != 0ull;
    }
    if (lane == 0) {
      wg_small[12 + hw] = n_wave;
      if (full) wg_small[3] = 1u;
    }
    __syncthreads();
    const uint32_t n = wg_small[12] + wg_small[13] + wg_small[14] + wg_small[15];
    const bool by_cell = wg_small[3] == 0u;
    if (by_cell) {
      uint32_t mine[PER], sum = 0;
#pragma unroll
      for (int j = 0; j < PER; ++j) { mine[j] = tid * PER < P ? cells[tid * PER + j] : 0u; sum += mine[j]; }
      const uint32_t upto = wave_scan_add(sum);
      if (lane == 63u) wg_small[8 + hw] = upto;
      __syncthreads();
      uint32_t at_cell = upto - sum;
#pragma unroll
      for (uint32_t h = 0; h < kBlock / 64; ++h) at_cell += h < hw ? wg_small[8 + h] : 0u;
      if (tid * PER < P) {
#pragma unroll
        for (int j = 0; j < PER; ++j) { cells[tid * PER + j] = at_cell; at_cell += mine[j]; }
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if (live >> u & 1u) { at[u] += cells[cell_of(end[u])]; key[at[u]] = key_of(u); }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        if (!(live >> u & 1u)) continue;
        const uint32_t c = cell_of(end[u]), lo = cells[c], hi = c + 1u < P ? cells[c + 1u] : n;
        const unsigned long long k = key_of(u);
        at[u] = lo;
        if (hi - lo > 1u) {
          // Each lane starts elsewhere in its cell: cells of 16 or 32 stages each lie a whole number of bank lines apart, and
          // lanes that all read the first key of theirs wait for one another (8192 tables of 16 x 64 whose regions end
          // together, 32 stages per cell: 314 us, 160 this way; with the stages in any order 369 and 149).
          const uint32_t n_cell = hi - lo, first = (lane * n_cell) >> 6;
          for (uint32_t m = 0; m < n_cell; m += 2u) {  // (two reads in flight; four gain nothing and take the registers of a workgroup per CU)
            unsigned long long other[2];
#pragma unroll
            for (uint32_t x = 0; x < 2u; ++x) {
              const uint32_t from = first + (m + x < n_cell ? m + x : 0u);
              other[x] = key[lo + (from < n_cell ? from : from - n_cell)];
            }
#pragma unroll
            for (uint32_t x = 0; x < 2u; ++x) at[u] += m + x < n_cell && other[x] < k ? 1u : 0u;
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if (live >> u & 1u) key[at[u]] = key_of(u);
      __syncthreads();
    } else {
      // The iterations of a region usually end one after the other, so that the keys of a region (a run of I
      // consecutive entries) are in order as they come; that is checked (an entry that is no stage has the
      // largest key: it must be behind the stages of its run).
      const bool runs = I >= 2u && (I & (I - 1u)) == 0u;  // runs that the merge steps below can start from
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if (tid + kBlock * u < P) key[tid + kBlock * u] = live >> u & 1u ? key_of(u) : ~0ull;
      __syncthreads();
      bool disorder = false;
      if (runs)
        for (uint32_t i = tid; i < N; i += kBlock)
          if ((i & (I - 1u)) != 0u) disorder = disorder || key[i - 1u] > key[i];
      if (__builtin_amdgcn_ballot_w64(disorder) != 0ull && lane == 0) wg_small[4] = 1u;
      __syncthreads();
      // Ascending sort by merging: blocks of k/2 keys in order become blocks of k.  The first step of a merge
      // compares key i of the lower block with key k/2 - 1 - i of the upper one (the smaller k/2 keys of the
      // two end up below, the larger above, each a rising-then-falling sequence), the steps after it are the
      // half-cleaners of a bitonic merge.  With every region's run in order the merging starts at blocks of I.
      // A thread takes the pairs t = tid, tid + 256, ..., so the 64 pairs of a hardware wave lie in one block of
      // 128 consecutive keys whenever the two keys of a pair are at most 64 apart (and, in a first step, the
      // blocks hold at most 128 keys): such steps touch no key of another wave, and since the LDS operations
      // of one wave take effect in order, two of them in a row need no workgroup barrier between them.
      auto between = [&](bool local_before, bool local_after) {
        if (local_before && local_after) { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier(); }
        else __syncthreads();
      };
      for (uint32_t k = (runs && wg_small[4] == 0u) ? 2u * I : 2u; k <= P; k <<= 1) {
        const uint32_t half = k >> 1;
        for (uint32_t t = tid; t < P / 2; t += kBlock) {
          const uint32_t blk = (t / half) * k, i = t & (half - 1u), lo = blk + i, hi = blk + k - 1u - i;
          const unsigned long long a = key[lo], b = key[hi];
          if (a > b) { key[lo] = b; key[hi] = a; }
        }
        // (the step after this one: the half-cleaner at distance half / 2, or the first step of the next size)
        between(k <= 128u, half >= 2u ? (half >> 1) <= 64u : 2u * k <= 128u);
        for (uint32_t j = half >> 1; j > 0; j >>= 1) {
          for (uint32_t t = tid; t < P / 2; t += kBlock) {
            const uint32_t lo = ((t & ~(j - 1u)) << 1) | (t & (j - 1u));  // the element of the pair with bit j clear
            const uint32_t hi = lo | j;
            const unsigned long long a = key[lo], b = key[hi];
            if (a > b) { key[lo] = b; key[hi] = a; }
          }
          between(j <= 64u, j >= 2u ? true : 2u * k <= 128u);
        }
      }
      __syncthreads();
    }
    // ---- 2: the stage each stage waited for (the stages are the first n keys) -----------------------
    uint32_t pred[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const uint32_t r = tid + kBlock * u;
      pred[u] = kNone;
      if (r < n) {
        const uint32_t s = start[(uint32_t)key[r]];
        uint32_t lo = 0, hi = n;  // first rank whose end exceeds s
        if (s < first_end) hi = 0;
        else if (s >= last_end) lo = n;
        else if (by_cell) {
          const uint32_t c = cell_of(s);
          lo = cells[c];
          hi = c + 1u < P ? cells[c + 1u] : n;
        }
        while (lo < hi) {
          const uint32_t mid = (lo + hi) >> 1;
          if ((uint32_t)(key[mid] >> 32) <= s) lo = mid + 1; else hi = mid;
        }
        const uint32_t c = lo < r ? lo : r;
        pred[u] = c ? c - 1u : kNone;
        jump1[r] = pred[u];
        if (r + 1u == n) mark[r] = 1;
      }
    }
    // ---- 3: mark the list that starts at the last stage --------------------------------------------
    uint32_t* cur = jump1;
    uint32_t* nxt = cells;
    for (uint32_t round = 0; (1u << round) < n; ++round) {
      __syncthreads();
      for (uint32_t r = tid; r < n; r += kBlock) {
        const uint32_t j = cur[r];
        // (a stage marked in this very round may already act: it only marks stages of the list)
        if (j != kNone && mark[r]) mark[j] = 1;
        nxt[r] = j != kNone ? cur[j] : kNone;
      }
      uint32_t* t = cur; cur = nxt; nxt = t;
    }
    __syncthreads();
    // ---- 4: totals ---------------------------------------------------------------------------------
    uint32_t my_n = 0;
    unsigned long long my_lat = 0, my_bub = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const uint32_t r = tid + kBlock * u;
      if (r >= n || !mark[r]) continue;
      const uint32_t idx = (uint32_t)key[r];
      const uint32_t s = start[idx], l = lat[idx];
      if (pred[u] != kNone) my_bub += s - (uint32_t)(key[pred[u]] >> 32);
      else wg_small[0] = s;  // the first stage of the path
      ++my_n; my_lat += l;
      const uint32_t region = idx / I;
      atomicAdd(&reg_tot[2 * region], 1ull);
      atomicAdd(&reg_tot[2 * region + 1], (unsigned long long)l);
    }
    if (__builtin_amdgcn_ballot_w64(my_n != 0u) != 0ull) {
      my_n = wave_total(my_n); my_lat = wave_total36(my_lat); my_bub = wave_total36(my_bub);
    }
    if (lane == 0 && my_n) {
      atomicAdd(&wg_tot[0], (unsigned long long)my_n);
      atomicAdd(&wg_tot[1], my_lat);
      atomicAdd(&wg_tot[2], my_bub);
    }
    __syncthreads();
    if (tid == 0) {
      u32x4 a, b;
      if (n) {
        const unsigned long long last = key[n - 1u];
        const uint32_t idx = (uint32_t)last;
        a = u32x4{(uint32_t)wg_tot[0], ((idx / I) << 16) | (idx % I), wg_small[0], (uint32_t)(last >> 32)};
        all_tot[0] += 1ull;
      } else {
        a = u32x4{0u, 0xFFFFFFFFu, 0u, 0u};
      }
      b = u32x4{(uint32_t)wg_tot[1], (uint32_t)(wg_tot[1] >> 32), (uint32_t)wg_tot[2], (uint32_t)(wg_tot[2] >> 32)};
      p.rows[2 * (size_t)wg] = a;
      p.rows[2 * (size_t)wg + 1] = b;
      all_tot[1] += wg_tot[0]; all_tot[2] += wg_tot[1]; all_tot[3] += wg_tot[2];
    }
    __syncthreads();
  }
  for (uint32_t i = tid; i < 2 * R; i += kBlock)
    if (reg_tot[i]) atomicAdd(&p.region[i], reg_tot[i]);
  if (tid < 4 && all_tot[tid]) atomicAdd(&p.hdr[3 + tid], all_tot[tid]);
}

struct LaunchCache { int dev = -1; uint32_t lds = 0; uint32_t max_grid = 0; };

// Every decoder workgroup adds its totals to the same few lines at its end, one after the other: 0.02 us each.  A
// recorded workgroup takes one of them 3.5 us and as long again for some 400 stages, twice that and more in the network:
// `times` as long as such an add.  With g decoder workgroups the sum of both is g + times * (n_wg / g), least at the root
// of n_wg * times, or next to it where every one of them has the same number.  All that are resident / so many: 2048
// workgroups of 64 stages 32.4 / 23.3 us (1024 of 2048), of 128 52.1 / 31.9.
inline uint32_t most_workgroups(uint32_t n_wg, uint32_t P) {
  const double times = 450.0 + P;
  const uint32_t turns = (uint32_t)sqrt((double)n_wg / times);
  auto cost = [&](uint32_t t) { return (double)n_wg / t + times * t; };
  const uint32_t t = turns < 1u ? 1u : (cost(turns + 1u) < cost(turns) ? turns + 1u : turns);
  return (n_wg + t - 1u) / t;
}
// Eight per CU take all its wave slots: 32768 workgroups of 64 stages 146 us, with seven 102, with six 111.
constexpr int kMaxPerCu = 7;

template <int PER>
kp_status launch(const CriticalParams& p, hipStream_t s) {
  const uint32_t lds = 25u * p.P + 16u * p.R + 24u + 64u + 32u;
  static thread_local LaunchCache cache;
  int dev = 0;
  KP_HIP_TRY(hipGetDevice(&dev));
  if (cache.dev != dev || cache.lds != lds) {
    KP_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kp_critical_main<PER>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    int per_cu = 0, cus = 0;
    KP_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kp_critical_main<PER>, kBlock, lds));
    if (per_cu < 1) return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "critical-path kernel does not fit one CU (LDS %u B)", lds);
    KP_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    cache.dev = dev; cache.lds = lds; cache.max_grid = (uint32_t)(per_cu < kMaxPerCu ? per_cu : kMaxPerCu) * (uint32_t)cus;
  }
  const uint32_t most = most_workgroups(p.n_wg, p.P);
  const uint32_t grid = cache.max_grid < most ? cache.max_grid : most;
  hipLaunchKernelGGL(kp_critical_main<PER>, dim3(grid), dim3(kBlock), lds, s, p);
  KP_HIP_TRY(hipGetLastError());
  return KP_OK;
}

}  // namespace

extern "C" size_t kp_critical_bytes(int n_wg, int n_regions) {
  if (n_wg < 0 || n_regions < 1 || n_regions > 128) return 0;
  return 64 + 16 * (size_t)n_regions + 32 * (size_t)n_wg;
}

extern "C" kp_status kp_stages_critical(const void* stages, int n_wg, int n_regions, int max_iter, void* out_paths,
                                        void* stream) {
  kp::clear_error();
  if (!stages || !out_paths) return kp::fail(KP_ERR_INVALID_ARG, "NULL argument");
  if (n_wg < 0 || n_regions < 1 || n_regions > 128 || max_iter < 1 || max_iter > 65535)
    return kp::fail(KP_ERR_INVALID_ARG, "n_wg=%d regions=%d max_iter=%d", n_wg, n_regions, max_iter);
  if (((uintptr_t)stages & 15u) || ((uintptr_t)out_paths & 15u))
    return kp::fail(KP_ERR_INVALID_ARG, "stages and out_paths must be 16-byte aligned");
  const uint64_t n_ent = (uint64_t)n_regions * (uint64_t)max_iter;
  if (n_ent > kMaxEntries)
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "%d regions x %d iterations exceed %u stages per workgroup", n_regions, max_iter,
                    kMaxEntries);
  hipStream_t s = static_cast<hipStream_t>(stream);
  uint8_t* out = static_cast<uint8_t*>(out_paths);
  CriticalParams p;
  p.table = reinterpret_cast<const u32x4*>(static_cast<const uint8_t*>(stages) + 32);
  p.hdr = reinterpret_cast<unsigned long long*>(out);
  p.region = p.hdr + 8;
  p.rows = reinterpret_cast<u32x4*>(out + 64 + 16 * (size_t)n_regions);
  p.n_wg = (uint32_t)n_wg; p.R = (uint32_t)n_regions; p.I = (uint32_t)max_iter; p.N = (uint32_t)n_ent;
  p.P = 64;
  while (p.P < p.N) p.P <<= 1;
  hipLaunchKernelGGL(kp_critical_init, dim3(1), dim3(256), 0, s, p.hdr, p.n_wg, p.R, p.I);
  KP_HIP_TRY(hipGetLastError());
  if (n_wg == 0) return KP_OK;
  if (p.P <= 256) return launch<1>(p, s);
  if (p.P == 512) return launch<2>(p, s);
  if (p.P == 1024) return launch<4>(p, s);
  if (p.P == 2048) return launch<8>(p, s);
  return launch<16>(p, s);
}
