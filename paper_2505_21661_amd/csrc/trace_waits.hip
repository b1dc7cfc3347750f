// GPU replay of the waits behind asynchronous operations (kp_trace_waits).
//
// Sec. 4.3 (trace replay, asynchronous instructions): with a START before the asynchronous launch
// (clock CLK0), an END right before the barrier that waits for it (CLK1) and a second START right
// after the barrier (CLK2), the wait is T_wait = CLK2 - CLK1 with the records' own cost cancelled,
// and the figure holds only while what is left of the operation at the barrier outlasts one record.
// This kernel finds every END whose successor in its wave is a START and reduces
//   gap   = (u32)(CLK2 - CLK1)                      per (workgroup, wave, region of the END),
//   gap <= rec_cost                                 counted as "uncovered",
//   whole = (u32)(CLK2 - CLK0) - rec_cost, >= 0     when the END is paired with a START at CLK0.
//
// One decoder workgroup stages one recorded workgroup in LDS, ordered by rank; the hardware waves
// share out the recorded waves in runs of consecutive ranks and walk them 128 ranks per round, two per
// lane.  A START takes what it needs to know about the rank below -- metadata, clock, whether that END is
// paired and with which clock -- from its own lane or the one below through DPP wave shifts (the last lane of
// the previous round stands in for lane 0).  An END that has not its START right below it looks further back in LDS
// (look_back); a START above an empty rank, which only damaged traces have, walks back to the record below it.
// Sums, extrema and the log2 histogram go to LDS atomics; totals live in LDS across the recorded workgroups of
// a persistent decoder workgroup.
// What bounds it: instruction issue.  Measured on 9000 workgroups of 3 waves x 1024 records: 144 us with the loads
// waited for, one rank per lane and runs cut by capacity instead of by what the wave holds; 82 us (2.7 TB/s).
#include "kp_stage.h"

#include <math.h>

namespace {

using namespace kp_stage;

struct WaitsLayout {  // offsets in u64 words
  size_t hist, cnt, sum, min, max, unc, acnt, asum, per, total;
};
__host__ __device__ inline WaitsLayout waits_layout(uint32_t n_wg, uint32_t W, uint32_t R) {
  WaitsLayout l;
  l.hist = 16;
  l.cnt = l.hist + (size_t)64 * R;
  l.sum = l.cnt + R; l.min = l.sum + R; l.max = l.min + R;
  l.unc = l.max + R; l.acnt = l.unc + R; l.asum = l.acnt + R;
  l.per = l.asum + R;
  l.total = l.per + (size_t)2 * n_wg * W * R;
  return l;
}
enum { H_WAITS = 0, H_UNCOVERED, H_ASYNC, H_NWG = 8, H_WAVES, H_NREG, H_CAP, H_COST };

constexpr uint32_t kNoId = 0xFFFFu;     // END << 7 | region of no record
constexpr uint32_t kHistStride = 65;  // regions that hit the same bin land in different LDS banks; word 64: the region's waits, at the end

// The per-(wave, region) sums exist in up to four copies, one per quarter of a hardware wave: lanes 16 apart tend
// to hold the same region, and LDS atomics of one instruction that hit one address are done one after the other.
constexpr uint32_t kMaxEntries = 1024;  // entries of those sums, copies included (one copy may exceed it)

struct WaitsLds {
  uint32_t hist, pw_pack, pw_max, pw_min, as_pack, unc, reg_sum, reg_max, reg_min, acnt, asum, total;
  uint32_t copies;
};
__host__ __device__ inline WaitsLds waits_lds(uint32_t from, uint32_t W, uint32_t R, uint32_t copies) {
  WaitsLds l;
  l.copies = copies;
  uint32_t o = from;
  l.hist = o; o = align16(o + R * kHistStride * 4);
  l.pw_pack = o; o = align16(o + W * R * 8 * copies);
  l.pw_max = o; o = align16(o + W * R * 4 * copies);
  l.pw_min = o; o = align16(o + W * R * 4 * copies);
  l.as_pack = o; o = align16(o + R * 8);
  l.unc = o; o = align16(o + R * 8);
  l.reg_sum = o; o = align16(o + R * 8);
  l.reg_max = o; o = align16(o + R * 4);
  l.reg_min = o; o = align16(o + R * 4);
  l.acnt = o; o = align16(o + R * 8);
  l.asum = o; o = align16(o + R * 8);
  l.total = o;
  return l;
}

// init: clear the totals, set min to all-ones, echo the geometry.
__global__ void kp_waits_init(uint64_t* out, uint32_t n_wg, uint32_t W, uint32_t R, uint32_t cap, uint32_t rec_cost) {
  const WaitsLayout l = waits_layout(n_wg, W, R);
  for (size_t i = threadIdx.x + (size_t)blockIdx.x * blockDim.x; i < l.per; i += (size_t)blockDim.x * gridDim.x) {
    uint64_t v = (i >= l.min && i < l.max) ? ~0ull : 0ull;
    if (i == H_NWG) v = n_wg;
    if (i == H_WAVES) v = W;
    if (i == H_NREG) v = R;
    if (i == H_CAP) v = cap;
    if (i == H_COST) v = rec_cost;
    out[i] = v;
  }
}

// (6 hardware waves per SIMD, i.e. 80 vector registers: 97 us against 102 with 85 and 122 with 64; with 8 units per thread
// 80 would be 16 too few: 1000 workgroups of 7 x 1024 43 us where 5 waves per SIMD take 33)
template <int BLOCK, int UNITS>
__global__ __launch_bounds__(BLOCK, BLOCK == 1024 ? 4 : (UNITS == 4 ? 6 : 5)) void kp_waits_main(Trace p, uint64_t* out_words, uint32_t parts, uint32_t copies, uint32_t add_head) {
  extern __shared__ __align__(16) unsigned char smem[];
  const Lds L = lds_layout(p.nrec);
  const WaitsLds X = waits_lds(L.end, p.W, p.R, copies);
  const uint2* rec = reinterpret_cast<const uint2*>(smem + L.rec);
  const u32x4* rec2 = reinterpret_cast<const u32x4*>(smem + L.rec);
  const uint32_t* sV = reinterpret_cast<const uint32_t*>(smem + L.v);
  uint32_t* hist = reinterpret_cast<uint32_t*>(smem + X.hist);
  unsigned long long* pw_pack = reinterpret_cast<unsigned long long*>(smem + X.pw_pack);
  uint32_t* pw_max = reinterpret_cast<uint32_t*>(smem + X.pw_max);
  uint32_t* pw_min = reinterpret_cast<uint32_t*>(smem + X.pw_min);
  unsigned long long* reg_sum = reinterpret_cast<unsigned long long*>(smem + X.reg_sum);
  uint32_t* reg_max = reinterpret_cast<uint32_t*>(smem + X.reg_max);
  uint32_t* reg_min = reinterpret_cast<uint32_t*>(smem + X.reg_min);
  unsigned long long* as_pack = reinterpret_cast<unsigned long long*>(smem + X.as_pack);  // this workgroup's whole operations: count << 46 | sum
  uint32_t* unc = reinterpret_cast<uint32_t*>(smem + X.unc);  // two per region, one per half of a hardware wave (64-bit counts: 97 us where this takes 93)
  unsigned long long* acnt = reinterpret_cast<unsigned long long*>(smem + X.acnt);
  unsigned long long* asum = reinterpret_cast<unsigned long long*>(smem + X.asum);

  const uint32_t tid = threadIdx.x, lane = tid & 63u, hw = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t W = p.W, R = p.R, cl2 = p.cap_log2;
  const WaitsLayout SL = waits_layout(p.n_wg, W, R);

  for (uint32_t i = tid; i < R * kHistStride; i += BLOCK) hist[i] = 0;
  for (uint32_t i = tid; i < W * R * copies; i += BLOCK) { pw_pack[i] = 0; pw_max[i] = 0; pw_min[i] = 0xFFFFFFFFu; }
  for (uint32_t i = tid; i < R; i += BLOCK) {
    reg_sum[i] = 0; reg_max[i] = 0; reg_min[i] = 0xFFFFFFFFu;
    unc[2u * i] = 0; unc[2u * i + 1u] = 0; as_pack[i] = 0; acnt[i] = 0; asum[i] = 0;
  }
  // stage_workgroup's first barrier orders these stores before any use

  InFlight<UNITS> coming;
  request_workgroup<BLOCK, UNITS>(p, blockIdx.x, coming);
  uint32_t iter = 0;
  for (uint32_t wg = blockIdx.x; wg < p.n_wg; wg += gridDim.x, ++iter) {
    stage_workgroup<BLOCK, UNITS>(p, smem, L, wg, iter, coming);
    request_workgroup<BLOCK, UNITS>(p, wg + gridDim.x < p.n_wg ? wg + gridDim.x : wg, coming);
    const uint32_t live_tag = live_tag_of(iter);
    // ---- walk: `parts` hardware waves share one recorded wave, each an equal run of consecutive rounds ----
    // Nothing but the look-back crosses from one run into the next, and the staged records of the
    // earlier run are all in LDS, so the runs are independent.
    if (hw < W * parts) {
      const uint32_t w = hw / parts, part = hw - w * parts;
      const uint32_t wofs = w << cl2, V = sV[w];
      const uint32_t rounds = (V + 127u) >> 7, plen = ((rounds + parts - 1u) / parts) << 7;
      const uint32_t k0 = part * plen, k1 = V < k0 + plen ? V : k0 + plen;
      const uint32_t copy = (lane >> 4) & (copies - 1u);
      // The START of an END with region `r` at rank `at`: the nearest record of its region below `from`, if that is one.
      auto find_start = [&](uint32_t from, uint32_t r, uint32_t& clock) -> bool {
        for (uint32_t kk = from; kk-- > 0;) {
          const uint2 rq = rec[wofs + kk];
          if (!is_live(rq.y, live_tag) || (rq.y & kMRegion) != r) continue;
          clock = rq.x;
          return !(rq.y & kMEnd);
        }
        return false;
      };
      // the rank just below the round: metadata byte (kNoId: no record) and clock; for an END, its START
      uint32_t carry_id = kNoId, carry_t = 0u, carry_paired = 0u, carry_start = 0u;
      if (k0 > 0u && k0 < k1) {  // (uniform)
        const uint2 r = rec[wofs + k0 - 1u];
        if (is_live(r.y, live_tag)) {
          carry_id = r.y & 0xFFu; carry_t = r.x;
          if (carry_id & kMEnd) carry_paired = find_start(k0 - 1u, carry_id & kMRegion, carry_start) ? 1u : 0u;
        }
      }
      // A wait: the START of this lane (clock after) above an END of region `a` (clock before), which is paired with
      // a START at `begin` or not.
      auto account = [&](uint32_t a, uint32_t before, uint32_t after, bool paired, uint32_t begin) __attribute__((always_inline)) {
        const uint32_t gap = after - before;
        const uint32_t e = (w * R + a) * copies + copy;
        atomicAdd(&pw_pack[e], (1ull << 46) | (unsigned long long)gap);
        atomicMax(&pw_max[e], gap);
        atomicMin(&pw_min[e], gap);
        atomicAdd(&hist[a * kHistStride + (gap ? 31 - __clz(gap) : 0)], 1u);
        if (gap <= p.rec_cost) atomicAdd(&unc[2u * a + (lane >> 5)], 1u);
        if (paired) {
          const uint32_t whole = after - begin;
          atomicAdd(&as_pack[a], (1ull << 46) | (unsigned long long)(whole > p.rec_cost ? whole - p.rec_cost : 0u));
        }
      };
      // 128 ranks per round, two neighbours per lane.  A lane holds at most one wait (a START above a START is none).
      u32x4 next = rec2[(wofs + (k0 + 2u * lane < k1 ? k0 + 2u * lane : 0u)) >> 1];  // one round ahead, to hide the LDS latency
      for (uint32_t kb = k0; kb < k1; kb += 128) {
        const uint32_t k = kb + 2u * lane;
        const u32x4 r = next;  // {clock, metadata} of the even rank and of the odd one
        next = rec2[(wofs + (k + 128u < k1 ? k + 128u : 0u)) >> 1];
        const uint32_t id0 = k < k1 && is_live(r.y, live_tag) ? r.y & 0xFFu : kNoId;
        const uint32_t id1 = k + 1u < k1 && is_live(r.w, live_tag) ? r.w & 0xFFu : kNoId;
        const uint32_t below_id = wave_shr1(id1, carry_id), below_t = wave_shr1(r.z, carry_t);
        // is the END at either rank paired, and with a START at which clock (x ^ y == kMEnd with END x: an END over its START)
        bool paired0 = (id0 ^ below_id) == kMEnd && id0 >= kMEnd, paired1 = (id1 ^ id0) == kMEnd && id1 >= kMEnd;
        uint32_t start0 = below_t, start1 = r.x;
        const bool end0 = (id0 & ~kMRegion) == kMEnd, open0 = end0 && !paired0;
        const bool open1 = (id1 & ~kMRegion) == kMEnd && !paired1 && id1 != id0;
        // a START above an empty rank
        const bool lost0 = id0 <= kMRegion && below_id == kNoId && k > 0u, lost1 = id1 <= kMRegion && id0 == kNoId;
        uint32_t far_id = kNoId, far_t = 0u, far_start = 0u;
        bool far_paired = false;
        if (__builtin_amdgcn_ballot_w64(open0 || open1 || lost0 || lost1) != 0ull) {
          look_back(rec2, (wofs + k) >> 1, k >> 1, live_tag, open0, id0, paired0, start0, open1, id1, paired1, start1);
          if (lost0 || lost1) {
            for (uint32_t kk = k; kk-- > 0;) {  // the record below it
              const uint2 rq = rec[wofs + kk];
              if (!is_live(rq.y, live_tag)) continue;
              far_id = rq.y & 0xFFu; far_t = rq.x;
              far_paired = (far_id & kMEnd) != 0u && find_start(kk, far_id & kMRegion, far_start);
              break;
            }
          }
        }
        // of the lane below: is its odd record a paired END, and with which START
        const uint32_t below_paired = wave_shr1(paired1 ? 1u : 0u, carry_paired), below_start = wave_shr1(start1, carry_start);
        carry_id = (uint32_t)__builtin_amdgcn_readlane((int)id1, 63);
        carry_t = (uint32_t)__builtin_amdgcn_readlane((int)r.z, 63);
        carry_paired = (uint32_t)__builtin_amdgcn_readlane((int)(paired1 ? 1u : 0u), 63);
        carry_start = (uint32_t)__builtin_amdgcn_readlane((int)start1, 63);
        const bool wait1 = id1 <= kMRegion && end0;                                // START over END in this lane
        const bool wait0 = id0 <= kMRegion && (below_id & ~kMRegion) == kMEnd;  // START over the END of the lane below
        const bool far = (far_id & ~kMRegion) == kMEnd;
        if (wait0 || wait1 || far)
          account((wait1 ? id0 : far ? far_id : below_id) & kMRegion, wait1 ? r.x : far ? far_t : below_t, wait1 || lost1 ? r.z : r.x,
                  wait1 ? paired0 : far ? far_paired : below_paired != 0u, wait1 ? start0 : far ? far_start : below_start);
      }
    }
    __syncthreads();
    // ---- per-(workgroup, wave, region) output, fold into running totals ------------------------------------
    for (uint32_t e = tid; e < W * R; e += BLOCK) {
      unsigned long long pk = 0ull;
      uint32_t mx = 0u, mn = 0xFFFFFFFFu;
      for (uint32_t c = 0; c < copies; ++c) {
        const uint32_t ec = e * copies + c;
        pk += pw_pack[ec];
        mx = pw_max[ec] > mx ? pw_max[ec] : mx;
        mn = pw_min[ec] < mn ? pw_min[ec] : mn;
        pw_pack[ec] = 0; pw_max[ec] = 0; pw_min[ec] = 0xFFFFFFFFu;
      }
      const uint32_t n = (uint32_t)(pk >> 46);
      const unsigned long long s = pk & ((1ull << 46) - 1);
      uint64_t* dst = out_words + SL.per + ((size_t)wg * W * R + e) * 2;
      dst[0] = s;
      dst[1] = (uint64_t)n | ((uint64_t)mx << 32);
      if (n) {
        const uint32_t r = e % R;
        atomicAdd(&reg_sum[r], s);
        atomicMax(&reg_max[r], mx);
        atomicMin(&reg_min[r], mn);
      }
    }
    for (uint32_t r = tid; r < R; r += BLOCK) {
      acnt[r] += as_pack[r] >> 46; asum[r] += as_pack[r] & ((1ull << 46) - 1);
      as_pack[r] = 0ull;
    }
    // No barrier here: what this tail reads and resets is next touched behind the barriers of the next workgroup's
    // staging, and nothing it touches belongs to the staging.
  }
  __syncthreads();

  // ---- flush this decoder workgroup's totals --------------------------------------------------------
  unsigned long long* out = reinterpret_cast<unsigned long long*>(out_words);
  for (uint32_t i = tid; i < R * 64; i += BLOCK) {  // one region per hardware wave; its waits are the sum of its bins
    const uint32_t v = hist[(i >> 6) * kHistStride + (i & 63u)];
    if (v) atomicAdd(&out[SL.hist + i], (unsigned long long)v);
    const uint32_t n = wave_sum(v);
    if (lane == 0) hist[(i >> 6) * kHistStride + 64u] = n;
  }
  __syncthreads();
  // The seven arrays of the regions lie one behind the other: one thread per word, so that the adds of a workgroup to a
  // line are one request (an array after the other: 20000 workgroups of 4 x 32 slots 95 us where this takes 82, 9000 of
  // 3 x 1024 89 / 85).
  for (uint32_t i = tid; i < 7u * R; i += BLOCK) {
    const uint32_t array = i / R, r = i - array * R;
    const unsigned long long n = hist[r * kHistStride + 64u];
    if (!n) continue;
    unsigned long long* to = &out[SL.cnt + i];
    if (array == 2u) { atomicMin(to, (unsigned long long)reg_min[r]); continue; }
    if (array == 3u) { atomicMax(to, (unsigned long long)reg_max[r]); continue; }
    const unsigned long long v = array == 0u ? n : array == 1u ? reg_sum[r] : array == 4u ? (unsigned long long)unc[2u * r] + unc[2u * r + 1u]
                                                        : array == 5u ? acnt[r] : asum[r];
    if (v) atomicAdd(to, v);
    if (!add_head) continue;
    if (array == 0u) atomicAdd(&out[H_WAITS], v);
    if (array == 4u && v) atomicAdd(&out[H_UNCOVERED], v);
    if (array == 5u && v) atomicAdd(&out[H_ASYNC], v);
  }
}

// The three header counts are the sums of the regions'.  Either every decoder workgroup adds its own (add_head), or a
// kernel behind them makes them (2 us).  The adds of all regions go to one line, which every workgroup visits, three
// times per region: with many of either the workgroups queue up there, unless they queue up just as long at the
// regions' own sums, which an odd number of regions, 2 and 6 leave across the lines.  Measured, added / kernel, us:
// 64 decoder workgroups x 16 regions 10.4 / 10.9, x 28 + 0.4 added, x 64 + 4.2; 128 x 8 11.8 / 11.6, x 12 12.3 / 13.1; 256 x 4 17.6 / 15.5,
// x 6 17.5 / 19.0, x 7 18.4 / 19.5, x 8 17.4 / 14.4, x 16 17.8 / 15.1; 1024 x 3 45.1 / 46.9, x 4 38.6 / 29.8, x 6 38.6 / 38.8,
// x 8 39.0 / 26.4, x 9 the same either way, x 10 + 4.4 added, x 16 39.8 / 27.8.  With more than nine regions the words of all
// arrays take two hardware waves, both of which add: 3000 recorded workgroups of 4 x 256 slots x 9 regions 40.9 / 41.2, x 11
// 46.5 / 40.7, x 13 46.3 / 38.2, x 15 46.8 / 38.2.
inline bool add_head_counts(uint32_t grid, uint32_t R) {
  return R <= 20u && (grid <= 128u || (R <= 9u && ((R & 1u) != 0u || R == 2u || R == 6u)));
}
__global__ void kp_waits_head(uint64_t* out, uint32_t n_wg, uint32_t W, uint32_t R) {
  const WaitsLayout l = waits_layout(n_wg, W, R);
  const uint32_t lane = threadIdx.x & 63u, which = threadIdx.x >> 6;  // one hardware wave per count
  const size_t from = which == H_WAITS ? l.cnt : (which == H_UNCOVERED ? l.unc : l.acnt);
  unsigned long long n = 0;
  for (uint32_t r = lane; r < R; r += 64u) n += out[from + r];
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) n += __shfl_xor(n, d, 64);
  if (lane == 0) out[which] = n;
}

// Every decoder workgroup adds its totals to the same few lines at its end, one after the other: 0.03 us each.  A
// recorded workgroup takes one of them 1.9 us and as long again for some 3000 record slots.  The sum of both is least
// where the decoder workgroups are the square root of the recorded ones times the ratio of the two, however many are
// resident.  All that are resident / so many: 509 workgroups of 8 x 64 slots 31.1 / 17.9 us (184 of 509), 2046 of 8 x 16
// 31.2 / 25.2 (365 of 768), 5461 of 3 x 16 68.4 / 45.5, 1024 of 4 x 1024 52.9 / 41.5; 9000 of 3 x 1024: all 768, 87.
// (To the nearest whole number of recorded workgroups for each: of 256, where some 240 are the least sum, a few would take
// a second one: 16 x 256 slots 29.2 us, 22.7 with all 256.)
inline uint32_t most_workgroups(uint32_t n_wg, uint32_t nrec) {
  const uint32_t each = (uint32_t)(sqrt((double)n_wg / (64.0 + nrec / 48.0)) + 0.5);
  return each > 1u ? (n_wg + each - 1u) / each : n_wg;
}

template <int BLOCK, int UNITS>
kp_status launch_waits_units(const Trace& p, uint64_t* out, const WaitsLds& X, hipStream_t s) {
  // hardware waves per recorded wave: as many as the block has, while a run keeps a round of 128 ranks
  uint32_t parts = (uint32_t)BLOCK / 64u / p.W;
  if (parts > (p.cap + 127u) / 128u) parts = (p.cap + 127u) / 128u;
  auto kern = kp_waits_main<BLOCK, UNITS>;
  static thread_local LaunchCache cache;
  uint32_t grid = 0;
  const kp_status st = resident_grid(kern, BLOCK, X.total, &cache, &grid);
  if (st != KP_OK) return st;
  const uint32_t most = most_workgroups(p.n_wg, p.nrec);
  if (grid > most) grid = most;
  const bool add_head = add_head_counts(grid, p.R);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(BLOCK), X.total, s, p, out, parts, X.copies, add_head ? 1u : 0u);
  KP_HIP_TRY(hipGetLastError());
  if (!add_head) {
    hipLaunchKernelGGL(kp_waits_head, dim3(1), dim3(192), 0, s, out, p.n_wg, p.W, p.R);
    KP_HIP_TRY(hipGetLastError());
  }
  return KP_OK;
}

template <int BLOCK>
kp_status launch_waits(const Trace& p, uint64_t* out, const WaitsLds& X, hipStream_t s) {
  if constexpr (BLOCK > 256) {  // (blocks of 256 hold less than 2048 records)
    if (p.nrec > 8u * BLOCK) return launch_waits_units<BLOCK, 8>(p, out, X, s);
  }
  return launch_waits_units<BLOCK, 4>(p, out, X, s);
}

kp_status waits_impl(const void* raw, size_t n, const kp_trace_hdr& h, void* out_waits, hipStream_t s) {
  Trace p;
  const kp_status st = trace_from_header(raw, n, h, out_waits, &p);
  if (st != KP_OK) return st;
  // Copies of the sums spread the atomics of one wave; each is cleared and added up per workgroup, which only pays
  // where there are more records than entries (16380 workgroups of 16 x 16 slots, 16 regions: 213 us with 4, 194 with 1).
  uint32_t copies = 4;
  while (copies > 1 && (copies * p.W * p.R > kMaxEntries || 2u * copies * p.W * p.R > p.nrec || waits_lds(lds_layout(p.nrec).end, p.W, p.R, copies).total > kMaxLds)) copies >>= 1;
  const WaitsLds X = waits_lds(lds_layout(p.nrec).end, p.W, p.R, copies);
  if (X.total > kMaxLds)
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "wait replay needs %u B of LDS for this geometry (limit %u)", X.total, kMaxLds);

  uint64_t* out = static_cast<uint64_t*>(out_waits);
  const WaitsLayout SL = waits_layout(p.n_wg, p.W, p.R);
  int init_blocks = (int)((SL.per + 255) / 256);
  if (init_blocks > 64) init_blocks = 64;
  hipLaunchKernelGGL(kp_waits_init, dim3(init_blocks), dim3(256), 0, s, out, p.n_wg, p.W, p.R, p.cap, p.rec_cost);
  KP_HIP_TRY(hipGetLastError());
  if (p.n_wg > 0) {
    const int block = block_threads(p.W, p.nrec);
    const kp_status ls = block == 1024 ? launch_waits<1024>(p, out, X, s)
                       : block == 512  ? launch_waits<512>(p, out, X, s)
                                       : launch_waits<256>(p, out, X, s);
    if (ls != KP_OK) return ls;
  }
  return KP_OK;
}

}  // namespace

extern "C" size_t kp_waits_bytes(int n_wg, int waves_per_wg, int n_regions) {
  if (n_wg < 0 || waves_per_wg < 1 || waves_per_wg > KP_MAX_WAVES || n_regions < 1 || n_regions > 128) return 0;
  return waits_layout((uint32_t)n_wg, (uint32_t)waves_per_wg, (uint32_t)n_regions).total * 8;
}

extern "C" kp_status kp_trace_waits_hdr(const void* raw, size_t n, const kp_trace_hdr* hdr_host,
                                        void* out_waits, void* stream) {
  kp::clear_error();
  if (!raw || !hdr_host || !out_waits) return kp::fail(KP_ERR_INVALID_ARG, "NULL argument");
  return waits_impl(raw, n, *hdr_host, out_waits, static_cast<hipStream_t>(stream));
}

extern "C" kp_status kp_trace_waits(const void* raw, size_t n, void* out_waits, void* stream) {
  kp::clear_error();
  if (!raw || !out_waits) return kp::fail(KP_ERR_INVALID_ARG, "NULL argument");
  kp_trace_hdr h;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const kp_status st = kp::read_header(raw, &h, s);
  if (st != KP_OK) return st;
  return waits_impl(raw, n, h, out_waits, s);
}
