// GPU timeline rows of the trace replay (kp_trace_pairs).
//
// The paper decodes the raw profile buffer into one struct per timed region instance, which
// front ends such as Chrome Trace turn into a timeline (Sec. 3.2), and ties loop iterations to
// the records for its iteration-based timing (Sec. 3.3 "Iteration-based Timing"); records are
// stored unpaired and aligned at replay (Sec. 4.2), and a constant record cost is subtracted
// (Sec. 4.3).  This kernel does that replay on the GPU: one row {start, dur, iter, region} per
// paired START/END of a (workgroup, wave), where iter counts the earlier pairs of the same region
// in that wave.
//
// One decoder workgroup stages one recorded workgroup in LDS as (clock, metadata) pairs, ordered by
// rank.  Then the hardware waves share out the recorded waves in runs of consecutive ranks and walk them
// 128 ranks per round, two per lane (a run above rank 0 first counts the pairs below it):
//   - an END is paired iff the nearest earlier record of its region is a START: by far the most often the
//     record right below it, in the same lane or the one below (a DPP wave shift).  An END that has another record
//     below it looks further back in LDS, two ranks per step, those of a round together (look_back);
//   - its row index is the running count of paired ENDs (ballot + popcount);
//   - its iteration index is the number of pairs of its region in earlier rounds, a counter in LDS, plus those in
//     lower lanes.
// What bounds it: instruction issue (one workgroup of this size per CU at a time, 16 hardware waves), then HBM.  So
// the next workgroup's records travel under the walk, and a lane takes two ranks: of a START and an END only one
// makes a row.  Measured on 4096 workgroups of 8 waves x 2048 records (0.54 GB read, 0.53 GB written): 495 us with
// the loads waited for, four ranks of look-back per record and byte-wide counters scanned over the lanes; 341 us
// with the loads ahead and ballots in their place, one rank per lane; 270 us with two; 245 us (4.4 TB/s) with what
// follows from the hardware wave's index in scalar registers and no code for more than two parts.  With 0.1 % of the records
// displaced 272 us, 260 with staging in fewer instructions, 250 with the lanes below counted by mbcnt and the region's bits
// matched three operands at a time.  (Non-temporal stores of the rows: 252 us, and whoever reads them next takes 15 % longer.)
#include "kp_stage.h"

namespace {

using namespace kp_stage;

constexpr uint32_t kBelowStride = 128;  // one counter per region
constexpr uint32_t kNoId = 0xFFFFu;     // END << 7 | region of no record

// First of the rounds that part i of n emits.  Of two parts the second also counts the pairs of the rounds below its run,
// which takes about two fifths of the time of emitting them where the regions follow one another: it gets three
// fifths of what the first one gets.  Three and more are equal and count their own rounds ahead of emitting them.
inline float share_of(uint32_t n) { return n == 2u ? 0.625f : 1.0f / (float)n; }
__device__ __forceinline__ uint32_t run_start(uint32_t rounds, uint32_t i, uint32_t n, float share) {
  return i >= n ? rounds : (uint32_t)((float)rounds * ((float)i * share) + 0.5f);
}

struct PairsOut {
  uint32_t* count;  // pairs per (workgroup, wave)
  u32x4* rows;      // cap/2 rows per (workgroup, wave)
};

// SHARED: more than two parts.
template <int BLOCK, int UNITS, bool SHARED>
__global__ __launch_bounds__(BLOCK) void kp_pairs_main(Trace p, PairsOut o, uint32_t parts, float share) {
  extern __shared__ __align__(16) unsigned char smem[];
  const Lds L = lds_layout(p.nrec);
  const u32x4* rec2 = reinterpret_cast<const u32x4*>(smem + L.rec);
  const uint32_t* sV = reinterpret_cast<const uint32_t*>(smem + L.v);
  uint32_t* below = reinterpret_cast<uint32_t*>(smem + L.end);  // per hardware wave: pairs per region below its run

  const uint32_t tid = threadIdx.x, lane = tid & 63u, hw = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t W = p.W, R = p.R, cap = p.cap, cl2 = p.cap_log2;
  uint32_t region_bits = 0; while ((1u << region_bits) < R) ++region_bits;
  const unsigned long long lt_mask = (1ull << lane) - 1ull;

  // the padding entries of the count array are part of the output: zero
  if (blockIdx.x == 0 && tid < ((0u - p.n_wg * W) & 3u)) o.count[(size_t)p.n_wg * W + tid] = 0u;

  InFlight<UNITS> coming;
  request_workgroup<BLOCK, UNITS>(p, blockIdx.x, coming);
  uint32_t iter = 0;
  for (uint32_t wg = blockIdx.x; wg < p.n_wg; wg += gridDim.x, ++iter) {
    stage_workgroup<BLOCK, UNITS>(p, smem, L, wg, iter, coming);
    request_workgroup<BLOCK, UNITS>(p, wg + gridDim.x < p.n_wg ? wg + gridDim.x : wg, coming);
    const uint32_t live_tag = live_tag_of(iter);
    // ---- walk: `parts` hardware waves share one recorded wave -------------------------------------------
    // Each emits the rows of a run of consecutive ranks, whose row and iteration indices continue those of the runs below.
    // Of two, the second counts the pairs below its run (in all and per region) with the same pairing rounds, and no wave
    // waits for another.  Of more, each counts those of its own run and adds up the runs below it: (1 + c) / n of the time
    // that one wave would need to emit all, c / (1 - (1 - c)^n) where each counts all runs below (c: the time of
    // counting a round over that of emitting it, 2/5 where regions follow one another, 4/5 and more where they lie inside one
    // another).  Each counting all below / its own: 512 workgroups of 1 x 16384 slots 113 / 42 us, regions three deep 277 / 68;
    // 2000 of 5 x 2048, three parts, 93.7 / 91.6 and 177 / 159.
    if (SHARED || hw < W * parts) {
      const bool walks = !SHARED || hw < W * parts;  // (a hardware wave without a run comes along to the barriers)
      const uint32_t w = walks ? hw / parts : 0u, part = walks ? hw - w * parts : 0u;
      const uint32_t wofs = w << cl2, V = walks ? sV[w] : 0u;
      const uint32_t rounds = (V + 127u) >> 7;
      const uint32_t k0 = run_start(rounds, part, parts, share) << 7, k_next = run_start(rounds, part + 1u, parts, share) << 7;
      const uint32_t k1 = V < k_next ? V : k_next;  // this wave emits ranks [k0, k1)
      const uint32_t c0 = SHARED ? k0 : 0u;         // and counts ranks [c0, c1)
      const uint32_t c1 = !SHARED ? (V < k0 ? V : k0) : (part + 1u < parts ? k1 : k0);
      uint32_t* seen = below + hw * kBelowStride;    // pairs of each region so far
      seen[lane] = 0u; seen[64u + lane] = 0u;        // (LDS operations of one wave complete in order)
      u32x4* my_rows = o.rows + ((size_t)wg * W + w) * (cap / 2);
      uint32_t n_rows = 0;
      uint32_t carry_id = kNoId, carry_t = 0u;  // the rank just below the round: metadata byte (kNoId: none) and clock
      // 128 ranks from kb, two neighbours per lane: which of this lane's are ENDs that are paired, and with what.
      uint32_t id0 = kNoId, id1 = kNoId, start0 = 0u, start1 = 0u;
      u32x4 r = {0u, 0u, 0u, 0u};  // {clock, metadata} of the even rank and of the odd one
      u32x4 next;  // one round ahead, to hide the LDS latency
      auto start_at = [&](uint32_t kb) __attribute__((always_inline)) {
        const uint32_t k = kb + 2u * lane;
        next = rec2[(wofs + (k < V ? k : 0u)) >> 1];
        if (kb != 0u && kb < V) {  // (uniform)
          const u32x4 under = rec2[(wofs + kb - 2u) >> 1];
          carry_id = is_live(under.w, live_tag) ? under.w & 0xFFu : kNoId;
          carry_t = under.z;
        }
      };
      start_at(c0);
      auto pair_128 = [&](uint32_t kb, uint32_t k_end, bool& paired0, bool& paired1) __attribute__((always_inline)) {
        const uint32_t k = kb + 2u * lane;
        r = next;
        next = rec2[(wofs + (k + 128u < V ? k + 128u : 0u)) >> 1];
        id0 = k < k_end && is_live(r.y, live_tag) ? r.y & 0xFFu : kNoId;
        id1 = k + 1u < k_end && is_live(r.w, live_tag) ? r.w & 0xFFu : kNoId;
        const uint32_t below_id = wave_shr1(id1, carry_id);
        start0 = wave_shr1(r.z, carry_t); start1 = r.x;
        carry_id = (uint32_t)__builtin_amdgcn_readlane((int)id1, 63);
        carry_t = (uint32_t)__builtin_amdgcn_readlane((int)r.z, 63);
        // an END carries kMEnd above its region, no record neither: x ^ y == kMEnd says "END over its START"
        paired0 = (id0 ^ below_id) == kMEnd && id0 >= kMEnd;
        paired1 = (id1 ^ id0) == kMEnd && id1 >= kMEnd;
        const bool open0 = (id0 & ~kMRegion) == kMEnd && !paired0;
        const bool open1 = (id1 & ~kMRegion) == kMEnd && !paired1 && id1 != id0;
        if (__builtin_amdgcn_ballot_w64(open0 || open1) != 0ull)
          look_back(rec2, (wofs + k) >> 1, k >> 1, live_tag, open0, id0, paired0, start0, open1, id1, paired1, start1);
      };
      // ---- count ------------------------------------------------------------------------------------------
      for (uint32_t kb = c0; kb < c1; kb += 128) {  // c1 is a multiple of 128 or the end of the wave
        bool paired0, paired1;
        pair_128(kb, c1, paired0, paired1);
        n_rows += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(paired0)) + (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(paired1));
        if (paired0) atomicAdd(&seen[id0 & kMRegion], 1u);
        if (paired1) atomicAdd(&seen[id1 & kMRegion], 1u);
      }
      if constexpr (SHARED) {
        __syncthreads();  // all runs are counted
        uint32_t lo = 0u, hi = 0u;
        for (uint32_t i = 0; i < part; ++i) {
          const uint32_t* of = seen - (part - i) * kBelowStride;
          lo += of[lane]; hi += of[64u + lane];
        }
        __syncthreads();  // and read by all that need them
        seen[lane] = lo; seen[64u + lane] = hi;
        n_rows = wave_total(lo + hi);
        carry_id = kNoId;  // (rank 0 has nothing below it)
        start_at(k0);
      }
      // ---- emit the rows of this run ------------------------------------------------------------------------
      auto row = [&](uint32_t j, uint32_t start, uint32_t end, uint32_t it, uint32_t region) __attribute__((always_inline)) {
        const uint32_t d_raw = end - start;
        my_rows[j] = u32x4{start, d_raw > p.rec_cost ? d_raw - p.rec_cost : 0u, it, region};
      };
      for (uint32_t kb = k0; kb < k1; kb += 128) {
        bool paired0, paired1;
        pair_128(kb, k1, paired0, paired1);
        const uint64_t pb0 = __builtin_amdgcn_ballot_w64(paired0), pb1 = __builtin_amdgcn_ballot_w64(paired1);
        // iteration index: pairs of this region in earlier rounds + on lower ranks of this round
        if ((pb0 & pb1) == 0ull) {  // at most one pair per lane (always so where every START is right below its END)
          const bool paired = paired0 || paired1;
          const uint32_t region = (paired1 ? id1 : id0) & kMRegion;
          const uint64_t pb = pb0 | pb1;
          uint32_t same_lo = (uint32_t)pb, same_hi = (uint32_t)(pb >> 32);  // the lanes whose pair has this lane's region
          for (uint32_t b = 0; b < region_bits; ++b) {
            const uint32_t bit = (uint32_t)__builtin_amdgcn_sbfe((int)region, b, 1u);  // 0 or all ones
            const uint64_t set = __builtin_amdgcn_ballot_w64(bit != 0u);
            same_lo &= ~((uint32_t)set ^ bit); same_hi &= ~((uint32_t)(set >> 32) ^ bit);
          }
          if (paired) {
            const uint32_t lower = __builtin_amdgcn_mbcnt_hi(same_hi, __builtin_amdgcn_mbcnt_lo(same_lo, 0u));
            const uint32_t it = seen[region] + lower;
            if ((uint32_t)(__popc(same_lo) + __popc(same_hi)) == lower + 1u) seen[region] = it + 1u;  // the region's last pair of the round
            row(__builtin_amdgcn_mbcnt_hi((uint32_t)(pb >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)pb, n_rows)),
                paired1 ? start1 : start0, paired1 ? r.z : r.x, it, region);
          }
          n_rows += (uint32_t)__popcll(pb);
        } else {
          uint64_t even0 = pb0, odd0 = pb1, even1 = pb0, odd1 = pb1;  // the pairs of even and of odd ranks with the region of this lane's even, odd rank
          for (uint32_t b = 0; b < region_bits; ++b) {
            const uint64_t even = __builtin_amdgcn_ballot_w64((id0 >> b) & 1u), odd = __builtin_amdgcn_ballot_w64((id1 >> b) & 1u);
            const uint64_t flip0 = ((id0 >> b) & 1u) ? 0ull : ~0ull, flip1 = ((id1 >> b) & 1u) ? 0ull : ~0ull;
            even0 &= even ^ flip0; odd0 &= odd ^ flip0;
            even1 &= even ^ flip1; odd1 &= odd ^ flip1;
          }
          const uint32_t j = n_rows + (uint32_t)__popcll(pb0 & lt_mask) + (uint32_t)__popcll(pb1 & lt_mask);
          const uint64_t le_mask = 2ull * lt_mask + 1ull;
          if (paired0)
            row(j, start0, r.x, seen[id0 & kMRegion] + (uint32_t)__popcll(even0 & lt_mask) + (uint32_t)__popcll(odd0 & lt_mask), id0 & kMRegion);
          if (paired1)
            row(j + (paired0 ? 1u : 0u), start1, r.z, seen[id1 & kMRegion] + (uint32_t)__popcll(even1 & le_mask) + (uint32_t)__popcll(odd1 & lt_mask), id1 & kMRegion);
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (LDS operations of one wave complete in order)
          if (paired0) atomicAdd(&seen[id0 & kMRegion], 1u);
          if (paired1) atomicAdd(&seen[id1 & kMRegion], 1u);
          n_rows += (uint32_t)__popcll(pb0) + (uint32_t)__popcll(pb1);
        }
      }
      // the wave with the last run knows the total
      if (lane == 0 && walks && part + 1u == parts) o.count[(size_t)wg * W + w] = n_rows;
    }
    __syncthreads();
  }
}

// Blocks of 256: six per CU.  Seven or eight, which the registers and the LDS of small rings leave room for, are slower
// (8, 7, 6, 5, 4 per CU): 10000 workgroups of 1 x 256 slots 22.9, 22.8, 18.9, 20.8, 22.6 us, 40000 of 2 x 32 68.8, 68.7, 56.2,
// 60.1, 66.0, 20000 of 1 x 1024 96.2, 96.1, 87.1, 89.6, 96.2; with two or three turns each 5000 of 4 x 256 26.9 / 27.5.
template <int BLOCK> constexpr int kMostPerCu = BLOCK == 256 ? 6 : 32;

template <int BLOCK, int UNITS, bool SHARED>
kp_status launch_pairs_parts(const Trace& p, const PairsOut& o, uint32_t lds_bytes, uint32_t parts, hipStream_t s) {
  auto kern = kp_pairs_main<BLOCK, UNITS, SHARED>;
  static thread_local LaunchCache cache;
  uint32_t grid = 0;
  const kp_status st = resident_grid(kern, BLOCK, lds_bytes, &cache, &grid, kMostPerCu<BLOCK>);
  if (st != KP_OK) return st;
  if (grid > p.n_wg) grid = p.n_wg;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(BLOCK), lds_bytes, s, p, o, parts, share_of(parts));
  KP_HIP_TRY(hipGetLastError());
  return KP_OK;
}

template <int BLOCK, int UNITS>
kp_status launch_pairs_units(const Trace& p, const PairsOut& o, uint32_t lds_bytes, hipStream_t s) {
  // hardware waves per recorded wave: as many as the block has, while a run keeps a round of 128 ranks
  uint32_t parts = (uint32_t)BLOCK / 64u / p.W;
  if (parts > (p.cap + 127u) / 128u) parts = (p.cap + 127u) / 128u;
  if constexpr (BLOCK != 512 || UNITS != 8) {  // (blocks of 512 cut one or two waves into more than two: 4096 records at most)
    if (parts > 2u) return launch_pairs_parts<BLOCK, UNITS, true>(p, o, lds_bytes, parts, s);
  }
  return launch_pairs_parts<BLOCK, UNITS, false>(p, o, lds_bytes, parts, s);
}

template <int BLOCK>
kp_status launch_pairs(const Trace& p, const PairsOut& o, uint32_t lds_bytes, hipStream_t s) {
  if constexpr (BLOCK > 256) {  // (blocks of 256 hold less than 2048 records)
    if (p.nrec > 8u * BLOCK) return launch_pairs_units<BLOCK, 8>(p, o, lds_bytes, s);
  }
  return launch_pairs_units<BLOCK, 4>(p, o, lds_bytes, s);
}

size_t count_bytes(size_t n_seg) { return ((n_seg + 3) / 4) * 16; }

kp_status pairs_impl(const void* raw, size_t n, const kp_trace_hdr& h, void* out_pairs, hipStream_t s) {
  Trace p;
  const kp_status st = trace_from_header(raw, n, h, out_pairs, &p);
  if (st != KP_OK) return st;
  const int block = block_threads(p.W, p.nrec);
  const uint32_t lds = lds_layout(p.nrec).end + (uint32_t)(block / 64) * kBelowStride * 4u;
  if (lds > kMaxLds)
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "timeline kernel needs %u B of LDS for this geometry (limit %u)", lds, kMaxLds);
  if (h.n_wg == 0) return KP_OK;

  uint8_t* out = static_cast<uint8_t*>(out_pairs);
  PairsOut o;
  o.count = reinterpret_cast<uint32_t*>(out);
  o.rows = reinterpret_cast<u32x4*>(out + count_bytes((size_t)p.n_wg * p.W));
  return block == 1024 ? launch_pairs<1024>(p, o, lds, s)
       : block == 512  ? launch_pairs<512>(p, o, lds, s)
                       : launch_pairs<256>(p, o, lds, s);
}

}  // namespace

extern "C" size_t kp_pairs_bytes(int n_wg, int waves_per_wg, int cap_per_wg) {
  if (n_wg < 0 || waves_per_wg < 1 || waves_per_wg > KP_MAX_WAVES || cap_per_wg < 0 || cap_per_wg % waves_per_wg) return 0;
  const size_t n_seg = (size_t)n_wg * waves_per_wg, cap_wave = (size_t)cap_per_wg / waves_per_wg;
  return count_bytes(n_seg) + n_seg * (cap_wave / 2) * sizeof(kp_pair_row);
}

extern "C" kp_status kp_trace_pairs_hdr(const void* raw, size_t n, const kp_trace_hdr* hdr_host,
                                        void* out_pairs, void* stream) {
  kp::clear_error();
  if (!raw || !hdr_host || !out_pairs) return kp::fail(KP_ERR_INVALID_ARG, "NULL argument");
  return pairs_impl(raw, n, *hdr_host, out_pairs, static_cast<hipStream_t>(stream));
}

extern "C" kp_status kp_trace_pairs(const void* raw, size_t n, void* out_pairs, void* stream) {
  kp::clear_error();
  if (!raw || !out_pairs) return kp::fail(KP_ERR_INVALID_ARG, "NULL argument");
  kp_trace_hdr h;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const kp_status st = kp::read_header(raw, &h, s);
  if (st != KP_OK) return st;
  return pairs_impl(raw, n, h, out_pairs, s);
}
