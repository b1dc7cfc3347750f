// Staging of one recorded workgroup in LDS, shared by the replay kernels that walk the records of
// each wave in order (timeline rows, asynchronous waits).
//
// The paper stores START/END records unpaired, per warp, in a ring whose tail survives, and aligns
// them at trace replay (Sec. 4.2 "SM-level Data Layout", "Shared Memory Circular Buffer"; Sec. 4.3).
// Here every record goes to position wave * cap_wave + rank, rank = seq - first surviving seq, as a
// (clock, metadata) pair, which undoes ring rotation and out-of-order flushes in O(1) per record.
// A sequence number that occurs twice must leave the later slot in place: only a record outside the
// slot of its seq can share it with another, so those are placed behind the others, by an exchange
// that says whether the rank was taken, and a workgroup with such a pair is scattered again.
// What bounds the scatter is instruction issue: where 128 records cannot belong to more than one
// recorded wave, everything about it is uniform and read from the lanes that hold the header's
// counts, and units without records are left out.
// Against every record placed as it came and the occupied ranks counted where one was displaced, wave, capacity and
// first seq read from LDS by every unit: 4096 workgroups of 8 x 2048 records, 0.1 % displaced, timeline 289 / 282 us, waits
// 224 / 211; waits of 9000 of 3 x 1024, partly filled, 90 / 88, 3000 of 16 x 512 88 / 84, 1000 of 12 x 512 31.6 / 31.0.
#pragma once
#include "kp_common.h"
#include "kp_wave.h"

namespace kp_stage {

using namespace kp_wave;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kSeqMask = 0xFFFFFu;
// staged metadata: bits 6:0 region, 7 END, 8 valid, 31:16 generation of the staging pass
constexpr uint32_t kMRegion = 0x7Fu, kMEnd = 0x80u, kMValid = 0x100u;
constexpr uint32_t kLiveMask = 0xFFFF0000u | kMValid;
constexpr uint32_t kMaxRecPerWg = 16384;
constexpr uint32_t kMaxLds = 160 * 1024;

struct Trace {
  const uint32_t* wg_hdrs;  // 32 words per recorded workgroup
  const u32x4* records;     // two records per 16-byte load
  uint32_t n_wg, W, R, cap, cap_log2, rec_cost, flush, nrec;
};

// LDS of the staging step: byte offsets from the start of dynamic shared memory.
struct Lds { uint32_t rec, tmp, v, first, end; };
__host__ __device__ inline uint32_t align16(uint32_t x) { return (x + 15u) & ~15u; }
__host__ __device__ inline Lds lds_layout(uint32_t nrec) {
  Lds l;
  uint32_t o = 0;
  l.rec = o; o = align16(o + nrec * 8);
  l.tmp = o; o = align16(o + 4 * 4);     // by parity of the pass: [0, 1] some seq occurs twice, [2, 3] a record outside the slot of its seq
  l.v = o; o = align16(o + 16 * 4);      // records held per wave
  l.first = o; o = align16(o + 16 * 4);  // first surviving seq per wave
  l.end = o;
  return l;
}

__device__ inline uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// The metadata tag of the records staged in pass `iter` of a persistent workgroup.  A staged word
// counts only if it carries the generation of its pass, so the staging area is cleared on the
// first pass and when the 16-bit generation wraps, not for every recorded workgroup.
__device__ __forceinline__ uint32_t live_tag_of(uint32_t iter) { return ((1u + iter % 0xFFFFu) << 16) | kMValid; }
__device__ __forceinline__ bool is_live(uint32_t m, uint32_t live_tag) { return (m & kLiveMask) == live_tag; }

// ENDs of two neighbouring ranks k and k + 1 (k even) whose START is not the record right below them: each looks for
// the nearest record of its region among the ranks below k, two ranks per step.  `at` is the index of ranks k, k + 1
// in rec2, `below` = k / 2; id is END << 7 | region, and a record found settles paired and start.
// An END inside another region looks three ranks back, so one iteration of two steps, which travel together, settles a
// round of regions inside regions.  A round that took them one per lane and asked for the lanes of a region with one
// ballot per bit, further back one lane at a time, against this: 1024 workgroups of 8 x 2048 records, regions three deep,
// timeline 199 / 117 us, waits 135 / 77; one region around 20 others 556 / 318 and 329 / 163.  Steps in fours: 126 us where
// two take 111; one END of a lane after the other: 133 us where both together take 117.
__device__ __forceinline__ void look_back(const u32x4* rec2, uint32_t at, uint32_t below, uint32_t live_tag, bool open0, uint32_t id0,
                                          bool& paired0, uint32_t& start0, bool open1, uint32_t id1, bool& paired1, uint32_t& start1) {
  constexpr uint32_t kSame = kLiveMask | kMRegion;
  if (!(open0 || open1) || below == 0u) return;
  const uint32_t want0 = live_tag | (id0 & kMRegion), want1 = live_tag | (id1 & kMRegion);
  for (uint32_t s = 1; s <= below && (open0 || open1); s += 2u) {
    const u32x4 va = rec2[at - s], vb = rec2[at - (s < below ? s + 1u : s)];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const u32x4 v = h ? vb : va;
      const bool odd0 = ((v.w ^ want0) & kSame) == 0u, odd1 = ((v.w ^ want1) & kSame) == 0u;
      if (open0 && (odd0 || ((v.y ^ want0) & kSame) == 0u)) {
        paired0 = ((odd0 ? v.w : v.y) & kMEnd) == 0u; start0 = odd0 ? v.z : v.x; open0 = false;
      }
      if (open1 && (odd1 || ((v.y ^ want1) & kSame) == 0u)) {
        paired1 = ((odd1 ? v.w : v.y) & kMEnd) == 0u; start1 = odd1 ? v.z : v.x; open1 = false;
      }
    }
  }
}

// The records of a recorded workgroup on their way to LDS: a thread's share in 16-byte units of two records
// (block_threads() makes it at most 8) and the header's record count of wave `thread`.  A persistent
// kernel requests the next workgroup before it walks the one in LDS, so that the loads travel under the walk
// (timeline of 4096 workgroups of 16384 records, one of them per CU at a time: 495 us with the loads waited
// for where they were issued).
// UNITS of them per thread, 4 where that is enough (a third more hardware waves fit a CU's registers).
// The thread index, opaque to the optimiser: without it the addresses of all units are computed once ahead of
// the loop over the workgroups and held in registers through the walks.
__device__ __forceinline__ uint32_t fresh_tid() { uint32_t t = threadIdx.x; asm volatile("" : "+v"(t)); return t; }
template <int UNITS> struct InFlight { u32x4 v[UNITS]; uint32_t total; };
template <int BLOCK, int UNITS>
__device__ __forceinline__ void request_workgroup(const Trace& p, uint32_t wg, InFlight<UNITS>& f) {
  const u32x4* recs = p.records + (size_t)wg * (p.nrec / 2);
  const uint32_t tid = fresh_tid(), n16 = p.nrec / 2;
  f.total = p.wg_hdrs[(size_t)32 * wg + 8 + (tid & 15u)];  // (first: staging begins with it)
#pragma unroll
  for (int u = 0; u < UNITS; ++u) {
    if (u * BLOCK >= n16) break;  // (uniform)
    const uint32_t i = tid + u * BLOCK;
    f.v[u] = __builtin_nontemporal_load(recs + (i < n16 ? i : n16 - 1u));
  }
}

// Stages the requested workgroup `wg`.  Every thread of the block calls it; it ends with a barrier, after
// which rec[w * cap + k] holds the record of rank k of wave w (live iff its metadata carries
// live_tag) and sV[w] the number of ranks of wave w.  The caller must put a barrier between its last
// read of the staging area and the next call.
template <int BLOCK, int UNITS>
__device__ __forceinline__ void stage_workgroup(const Trace& p, unsigned char* smem, const Lds& L, uint32_t wg,
                                                uint32_t iter, const InFlight<UNITS>& f) {
  uint2* rec = reinterpret_cast<uint2*>(smem + L.rec);
  uint32_t* recw = reinterpret_cast<uint32_t*>(smem + L.rec);  // word 2p = clock, 2p+1 = metadata
  uint32_t* tmp = reinterpret_cast<uint32_t*>(smem + L.tmp);
  uint32_t* sV = reinterpret_cast<uint32_t*>(smem + L.v);
  uint32_t* sFirst = reinterpret_cast<uint32_t*>(smem + L.first);
  const uint32_t tid = fresh_tid(), lane = tid & 63u;
  const uint32_t W = p.W, R = p.R, cap = p.cap, nrec = p.nrec, capm = cap - 1, cl2 = p.cap_log2;
  const uint32_t live_tag = live_tag_of(iter);
  uint32_t* const twice = tmp + (iter & 1u);         // some seq occurs twice
  uint32_t* const displaced = tmp + 2u + (iter & 1u);  // a record is not in the slot of its seq

  if ((live_tag >> 16) == 1u) {
    u32x4* z = reinterpret_cast<u32x4*>(rec);
    for (uint32_t i = tid; i < nrec / 2; i += BLOCK) z[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid < 4u) tmp[tid] = 0u;
    __syncthreads();
  }
  if (tid < 16u) {
    const uint32_t T = tid < W ? f.total : 0u;
    const uint32_t V = T < cap ? T : cap;
    sV[tid] = V;
    sFirst[tid] = p.flush ? 0u : T - V;
  }
  if (tid == 64u) { tmp[(iter + 1u) & 1u] = 0u; tmp[2u + ((iter + 1u) & 1u)] = 0u; }  // the flags of the next pass
  // ---- scatter by rank --------------------------------------------------------------------------
  // Records in the slot of their own seq have distinct seq modulo the ring size, hence distinct ranks.  The others
  // (bit 2u + h of `moved`: record h of unit u) wait until those are in place.
  uint32_t moved = 0;
  // Two neighbouring records from slot s0 of recorded wave w, which holds V records, from seq `first` on.
  auto accept = [&](int u, uint32_t w, uint32_t V, uint32_t first, uint32_t s0) __attribute__((always_inline)) {
#pragma unroll
    for (uint32_t h = 0; h < 2u; ++h) {
      const uint32_t tag = h ? f.v[u].z : f.v[u].x, pay = h ? f.v[u].w : f.v[u].y;
      const uint32_t k = (tag - first) & kSeqMask;  // the low 20 bits of tag - first are those of seq - first
      const bool good = s0 + h < V && k < V && ((tag >> 20) & 0xFu) == w && ((tag >> 24) & 0x7Fu) < R;
      const bool home = ((tag ^ (s0 + h)) & capm) == 0u;
      if (good && home) rec[(w << cl2) + k] = make_uint2(pay, (tag >> 24) | live_tag);  // region and END flag sit in the tag as in the metadata
      moved |= good && !home ? 1u << (2u * (uint32_t)u + h) : 0u;
    }
  };
  const uint32_t n16 = nrec / 2;
  const uint32_t hw = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  // Hardware waves without a record leave at once: of 64 slots only one wave has any (waits of 65535 workgroups of 2 x 32
  // slots 124 / 118 us, 60000 of 4 x 16 126 / 118; timeline of the former 88 / 79).
  if (cap >= 128u && nrec > 256u) {  // the 128 records of a hardware wave's unit are one recorded wave's: all about it is uniform (65535 workgroups of 2 x 128: 129.6 / 128.1 the other way)
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      if (u * BLOCK >= n16) break;  // (uniform)
      const uint32_t f0 = 128u * (hw + u * (BLOCK / 64)), w = f0 >> cl2;
      if (f0 >= nrec) break;
      const uint32_t T = (uint32_t)__builtin_amdgcn_readlane((int)f.total, (int)w);
      const uint32_t V = T < cap ? T : cap;
      if ((f0 & capm) < V) accept(u, w, V, p.flush ? 0u : T - V, (f0 & capm) + 2u * lane);
    }
  } else {
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      if (128u * (hw + u * (BLOCK / 64)) >= nrec) break;
      const uint32_t f0 = 2u * (tid + u * BLOCK), w = f0 < nrec ? f0 >> cl2 : 0u;
      const uint32_t T = (uint32_t)__shfl((int)f.total, (int)w, 64);
      const uint32_t V = f0 < nrec ? (T < cap ? T : cap) : 0u;
      accept(u, w, V, p.flush || T < cap ? 0u : T - cap, f0 & capm);
    }
  }
  if (moved != 0u) *displaced = 1u;  // (asked of the wave by a ballot: 1 % slower)
  __syncthreads();
  if (*displaced == 0u) return;
  // ---- the others: one whose rank is taken shares its seq with another record --------------------------
  {
    bool taken = false;
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
#pragma unroll
      for (uint32_t h = 0; h < 2u; ++h) {
        if (!((moved >> (2u * (uint32_t)u + h)) & 1u)) continue;
        const uint32_t tag = h ? f.v[u].z : f.v[u].x, w = 2u * (tid + u * BLOCK) >> cl2;
        const uint32_t at = (w << cl2) + ((tag - sFirst[w]) & kSeqMask);
        taken = is_live(atomicExch(&recw[2u * at + 1u], (tag >> 24) | live_tag), live_tag) || taken;
        recw[2u * at] = h ? f.v[u].w : f.v[u].y;
      }
    }
    if (taken) *twice = 1u;
  }
  __syncthreads();
  if (*twice != 0u) {
    // Rare: some seq occurs twice.  The later slot must win, so redo this workgroup's scatter: the metadata words take the
    // largest slot of their rank first (a slot's number stays below every live tag), and the records of those slots follow.
    // 512 workgroups of 1 x 2048 slots, two such records each: timeline 301 and
    // waits 880 us with one thread per wave in slot order, 15 and 33 us this way.
    __syncthreads();
    for (uint32_t i = tid; i < nrec; i += BLOCK) recw[2 * i + 1] = 0;
    const uint2* recs = reinterpret_cast<const uint2*>(p.records) + (size_t)wg * nrec;
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
      __syncthreads();
      for (uint32_t i = tid; i < nrec; i += BLOCK) {
        const uint2 r = recs[i];
        const uint32_t w = i >> cl2, s = i & capm, V = sV[w], k = (r.x - sFirst[w]) & kSeqMask;
        if (s >= V || k >= V || ((r.x >> 20) & 0xFu) != w || ((r.x >> 24) & 0x7Fu) >= R) continue;
        uint32_t* meta = &recw[2u * ((w << cl2) + k) + 1u];
        if (pass == 0) atomicMax(meta, s + 1u);
        else if (*meta == s + 1u) rec[(w << cl2) + k] = make_uint2(r.y, (r.x >> 24) | live_tag);
      }
    }
    __syncthreads();
  }
}

// Host-side checks common to the replay entry points; fills `t` from a validated header.
inline kp_status trace_from_header(const void* raw, size_t n, const kp_trace_hdr& h, const void* out, Trace* t) {
  if (h.magic != KP_TRACE_MAGIC || h.version != KP_TRACE_VERSION)
    return kp::fail(KP_ERR_BAD_TRACE, "trace header: bad magic/version (%08x, %u)", h.magic, h.version);
  if (h.waves_per_wg < 1 || h.waves_per_wg > KP_MAX_WAVES || h.n_regions < 1 || h.n_regions > 128 ||
      !kp::is_pow2(h.cap_wave) || h.cap_wave < 2)
    return kp::fail(KP_ERR_BAD_TRACE, "trace header: waves=%u regions=%u cap_wave=%u", h.waves_per_wg, h.n_regions, h.cap_wave);
  if ((size_t)h.n_wg * h.waves_per_wg * h.cap_wave != n)
    return kp::fail(KP_ERR_BAD_TRACE, "trace header describes %zu record slots, caller passed %zu",
                    (size_t)h.n_wg * h.waves_per_wg * h.cap_wave, n);
  if ((h.flags & ~(KP_FLAG_FLUSH | KP_FLAG_REALTIME | KP_FLAG_HW_IDS)) != 0) return kp::fail(KP_ERR_BAD_TRACE, "trace header: unknown flags %x", h.flags);
  const uint32_t nrec = h.waves_per_wg * h.cap_wave;
  if (nrec > kMaxRecPerWg)
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "%u records per workgroup exceed the LDS staging limit %u", nrec, kMaxRecPerWg);
  if (((uintptr_t)raw & 15u) || ((uintptr_t)out & 15u))
    return kp::fail(KP_ERR_INVALID_ARG, "raw and the output block must be 16-byte aligned");
  const uint8_t* base = static_cast<const uint8_t*>(raw);
  t->wg_hdrs = reinterpret_cast<const uint32_t*>(base + sizeof(kp_trace_hdr));
  t->records = reinterpret_cast<const u32x4*>(base + sizeof(kp_trace_hdr) + sizeof(kp_wg_hdr) * (size_t)h.n_wg);
  t->n_wg = h.n_wg; t->W = h.waves_per_wg; t->R = h.n_regions; t->cap = h.cap_wave;
  t->cap_log2 = 0; while ((1u << t->cap_log2) < h.cap_wave) ++t->cap_log2;
  t->rec_cost = h.rec_cost; t->flush = h.flags & KP_FLAG_FLUSH; t->nrec = nrec;
  return KP_OK;
}

// One hardware wave per recorded wave, and enough threads to stage the records in 8 units each.
inline int block_threads(uint32_t W, uint32_t nrec) {
  return (W > 8 || nrec >= 8192) ? 1024 : ((W > 4 || nrec >= 2048) ? 512 : 256);
}

// Grid of a persistent kernel: as many workgroups as stay resident, and not more than `most_per_cu` of them.
struct LaunchCache { int dev = -1; uint32_t lds = 0; uint32_t max_grid = 0; };
template <typename Kernel>
kp_status resident_grid(Kernel kern, int block, uint32_t lds_bytes, LaunchCache* cache, uint32_t* grid, int most_per_cu = 32) {
  int dev = 0;
  KP_HIP_TRY(hipGetDevice(&dev));
  if (cache->dev != dev || cache->lds != lds_bytes) {
    KP_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes));
    int per_cu = 0, cus = 0;
    KP_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, block, lds_bytes));
    if (per_cu < 1) return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "replay kernel does not fit one CU (LDS %u B)", lds_bytes);
    KP_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    cache->dev = dev; cache->lds = lds_bytes; cache->max_grid = (uint32_t)(per_cu < most_per_cu ? per_cu : most_per_cu) * (uint32_t)cus;
  }
  *grid = cache->max_grid;
  return KP_OK;
}

}  // namespace kp_stage
