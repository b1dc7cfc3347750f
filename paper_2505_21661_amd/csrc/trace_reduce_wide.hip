// Statistics decoder for wide geometries: more than 32 regions (the tag holds 128) or more records
// per workgroup than the LDS-resident decoder stages at once.
//
// Same replay as there (Sec. 4.2: per-wave rings whose tail survives; Sec. 4.3: records are stored
// unpaired and aligned at replay, the constant record cost is subtracted), same statistics block, in
// several passes over a recorded workgroup's records, which stay in HBM:
//   0  every slot is checked once (fields, slot against seq).  Only a workgroup with a record outside
//      the slot of its seq needs more: those records go on a list, sorted by wave and rank, which the
//      passes below look into beside the slot a rank belongs in (the later slot wins); a workgroup with
//      more such records than the list holds scans all its slots into a rank -> slot table (atomic max)
//      for every range of ranks instead;
//   1  pairing (an END is paired iff the nearest earlier record of its wave and region is a START):
//      the hardware waves share out the recorded waves in runs of consecutive ranks and walk them 64
//      ranks at a time, one per lane; the lanes that hold a lane's region come from one ballot per bit
//      of the region number, the last record of every region in the ranks before from a table in LDS
//      (only where some END does not have its START right below it).  A run does not know what came before
//      it, so it also keeps the ENDs that found no earlier record of their region, and one thread per
//      (wave, region) joins the runs afterwards.  Durations go to the histogram and to
//      the (wave, region) rows with atomics; a paired START and END each set their bit in a bitmap of the
//      workgroup's ranks;
//   2  overlap, a window of time at a time: every wave offers its next range of ranks, the window
//      ends at the earliest last clock among the waves that have more to offer, and the marked records
//      inside the window are sorted by clock: a counting sort into as many cells of time as the window
//      has places, then lanes take consecutive records and finish the order in registers (with fuller
//      cells: every record counts the records of its cell that come before it).  The number of waves that
//      have each region open is kept bit-sliced (plane k = bit k of every region's count): each lane's net
//      change, a scan over lanes and hardware waves, the state before each lane's records.  The total time
//      two regions are both open is the sum over the ends of their common stretches minus the sum over
//      the beginnings; a common stretch of a and b begins when one of them opens while the other is
//      open and ends when one closes while the other is open, so every event that opens or closes a region adds its clock, signed, to the sums of that
//      region with every open region (modulo 2^64: the total is exact).
// Nothing but the inputs and the statistics block is touched in HBM.
//
// What bounds it: the latency of its steps (the hardware waves are in lockstep between some ten barriers per window),
// then LDS and instruction issue in about equal parts.  So two decoder workgroups share a CU where there is work for them
// (launch_wide), a window is as large as LDS then allows, the order is finished in registers, and nothing is done per region.  Of
// the 675 us that 1024 workgroups of 8 x 4096 records with 48 regions take one workgroup to a CU, pass 0 is 57 (what reading them
// once takes), pass 1 122, looking at the windows and counting cells 134, sorting 111, the sweep 135, the sums of the region
// pairs 114; two to a CU 627.  Before: measured
// on 1024 workgroups of 8 waves x 4096 records with 48 regions (268 MB), merging 2048 records at a time in LDS and
// walking the regions one by one in the sweep before: 2594 -> 685 us (passes 0 and 1: 640 -> 187 us, of which 220 us
// were a device-wide fence per workgroup; the sweep: 220 us, half of it the sums of the region pairs).  Keys of 64
// bits in the register sort: 698 us.  Requesting a window's records under the sweep before it: 743 us (registers).
#include "kp_reduce.h"
#include "kp_stage.h"

#include <type_traits>

namespace {

using namespace kp_reduce;

constexpr uint32_t kWavesMost = 16;         // hardware waves of a decoder workgroup, at most
constexpr uint32_t kTableMin = 11, kTableMax = 14;  // ranks whose winning slots pass 1 looks up at a time: log2, what LDS has room for
constexpr uint32_t kAreaMin = 32768;        // LDS that the passes share at least
constexpr uint32_t kListMin = 512, kListMax = 8192;  // records outside the slot of their seq that a workgroup can list: what LDS has room for
constexpr uint32_t kMaxCell = 64;           // fullest time cell in which records are ranked by comparing each with each
constexpr uint32_t kSeqMask = 0xFFFFFu;
constexpr uint32_t kBins = 32;              // a duration has 32 bits: bins from there on stay empty
constexpr uint32_t kHistStride = kBins + 1; // an odd number of words apart: equal bins of different regions, different banks
constexpr uint32_t kMaxPlanes = 4 * 5;      // words of a bit-sliced count of every region the tag can name
constexpr uint64_t kNoKey = ~0ull;
constexpr uint32_t kNoId = 0xFFFFu;          // END << 7 | region of no record
constexpr uint32_t kMaxLds = 160 * 1024;    // of a CU

// per-workgroup temporaries (u32 words in LDS)
enum { T_FIELDVALID = 0, T_DISORDER, T_OCCUPIED, T_WINNER_DISORDER, T_NONMONO, T_PAIRS, T_ENDS, T_WINDOW_BEGIN,
       T_WINDOW_END, T_WINDOW_LAST, T_MAXCELL, T_EVENTS, T_LISTED, T_COUNT };

struct WideLds {  // byte offsets
  uint32_t last, head, rows, row_min, table;  // pass 1
  uint32_t cells, totals;                     // pass 2, behind the keys, which start at 0
  uint32_t bitmap, otri, hist, reg_sum, reg_max, reg_min, ctr, tmp, vf, pos, adv, edge, list, total;
  uint32_t per_lane, split_log2, rows_in_lds, list_cap, table_log2;
};
inline uint32_t up16(uint32_t x) { return (x + 15u) & ~15u; }
// LDS byte address of a place of the sorted sequence: 16 bytes of padding after every 256, so that lanes that
// read 8 consecutive places each, 64 bytes apart, spread over all banks.
__host__ __device__ constexpr uint32_t key_at(uint32_t place) { return place * 8u + ((place >> 5) << 4); }

// block: threads of a decoder workgroup; per_cu: decoder workgroups that share the LDS of a CU; per_lane: records of a window
// per lane; split_log2: runs per recorded wave in pass 1
WideLds lay_out(uint32_t block, uint32_t per_cu, uint32_t W, uint32_t R, uint32_t nrec, uint32_t per_lane, uint32_t split_log2, bool rows_in_lds) {
  const uint32_t max_lds = kMaxLds / per_cu;
  WideLds l;
  l.per_lane = per_lane; l.split_log2 = split_log2; l.rows_in_lds = rows_in_lds ? 1u : 0u;
  const uint32_t runs_bytes = (W << split_log2) * R * 8u;
  l.last = 0;
  l.head = l.last + runs_bytes;
  l.rows = up16(l.head + (split_log2 ? runs_bytes : 0u));
  l.row_min = l.rows + (rows_in_lds ? W * R * 16u : 0u);
  l.table = up16(l.row_min + (rows_in_lds ? W * R * 4u : 0u));
  const uint32_t pass1 = l.table + (4u << kTableMin);
  l.cells = key_at(block * per_lane);
  l.totals = l.cells + block * per_lane * 2u;
  const uint32_t pass2 = l.totals + kWavesMost * kMaxPlanes * 4u;
  uint32_t area = pass1 > pass2 ? pass1 : pass2;
  area = area > kAreaMin / per_cu ? area : kAreaMin / per_cu;
  l.table_log2 = kTableMin;
  while (l.table_log2 < kTableMax && l.table + (8u << l.table_log2) <= area) ++l.table_log2;
  l.bitmap = up16(area);
  l.otri = up16(l.bitmap + ((nrec + 31) / 32) * 4);
  l.hist = l.otri + R * (R + 1) / 2 * 8;
  l.reg_sum = up16(l.hist + R * kHistStride * 4);
  l.reg_max = l.reg_sum + R * 8;
  l.reg_min = l.reg_max + R * 4;
  l.ctr = up16(l.reg_min + R * 4);
  l.tmp = l.ctr + 16 * 8;
  l.vf = l.tmp + 16 * 4;
  static_assert(T_COUNT <= 16, "temporaries");
  l.pos = l.vf + 32 * 8;
  l.adv = l.pos + 16 * 4;
  l.edge = l.adv + 16 * 4;
  l.list = l.edge + kWavesMost * 16;
  l.list_cap = kListMin;
  while (l.list_cap < kListMax && l.list + l.list_cap * 2 * 8 <= max_lds) l.list_cap *= 2;  // what is left
  l.total = l.list + l.list_cap * 8;
  return l;
}
// Runs that a recorded wave is cut into in pass 1 (log2): as many as there are hardware waves for, while a run keeps 256 ranks.
inline uint32_t split_log2(uint32_t block, uint32_t W, uint32_t cap) {
  uint32_t most = 0;
  while ((W << (most + 1)) <= block / 64u && (cap >> (most + 1)) >= 256u) ++most;
  return most;
}
// The largest window that LDS has room for (beside a list of twice the smallest size), with the rows of the
// (wave, region) sums in LDS and the recorded waves cut into as many runs as there are hardware waves for;
// failing that with fewer runs; the smallest window also with the rows in HBM.
WideLds wide_lds(uint32_t block, uint32_t per_cu, uint32_t W, uint32_t R, uint32_t cap) {
  const uint32_t max_lds = kMaxLds / per_cu, most = split_log2(block, W, cap);
  for (uint32_t per_lane = 8; per_lane >= 2; per_lane >>= 1) {
    for (uint32_t split = most + 1; split-- > 0;) {
      const WideLds l = lay_out(block, per_cu, W, R, W * cap, per_lane, split, true);
      if (l.total <= max_lds && (per_lane == 2 || l.list_cap > kListMin)) return l;
    }
  }
  return lay_out(block, per_cu, W, R, W * cap, 2, 0, false);
}

struct WideParams {
  const uint32_t* wg_hdrs;  // 32 words per recorded workgroup
  const uint2* records;     // {tag, payload}
  uint64_t* out;
  uint32_t n_wg, W, R, cap, cap_log2, rec_cost, flush, nrec;
  uint32_t waves_log2;      // ceil(log2 W): a window offers (window places >> this) ranks of every wave
  WideLds lds;
};

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// Bit-sliced counters of up to 32 NW regions: plane k of word w holds bit k of the counts of regions 32 w ..
template <int NW, int P> struct Planes { uint32_t at[NW][P]; };
template <int NW, int P>
__device__ __forceinline__ void planes_add(Planes<NW, P>& a, const Planes<NW, P>& b) {
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const uint32_t s = a.at[w][k] ^ b.at[w][k], g = a.at[w][k] & b.at[w][k];
      a.at[w][k] = s ^ c;
      c = g | (s & c);
    }
  }
}
// count of `region` += 1, or -= 1 where down is all ones; nothing where on is zero
template <int NW, int P>
__device__ __forceinline__ void planes_step(Planes<NW, P>& p, uint32_t region, uint32_t on, uint32_t down) {
  const uint32_t bit = on << (region & 31u);
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    uint32_t carry = (NW == 1 || (region >> 5) == (uint32_t)w) ? bit : 0u;
#pragma unroll
    for (int k = 0; k < P; ++k) { const uint32_t o = p.at[w][k]; p.at[w][k] = o ^ carry; carry &= o ^ down; }
  }
}
template <int NW, int P>
__device__ __forceinline__ uint32_t planes_any(const Planes<NW, P>& p, int w) {  // regions of word w with a count above zero
  uint32_t v = p.at[w][0];
#pragma unroll
  for (int k = 1; k < P; ++k) v |= p.at[w][k];
  return v;
}
template <int STEP, int NW, int P>
__device__ __forceinline__ void planes_scan_step(Planes<NW, P>& p) {
  Planes<NW, P> o;
#pragma unroll
  for (int w = 0; w < NW; ++w)
#pragma unroll
    for (int k = 0; k < P; ++k) o.at[w][k] = scan_src<STEP>(p.at[w][k]);
  planes_add<NW, P>(p, o);
}

// kBlock: threads; E: records of a window per lane; NW: 32-bit words that hold one bit per region; P: bits of a count of waves.
template <int kBlock, int E, int NW, int P>
__global__ __launch_bounds__(kBlock, 4) void kp_reduce_wide(WideParams p) {
  constexpr uint32_t kWavesHw = kBlock / 64;
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr uint32_t K = kBlock * E;  // places of a window
  // [run][region] its last record: (rank + 1) << 33 | END << 32 | clock, 0 for none; so the latest is the largest
  unsigned long long* last_all = reinterpret_cast<unsigned long long*>(smem + p.lds.last);
  uint2* head_all = reinterpret_cast<uint2*>(smem + p.lds.head);        // {clock, 1 << 31 | rank} of its first record if that is an END (waves cut into runs)
  uint32_t* table1 = reinterpret_cast<uint32_t*>(smem + p.lds.table);   // rank -> winning slot + 1, 2^table_log2 ranks at a time (pass 1)
  uint32_t* table2 = reinterpret_cast<uint32_t*>(smem);                 // the same for the ranks a window looks at (before its keys are written)
  uint32_t* cells = reinterpret_cast<uint32_t*>(smem + p.lds.cells);    // cell c: half (c & 1) of word c >> 1
  // the records outside the slot of their seq: (wave << 20 | rank) << 20 | slot, sorted
  unsigned long long* list = reinterpret_cast<unsigned long long*>(smem + p.lds.list);
  uint32_t* rows_lds = reinterpret_cast<uint32_t*>(smem + p.lds.rows);  // {u64 sum; u32 n; u32 max} per (wave, region), if p.lds.rows_in_lds
  uint32_t* row_min = reinterpret_cast<uint32_t*>(smem + p.lds.row_min);
  uint32_t* bitmap = reinterpret_cast<uint32_t*>(smem + p.lds.bitmap);  // bit wave * cap + rank: the record is a paired START or END
  unsigned long long* otri = reinterpret_cast<unsigned long long*>(smem + p.lds.otri);  // pair (a <= b) at b (b + 1) / 2 + a
  uint32_t* hist = reinterpret_cast<uint32_t*>(smem + p.lds.hist);
  unsigned long long* reg_sum = reinterpret_cast<unsigned long long*>(smem + p.lds.reg_sum);
  uint32_t* reg_max = reinterpret_cast<uint32_t*>(smem + p.lds.reg_max);
  uint32_t* reg_min = reinterpret_cast<uint32_t*>(smem + p.lds.reg_min);
  uint32_t* totals = reinterpret_cast<uint32_t*>(smem + p.lds.totals);  // [hardware wave][plane]: net change over its records of the window
  unsigned long long* ctr = reinterpret_cast<unsigned long long*>(smem + p.lds.ctr);
  uint32_t* tmp = reinterpret_cast<uint32_t*>(smem + p.lds.tmp);
  uint2* sVF = reinterpret_cast<uint2*>(smem + p.lds.vf);               // per wave: records held, first surviving seq
  uint32_t* pos = reinterpret_cast<uint32_t*>(smem + p.lds.pos);        // per wave: first rank of the range in LDS
  uint32_t* adv = reinterpret_cast<uint32_t*>(smem + p.lds.adv);        // per wave: ranks the window took
  uint32_t* edge = reinterpret_cast<uint32_t*>(smem + p.lds.edge);      // pass 1, per run: 1 if it holds a record, first clock, last clock and id; pass 2: records in the cells of each hardware wave
  // hi (hi + 1), which is even: the bytes of hi (hi + 1) / 2 places are four times as many.  (A 32-bit product, which the compiler
  // makes of it, takes four times as long as this instruction:
  // 1024 workgroups of 8 x 4096 slots, 48 regions 632 -> 621 us, 300 of 16 x 2048, 128 regions 780 -> 768.)
  auto pair_sum = [&](uint32_t lo, uint32_t hi) {
    uint32_t twice;
    asm("v_mad_u32_u24 %0, %1, %1, %1" : "=v"(twice) : "v"(hi));
    return reinterpret_cast<unsigned long long*>(smem + p.lds.otri + (twice << 2) + (lo << 3));
  };
  auto key = [&](uint32_t place) -> unsigned long long& { return *reinterpret_cast<unsigned long long*>(smem + key_at(place)); };

  const uint32_t tid_k = threadIdx.x;
  uint32_t tid = tid_k, lane = tid & 63u, hw = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  // A copy of the thread index that the optimiser cannot see through: without it address arithmetic of all
  // passes is done ahead of the loops and held in registers through them.
  auto fresh_tid = [&]() { tid = tid_k; asm volatile("" : "+v"(tid)); lane = tid & 63u; };
  const uint32_t W = p.W, R = p.R, cap = p.cap, capm = cap - 1u, cl2 = p.cap_log2, nrec = p.nrec;
  constexpr uint32_t kPlacesLog2 = (E == 8 ? 3u : E == 4 ? 2u : 1u) + (kBlock == 1024 ? 10u : kBlock == 512 ? 9u : 8u);
  static_assert(K == 1u << kPlacesLog2, "places of a window");
  const uint32_t rsh = kPlacesLog2 - p.waves_log2, C = 1u << rsh;  // a window looks at C ranks of every wave
  const uint32_t tsh = p.lds.table_log2 - p.waves_log2, Ct = 1u << tsh;                        // table1: Ct ranks of every wave
  uint32_t region_bits = 0; while ((1u << region_bits) < R) ++region_bits;
  const StatsLayout SL = stats_layout(p.n_wg, W, R);
  if (p.out[H_STATUS] != 0) return;  // device header did not match the launch geometry

  for (uint32_t i = tid; i < R * kHistStride; i += kBlock) hist[i] = 0;
  for (uint32_t i = tid; i < R * (R + 1) / 2; i += kBlock) otri[i] = 0;
  for (uint32_t i = tid; i < R; i += kBlock) { reg_sum[i] = 0; reg_max[i] = 0; reg_min[i] = 0xFFFFFFFFu; }
  if (tid < 16) ctr[tid] = 0;
  __syncthreads();

  for (uint32_t wg = blockIdx.x; wg < p.n_wg; wg += gridDim.x) {
    const uint32_t* wh = p.wg_hdrs + (size_t)32 * wg;
    const uint2* recs = p.records + (size_t)wg * nrec;
    __syncthreads();  // every wave is done with the workgroup before
    fresh_tid();

    // ---- workgroup header ------------------------------------------------------------------------
    if (tid <= KP_MAX_WAVES) {  // (entries from W up: no records)
      const uint32_t T = tid < W ? wh[8 + tid] : 0u;
      const uint32_t V = T < cap ? T : cap;
      sVF[tid] = make_uint2(V, p.flush ? 0u : T - V);
      if (tid < W) {
        atomicAdd(&ctr[H_DROPPED], (unsigned long long)(T - V));
        atomicAdd(&ctr[H_SLOTS_VALID], (unsigned long long)V);
      }
    }
    if (tid < T_COUNT) tmp[tid] = 0;
    for (uint32_t i = tid; i < (nrec + 31u) / 32u; i += kBlock) bitmap[i] = 0;
    for (uint32_t e = tid; e < (W << p.lds.split_log2) * R; e += kBlock) {  // no last record of (run, region) yet, and no first
      last_all[e] = 0ull;
      if (p.lds.split_log2) head_all[e] = make_uint2(0u, 0u);
    }
    for (uint32_t e = tid; e < W * R; e += kBlock) {
      // pass 1 adds every pair to its row with atomics: in LDS, or in the statistics block itself
      if (p.lds.rows_in_lds) {
        reinterpret_cast<uint4*>(rows_lds)[e] = make_uint4(0u, 0u, 0u, 0u);
        row_min[e] = 0xFFFFFFFFu;
      } else {
        uint64_t* row = p.out + SL.per + ((size_t)wg * W * R + e) * 2;  // (stored where the atomics act)
        __hip_atomic_store(&row[0], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&row[1], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (tid < kWavesMost) edge[4u * tid] = 0u;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the rows are cleared before any wave adds to them
    __syncthreads();
    uint32_t held = 0, max_v = 0;
    for (uint32_t w = 0; w < W; ++w) {
      const uint32_t V = sVF[w].x;
      held += V;
      max_v = V > max_v ? V : max_v;
    }
    const bool span_overflow = (((uint64_t)wh[4] | ((uint64_t)wh[5] << 32)) - ((uint64_t)wh[2] | ((uint64_t)wh[3] << 32))) >> 32 != 0;

    // A record that passes the checks of its fields: its rank, else all ones.
    auto rank_of = [&](uint2 rec, uint32_t w, uint32_t s) -> uint32_t {
      const uint2 vf = sVF[w];
      const uint32_t k = (rec.x - vf.y) & kSeqMask;  // the low 20 bits of tag - first are those of seq - first
      const bool good = s < vf.x && k < vf.x && ((rec.x >> 20) & 0xFu) == w && ((rec.x >> 24) & 0x7Fu) < R;
      return good ? k : 0xFFFFFFFFu;
    };

    // ---- pass 0: every slot once -------------------------------------------------------------------
    {
      uint32_t c_field = 0, c_dis = 0;
      const uint4* units = reinterpret_cast<const uint4*>(recs);  // two records each
      for (uint32_t i0 = tid; i0 < nrec / 2u; i0 += 4u * kBlock) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = units[i0 + u * kBlock < nrec / 2u ? i0 + u * kBlock : i0];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (i0 + u * kBlock >= nrec / 2u) continue;
#pragma unroll
          for (uint32_t h = 0; h < 2u; ++h) {
            const uint32_t i = 2u * (i0 + u * kBlock) + h, w = i >> cl2, s = i & capm;
            const uint2 rec = h ? make_uint2(v[u].z, v[u].w) : make_uint2(v[u].x, v[u].y);
            const uint32_t k = rank_of(rec, w, s);
            const bool good = k != 0xFFFFFFFFu;
            c_field += good ? 1u : 0u;
            if (good && ((rec.x ^ s) & capm) != 0u) {
              ++c_dis;
              const uint32_t at = atomicAdd(&tmp[T_LISTED], 1u);
              if (at < p.lds.list_cap) list[at] = ((unsigned long long)((w << 20) | k) << 20) | s;
            }
          }
        }
      }
      c_field = wave_sum(c_field);
      c_dis = wave_sum(c_dis);
      if (lane == 0) {
        if (c_field) atomicAdd(&tmp[T_FIELDVALID], c_field);
        if (c_dis) atomicAdd(&tmp[T_DISORDER], c_dis);
      }
    }
    __syncthreads();
    // Records that all sit in the slot of their own seq have distinct seq modulo the ring size, hence
    // distinct ranks, and rank k of a wave is in slot (first + k) mod cap.
    const bool displaced = tmp[T_DISORDER] != 0u;
    // A workgroup with such records: which slot holds rank k (the later slot wins) comes from the sorted
    // list of those records, next to the slot the rank belongs in; a workgroup with more of them than the
    // list holds scans all its slots into a rank -> slot table, a range of ranks at a time: as large a range as LDS has
    // room for, four loads in flight per thread (64 workgroups of 8 x 8192 with a tenth of the neighbours swapped: 1880 us
    // with ranges of 2048 ranks, one load at a time and a further scan that counted the winners; 496 us).
    const bool listed = displaced && tmp[T_LISTED] <= p.lds.list_cap, tabled = displaced && !listed;
    const uint32_t n_listed = listed ? tmp[T_LISTED] : 0u;
    if (listed) {
      // sorted (bitonic) over the smallest power of two of places that holds it
      uint32_t n_sort = kListMin;
      while (n_sort < n_listed) n_sort <<= 1;
      for (uint32_t i = tid; i < n_sort; i += kBlock) {
        if (i >= n_listed) list[i] = kNoKey;
      }
      __syncthreads();
      for (uint32_t size = 2; size <= n_sort; size <<= 1) {
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
          for (uint32_t i = tid; i < n_sort / 2u; i += kBlock) {
            const uint32_t lo = ((i & ~(stride - 1u)) << 1) | (i & (stride - 1u)), hi = lo | stride;
            const bool up = (lo & size) == 0u;
            const unsigned long long x = list[lo], y = list[hi];
            if ((x > y) == up) { list[lo] = y; list[hi] = x; }
          }
          __syncthreads();
        }
      }
    }
    // first place of the sorted list whose (wave << 20 | rank) is not below `prefix`
    auto list_lower_bound = [&](uint32_t prefix) -> uint32_t {
      uint32_t lo = 0, hi = n_listed;
      while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if ((uint32_t)(list[mid] >> 20) < prefix) lo = mid + 1u; else hi = mid;
      }
      return lo;
    };

    // The ranks pos[w] .. pos[w] + (1 << sh) of every wave: which slot holds each (the later slot wins).
    auto build_table = [&](uint32_t* table, uint32_t places, uint32_t sh) {
      __syncthreads();  // pos[] is written, the table's last readers are done
      for (uint32_t i = tid; i < places; i += kBlock) table[i] = 0;
      __syncthreads();
      const uint4* units = reinterpret_cast<const uint4*>(recs);  // two records each
      for (uint32_t i0 = tid; i0 < nrec / 2u; i0 += 4u * kBlock) {  // (the loads of an iteration are in flight together)
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = units[i0 + u * kBlock < nrec / 2u ? i0 + u * kBlock : i0];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t i = 2u * (i0 + u * kBlock), w = i < nrec ? i >> cl2 : 0u, s = i & capm;
          const uint32_t first = sVF[w].y, from = pos[w];
#pragma unroll
          for (uint32_t h = 0; h < 2u; ++h) {
            const uint2 rec = h ? make_uint2(v[u].z, v[u].w) : make_uint2(v[u].x, v[u].y);
            const uint32_t d = ((rec.x - first) & kSeqMask) - from;  // (most records are of another range)
            if (i < nrec && d < (1u << sh) && rank_of(rec, w, s + h) != 0xFFFFFFFFu) atomicMax(&table[(w << sh) + d], s + h + 1u);
          }
        }
      }
      __syncthreads();
    };

    uint32_t n_occupied = 0, n_disorder = 0;
    // ---- pass 1: pairing, durations, per-(wave, region) statistics, monotonicity ---------------------
    // Hardware wave (w << split) + i takes run i of recorded wave w, 64 consecutive ranks at a time, one per
    // lane.  The nearest earlier record of a lane's (wave, region) is the highest lower lane with the same
    // region (the lanes with a lane's region: one ballot per bit of the region number) or, when there is none,
    // the last record of that region in the ranks before, which the run keeps in a table of its own.
    // (a workgroup that looks its winning slots up in a table does not cut its waves into runs)
    {
      const uint32_t split = tabled ? 0u : p.lds.split_log2;
      uint32_t n_pairs = 0, n_ends = 0, nonmono = 0, occupied = 0, moved = 0;  // (the same in all lanes)
      uint32_t w_here = 0, run = 0;
      unsigned long long* last = last_all;
      uint2* head = head_all;
      bool carry_has = false;
      uint32_t carry_ts = 0, first_ts = 0, carry_id = kNoId;  // the run's last record so far: clock, END << 7 | region; clock of its first
      const uint64_t below = (1ull << lane) - 1ull;
      // the duration of a pair into the histogram and its row
      auto account = [&](uint32_t w, uint32_t r, uint32_t d_raw) {
        const uint32_t d = d_raw > p.rec_cost ? d_raw - p.rec_cost : 0u;
        atomicAdd(&hist[r * kHistStride + (31 - __clz(d | 1u))], 1u);
        // row {u64 sum; u32 n; u32 max}, cleared above
        if (p.lds.rows_in_lds) {
          uint32_t* row = rows_lds + (w * R + r) * 4u;
          atomicAdd(reinterpret_cast<unsigned long long*>(row), (unsigned long long)d);
          atomicAdd(row + 2, 1u);
          atomicMax(row + 3, d);
          atomicMin(&row_min[w * R + r], d);
        } else {
          uint64_t* row = p.out + SL.per + (((size_t)wg * W + w) * R + r) * 2u;
          atomicAdd(reinterpret_cast<unsigned long long*>(row), (unsigned long long)d);
          atomicAdd(reinterpret_cast<uint32_t*>(row) + 2, 1u);
          atomicMax(reinterpret_cast<uint32_t*>(row) + 3, d);
          atomicAdd(&reg_sum[r], (unsigned long long)d);
          atomicMax(&reg_max[r], d);
          atomicMin(&reg_min[r], d);
        }
      };
      auto mark = [&](uint32_t bit) { atomicOr(&bitmap[bit >> 5], 1u << (bit & 31u)); };
      auto group = [&](uint32_t k0, bool ok, uint2 rec) {  // this lane: rank k0 + lane, its record if ok
        const uint32_t k = k0 + lane, id = rec.x >> 24, r = id & 0x7Fu, ts = rec.y;
        const bool is_end = ok && id >= 0x80u;
        const uint64_t there = __builtin_amdgcn_ballot_w64(ok), ends = __builtin_amdgcn_ballot_w64(is_end);
        if (there == 0ull) return;
        occupied += (uint32_t)__popcll(there);
        n_ends += (uint32_t)__popcll(ends);
        // the record before each (clocks must not decrease from one to the next), by far the most often also
        // the nearest one of an END's region
        uint32_t start_ts = wave_shr1(ts, carry_ts), before_id = wave_shr1(id, carry_id);
        const bool gaps = (there & (there + 1ull)) != 0ull;  // (uniform) a rank without a record
        if (gaps) {
          const uint64_t lower = there & below;
          const uint32_t from_ts = (uint32_t)__shfl((int)ts, lower ? 63 - (int)__builtin_clzll(lower) : 0, 64);
          start_ts = lower ? from_ts : carry_ts;
          before_id = kNoId;
        }
        nonmono += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(ok && ts < start_ts));  // (0 before the run's first record)
        if (!carry_has) first_ts = (uint32_t)__builtin_amdgcn_readlane((int)ts, (int)__builtin_ctzll(there));
        const int top = 63 - (int)__builtin_clzll(there);
        carry_ts = (uint32_t)__builtin_amdgcn_readlane((int)ts, top);
        carry_id = (uint32_t)__builtin_amdgcn_readlane((int)id, top);
        carry_has = true;
        bool pair = is_end && before_id == r;
        const uint64_t near = __builtin_amdgcn_ballot_w64(pair);
        const uint32_t b0 = w_here * cap + k0;
        if (ends & ~near) {
          uint64_t same = there;
          for (uint32_t b = 0; b < region_bits; ++b) {
            const uint64_t set = __builtin_amdgcn_ballot_w64(ok && ((r >> b) & 1u));
            same &= ((r >> b) & 1u) ? set : ~set;
          }
          const uint64_t lower = same & below;
          const int src = lower ? 63 - (int)__builtin_clzll(lower) : 0;
          const uint32_t far_ts = (uint32_t)__shfl((int)ts, src, 64);
          if (is_end && !pair) {
            bool start = lower != 0ull && !((ends >> src) & 1ull);
            uint32_t at = k0 + (uint32_t)src;
            start_ts = far_ts;
            if (lower == 0ull) {
              const unsigned long long c = last[r];
              start = c != 0ull && !((c >> 32) & 1ull);
              at = (uint32_t)(c >> 33) - 1u;
              start_ts = (uint32_t)c;
              if (c == 0ull && run) head[r] = make_uint2(ts, 0x80000000u | k);  // the run's first record of the region: decided when the runs are joined
            }
            if (start) mark(w_here * cap + at);
            pair = start;
          }
        }
        if (ok) atomicMax(&last[r], ((unsigned long long)(((k + 1u) << 1) | (is_end ? 1u : 0u)) << 32) | ts);
        const uint64_t pairs = __builtin_amdgcn_ballot_w64(pair);
        n_pairs += (uint32_t)__popcll(pairs);
        if (pair) account(w_here, r, ts - start_ts);
        // both records of a pair are marked (those found further back: above)
        if (cap >= 64u) {  // (the ranks then start at a word of the bitmap)
          const uint64_t marks = pairs | (near >> 1);
          if (lane < 2u) atomicOr(&bitmap[(b0 >> 5) + lane], lane ? (uint32_t)(marks >> 32) : (uint32_t)marks);
          if (lane == 2u && (near & 1ull)) mark(b0 - 1u);
        } else if (pair) {
          mark(b0 + lane);
          if ((near >> lane) & 1ull) mark(b0 + lane - 1u);
        }
      };
      auto take_run = [&](uint32_t id) {
        w_here = id >> split; run = id & ((1u << split) - 1u);
        last = last_all + id * R;
        head = head_all + id * R;
      };
      auto keep_edge = [&](uint32_t id) {
        if (lane == 0 && w_here < W) *reinterpret_cast<uint4*>(edge + 4u * id) = make_uint4(carry_has ? 1u : 0u, first_ts, carry_ts, carry_id);
      };
      // (runs may outnumber the hardware waves where these are fewer than the recorded ones)
      const bool several = kWavesHw != kWavesMost && tabled && W > kWavesHw;
      const uint32_t n_runs = kWavesHw == kWavesMost || several ? 1u : W << split;
      for (uint32_t run0 = 0; run0 < n_runs; run0 += kWavesHw) {
      const uint32_t id = run0 + hw;
      take_run(id);
      carry_has = false; carry_ts = 0u; first_ts = 0u; carry_id = kNoId;
      const uint32_t V = w_here < W ? sVF[w_here].x : 0u;
      if (!tabled) {
        // rank k belongs in slot (first + k) mod cap; nothing is shared with the other runs
        const uint32_t first = sVF[w_here < W ? w_here : 0u].y;
        const uint32_t k_begin = run * (cap >> split), k_end = V < k_begin + (cap >> split) ? V : k_begin + (cap >> split);
        uint32_t cursor = 0, cursor_end = 0;  // this run's stretch of the sorted list
        if (listed && w_here < W) {
          cursor = list_lower_bound((w_here << 20) | k_begin);
          cursor_end = list_lower_bound(k_begin + (cap >> split) < (1u << 20) ? (w_here << 20) | (k_begin + (cap >> split)) : (w_here + 1u) << 20);
        }
        const uint2* seg = recs + (size_t)(w_here < W ? w_here : 0u) * cap;
        uint2 ahead[4];  // the records of the next 256 ranks are on their way while 64 are walked
        auto request = [&](uint32_t k0) -> uint2 { const uint32_t k = k0 + lane; return seg[k < k_end ? (first + k) & capm : 0u]; };
#pragma unroll
        for (int g = 0; g < 4; ++g) ahead[g] = k_begin < k_end ? request(k_begin + 64u * g) : make_uint2(0u, 0u);
#pragma unroll 1
        for (uint32_t k0 = k_begin; k0 < k_end; k0 += 64u) {
          const uint32_t k = k0 + lane;
          uint32_t slot = (first + k) & capm;
          uint2 rec = ahead[0];
          ahead[0] = ahead[1]; ahead[1] = ahead[2]; ahead[2] = ahead[3];
          ahead[3] = request(k0 + 256u);
          bool ok = k < k_end && rank_of(rec, w_here, slot) == k;
          if (cursor < cursor_end && ((uint32_t)(list[cursor] >> 20) & kSeqMask) < k0 + 64u) {
            // listed records whose rank is among these: a later slot displaces an earlier one
            bool moved_here = false;
            while (cursor < cursor_end) {
              const unsigned long long entry = list[cursor];
              const uint32_t rank = (uint32_t)(entry >> 20) & kSeqMask, s = (uint32_t)entry & 0xFFFFFu;
              if (rank >= k0 + 64u) break;
              ++cursor;
              if (rank == k && (!ok || s > slot)) { slot = s; ok = true; moved_here = true; }
            }
            if (moved_here) rec = seg[slot];
          }
          if (displaced) moved += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(ok && ((rec.x ^ slot) & capm) != 0u));
          group(k0, ok, rec);
        }
      } else {
        for (uint32_t k0 = 0; k0 < max_v; k0 += Ct) {
          if (tid < 16) pos[tid] = k0;
          build_table(table1, 1u << p.lds.table_log2, tsh);
          // A table holds a range of ranks of all waves, and takes a look at every slot.  So it is made once, and a hardware wave that
          // has several waves walks the range in one after the other, with each one's last record kept beside its edges.  (Each through
          // all ranges, the tables made anew for it: 1000 workgroups of 16 x 1024 slots, 40 regions, a third of the neighbours swapped
          // 613 us, 558 this way; 500 of 16 x 2048, 24 regions 594 / 536.  Where each has one wave nothing is reloaded: 563 / 566
          // for 1000 of 8 x 1024, 585 if it is.)
          for (uint32_t id_t = hw;;) {
            const uint32_t V_t = id_t < W ? sVF[id_t].x : 0u;
#pragma unroll 1
            for (uint32_t j0 = 0; j0 < Ct && k0 + j0 < V_t; j0 += 64u) {
              const uint32_t t = table1[(id_t << tsh) + j0 + lane];
              const uint2 rec = recs[(size_t)id_t * cap + (t ? t - 1u : 0u)];
              moved += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(t != 0u && ((rec.x ^ (t - 1u)) & capm) != 0u));
              group(k0 + j0, t != 0u, rec);
            }
            if (!several) break;
            keep_edge(id_t);
            id_t += kWavesHw;
            const bool back = id_t >= W;  // to the first, for the next range
            if (back) id_t = hw;
            take_run(id_t);
            auto kept = [&](uint32_t i) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)edge[4u * id_t + i]); };
            carry_has = kept(0u) != 0u; first_ts = kept(1u); carry_ts = carry_has ? kept(2u) : 0u; carry_id = carry_has ? kept(3u) : kNoId;
            if (back) break;
          }
        }
      }
      keep_edge(id);
      }
      if (lane == 0) {
        if (n_pairs) atomicAdd(&tmp[T_PAIRS], n_pairs);
        if (n_ends) atomicAdd(&tmp[T_ENDS], n_ends);
        if (nonmono) atomicAdd(&tmp[T_NONMONO], nonmono);
        if (occupied) atomicAdd(&tmp[T_OCCUPIED], occupied);
        if (moved) atomicAdd(&tmp[T_WINNER_DISORDER], moved);
      }
      __syncthreads();
      // Join the runs of a wave, region by region.
      n_pairs = 0;  // (from here on each lane's own)
      for (uint32_t e = tid; e < W * R; e += kBlock) {
        const uint32_t w = e / R, r = e - w * R;
        unsigned long long before = 0ull;
        for (uint32_t i = 0; i + 1u < (1u << split); ++i) {
          const unsigned long long l = last_all[((w << split) + i) * R + r];
          if (l) before = l;
          const uint2 h = head_all[((w << split) + i + 1u) * R + r];  // an END that found no earlier record in its own run
          if (h.y && before && !((before >> 32) & 1ull)) {
            ++n_pairs;
            account(w, r, h.x - (uint32_t)before);
            mark(w * cap + (uint32_t)(before >> 33) - 1u);
            mark(w * cap + (h.y & kSeqMask));
          }
        }
        if (p.lds.rows_in_lds) {  // (nobody else adds to this row any more)
          const uint64_t sum = reinterpret_cast<const uint64_t*>(rows_lds)[2u * e], n_max = reinterpret_cast<const uint64_t*>(rows_lds)[2u * e + 1u];
          uint64_t* row = p.out + SL.per + ((size_t)wg * W * R + e) * 2;
          row[0] = sum;
          row[1] = n_max;
          if ((uint32_t)n_max) {
            atomicAdd(&reg_sum[r], (unsigned long long)sum);
            atomicMax(&reg_max[r], (uint32_t)(n_max >> 32));
            atomicMin(&reg_min[r], row_min[e]);
          }
        }
      }
      nonmono = 0;
      if (tid < W) {
        bool has = false;
        uint32_t ts = 0;
        for (uint32_t i = 0; i < (1u << split); ++i) {
          const uint32_t* at = edge + 4u * ((tid << split) + i);
          if (!at[0]) continue;
          nonmono += has && at[1] < ts ? 1u : 0u;
          has = true; ts = at[2];
        }
      }
      n_pairs = wave_sum(n_pairs); nonmono = wave_sum(nonmono);
      if (lane == 0) {
        if (n_pairs) atomicAdd(&tmp[T_PAIRS], n_pairs);
        if (nonmono) atomicAdd(&tmp[T_NONMONO], nonmono);
      }
      n_occupied = tmp[T_OCCUPIED];
      n_disorder = tmp[T_WINNER_DISORDER];
    }
    const uint32_t wg_invalid = held - n_occupied;  // slots that hold a record and did not make it into the ordered sequence
    __syncthreads();
    const bool eligible = !span_overflow && wg_invalid == 0u && tmp[T_NONMONO] == 0u;
    if (tid == 0) {
      ctr[H_INVALID] += wg_invalid;
      ctr[H_DISORDER] += n_disorder;
      ctr[H_NONMONO] += tmp[T_NONMONO];
      ctr[H_PAIRS] += tmp[T_PAIRS];
      ctr[H_ORPHAN_START] += n_occupied - tmp[T_ENDS] - tmp[T_PAIRS];  // every START and END is paired or an orphan
      ctr[H_ORPHAN_END] += tmp[T_ENDS] - tmp[T_PAIRS];
      ctr[H_SPAN_OVF] += span_overflow ? 1u : 0u;
      ctr[H_OVERLAP_WGS] += eligible ? 1u : 0u;
    }
    if (!eligible) continue;  // (the same in every thread)

    // ---- pass 2: region-pair overlap -----------------------------------------------------------------
    // Every rank below a wave's record count holds a record here and the clocks of a wave do not decrease.
    if (tid < 16) pos[tid] = 0;
    Planes<NW, P> open_now;  // waves that have each region open at the window's start (the same in all threads)
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
      for (int k = 0; k < P; ++k) open_now.at[w][k] = 0u;
    for (uint32_t round = 0; round <= nrec; ++round) {  // (every window takes at least one record: the bound is never reached)
      __syncthreads();
      fresh_tid();
      bool more = false;
      for (uint32_t w = 0; w < W; ++w) more = more || pos[w] < sVF[w].x;
      if (!more) break;
      if (tabled) build_table(table2, K, rsh);
      if (tid == 0) { tmp[T_WINDOW_BEGIN] = 0xFFFFFFFFu; tmp[T_WINDOW_END] = 0xFFFFFFFFu; tmp[T_WINDOW_LAST] = 0u; tmp[T_MAXCELL] = 0u; }
      if (tid < 16) adv[tid] = 0;
#pragma unroll
      for (int x = 0; x < E / 2; ++x) cells[tid + x * kBlock] = 0u;
      __syncthreads();
      // ---- the records this window looks at: place idx is (wave idx >> rsh, rank pos + (idx & (C - 1))) ----
      uint2 rec[E];
#pragma unroll
      for (int x = 0; x < E; ++x) {
        const uint32_t idx = tid + x * kBlock, w = idx >> rsh, k = pos[w & 15u] + (idx & (C - 1u));
        const uint2 vf = sVF[w];  // (no records from wave W up)
        const uint32_t s = tabled ? table2[idx] - 1u : (vf.y + k) & capm;
        rec[x] = recs[k < vf.x ? (size_t)w * cap + s : (size_t)0];
      }
      bool ok[E];
#pragma unroll
      for (int x = 0; x < E; ++x) {
        const uint32_t idx = tid + x * kBlock, w = idx >> rsh, j = idx & (C - 1u), k = pos[w & 15u] + j;
        const uint2 vf = sVF[w];
        ok[x] = k < vf.x;  // (every such rank holds a record here)
        if (ok[x] && !tabled && rank_of(rec[x], w, (vf.y + k) & capm) != k) {  // the rank's record is on the list
          const uint32_t at = list_lower_bound((w << 20) | k);
          ok[x] = at < n_listed && (uint32_t)(list[at] >> 20) == ((w << 20) | k);
          if (ok[x]) rec[x] = recs[(size_t)w * cap + ((uint32_t)list[at] & 0xFFFFFu)];
        }
        if (ok[x]) {
          const uint32_t left = vf.x - k;  // records of the wave from this one on
          if (j == 0u) atomicMin(&tmp[T_WINDOW_BEGIN], rec[x].y);
          if (j == C - 1u || left == 1u) atomicMax(&tmp[T_WINDOW_LAST], rec[x].y);
          // a wave with records beyond this range: the window cannot reach past the range's last clock
          if (j == C - 1u && left > 1u) atomicMin(&tmp[T_WINDOW_END], rec[x].y);
        }
      }
      __syncthreads();
      // ---- counting sort of the marked records inside the window into K cells of time ---------------------
      const uint32_t t_begin = tmp[T_WINDOW_BEGIN];
      const uint32_t t_end = tmp[T_WINDOW_END] < tmp[T_WINDOW_LAST] ? tmp[T_WINDOW_END] : tmp[T_WINDOW_LAST];
      // (a product and a conversion that never decrease with the clock: the cells follow one another in time)
      const float scale = (float)K / ((float)(t_end - t_begin) + 1.0f);
      uint32_t ca[E];  // cell | arrival in the cell << 16; all ones: no event
#pragma unroll
      for (int x = 0; x < E; ++x) {
        const uint32_t idx = tid + x * kBlock, w = idx >> rsh, j = idx & (C - 1u);
        const bool inside = ok[x] && rec[x].y <= t_end;  // the records inside are the first ones of the range
        const uint64_t taken = __builtin_amdgcn_ballot_w64(inside);
        // (a wave offers at least 128 ranks, so that the 64 places of a hardware wave are one recorded wave's)
        if (lane == 0u && taken) atomicAdd(&adv[w], (uint32_t)__popcll(taken));
        const uint32_t b = (w & 15u) * cap + pos[w & 15u] + j;
        const bool event = inside && ((bitmap[inside ? b >> 5 : 0u] >> (b & 31u)) & 1u);
        uint32_t c = (uint32_t)((float)(rec[x].y - t_begin) * scale);
        c = c < K - 1u ? c : K - 1u;
        const uint32_t sh = (c & 1u) << 4;
        ca[x] = 0xFFFFFFFFu;
        if (event) ca[x] = c | (((atomicAdd(&cells[c >> 1], 1u << sh) >> sh) & 0xFFFFu) << 16);
      }
      __syncthreads();
      {  // exclusive prefix sum over the cell counters, E cells per thread
        uint32_t wv[E / 2], run = 0, fullest = 0;
#pragma unroll
        for (int i = 0; i < E / 2; ++i) {
          const uint32_t v = cells[tid * (E / 2) + i], lo = v & 0xFFFFu, hi = v >> 16;
          fullest = lo > fullest ? lo : fullest;
          fullest = hi > fullest ? hi : fullest;
          wv[i] = run | ((run + lo) << 16);
          run += lo + hi;
        }
        const uint32_t incl = wave_scan_add(run);
        uint32_t* share = edge;  // records in the cells of each hardware wave
        if (lane == 63u) share[hw] = incl;
        if (__builtin_amdgcn_ballot_w64(fullest > 8u)) { if (fullest > 8u) atomicMax(&tmp[T_MAXCELL], fullest); }
        __syncthreads();
        uint32_t below = (lane & 15u) < hw ? share[lane & 15u] : 0u;  // lane h of a row takes wave h's
        below += scan_src<0>(below); below += scan_src<1>(below); below += scan_src<2>(below); below += scan_src<3>(below);
        const uint32_t base = incl - run + (uint32_t)__builtin_amdgcn_readlane((int)below, 15);
#pragma unroll
        for (int i = 0; i < E / 2; ++i) cells[tid * (E / 2) + i] = wv[i] + base * 0x00010001u;
        if (tid == kBlock - 1u) tmp[T_EVENTS] = base + run;
      }
      __syncthreads();
      const uint32_t n_events = tmp[T_EVENTS];
      auto cell_start = [&](uint32_t c) -> uint32_t { return c < K ? (cells[c >> 1] >> ((c & 1u) << 4)) & 0xFFFFu : n_events; };
      // clock << 8 | region << 1 | END: records with equal keys are interchangeable
      auto key_of = [&](int x) -> unsigned long long { return ((unsigned long long)rec[x].y << 8) | (((rec[x].x >> 24) & 0x7Fu) << 1) | (rec[x].x >> 31); };
      const uint32_t g0 = tid * E;
      uint32_t clock[E], info[E];  // this lane's records of the sequence; info: region << 1 | END, bit 8 set: none
      // Windows of less than 2^24 ticks with at most 9 records per cell, with 8 records per lane: the order is
      // finished in registers, on keys of 32 bits that start at the window.  (9: see below.)
      const bool in_lanes = E == 8 && tmp[T_MAXCELL] <= 9u && t_end - t_begin < (1u << 24) - 1u;  // (uniform)
      if (!in_lanes) {
#pragma unroll
        for (int x = 0; x < E; ++x) {
          if (ca[x] != 0xFFFFFFFFu) key(cell_start(ca[x] & 0xFFFFu) + (ca[x] >> 16)) = key_of(x);
        }
      }
      if (in_lanes) {
        // A cell of at most 9 records lies in at most two neighbouring lanes.  The lane sorts its own places; then
        // lanes 2m and 2m + 1 merge (the lower lane keeps the lower 8 of the 16), and after that lanes 2m + 1 and
        // 2m + 2.  The second merge moves no record across the boundary the first one settled: what it hands down
        // to lane 2m + 1 belongs to the cell across the boundary above, which has no record in lane 2m (it would
        // hold 10).
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        // word of a place: 4 words of padding after every 64
        auto word = [&](uint32_t place) -> uint32_t* { return reinterpret_cast<uint32_t*>(smem) + place + ((place >> 6) << 2); };
        auto lane_at = [&](uint32_t t) -> u32x4* { return reinterpret_cast<u32x4*>(word(t * E)); };
#pragma unroll
        for (int x = 0; x < E; ++x) {
          if (ca[x] != 0xFFFFFFFFu) *word(cell_start(ca[x] & 0xFFFFu) + (ca[x] >> 16)) = ((rec[x].y - t_begin) << 8) | (uint32_t)(key_of(x) & 0xFFu);
        }
        __syncthreads();
        uint32_t own[E];
        {
          const u32x4* at = lane_at(tid);
#pragma unroll
          for (int i = 0; i < E; ++i) own[i] = g0 + i < n_events ? at[i / 4][i % 4] : 0xFFFFFFFFu;
        }
        network_sort<E>(own);
#pragma unroll
        for (uint32_t round2 = 0; round2 < 2u; ++round2) {
#pragma unroll
          for (int i = 0; i < E / 4; ++i) lane_at(tid)[i] = u32x4{own[4 * i], own[4 * i + 1], own[4 * i + 2], own[4 * i + 3]};
          __syncthreads();
          const bool upper = ((tid ^ round2) & 1u) != 0u;  // this lane keeps the upper half of the merge
          const bool alone = round2 == 1u && (tid == 0u || tid + 1u == (uint32_t)kBlock);
          const u32x4* partner = lane_at(alone ? tid : (upper ? tid - 1u : tid + 1u));
          const uint32_t neutral = upper ? 0u : 0xFFFFFFFFu;
          u32x4 other[E / 4 ? E / 4 : 1];
#pragma unroll
          for (int i = 0; i < E / 4; ++i) other[i] = partner[i];
#pragma unroll
          for (int i = 0; i < E; ++i) {
            const uint32_t y = alone ? neutral : other[(E - 1 - i) / 4][(E - 1 - i) % 4];
            const uint32_t lo = own[i] < y ? own[i] : y, hi = own[i] < y ? y : own[i];
            own[i] = upper ? hi : lo;
          }
          bitonic_merge<E>(own);
          if (round2 == 0u) __syncthreads();  // every lane has read its partner's records before they are overwritten
        }
#pragma unroll
        for (int i = 0; i < E; ++i) {
          clock[i] = t_begin + (own[i] >> 8);
          info[i] = g0 + i < n_events ? own[i] & 0xFFu : 0x100u;
        }
      } else if (tmp[T_MAXCELL] <= kMaxCell) {
        __syncthreads();
        // place inside the cell: the records with a smaller key, or with the same one and an earlier arrival
        // (all of a lane's records together, so that their reads are in flight together)
        uint32_t nm[E];  // records in the cell (0: this one is no event) | arrival << 16
        uint32_t most = 0;
#pragma unroll
        for (int x = 0; x < E; ++x) {
          const bool event = ca[x] != 0xFFFFFFFFu;
          const uint32_t c = event ? ca[x] & 0xFFFFu : 0u, s0 = cell_start(c), n = event ? cell_start(c + 1u) - s0 : 0u;
          nm[x] = n | (ca[x] & 0xFFFF0000u);
          ca[x] = s0;
          most = n > most ? n : most;
        }
        uint32_t place[E];
#pragma unroll
        for (int x = 0; x < E; ++x) place[x] = ca[x];
        for (uint32_t it = 0; __builtin_amdgcn_ballot_w64(it < most); ++it) {
#pragma unroll
          for (int x = 0; x < E; ++x) {
            const uint32_t n = nm[x] & 0xFFFFu;
            const unsigned long long other = key(it < n ? ca[x] + it : 0u), mine = key_of(x);
            place[x] += (it < n && (other < mine || (other == mine && it < (nm[x] >> 16)))) ? 1u : 0u;
          }
        }
        __syncthreads();
#pragma unroll
        for (int x = 0; x < E; ++x) {
          if (nm[x] & 0xFFFFu) key(place[x]) = key_of(x);
        }
        __syncthreads();
      } else {
        // many records in one cell (waves in lockstep, or a few far apart from the rest): all places, bitonic
        uint32_t n_sort = 64u;
        while (n_sort < n_events) n_sort <<= 1;
        for (uint32_t i = n_events + tid; i < n_sort; i += kBlock) key(i) = kNoKey;
        __syncthreads();
        // A thread takes 8 places at a time, so that up to three steps in a row stay in registers: 33 passes over 8192 places
        // instead of 91.  64 workgroups of 8 x 8192, 16 regions, all records at one clock: 826 us with 91 passes, 583 this way
        // (713 with windows of 2048 whose runs were merged); bursts of 64 records: 896 / 645 (831).
        const bool mine8 = tid < n_sort / 8u;
        unsigned long long v[8];
        auto exchange = [&](int bit) {  // the step over 2^bit of this thread's places
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            if (!((i >> bit) & 1)) {
              const int j = i | (1 << bit);
              const unsigned long long x = v[i], y = v[j];
              v[i] = x < y ? x : y;
              v[j] = x < y ? y : x;
            }
          }
        };
        for (uint32_t l = 3; (1u << l) <= n_sort; ++l) {  // blocks of 2^l in order, every second one falling
          for (uint32_t todo = l; todo != 0u;) {             // steps of this size that are left
            const uint32_t steps = todo < 3u ? todo : 3u, low = steps == 3u ? todo - 3u : 0u;  // the thread's places are 2^low apart
            if (mine8) {
              const uint32_t first = ((tid >> low) << (low + 3u)) | (tid & ((1u << low) - 1u));
              const unsigned long long turn = (first >> l) & 1u ? ~0ull : 0ull;  // a falling block: the complements rise
#pragma unroll
              for (uint32_t i = 0; i < 8u; ++i) v[i] = key(first + (i << low)) ^ turn;
              if (l == 3u) network_sort<8>(v);
              else {
                if (steps == 3u) exchange(2);
                if (steps >= 2u) exchange(1);
                exchange(0);
              }
#pragma unroll
              for (uint32_t i = 0; i < 8u; ++i) key(first + (i << low)) = v[i] ^ turn;
            }
            todo -= steps;
            __syncthreads();
          }
        }
      }
      if (!in_lanes) {
#pragma unroll
        for (int i = 0; i < E; ++i) {
          const unsigned long long v = key(g0 + i);
          clock[i] = (uint32_t)(v >> 8);
          info[i] = g0 + i < n_events ? (uint32_t)v & 0xFFu : 0x100u;
        }
      }
      // ---- sweep ---------------------------------------------------------------------------------------------
      const bool in_slab = hw * 64u * E < n_events;  // (uniform in the wave)
      Planes<NW, P> change;
#pragma unroll
      for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int k = 0; k < P; ++k) change.at[w][k] = 0u;
      auto step = [&](Planes<NW, P>& pl, int i) { planes_step<NW, P>(pl, info[i] >> 1, info[i] < 0x100u ? 1u : 0u, 0u - (info[i] & 1u)); };
      if (in_slab) {
#pragma unroll
        for (int i = 0; i < E; ++i) step(change, i);
        planes_scan_step<0, NW, P>(change); planes_scan_step<1, NW, P>(change); planes_scan_step<2, NW, P>(change);
        planes_scan_step<3, NW, P>(change); planes_scan_step<4, NW, P>(change); planes_scan_step<5, NW, P>(change);
      }
      if (lane == 63u) {
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
          for (int k = 0; k < P; ++k) totals[hw * kMaxPlanes + w * P + k] = change.at[w][k];
      }
      __syncthreads();
      Planes<NW, P> state = open_now;  // before this lane's records
      {
        // the net change of the hardware waves below, and of all of them: lane h of a row takes wave h's
        Planes<NW, P> sum, below;
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
          for (int k = 0; k < P; ++k) sum.at[w][k] = kWavesHw == 16u || (lane & 15u) < kWavesHw ? totals[(lane & 15u) * kMaxPlanes + w * P + k] : 0u;
        planes_scan_step<0, NW, P>(sum); planes_scan_step<1, NW, P>(sum); planes_scan_step<2, NW, P>(sum); planes_scan_step<3, NW, P>(sum);
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
          for (int k = 0; k < P; ++k) {
            below.at[w][k] = hw ? (uint32_t)__builtin_amdgcn_readlane((int)sum.at[w][k], (int)(hw - 1u)) : 0u;
            sum.at[w][k] = (uint32_t)__builtin_amdgcn_readlane((int)sum.at[w][k], 15);
            change.at[w][k] = wave_shr1(change.at[w][k], 0u);  // of the lanes below
          }
        planes_add<NW, P>(open_now, sum);
        if (in_slab) {
          planes_add<NW, P>(state, below);
          planes_add<NW, P>(state, change);
        }
      }
      if (in_slab) {
#pragma unroll
        for (int i = 0; i < E; ++i) {
          const uint32_t r = info[i] >> 1, down = 0u - (info[i] & 1u);
          uint32_t open[NW];  // the regions open on the side of the event where its own count is lower
#pragma unroll
          for (int w = 0; w < NW; ++w) open[w] = planes_any<NW, P>(state, w);
          step(state, i);
          bool own = false;
#pragma unroll
          for (int w = 0; w < NW; ++w) {
            const uint32_t after = planes_any<NW, P>(state, w);
            open[w] = down ? after : open[w];
            if (NW == 1 || (r >> 5) == (uint32_t)w) own = (open[w] >> (r & 31u)) & 1u;
          }
          // the region opens (no wave had it open) or closes (the last wave that had it open)
          if (info[i] < 0x100u && !own) {
            const unsigned long long val = down ? (unsigned long long)clock[i] : 0ull - (unsigned long long)clock[i];
            atomicAdd(pair_sum(r, r), val);  // the time the region is open at all
#pragma unroll
            for (int w = 0; w < NW; w += 2) {
              std::conditional_t<NW == 1, uint32_t, uint64_t> set = open[w];  // (64 bits at a time, but for one word: 472 -> 449 us for 500 of 8 x 8192)
              if constexpr (NW > 1) set |= (uint64_t)open[w + 1] << 32;
              while (set) {
                const uint32_t b = NW == 1 ? (uint32_t)__builtin_ctz((uint32_t)set) : 32u * w + (uint32_t)__builtin_ctzll(set);
                set &= set - 1u;
                atomicAdd(pair_sum(r < b ? r : b, r < b ? b : r), val);
              }
            }
          }
        }
      }
      if (tid < W) pos[tid] += adv[tid];
    }
  }
  __syncthreads();

  // ---- flush this decoder workgroup's totals ----------------------------------------------------
  unsigned long long* out = reinterpret_cast<unsigned long long*>(p.out);
  for (uint32_t i = tid; i < R * kBins; i += kBlock) {
    const uint32_t r = i / kBins, bin = i % kBins, h = hist[r * kHistStride + bin];
    if (h) atomicAdd(&out[SL.hist + r * 64u + bin], (unsigned long long)h);
  }
  for (uint32_t i = tid; i < R * R; i += kBlock) {
    const uint32_t a = i / R, b = i - a * R;
    if (a <= b && otri[b * (b + 1u) / 2u + a]) atomicAdd(&out[SL.F + i], otri[b * (b + 1u) / 2u + a]);
  }
  for (uint32_t r = tid; r < R; r += kBlock) {
    if (reg_min[r] != 0xFFFFFFFFu || reg_max[r] || reg_sum[r]) {
      atomicAdd(&out[SL.sum + r], reg_sum[r]);
      atomicMax(&out[SL.max + r], (unsigned long long)reg_max[r]);
      atomicMin(&out[SL.min + r], (unsigned long long)reg_min[r]);
    }
  }
  if (tid < H_STATUS && ctr[tid]) atomicAdd(&out[tid], ctr[tid]);
}

}  // namespace

namespace kp_reduce {

kp_status wide_supported(const kp_trace_hdr& h) {
  const uint32_t nrec = h.waves_per_wg * h.cap_wave;
  // What the smallest form needs with 64 bins per histogram row: the limits are those from before the rows had 32.
  const uint32_t need = lay_out(1024u, 1u, h.waves_per_wg, h.n_regions, nrec, 2u, 0u, false).list + kListMin * 8u + h.n_regions * (64u - kBins) * 4u;
  if (need > kMaxLds)
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE,
                    "%u record slots per workgroup with %u regions: the decoder needs %u B of LDS (limit %u)", nrec,
                    h.n_regions, need, kMaxLds);
  return KP_OK;
}

namespace {

template <int BLOCK, int E, int NW, int P>
kp_status launch(const WideParams& p, hipStream_t s) {
  auto kern = kp_reduce_wide<BLOCK, E, NW, P>;
  static thread_local kp_stage::LaunchCache cache;
  uint32_t grid = 0;
  const kp_status st = kp_stage::resident_grid(kern, BLOCK, p.lds.total, &cache, &grid);
  if (st != KP_OK) return st;
  if (grid > p.n_wg) grid = p.n_wg;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(BLOCK), p.lds.total, s, p);
  KP_HIP_TRY(hipGetLastError());
  return KP_OK;
}
template <int BLOCK, int E>
kp_status launch_words(const WideParams& p, hipStream_t s) {
  // (What no geometry comes with is not built: with up to 32 regions it is more than 16384 slots; with 16 waves and two records per
  // lane more than 64 regions; with 16 waves and more than 64 regions three workgroups do not share a CU's LDS.)
  constexpr bool small = BLOCK < 1024 && BLOCK * E <= 2048;
  if (p.W == 16) {  // counts up to 16
    if constexpr (!small && E != 2) { if (p.R <= 32) return launch<BLOCK, E, 1, 5>(p, s); }
    if constexpr (E != 2) { if (p.R <= 64) return launch<BLOCK, E, 2, 5>(p, s); }
    if constexpr (BLOCK != 256) { if (p.R > 64) return launch<BLOCK, E, 4, 5>(p, s); }
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "no decoder for 16 waves, %u regions and %u record slots per workgroup", p.R, p.nrec);
  }
  if constexpr (!small) { if (p.R <= 32) return launch<BLOCK, E, 1, 4>(p, s); }
  return p.R <= 64 ? launch<BLOCK, E, 2, 4>(p, s) : launch<BLOCK, E, 4, 4>(p, s);
}

}  // namespace

kp_status launch_wide(const uint32_t* wg_hdrs, const void* records, uint64_t* out, const kp_trace_hdr& h,
                      hipStream_t s) {
  const kp_status ok = wide_supported(h);
  if (ok != KP_OK) return ok;
  WideParams p;
  p.wg_hdrs = wg_hdrs;
  p.records = static_cast<const uint2*>(records);
  p.out = out;
  p.n_wg = h.n_wg; p.W = h.waves_per_wg; p.R = h.n_regions; p.cap = h.cap_wave;
  p.cap_log2 = 0; while ((1u << p.cap_log2) < p.cap) ++p.cap_log2;
  p.rec_cost = h.rec_cost; p.flush = h.flags & KP_FLAG_FLUSH;
  p.nrec = p.W * p.cap;
  p.waves_log2 = 0; while ((1u << p.waves_log2) < p.W) ++p.waves_log2;
  uint32_t wgs = 0;
  const kp_status known = wgs_of_256_cus(p.n_wg, &wgs);
  if (known != KP_OK) return known;
  // How many threads take a recorded workgroup (numbers of workgroups are those on 256 CUs).  1024, and windows of 8192 places, are
  // all that fits one CU.  With more recorded workgroups than CUs two of 512 threads, with 4096 places each, hide each other's barriers and
  // LDS round trips: 1024 workgroups of 8 x 4096 slots, 48 regions 675 -> 627 us, 1000 of 16 x 2048, 16 regions 772 -> 743, 2000 of
  // 8 x 2048, 64 regions 829 -> 699, 3000 of 4 x 1024, 64 regions 428 -> 285, 257 of 8 x 4096 359 -> 332, 512 of 3 x 8192 the same;
  // with no more of them than CUs it is one workgroup's chain of steps: 100 of 8 x 4096 172 against 235 us, 200 of 16 x 512 82 / 118.
  // Up to 2048 slots one window of 2048 places holds all there are: three workgroups of 256 threads where LDS has room
  // (1024 threads / 512 / 256, us: 4000 of 8 x 256, 40 regions 394 / 226 / 185, 4000 of 1 x 256 300 / 160 / 123), else, and with few
  // workgroups, 512 threads with four records each (100 of 2 x 256 27.0 -> 24.2, 256 of 2 x 512, 64 regions 38.8 -> 36.5, 1021 of
  // 8 x 256, 64 regions 146 -> 92).
  if (p.nrec <= 2048u && wgs > 256u) {
    p.lds = lay_out(256u, 3u, p.W, p.R, p.nrec, 8u, 0u, true);
    if (p.lds.total <= kMaxLds / 3u) return launch_words<256, 8>(p, s);
  }
  if (p.nrec <= 2048u) {
    const uint32_t per_cu = wgs > 256u ? 2u : 1u;
    p.lds = lay_out(512u, per_cu, p.W, p.R, p.nrec, 4u, split_log2(512u, p.W, p.cap), true);
    if (p.lds.total <= kMaxLds / per_cu) return launch_words<512, 4>(p, s);
  }
  // (With more than one window each, two of them take 1.9 times as long as one of 1024 threads alone and one that is left over
  // 1.4 times: a last turn of at most one to a CU pays only behind three full ones.  582 of 7 x 1024, 64 regions 110 us, 126 this way.)
  const bool full_turns = p.nrec <= 4096u || wgs >= 1536u || (wgs - 1u) % 512u >= 256u;
  // (One window of 8192 places is better than two or three of 4096: 1362 of 12 x 512, 40 regions 210 us against 231.)
  const bool one_large = p.cap <= (8192u >> p.waves_log2) && p.cap > (4096u >> p.waves_log2);
  if (wgs > 256u && full_turns && !one_large) {
    p.lds = wide_lds(512u, 2u, p.W, p.R, p.cap);
    if (p.lds.total <= kMaxLds / 2u && p.lds.per_lane == 8u) return launch_words<512, 8>(p, s);
  }
  // (one window of 4096 places, four records a lane, where three quarters of it hold all: 170 of 12 x 256 slots, 100 regions 65.0 ->
  // 61.6 us, 600 of 5 x 512, 100 regions 140 -> 132; of 8192 with full ones: 100 of 16 x 256 80.8 -> 80.1)
  if (p.nrec <= 3072u) {
    p.lds = lay_out(1024u, 1u, p.W, p.R, p.nrec, 4u, split_log2(1024u, p.W, p.cap), true);
    if (p.lds.total <= kMaxLds) return launch_words<1024, 4>(p, s);
  }
  p.lds = wide_lds(1024u, 1u, p.W, p.R, p.cap);
  return p.lds.per_lane == 8 ? launch_words<1024, 8>(p, s) : (p.lds.per_lane == 4 ? launch_words<1024, 4>(p, s) : launch_words<1024, 2>(p, s));
}

}  // namespace kp_reduce
