// GPU trace decode / pair / reduce (kp_trace_reduce).
//
// The paper stores START/END records unpaired, per warp, in a ring whose tail survives, and
// aligns them at "trace replay" on the host (Sec. 4.2 "SM-level Data Layout", "Shared Memory
// Circular Buffer"; Sec. 4.3).  Here replay runs on the GPU: one persistent decoder workgroup
// takes one recorded workgroup at a time.
//   A  every lane holds the records of NR / 2 rounds of 128 consecutive slots, two neighbours per round, and checks that
//      they are the ones that belong there (seq against slot).  One that is not goes to its slot through LDS, in O(1), which
//      undoes out-of-order flushes; ring rotation is a question of which slot is the oldest.  The records of the next
//      workgroup are requested before the results of the current one are written;
//   B  an END is paired iff the nearest earlier record of its (wave, region) is a START --
//      usually the slot just below, in the same lane or the lane below (DPP), four records at a time on their packed
//      metadata bytes; the others look through the records in LDS, where they are put only if some END has to;
//      d = (u32)(ts_end - ts_start) minus the constant record cost (Sec. 4.3) goes to the
//      per-(wave, region) sums and the log2 histogram with LDS atomics;
//   C  the paired records of all waves are sorted by clock: counting sort into time cells (one
//      LDS atomic per record gives cell and arrival slot) and a prefix sum over the cells put
//      them in cell order;
//   D  every lane takes NR (4 or 16) consecutive records of that sequence and finishes the order in
//      registers (a sorting network over its own records, then a merge of its outer halves with
//      the neighbouring lanes').  A first pass gives each lane's net change in the number of waves that have each region
//      open, a prefix sum over lanes and waves (one 64-bit number with four bits per region, up to 15 waves) the state at
//      the start of each lane's stretch, and a second pass, on bit-sliced counts (plane k = bit k of every region's count),
//      the set of open regions after every record.  The time two regions
//      are both open is the sum over the stretches between records of length * open(a) * open(b):
//      a matrix product, taken by the matrix cores 64 stretches at a time;
//   E  the per-(workgroup, wave, region) results go to HBM and into running totals, which live in
//      LDS and reach HBM once per decoder workgroup.
// What bounds it is instruction issue: 2.5 vector instructions per record (3.2 with every record scattered to LDS by its
// rank and read back, one round at a time in B, planes in the prefix sum): 16384 workgroups of 8 x 2048 records 1775 -> 1550
// us; 4000 of 4 x 1024, wrapped 125 -> 114; 256 of 8 x 512 28.7 -> 27.1; 512 of 8 x 2048, regions three deep 389 -> 219.
// A kernel of its own per class of ring sizes (RINGS), and for more than 16 regions (MANY), instead of one that chooses:
// 16384 of 8 x 2048 1562 -> 1495, 8191 of 2 x 4096 889 -> 856, 8192 of 16 x 32 74.0 -> 70.1, 64 of 4 x 128 16.4 -> 15.5, 65534 of 7 x 128,
// 32 regions 1325 -> 1289.
// Traces outside what the register sort covers (more than 16 regions, a span of 2^26 ticks or
// more, a time cell with more than NR + 1 records) rank the records inside their cell by comparing
// clocks and add every switch of a region to the region-pair sums with LDS atomics.
// A workgroup with a corrupt record (bad field, duplicated seq) has holes in its ranks; it is rare,
// takes no part in the overlap statistics and is paired by a plain serial walk per (wave, region).
#include "kp_reduce.h"

#include <type_traits>

namespace {

using namespace kp_reduce;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kSeqMask = 0xFFFFFu;
// staged metadata byte: bits 5:0 region (63 = no record), 6 paired, 7 END
constexpr uint32_t kRegion = 0x3Fu, kEmpty = 0x3Fu, kPaired = 0x40u, kEnd = 0x80u;
constexpr uint32_t kMaxRecPerWg = 16384;
constexpr uint32_t kMaxLds = 160 * 1024;
constexpr uint32_t kBins = 32, kHistStride = 33;  // (durations have 32 bits) histogram rows an odd number of words apart: equal bins of different regions, different banks

// rings of less than 128 slots; of 128 and more, so that a round is one recorded wave's, but less than a hardware wave's share; of at
// least that share; either of the last two
enum { kSmall, kPart, kWhole, kAny };
// steps after which kp_trace_reduce_steps can leave a workgroup
enum { kStepOrdered = 1, kStepPaired, kStepCounted, kStepCellSums, kStepPlaced, kStepRanked, kStepSorted, kStepSwept };

// A condition that seldom holds: what hangs on it is kept out of the straight line of instructions, which a launch of few
// workgroups has to fetch before it can run.
__device__ __forceinline__ bool rare(bool x) { return __builtin_expect(x, false); }

// per-workgroup temporaries (u32 words in LDS)
enum { T_BAD = 0, T_DISORDER, T_UNFILLED, T_NONMONO, T_PAIRS, T_STARTS, T_ENDS,
       T_EVENTS, T_MARKS, T_DEEP, T_WIDE, T_MAXCELL, T_ZERO, T_HELD, T_COUNT };  // T_HELD stays last

struct DecodeParams {
  const uint32_t* wg_hdrs;  // 32 words per recorded workgroup
  const u32x4* records;     // two records per 16-byte load
  uint64_t* out;
  uint32_t n_wg, W, R, cap, cap_log2, rec_cost, flush;
  uint32_t nrec;            // record slots per recorded workgroup
  uint32_t ncopy;           // copies of the per-(wave, region) sums: 1, 2 or 4
  uint32_t stop_after;      // 0: everything; else leave each workgroup after this step (timing only), see kStep*
};

__host__ __device__ constexpr uint32_t align16(uint32_t x) { return (x + 15u) & ~15u; }
constexpr uint32_t kMaxPerWave = 1024;  // entries of the per-(wave, region) sums, copies included

// LDS of a decoder workgroup, byte offsets.  Every array is sized for the largest geometry the kernel takes (RMAX regions,
// PERWAVE entries of the per-(wave, region) sums), so that all addresses are compile-time constants.  A team of BLOCK
// threads decodes one recorded workgroup at a time in arrays of its own; the TEAMS teams of a decoder workgroup share the
// running totals.
template <int BLOCK, int NR, int TEAMS, int RMAX, int PERWAVE>
struct Lds {
  static constexpr uint32_t npos = BLOCK * NR, ncell = BLOCK * 16;
  // (What is addressed by a computed index stands in the first 64 KiB: its base then fits the instruction.)
  // of all teams
  static constexpr uint32_t hist = 0;
  static constexpr uint32_t teams = align16(hist + RMAX * kHistStride * 4);
  // of every team, from the start of its block on
  static constexpr uint32_t pw_pack = 0;
  static constexpr uint32_t pw_max = pw_pack + PERWAVE * 8;
  static constexpr uint32_t pw_min = pw_max + PERWAVE * 4;
  static constexpr uint32_t cells = pw_min + PERWAVE * 4;                  // one 16-bit counter per time cell + the total
  static constexpr uint32_t clk = align16(cells + (ncell / 2 + 4) * 4);    // 4 words of padding after every 64
  static constexpr uint32_t meta = align16(clk + (npos + npos / 16) * 4);
  static constexpr uint32_t tmp = align16(meta + npos + 16);
  static constexpr uint32_t misc = align16(tmp + T_COUNT * 4);
  static constexpr uint32_t vf = misc + 4 * 4;
  static constexpr uint32_t ring_end = vf + (KP_MAX_WAVES + 1) * 8;
  static constexpr uint32_t wtot = ring_end + KP_MAX_WAVES * 8;
  static constexpr uint32_t ptot = wtot + 16 * 4;
  static constexpr uint32_t wave_end = ptot;                               // (done with before ptot is written)
  static constexpr uint32_t oacc32 = align16(ptot + (BLOCK / 64) * 8 * 4);
  static constexpr uint32_t team = align16(oacc32 + RMAX * (RMAX + 1) * 4);
  // of all teams
  static constexpr uint32_t ctr = teams + TEAMS * team;
  static constexpr uint32_t oacc = ctr + 16 * 8;
  static constexpr uint32_t reg_sum = oacc + RMAX * RMAX * 8;
  static constexpr uint32_t reg_max = reg_sum + RMAX * 8;
  static constexpr uint32_t reg_min = reg_max + RMAX * 4;
  static constexpr uint32_t total = align16(reg_min + RMAX * 4);
  static_assert(total <= kMaxLds, "decoder LDS exceeds one CU");
  // waves per SIMD that this leaves room for, at most the four for which 128 registers do
  static constexpr int waves = (int)(kMaxLds / total) * (BLOCK * TEAMS / 64) / 4;
  static constexpr int waves_per_simd = waves < 1 ? 1 : waves > 4 ? 4 : waves;
};

// All threads of a team.  Where that is one wave its LDS operations are done in order, and only the compiler has to be held.
template <int BLOCK>
__device__ __forceinline__ void team_sync() {
  if constexpr (BLOCK == 64) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// Word of the clock array that holds position i: 4 words of padding after every 64, so that the
// 64 lanes of a wave reading 16 consecutive words each (64 bytes apart) spread over all banks.
__device__ __forceinline__ uint32_t clk_word(uint32_t i) { return i + ((i >> 6) << 2); }

// a += b for bit-sliced numbers: plane k holds bit k of 32 independent counters, modulo 2^PLANES.
template <int PLANES>
__device__ __forceinline__ void planes_add(uint32_t (&a)[PLANES], const uint32_t (&b)[PLANES]) {
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < PLANES; ++k) {
    const uint32_t s = a[k] ^ b[k];
    const uint32_t g = a[k] & b[k];
    a[k] = s ^ c;
    c = g | (s & c);
  }
}

// counter[bit of x] += 1 (up = all ones) or -= 1 (up = 0); x is zero or one-hot.
template <int PLANES>
__device__ __forceinline__ void planes_step(uint32_t (&pl)[PLANES], uint32_t x, uint32_t up) {
  uint32_t carry = x;
#pragma unroll
  for (int k = 0; k < PLANES; ++k) { const uint32_t o = pl[k]; pl[k] = o ^ carry; carry = __builtin_amdgcn_bitop3_b32(carry, o, up, 0x90); }  // carry & ~(o ^ up), which the compiler would make two instructions of
}

// The sweep works on one word per record of the sequence: clock << 6 | START << 5 | region; records with
// equal words are interchangeable.  Of the records of one clock the ENDs come first: pairs of length 0 are not in the
// sequence, so every END meets a count that has its START in it, and no count ever exceeds the number of waves, whichever
// waves end a region and start it again on that clock.  A place past the end of the sequence holds `fake`: the largest
// clock of the workgroup with a region number that no record has, so that it sorts last, opens no
// region and the stretch in front of it has an honest length.
// Fields of such a word.
__device__ __forceinline__ uint32_t key_clock(uint32_t k) { return k >> 6; }
__device__ __forceinline__ uint32_t key_region_bit(uint32_t k) { return 1u << (k & 31u); }  // bit 31 for a place past the end: above every region
__device__ __forceinline__ uint32_t key_start_mask(uint32_t k) { return (uint32_t)__builtin_amdgcn_sbfe((int)k, 5, 1); }  // all ones for a START

// Eight 4-bit numbers as planes: byte k of the result holds bit k of each.  Bit 4 r + k goes to 8 k + r: the five index
// bits r2 r1 r0 k1 k0 become k1 k0 r2 r1 r0, by four exchanges of two of them.
__device__ __forceinline__ uint32_t planes_of_nibbles(uint32_t x) {
  auto exchange = [&](int d, uint32_t m) { const uint32_t t = ((x >> d) ^ x) & m; x ^= t ^ (t << d); };
  exchange(14, 0x0000CCCCu);
  exchange(7, 0x00AA00AAu);
  exchange(2, 0x0C0C0C0Cu);
  exchange(1, 0x22222222u);
  return x;
}

// The NR records of the clock-sorted sequence that lane `tid` of the sweep owns, from a sequence that
// is only ordered cell by cell (inside a cell the records stand in arrival order).  Cells follow one
// another in clock order, so sorting the words sorts every cell and moves no record out of its cell.
template <int NR>
__device__ __forceinline__ void load_run(const uint32_t* clk, uint32_t lane_of_sweep, uint32_t (&key)[NR]) {
  const u32x4* at = reinterpret_cast<const u32x4*>(clk + clk_word(lane_of_sweep * NR));
#pragma unroll
  for (int x = 0; x < NR / 4; ++x) {
    const u32x4 v = at[x];
    key[4 * x] = v.x; key[4 * x + 1] = v.y; key[4 * x + 2] = v.z; key[4 * x + 3] = v.w;
  }
}
template <int NR>
__device__ __forceinline__ void store_run(uint32_t* clk, uint32_t lane_of_sweep, const uint32_t (&key)[NR]) {
  u32x4* at = reinterpret_cast<u32x4*>(clk + clk_word(lane_of_sweep * NR));
#pragma unroll
  for (int x = 0; x < NR / 4; ++x) at[x] = u32x4{key[4 * x], key[4 * x + 1], key[4 * x + 2], key[4 * x + 3]};
}
template <int NR>
__device__ __forceinline__ void load_and_sort_own(const uint32_t* clk, uint32_t tid, uint32_t n_events, uint32_t fake, uint32_t (&key)[NR]) {
  load_run<NR>(clk, tid, key);
  if (__builtin_amdgcn_ballot_w64(tid * NR + NR > n_events)) {
#pragma unroll
    for (int y = 0; y < NR; ++y) key[y] = tid * NR + y < n_events ? key[y] : fake;
  }
  network_sort<NR>(key);
}

// Form for cells of at most NR / 2 + 1 records: the lane sorts its own NR places and puts them back; a cell that
// lies across the boundary to the next lane then has at most NR / 2 records on either side, all of them in
// the upper half here and in the lower half there, so merging these two halves (both sorted) and
// handing the lower ones back to this lane, the upper ones to the next one finishes the job.  Each lane does
// that for its lower half with the lane below and for its upper half with the lane above: the larger
// (smaller) of element i of one run and element NR / 2 - 1 - i of the other are the upper (lower) ones of the two
// runs, in rising-then-falling order.  Contains one barrier of the team.
template <int BLOCK, int NR>
__device__ __forceinline__ void sorted_own(uint32_t* clk, uint32_t tid, uint32_t n_events, uint32_t fake, uint32_t (&key)[NR]) {
  constexpr int H = NR / 2;
  load_and_sort_own<NR>(clk, tid, n_events, fake, key);
  store_run<NR>(clk, tid, key);
  team_sync<BLOCK>();
  uint32_t below[NR], above[NR];  // (the halves that are not used are not loaded)
  load_run<NR>(clk, tid > 0 ? tid - 1 : 0, below);
  load_run<NR>(clk, tid + 1 < BLOCK ? tid + 1 : tid, above);
  const uint32_t lo_gate = tid > 0 ? 0xFFFFFFFFu : 0u;           // no lane below: nothing comes up
  const uint32_t hi_fill = tid + 1 < BLOCK ? 0u : 0xFFFFFFFFu;  // no lane above: nothing comes down
  uint32_t lo[H], hi[H];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const uint32_t bw = below[H + i] & lo_gate, aw = above[H - 1 - i] | hi_fill;
    lo[i] = key[H - 1 - i] > bw ? key[H - 1 - i] : bw;  // the upper ones of (upper half below, own lower half)
    hi[i] = key[H + i] < aw ? key[H + i] : aw;          // the lower ones of (own upper half, lower half above)
  }
  bitonic_merge<H>(lo);
  bitonic_merge<H>(hi);
#pragma unroll
  for (int i = 0; i < H; ++i) { key[i] = lo[i]; key[H + i] = hi[i]; }
}

// Form for cells of up to NR + 1 records: a cell then lies in at most two neighbouring lanes, with up to NR
// records in either.  The lane sorts its own places; then lanes 2m and 2m + 1 merge their runs (the
// lower lane keeps the lower NR, the upper lane the upper NR), and after that lanes 2m + 1 and
// 2m + 2 do the same.  The second merge moves no record across the boundary the first one settled: what
// it hands down to lane 2m + 1 belongs to the cell that lies across the boundary above, and that cell
// has no record in lane 2m (it would hold NR + 2).  Contains three barriers of the team.
template <int BLOCK, int NR>
__device__ __forceinline__ void sorted_pairs(uint32_t* clk, uint32_t tid, uint32_t n_events, uint32_t fake, uint32_t (&key)[NR]) {
  load_and_sort_own<NR>(clk, tid, n_events, fake, key);
#pragma unroll
  for (int round = 0; round < 2; ++round) {
    store_run<NR>(clk, tid, key);
    team_sync<BLOCK>();
    // round 0: partner of lane t is t ^ 1; round 1: the other neighbour (the first and the last lane have none)
    const bool upper = ((tid ^ (uint32_t)round) & 1u) != 0u;  // this lane keeps the upper ones of the merge
    const bool alone = round == 1 && (tid == 0u || tid + 1u == BLOCK);
    uint32_t pw[NR];
    load_run<NR>(clk, alone ? tid : upper ? tid - 1u : tid + 1u, pw);
    // the larger (smaller) of element i of one run and element NR - 1 - i of the other: the upper (lower) ones
    const uint32_t neutral = upper ? 0u : 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const uint32_t x = key[i], y = alone ? neutral : pw[NR - 1 - i];
      const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
      key[i] = upper ? hi : lo;
    }
    bitonic_merge<NR>(key);
    if (round == 0) team_sync<BLOCK>();  // every lane has read its partner's run before it is overwritten
  }
}

// ------------------------------------------------------------------------------------------
// init: clear the global totals, set min to all-ones, check the device header against the
// geometry the launch was sized for.
__global__ void kp_reduce_init(const uint32_t* trace_hdr, uint64_t* out, uint32_t n_wg, uint32_t W,
                               uint32_t R, uint32_t cap, uint32_t flags) {
  const StatsLayout l = stats_layout(n_wg, W, R);
  for (size_t i = threadIdx.x + (size_t)blockIdx.x * blockDim.x; i < l.per; i += (size_t)blockDim.x * gridDim.x)
    out[i] = (i >= l.min && i < l.max) ? ~0ull : 0ull;
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const bool ok = trace_hdr[0] == KP_TRACE_MAGIC && trace_hdr[1] == KP_TRACE_VERSION &&
                    trace_hdr[2] == n_wg && trace_hdr[3] == W && trace_hdr[4] == R &&
                    trace_hdr[5] == cap && trace_hdr[7] == flags;
    out[H_STATUS] = ok ? 0ull : 1ull;
    out[H_NWG] = n_wg; out[H_WAVES] = W; out[H_NREG] = R; out[H_CAP] = cap;
  }
}

// derive (one workgroup, a kernel of its own behind the main one): the figures that follow from the totals.  The
// pairs of a region are the sum of its histogram, the region-pair sums stand in the upper triangle of the F area (away
// from the sums and extrema: atomics of many workgroups on one line wait for one another) and are mirrored into O,
// U is the diagonal, F = O / U.
// Having the last of few decoder workgroups do this instead gains nothing that would pay for the count: 64
// workgroups of 4 x 128 records, 3 regions 20.9 us this way and 21.3 counted; 64 of 4 x 256, 16 regions 24.4 and
// 27.2; 64 of 8 x 512, 5 regions 25.7 and 25.1; 256 of them 32.3 and 33.0.
__global__ __launch_bounds__(1024) void kp_reduce_derive(uint64_t* out, uint32_t n_wg, uint32_t W, uint32_t R) {
  const StatsLayout l = stats_layout(n_wg, W, R);
  // Up to 32 regions: one element per thread, requested ahead of the histograms and read before any is written, so that
  // there is one way to memory and back.
  uint64_t o = 0, u = 0;
  const uint32_t at = threadIdx.x, at_a = at / R, at_b = at - at_a * R;
  if (R <= 32u && at < R * R) {
    o = out[l.F + (at_a <= at_b ? at : at_b * R + at_a)];
    u = out[l.F + at_a * R + at_a];
  }
  for (uint32_t i = threadIdx.x; i < ((R * 16u + 63u) & ~63u); i += blockDim.x) {  // 16 lanes per region
    const uint32_t r = i >> 4, part = i & 15u;
    uint64_t n = 0;
    if (r < R) {
      const uint64_t* bins = out + l.hist + (size_t)r * 64 + part;
      n = bins[0] + bins[16] + bins[32] + bins[48];
    }
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) n += __shfl_xor((unsigned long long)n, d, 64);
    if (r < R && part == 0u) out[l.cnt + r] = n;
  }
  if (R <= 32u) {
    __syncthreads();
    if (at < R * R) {
      out[l.O + at] = o;
      if (at_a == at_b) out[l.U + at_a] = o;
      reinterpret_cast<double*>(out)[l.F + at] = u ? (double)o / (double)u : 0.0;
    }
    return;
  }
  for (uint32_t i = threadIdx.x; i < R * R; i += blockDim.x) {
    const uint32_t a = i / R, b = i - a * R;
    const uint64_t o = out[l.F + (a <= b ? i : b * R + a)];
    out[l.O + i] = o;
    if (a == b) out[l.U + a] = o;
  }
  __syncthreads();  // (a workgroup's own global stores are visible to it after the barrier)
  for (uint32_t i = threadIdx.x; i < R * R; i += blockDim.x) {
    const uint64_t u = out[l.U + i / R], o = out[l.O + i];
    reinterpret_cast<double*>(out)[l.F + i] = u ? (double)o / (double)u : 0.0;
  }
}

// ------------------------------------------------------------------------------------------
// Position p = wave*cap_wave + slot.  Hardware wave h of the decoder
// owns the 64 * NR positions from 64 * NR * h on, and lane l takes 128 j + 2 l of them and the one above it in round j,
// so that neighbouring lanes hold neighbouring slots.
// RINGS: slots of a ring.  MANY: more than 16 regions, which
// the register sort does not take.
template <int BLOCK, int NR, int TEAMS, int PLANES, int RMAX, int PERWAVE, int RINGS, bool MANY>
__global__ __launch_bounds__(BLOCK * TEAMS, (Lds<BLOCK, NR, TEAMS, RMAX, PERWAVE>::waves_per_simd)) void kp_reduce_main(DecodeParams p) {
  using L = Lds<BLOCK, NR, TEAMS, RMAX, PERWAVE>;
  constexpr bool SMALL = RINGS == kSmall;
  constexpr uint32_t kWaveSpan = 64 * NR;      // positions per hardware wave
  constexpr uint32_t kMaxCellWindow = NR + 1;  // fullest time cell the sweep's register sort covers
  static_assert(TEAMS == 1 || BLOCK == 64, "teams of more than one wave have no barrier of their own");
  __shared__ __align__(16) unsigned char shared[L::total];
  const uint32_t team = TEAMS == 1 ? 0u : (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t n_teams = TEAMS == 1 ? 1u : blockDim.x >> 6;  // (as many as the launch asked for)
  unsigned char* smem = shared + L::teams + team * L::team;
  uint32_t* clk = reinterpret_cast<uint32_t*>(smem + L::clk);
  uint8_t* meta = smem + L::meta;
  uint32_t* cells = reinterpret_cast<uint32_t*>(smem + L::cells);  // cell c: half (c & 1) of word c >> 1
  uint32_t* hist = reinterpret_cast<uint32_t*>(shared + L::hist);
  unsigned long long* oacc = reinterpret_cast<unsigned long long*>(shared + L::oacc);
  uint32_t* oacc32 = reinterpret_cast<uint32_t*>(smem + L::oacc32);  // this workgroup's sums modulo 2^32
  unsigned long long* reg_sum = reinterpret_cast<unsigned long long*>(shared + L::reg_sum);
  uint32_t* reg_max = reinterpret_cast<uint32_t*>(shared + L::reg_max);
  uint32_t* reg_min = reinterpret_cast<uint32_t*>(shared + L::reg_min);
  unsigned long long* pw_pack = reinterpret_cast<unsigned long long*>(smem + L::pw_pack);
  uint32_t* pw_max = reinterpret_cast<uint32_t*>(smem + L::pw_max);
  uint32_t* pw_min = reinterpret_cast<uint32_t*>(smem + L::pw_min);
  unsigned long long* ctr = reinterpret_cast<unsigned long long*>(shared + L::ctr);
  uint32_t* tmp = reinterpret_cast<uint32_t*>(smem + L::tmp);
  uint32_t* misc = reinterpret_cast<uint32_t*>(smem + L::misc);  // [0] span overflow, [1] cell scale, [2] span
  uint2* sVF = reinterpret_cast<uint2*>(smem + L::vf);           // per wave: records held, first surviving seq
  uint2* ring_end = reinterpret_cast<uint2*>(smem + L::ring_end);  // per wave: clock and metadata in the last slot of its ring
  uint2* wave_end = reinterpret_cast<uint2*>(smem + L::wave_end);  // the same of the last position of each hardware wave
  uint32_t* wtot = reinterpret_cast<uint32_t*>(smem + L::wtot);
  uint32_t* ptot = reinterpret_cast<uint32_t*>(smem + L::ptot);

  auto seldom = [](bool x) -> bool { return NR == 4 || SMALL ? x : rare(x); };  // (where a ring begins or ends: in most rounds of small workgroups)
  constexpr uint32_t NPOS = L::npos, NCELL = L::ncell;
  constexpr uint32_t kSlotShift = (BLOCK == 1024 ? 14 : BLOCK == 512 ? 13 : BLOCK == 256 ? 12 : BLOCK == 128 ? 11 : 10) + 4;
  // The last four words of the clock array are padding that no position maps to, and the metadata
  // array has 16 spare bytes: stores of lanes that have nothing to store go there instead of branching.
  constexpr uint32_t kSpareWord = NPOS + NPOS / 16 - 1;
  const uint32_t tid_k = TEAMS == 1 ? threadIdx.x : threadIdx.x & 63u;  // in the team
  // The kernel arguments arrive as one block of scalar registers.  Each one used in the loop gets a
  // register of its own through an opaque move: when scalar registers run short the compiler then parks
  // and fetches single values instead of the whole block.
  auto own_reg = [](uint32_t x) -> uint32_t { uint32_t y; asm("s_mov_b32 %0, %1" : "=s"(y) : "s"(x)); return y; };
  const uint32_t W = own_reg(p.W), R = own_reg(p.R), cap = own_reg(p.cap), nrec = own_reg(p.nrec);
  const uint32_t capm = cap - 1, cl2 = own_reg(p.cap_log2);
  const uint32_t n_wg = own_reg(p.n_wg), n_copies = own_reg(p.ncopy), stop_after = own_reg(p.stop_after);
  const uint32_t rec_cost = own_reg(p.rec_cost), flush = own_reg(p.flush);
  const StatsLayout SL = stats_layout(n_wg, W, R);
  const uint64_t status = p.out[H_STATUS];  // (needed behind the first requests only)

  const uint32_t n_threads = TEAMS == 1 ? (uint32_t)BLOCK : blockDim.x;
  for (uint32_t i = threadIdx.x; i < R * kHistStride; i += n_threads) hist[i] = 0;
  for (uint32_t i = threadIdx.x; i < R * R; i += n_threads) oacc[i] = 0;
  for (uint32_t i = tid_k; i < R * (R | 1u); i += BLOCK) oacc32[i] = 0;
  for (uint32_t i = threadIdx.x; i < R; i += n_threads) { reg_sum[i] = 0; reg_max[i] = 0; reg_min[i] = 0xFFFFFFFFu; }
  for (uint32_t i = tid_k; i < n_copies * W * R; i += BLOCK) { pw_pack[i] = 0; pw_max[i] = 0; pw_min[i] = 0xFFFFFFFFu; }
  if (threadIdx.x < 16) ctr[threadIdx.x] = 0;
  __syncthreads();

  auto clear_meta = [&](uint32_t t) __attribute__((always_inline)) {  // no record: the NR metadata bytes of thread t
    if constexpr (NR == 16) reinterpret_cast<u32x4*>(meta)[t] = u32x4{0x3F3F3F3Fu, 0x3F3F3F3Fu, 0x3F3F3F3Fu, 0x3F3F3F3Fu};
    else reinterpret_cast<uint32_t*>(meta)[t] = 0x3F3F3F3Fu;
  };
  auto load_meta = [&](uint32_t t, uint32_t (&w)[NR / 4]) __attribute__((always_inline)) {
    if constexpr (NR == 16) {
      const u32x4 v = reinterpret_cast<const u32x4*>(meta)[t];
      w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    } else {
      w[0] = reinterpret_cast<const uint32_t*>(meta)[t];
    }
  };

  // The records of a workgroup (NR / 2 16-byte units, two records each, per thread) and the words of its
  // header are requested one workgroup ahead, before the previous workgroup's results are written, so
  // that the memory latency runs under that tail and under the clearing of the staging state.
  u32x4 v[NR / 2];
  uint32_t h_total;  // lane & 15 -> records written by that wave
  uint2 h_begin, h_end;
  constexpr int kEarly = NR / 2 * 3 / 4 > 1 ? NR / 2 * 3 / 4 : NR / 2;  // units requested before the matrix products of the sweep of the workgroup before
  auto request_units = [&](uint32_t g, uint32_t t, auto first, auto last) {
    const u32x4* recs = p.records + (size_t)g * (nrec / 2);
    const uint32_t t_first = (t >> 6) * (kWaveSpan / 2u) + (t & 63u);
#pragma unroll
    for (int u = decltype(first)::value; u < decltype(last)::value; ++u) {
      const uint32_t i = t_first + 64u * u;
      v[u] = __builtin_nontemporal_load(recs + (i < nrec / 2 ? i : nrec / 2 - 1));
    }
  };
  auto request_header = [&](uint32_t g, uint32_t t) {
    const uint32_t* whn = p.wg_hdrs + (size_t)32 * g;
    h_total = whn[8 + (t & 15u)];
    h_begin = *reinterpret_cast<const uint2*>(whn + 2);
    h_end = *reinterpret_cast<const uint2*>(whn + 4);
  };
  const uint32_t first_wg = blockIdx.x + team * gridDim.x, stride = gridDim.x * n_teams;
  {
    const uint32_t at = TEAMS == 1 || first_wg < n_wg ? first_wg : n_wg - 1u;  // (a team without a workgroup asks all the same)
    request_units(at, tid_k, std::integral_constant<int, 0>{}, std::integral_constant<int, kEarly>{});
    request_header(at, tid_k);
  }
  if (status != 0) return;  // device header did not match the launch geometry

  for (uint32_t wg = first_wg; wg < n_wg; wg += stride) {
    // A fresh copy of the thread index per workgroup that the optimiser cannot see through: without it
    // the address arithmetic of all rounds is computed once before the loop and held in registers
    // for the whole kernel.
    uint32_t tid = tid_k;
    asm volatile("" : "+v"(tid));
    const uint32_t lane = tid & 63u, hw = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t pbase = hw * kWaveSpan;
    const uint32_t qe = pbase + 2u * lane;     // even position of round 0; round j: qe + 128 j
    // its clock word; round j: cwe + 136 j (pbase is a multiple of 64, lanes 32.. are past one padding)
    const uint32_t cwe = qe + (pbase >> 4) + ((lane >> 5) << 2);
    // the last units of this workgroup's records: they travel while the staging state is cleared
    request_units(wg, tid, std::integral_constant<int, kEarly>{}, std::integral_constant<int, NR / 2>{});
    // ---- workgroup header, clear the staging state -----------------------------------------------
    if (tid <= KP_MAX_WAVES) {  // (entries from W up: no records)
      const uint32_t T = tid < W ? h_total : 0u;
      const uint32_t V = T < cap ? T : cap;
      sVF[tid] = make_uint2(V, flush ? 0u : (T - V) & kSeqMask);
      atomicAdd(&ctr[H_DROPPED], (unsigned long long)(T - V));
      atomicAdd(&ctr[H_SLOTS_VALID], (unsigned long long)V);
    }
    if (tid < 64) {  // clear the temporaries; the last one takes the records the waves hold together
      const uint32_t held = wave_scan_add(tid < W ? (h_total < cap ? h_total : cap) : 0u);
      if (tid >= 64 - T_COUNT) tmp[tid - (64 - T_COUNT)] = tid == 63u ? held : 0u;
    }
    if (tid == 32) {
      const uint64_t tb = (uint64_t)h_begin.x | ((uint64_t)h_begin.y << 32);
      const uint64_t te = (uint64_t)h_end.x | ((uint64_t)h_end.y << 32);
      const uint64_t sp = te - tb;
      // 16 times the cell of clock t: t * scale, i.e. the span divided into NCELL cells (clamped below).  Any
      // scale near 16 * NCELL / (span + 1) orders the cells by time.
      const float scale = (float)(16u * NCELL) / ((float)(uint32_t)sp + 1.0f);
      misc[0] = (sp >> 32) ? 1u : 0u;
      misc[1] = __builtin_bit_cast(uint32_t, scale);
      misc[2] = (uint32_t)sp;
    }
    clear_meta(tid);
    reinterpret_cast<u32x4*>(cells)[2 * tid] = u32x4{0u, 0u, 0u, 0u};
    reinterpret_cast<u32x4*>(cells)[2 * tid + 1] = u32x4{0u, 0u, 0u, 0u};
    if (tid == 0) reinterpret_cast<u32x4*>(cells)[2 * BLOCK] = u32x4{0u, 0u, 0u, 0u};
    team_sync<BLOCK>();

    uint32_t wg_invalid = 0;
    bool eligible = false;
    uint32_t products = 0;  // digits of the stretch lengths when the sweep hands its sets to the matrix cores, else 0
    const uint32_t wg_ahead = wg + stride < n_wg ? wg + stride : wg;  // (the last one asks for its own again)
    do {  // (left early only when single steps are timed)
    // ---- A: every record to its place --------------------------------------------------------------
    // Places are slots: rank k of a wave belongs in slot (first + k) mod capacity, and a record is nearly always there.
    // So the records stay in the registers they were loaded into, and a lane checks that its two of a round are the ones
    // expected.  A round in which some record is not looks at every one of them: a record that belongs elsewhere is left
    // in LDS at its place, and a place whose own record is missing looks there behind the barrier.
    // Round j: the even position qe + 128 j and the one above it.  A place without a record holds the largest clock: it
    // never counts as a step back in time.
    uint32_t t[NR], mq[NR / 4];  // clocks; metadata bytes, record i in byte i & 3 of word i >> 2
    uint32_t holes = 0;          // bit i: place i has a slot that holds a record, but not its own
    uint32_t oldest = 0;         // (small rings) bits j, 8 + j, 16 + j: the even place of round j is rank 0, rank 1, the last one
    // Rings of at least 128 slots: a round is one recorded wave's, and what there is to know of that is uniform; of at least
    // a hardware wave's share: so are all its rounds.
    const bool whole_rings = RINGS == kWhole || (RINGS == kAny && cap >= kWaveSpan);
    const uint32_t wave_here = pbase >> cl2;
    uint32_t held_here = 0, first_here = 0;  // records held by that wave, its first surviving seq (of 20 bits)
    if (whole_rings && wave_here < W) {
      const uint32_t T = (uint32_t)__builtin_amdgcn_readlane((int)h_total, (int)wave_here);
      held_here = T < cap ? T : cap;
      first_here = flush ? 0u : (T - held_here) & kSeqMask;
    }
    const uint32_t slot_here = pbase & capm;
    const uint32_t to_oldest = (first_here - slot_here) & capm;  // slots from the hardware wave's first place to the oldest record
    auto set_round = [&](int j, uint32_t t0, uint32_t t1, uint32_t m2) __attribute__((always_inline)) {
      t[2 * j] = t0; t[2 * j + 1] = t1;
      if (j & 1) mq[j >> 1] |= m2 << 16; else mq[j >> 1] = m2;
    };
    // What others need to know of the records here: the last one of the hardware wave and those at the ends of rings.
    auto publish_ends = [&]() __attribute__((always_inline)) {
      const uint2 e = make_uint2(t[NR - 1], mq[NR / 4 - 1] >> 24);
      if (lane == 63u) wave_end[hw] = e;
      if (whole_rings) {
        if (((pbase + kWaveSpan) & capm) == 0u && wave_here < W && lane == 63u) ring_end[wave_here] = e;
      } else {
#pragma unroll
        for (int j = 0; j < NR / 2; ++j) {
          const uint32_t q = qe + 128u * j;
          if (((q + 2u) & capm) == 0u && q < nrec) ring_end[q >> cl2] = make_uint2(t[2 * j + 1], (mq[j >> 1] >> (16 * (j & 1) + 8)) & 0xFFu);
        }
      }
    };
    {
      uint32_t c_bad = 0, c_dis = 0;
      // e0, e1: the low 24 bits of the tags if both records are in place; not exact in every lane where seq wraps inside the
      // ring or the ring begins inside the round, which the caller says.  The records are looked at in any case if not `whole` (some
      // place has no record) or `look` is not 0, and if one names a region from `above` on.
      auto check = [&](int j, uint32_t w, uint32_t V, uint32_t first, uint32_t s0, bool whole, uint32_t look, bool exact, uint32_t above, uint32_t e0, uint32_t e1) __attribute__((always_inline)) {
        const uint32_t tag0 = v[j].x, tag1 = v[j].z;
        const uint32_t wrong = ((tag0 ^ e0) | (tag1 ^ e1)) & 0xFFFFFFu;
        const uint32_t r0 = tag0 & 0x7F000000u, r1 = tag1 & 0x7F000000u;
        uint32_t t0 = v[j].y, t1 = v[j].w, m2 = __builtin_amdgcn_perm(tag1, tag0, 0x0C0C0703u);  // END flag and region of both
        if (seldom(!whole || (look | __builtin_amdgcn_ballot_w64(wrong != 0u) | __builtin_amdgcn_ballot_w64((r0 > r1 ? r0 : r1) >= above)) != 0ull)) {
          bool home0 = s0 < V, home1 = s0 + 1u < V;
          if (!exact) above = 0u;
          const bool odd0 = ((tag0 ^ e0) & 0xFFFFFFu) != 0u || r0 >= above, odd1 = ((tag1 ^ e1) & 0xFFFFFFu) != 0u || r1 >= above;
          if (rare(__builtin_amdgcn_ballot_w64((home0 && odd0) || (home1 && odd1)) != 0ull)) {
            // rank: the low 20 bits of tag - first are those of seq - first
            const uint32_t n0 = (tag0 - first) & kSeqMask, n1 = (tag1 - first) & kSeqMask;
            const bool good0 = s0 < V && n0 < V && ((tag0 >> 20) & 0xFu) == w && r0 < (R << 24);
            const bool good1 = s0 + 1u < V && n1 < V && ((tag1 >> 20) & 0xFu) == w && r1 < (R << 24);
            home0 = good0 && ((tag0 ^ s0) & capm) == 0u;
            home1 = good1 && ((tag1 ^ (s0 + 1u)) & capm) == 0u;
            const uint32_t q = qe + 128u * j - s0;  // first position of the recorded wave
            if (good0 && !home0) { const uint32_t to = q + (tag0 & capm); clk[clk_word(to)] = t0; meta[to] = (uint8_t)(tag0 >> 24); ++c_dis; }
            if (good1 && !home1) { const uint32_t to = q + (tag1 & capm); clk[clk_word(to)] = t1; meta[to] = (uint8_t)(tag1 >> 24); ++c_dis; }
            c_bad += (s0 < V && !good0 ? 1u : 0u) + (s0 + 1u < V && !good1 ? 1u : 0u);
            holes |= (s0 < V && !home0 ? 1u << (2 * j) : 0u) | (s0 + 1u < V && !home1 ? 2u << (2 * j) : 0u);
          }
          t0 = home0 ? t0 : 0xFFFFFFFFu;
          t1 = home1 ? t1 : 0xFFFFFFFFu;
          m2 = (home0 ? m2 & 0xFFu : kEmpty) | (home1 ? m2 & 0xFF00u : kEmpty << 8);
        }
        set_round(j, t0, t1, m2);
      };
      if (whole_rings) {
        const uint32_t tag_here = (wave_here << 20) + first_here + ((slot_here - first_here) & capm) + 2u * lane;
        // rounds in which the expected tags are not exact, and with those that have a place without a record
        const uint32_t inexact = first_here + capm > kSeqMask ? 0xFFFFFFFFu : (to_oldest & 127u) != 0u && to_oldest < kWaveSpan ? 1u << (to_oldest >> 7) : 0u;
        const uint32_t full = held_here > slot_here ? (held_here - slot_here) >> 7 : 0u;
        const uint32_t look = inexact | (full < NR / 2 ? 0xFFFFFFFFu << full : 0u);
#pragma unroll
        for (int j = 0; j < NR / 2; ++j) {
          const uint32_t e0 = tag_here + (128u * j - (to_oldest != 0u && 128u * j >= to_oldest ? cap : 0u));
          check(j, wave_here, held_here, first_here, slot_here + 128u * j + 2u * lane, true, look & (1u << j), (inexact & (1u << j)) == 0u, R << 24, e0, e0 + 1u);
        }
      } else if (!SMALL) {
#pragma unroll
        for (int j = 0; j < NR / 2; ++j) {
          const uint32_t p0 = pbase + 128u * j, w = p0 >> cl2, slot = p0 & capm;
          const uint32_t T = (uint32_t)__builtin_amdgcn_readlane((int)h_total, (int)(w & 15u));
          const uint32_t V = w >= W ? 0u : T < cap ? T : cap, first = flush ? 0u : (T - V) & kSeqMask;
          if (rare(slot >= V)) {
            set_round(j, 0xFFFFFFFFu, 0xFFFFFFFFu, kEmpty | (kEmpty << 8));
          } else {
            const uint32_t k0 = (slot - first + 2u * lane) & capm, base = (w << 20) + first;
            check(j, w, V, first, slot + 2u * lane, slot + 128u <= V, 0u, true, first + capm <= kSeqMask ? R << 24 : 0u, base + k0, base + ((k0 + 1u) & capm));
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < NR / 2; ++j) {
          const uint32_t q = qe + 128u * j, s0 = q & capm, wv = q >> cl2, w = wv < KP_MAX_WAVES ? wv : KP_MAX_WAVES;  // (entry KP_MAX_WAVES: no records)
          const uint2 vf = sVF[w];
          const uint32_t k0 = (s0 - vf.y) & capm;
          const uint32_t e0 = (w << 20) | ((vf.y + k0) & kSeqMask), e1 = (w << 20) | ((vf.y + ((k0 + 1u) & capm)) & kSeqMask);
          oldest |= (k0 == 0u ? 1u << j : 0u) | (k0 == 1u ? 0x100u << j : 0u) | (k0 == capm ? 0x10000u << j : 0u);
          check(j, w, vf.x, vf.y, s0, __builtin_amdgcn_ballot_w64(s0 + 1u >= vf.x) == 0ull, 0u, true, R << 24, e0, e1);
        }
      }
      publish_ends();
      if (__builtin_amdgcn_ballot_w64((c_bad | c_dis) != 0u)) {
        if (c_bad) atomicAdd(&tmp[T_BAD], c_bad);
        if (c_dis) atomicAdd(&tmp[T_DISORDER], c_dis);
      }
    }
    team_sync<BLOCK>();
    if (stop_after == kStepOrdered) break;

    // ---- records outside the slot of their seq -----------------------------------------------------
    wg_invalid = tmp[T_BAD];  // slots that hold a record and did not make it into the ordered sequence
    if (rare(tmp[T_DISORDER] != 0u)) {
      uint32_t left = 0;
#pragma unroll
      for (int j = 0; j < NR / 2; ++j) {
        const uint32_t mine = (holes >> (2 * j)) & 3u;
        if (__builtin_amdgcn_ballot_w64(mine != 0u) == 0ull) continue;
        const uint32_t there = *reinterpret_cast<const uint16_t*>(meta + qe + 128u * j);
        const uint2 tt = *reinterpret_cast<const uint2*>(clk + cwe + 136u * j);
        const bool take0 = (mine & 1u) && (there & 0x3Fu) != kEmpty, take1 = (mine & 2u) && ((there >> 8) & 0x3Fu) != kEmpty;
        left += __popc(mine) - (take0 ? 1u : 0u) - (take1 ? 1u : 0u);
        if (take0) t[2 * j] = tt.x;
        if (take1) t[2 * j + 1] = tt.y;
        const uint32_t bytes = (take0 ? 0xFFu : 0u) | (take1 ? 0xFF00u : 0u);
        mq[j >> 1] = (mq[j >> 1] & ~(bytes << (16 * (j & 1)))) | ((there & bytes) << (16 * (j & 1)));
      }
      publish_ends();
      if (left) atomicAdd(&tmp[T_UNFILLED], left);
      team_sync<BLOCK>();
      wg_invalid = tmp[T_UNFILLED];
      // Every slot without its own record holds a bad one or one that belongs elsewhere: as many places are left without a
      // record as there are bad ones, unless some record found its place taken.
      if (rare(wg_invalid != tmp[T_BAD])) {
        // Rare: some seq occurs twice.  The later slot must win, so this workgroup's records are placed again in slot
        // order, one thread per wave.
        team_sync<BLOCK>();
        clear_meta(tid);
        {
          uint32_t ones[NR];
#pragma unroll
          for (int i = 0; i < NR; ++i) ones[i] = 0xFFFFFFFFu;
          store_run<NR>(clk, tid, ones);
        }
        if (tid == 0) { tmp[T_DISORDER] = 0; tmp[T_UNFILLED] = tmp[T_HELD]; }
        team_sync<BLOCK>();
        if (tid < W) {
          const uint32_t w = tid, V = sVF[w].x, first = sVF[w].y;
          const uint32_t* seg = reinterpret_cast<const uint32_t*>(p.records) + ((size_t)wg * nrec + (size_t)w * cap) * 2;
          for (uint32_t s = 0; s < V; ++s) {
            const uint32_t tag = seg[2 * s];
            const uint32_t k = (tag - first) & kSeqMask, region = (tag >> 24) & 0x7Fu, at = w * cap + (tag & capm);
            if (k >= V || ((tag >> 20) & 0xFu) != w || region >= R) continue;
            // the clock word remembers the winning slot for now
            clk[clk_word(at)] = s;
            meta[at] = (uint8_t)(tag >> 24);
          }
          uint32_t dis = 0, occ = 0;
          for (uint32_t k = 0; k < V; ++k) {
            const uint32_t at = w * cap + k;
            if ((meta[at] & kRegion) == kEmpty) continue;
            const uint32_t s = clk[clk_word(at)];
            dis += s != k;
            clk[clk_word(at)] = seg[2 * s + 1];
            ++occ;
          }
          atomicAdd(&tmp[T_DISORDER], dis);
          atomicSub(&tmp[T_UNFILLED], occ);
        }
        team_sync<BLOCK>();
        wg_invalid = tmp[T_UNFILLED];
#pragma unroll
        for (int j = 0; j < NR / 2; ++j) {
          const uint2 tt = *reinterpret_cast<const uint2*>(clk + cwe + 136u * j);
          const uint32_t m2 = *reinterpret_cast<const uint16_t*>(meta + qe + 128u * j);
          t[2 * j] = tt.x; t[2 * j + 1] = tt.y;
          mq[j >> 1] = j & 1 ? (mq[j >> 1] & 0xFFFFu) | (m2 << 16) : m2;
        }
        publish_ends();
        team_sync<BLOCK>();
      }
    }
    const uint32_t n_occupied = tmp[T_HELD] - wg_invalid;
    auto meta_of = [&](int i) -> uint32_t { return (mq[i >> 2] >> (8 * (i & 3))) & 0xFFu; };
    auto set_paired = [&](int i, uint32_t yes) { mq[i >> 2] |= (yes << 6) << (8 * (i & 3)); };  // yes: 0 or 1

    // One pair: duration into the per-(wave, region) sums and the histogram.  The sums exist in up to
    // four copies, one per quarter of the wave: lanes 16 apart tend to hold the same region, and LDS
    // atomics of one instruction that hit one address are processed one after the other.
    const uint32_t copy = (lane >> 4) & (n_copies - 1u);
    uint32_t shortest = 0xFFFFFFFFu;
    auto account_row = [&](uint32_t row, uint32_t region, uint32_t d_raw) __attribute__((always_inline)) {  // row: wave * R
      shortest = d_raw < shortest ? d_raw : shortest;
      const uint32_t d = d_raw > rec_cost ? d_raw - rec_cost : 0u;
      const uint32_t e = __umul24(row + region, n_copies) + copy;
      atomicAdd(&pw_pack[e], (1ull << 46) | (unsigned long long)d);
      atomicMax(&pw_max[e], d);
      atomicMin(&pw_min[e], d);
      atomicAdd(&hist[__umul24(region, kHistStride) + (31 - __clz(d | 1u))], 1u);
    };
    auto account_pair = [&](uint32_t w, uint32_t region, uint32_t d_raw) { account_row(__umul24(w, R), region, d_raw); };

    uint32_t deep = 0;  // bit i: place i holds an END that has to look further down than one rank
    if (!rare(wg_invalid != 0u)) {
      // ---- B: pairing, durations, per-(wave,region) statistics, monotonicity ------------------------
      // Every slot that a wave's record count covers holds a record here.  An END is paired iff the nearest
      // earlier record of its (wave, region) is a START; every START that is not claimed this way is an
      // orphan, so only ENDs search.  In traces of kernels whose regions follow one another the START
      // sits one rank below: in the lane's own even position, or, for an END in the even position, in
      // the odd position of the lane below (DPP; lane 0 takes the last lane of the round before, or what the
      // hardware wave or the end of the ring before it left in LDS).  Both positions of a round are tested at once on
      // the two metadata bytes side by side.  An END whose lower neighbour belongs to another region looks further
      // behind the barrier, where all records are in LDS.
      // A START learns that it is paired from its END: in the same lane directly, one lane up through a
      // DPP shift of the claims, and otherwise through a mark at its place in LDS that is read back after the barrier.
      uint32_t n_nonmono = 0;  // wave-uniform count
      bool marked = false;
      auto count = [](bool b) -> uint32_t { return (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(b)); };
      uint2 below = wave_end[hw ? hw - 1u : 0u];
      if (slot_here == 0u) below = ring_end[wave_here & 15u];
      // Masks of rounds: those in which a ring begins (but for the first, whose record below is known), and those that may
      // hold the oldest record of a ring.
      uint32_t begins_in = 0u, oldest_in = 0u;
      uint2 last_of = make_uint2(0u, 0u);  // lane w & 15: the record in the last slot of wave w's ring
      if (whole_rings) {
        oldest_in = to_oldest < kWaveSpan ? 1u << (to_oldest >> 7) : 0u;
      } else if (SMALL) {
        begins_in = oldest_in = 0xFFFFFFFFu;
      } else {
        last_of = ring_end[lane & 15u];
#pragma unroll
        for (int j = 0; j < NR / 2; ++j) {
          const uint32_t p0 = pbase + 128u * j, T = (uint32_t)__builtin_amdgcn_readlane((int)h_total, (int)((p0 >> cl2) & 15u));
          const uint32_t rot = flush || T < cap ? 0u : T & capm;  // (first surviving seq modulo capacity: T - capacity)
          begins_in |= j != 0 && (p0 & capm) == 0u ? 1u << j : 0u;
          oldest_in |= rot - (p0 & capm) < 128u ? 1u << j : 0u;
        }
      }
      uint32_t odd_before = below.y << 16;  // the odd positions' metadata of the two rounds before: lane 63's are the ones below lane 0
#pragma unroll
      for (int x = 0; x < NR / 4; ++x) {
        // Rounds 2 x and 2 x + 1 side by side: bytes 0 and 1 the even and the odd position of the first, 2 and 3 of the second.
        const uint32_t m4 = mq[x], odd = (m4 >> 8) & 0x00FF00FFu;
        const uint32_t edge = __builtin_amdgcn_alignbit(odd, odd_before, 16);
        const uint32_t pm = wave_shr1(odd, x == 0 ? (odd_before >> 16) | (wave_ror1(odd) << 16) : wave_ror1(edge));
        odd_before = odd;
        uint32_t p4 = ((m4 << 8) & 0xFF00FF00u) | pm;  // the record one rank below each of the four
        uint32_t pt[2], own_t[2];                      // the clock one rank below the even position, the odd position
        uint32_t search = 0x80808080u;                 // bits of the positions that may have to look further down
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int j = 2 * x + h;
          pt[h] = wave_shr1(t[2 * j + 1], j == 0 ? below.x : wave_ror1(t[j == 0 ? 0 : 2 * j - 1]));
          own_t[h] = t[2 * j];
          if (seldom((begins_in >> j) & 1u)) {  // the record below the first slot of a ring is the one in its last
            const uint32_t q = qe + 128u * j, w = SMALL ? q >> cl2 : (pbase + 128u * j) >> cl2;
            const uint2 e = SMALL ? ring_end[w & 15u] : make_uint2((uint32_t)__builtin_amdgcn_readlane((int)last_of.x, (int)(w & 15u)),
                                                                    (uint32_t)__builtin_amdgcn_readlane((int)last_of.y, (int)(w & 15u)));
            if ((q & capm) == 0u) {
              pt[h] = e.x;
              p4 = (p4 & ~(0xFFu << (16 * h))) | (e.y << (16 * h));
            }
          }
          if (seldom((oldest_in >> j) & 1u)) {  // nothing below rank 0, nothing to look for below rank 1
            bool lowest0, lowest1, second0;
            if constexpr (SMALL) {
              lowest0 = (oldest >> j) & 1u; second0 = (oldest >> (8 + j)) & 1u; lowest1 = (oldest >> (16 + j)) & 1u;
            } else {
              const uint32_t p0 = pbase + 128u * j, s0 = (p0 & capm) + 2u * lane, T = (uint32_t)__builtin_amdgcn_readlane((int)h_total, (int)((p0 >> cl2) & 15u));
              const uint32_t rot = flush || T < cap ? 0u : T & capm;
              lowest0 = s0 == rot; lowest1 = s0 + 1u == rot; second0 = s0 == ((rot + 1u) & capm);
            }
            p4 |= (lowest0 ? kEmpty << (16 * h) : 0u) | (lowest1 ? kEmpty << (16 * h + 8) : 0u);  // (region 63)
            pt[h] = lowest0 ? 0u : pt[h];
            own_t[h] = lowest1 ? 0u : own_t[h];
            search &= ~((lowest0 || second0 ? 0x80u << (16 * h) : 0u) | (lowest1 || lowest0 ? 0x8000u << (16 * h) : 0u));
          }
          // (a position without a record holds the largest clock, and so do all above it in its wave)
          n_nonmono += count(t[2 * j] < pt[h]) + count(t[2 * j + 1] < own_t[h]);
          asm volatile("" : "+s"(n_nonmono));  // (counted here: kept for later the two masks would be parked in vector registers)
        }
        const uint32_t x4 = m4 ^ p4;
        // bit 7 of each byte: that byte of the argument is not zero
        auto nonzero7 = [](uint32_t v) -> uint32_t { return ((v & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v; };
        const uint32_t end4 = m4 & 0x80808080u;                                   // is an END (no record: 0)
        const uint32_t differ4 = nonzero7(x4 & 0x3F3F3F3Fu) & end4 & search;      // END, other region one rank below
        const uint32_t near4 = ~nonzero7((x4 & 0xBFBFBFBFu) ^ 0x80808080u) & end4;  // END, START of its region one rank below
        // as END, or as the START of the odd position; the mark of an END sits one bit above its flag
        mq[x] = m4 | (near4 >> 1) | ((near4 >> 9) & 0x00400040u);
        if (rare(__builtin_amdgcn_ballot_w64(differ4 != 0u) != 0ull))
          deep |= (((differ4 >> 7) & 1u) | ((differ4 >> 14) & 2u) | ((differ4 >> 21) & 4u) | ((differ4 >> 28) & 8u)) << (4 * x);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int j = 2 * x + h;
          const uint32_t q = qe + 128u * j;  // even position; the odd one is q + 1
          const bool e0 = (near4 & (0x80u << (16 * h))) != 0u, e1 = (near4 & (0x8000u << (16 * h))) != 0u;
          // a START that is not in the lane below: in the last place of a hardware wave, or of a ring
          if (j == 0 && !SMALL) {
            if (e0 && lane == 0u) { meta[slot_here == 0u ? q + capm : q - 1u] = (uint8_t)kPaired; marked = !whole_rings; }
          } else if (seldom((begins_in >> j) & 1u)) {
            if (e0 && (q & capm) == 0u) { meta[q + capm] = (uint8_t)kPaired; marked = true; }
          }
          uint32_t row = ((pbase + 128u * j) >> cl2) * R;
          if constexpr (SMALL) row = __umul24(q >> cl2, R);
          const uint32_t m0 = (m4 >> (16 * h)) & kRegion, m1 = (m4 >> (16 * h + 8)) & kRegion;
          const uint32_t d0 = t[2 * j] - pt[h], d1 = t[2 * j + 1] - t[2 * j];
          if (e0 || e1) account_row(row, e1 ? m1 : m0, e1 ? d1 : d0);  // (never both: what the odd one is paired with is a START)
        }
      }
      // A START in an odd position that the even position of the lane above claimed (lane 63: that of lane 0 in the next
      // round): the END there carries both flags.  Two rounds at a time.
      uint32_t claim[NR / 4 + 1];  // bits 7 and 23: the even position's END is paired
#pragma unroll
      for (int x = 0; x < NR / 4; ++x) {
        claim[x] = mq[x] & (mq[x] << 1) & 0x00800080u;
        if (seldom(begins_in != 0u))  // (where a ring begins the START is elsewhere)
          claim[x] &= (((qe + 256u * x) & capm) ? 0x80u : 0u) | (((qe + 256u * x + 128u) & capm) ? 0x800000u : 0u);
      }
      claim[NR / 4] = 0u;
#pragma unroll
      for (int x = 0; x < NR / 4; ++x) {
        const uint32_t now = (uint32_t)__builtin_amdgcn_readlane((int)claim[x], 0), next = (uint32_t)__builtin_amdgcn_readlane((int)claim[x + 1], 0);
        const uint32_t above = (uint32_t)__builtin_amdgcn_update_dpp((int)((now >> 16) | (next << 16)), (int)claim[x], 0x130, 0xF, 0xF,
                                                                     false);  // wave_shl:1
        mq[x] |= above << 7;
      }
      // ENDs, and ENDs that are paired (the flag sits one bit below): counted on the packed bytes
      uint32_t n_ends = 0, n_pairs = 0;
#pragma unroll
      for (int x = 0; x < NR / 4; ++x) {
        n_ends += __popc(mq[x] & 0x80808080u);
        n_pairs += __popc(mq[x] & (mq[x] << 1) & 0x80808080u);
      }
      n_pairs = wave_scan_add(n_ends | (n_pairs << 16));  // both at most 1024 per wave
      const bool any_marked = __builtin_amdgcn_ballot_w64(marked) != 0, any_zero = __builtin_amdgcn_ballot_w64(shortest == 0u) != 0;
      const bool any_deep = __builtin_amdgcn_ballot_w64(deep != 0u) != 0;
      if (lane == 0u) {
        if (any_marked) tmp[T_MARKS] = 1u;
        if (any_deep) tmp[T_DEEP] = 1u;
        if (any_zero) tmp[T_ZERO] = 1u;
        if (n_nonmono) atomicAdd(&tmp[T_NONMONO], n_nonmono);
      }
      if (lane == 63u) {
        atomicAdd(&tmp[T_PAIRS], n_pairs >> 16);
        atomicAdd(&tmp[T_ENDS], n_pairs & 0xFFFFu);
      }
      if (tid == 0) tmp[T_STARTS] = n_occupied;  // records; orphans = records - ENDs - pairs, ENDs - pairs
    }
    team_sync<BLOCK>();
    // marks left by ENDs of other hardware waves (only the last position can have one) and at the ends of short rings
    auto read_marks = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < NR / 2; ++j)
        mq[j >> 1] |= ((uint32_t)*reinterpret_cast<const uint16_t*>(meta + qe + 128u * j) & 0x4040u) << (16 * (j & 1));
    };
    if (wg_invalid == 0u) {
      set_paired(NR - 1, ((uint32_t)meta[qe + 128u * (NR / 2 - 1) + 1u] >> 6) & 1u);
      if (rare(tmp[T_MARKS] != 0u)) read_marks();
    }
    if (rare(wg_invalid != 0u || tmp[T_DEEP] != 0u || tmp[T_ZERO] != 0u)) {
      // Whoever looks further than one rank needs the other lanes' records: all of them to LDS, each at its position.
#pragma unroll
      for (int j = 0; j < NR / 2; ++j) {
        *reinterpret_cast<uint2*>(clk + cwe + 136u * j) = make_uint2(t[2 * j], t[2 * j + 1]);
        *reinterpret_cast<uint16_t*>(meta + qe + 128u * j) = (uint16_t)(mq[j >> 1] >> (16 * (j & 1)));
      }
      team_sync<BLOCK>();
      if (wg_invalid != 0u) {
        // ---- B, workgroup with holes: the definition, one thread per (wave, region) -----------------
        for (uint32_t e = tid; e < W * R; e += BLOCK) {
          const uint32_t w = e / R, r = e - w * R, V = sVF[w].x, first = sVF[w].y;
          bool have_prev = false;
          uint32_t prev_m = 0, prev_t = 0, n_pairs = 0, n_starts = 0, n_ends = 0;
          for (uint32_t k = 0; k < V; ++k) {
            const uint32_t at = w * cap + ((first + k) & capm), mm = meta[at];
            if ((mm & kRegion) != r) continue;
            const uint32_t ts = clk[clk_word(at)];
            if (mm & kEnd) {
              ++n_ends;
              if (have_prev && !(prev_m & kEnd)) { ++n_pairs; account_pair(w, r, ts - prev_t); }
            } else {
              ++n_starts;
            }
            have_prev = true; prev_m = mm; prev_t = ts;
          }
          if (n_pairs) atomicAdd(&tmp[T_PAIRS], n_pairs);
          if (n_starts + n_ends) atomicAdd(&tmp[T_STARTS], n_starts + n_ends);
          if (n_ends) atomicAdd(&tmp[T_ENDS], n_ends);
        }
        for (uint32_t w = tid; w < W; w += BLOCK) {
          const uint32_t V = sVF[w].x, first = sVF[w].y;
          bool have_prev = false;
          uint32_t prev_t = 0, n = 0;
          for (uint32_t k = 0; k < V; ++k) {
            const uint32_t at = w * cap + ((first + k) & capm);
            if ((meta[at] & kRegion) == kEmpty) continue;
            const uint32_t ts = clk[clk_word(at)];
            n += (have_prev && ts < prev_t) ? 1u : 0u;
            have_prev = true; prev_t = ts;
          }
          if (n) atomicAdd(&tmp[T_NONMONO], n);
        }
        team_sync<BLOCK>();
      } else if (tmp[T_DEEP] != 0u) {
        // ---- B, regions inside regions: down the ranks to the nearest record of the END's region -----
        // (each lane takes its ENDs one after the other, four ranks at a step.  All lanes' END of one place at a time, rank by
        // rank: 512 turns of nested regions, three deep, 8 x 2048 records 409 us, 500 of 8 x 512 78.0.)
        shortest = 0xFFFFFFFFu;
        uint32_t found = 0;
        while (deep != 0u) {
          const uint32_t i = (uint32_t)__builtin_ctz(deep);
          deep &= deep - 1u;
          const uint32_t q = qe + 128u * (i >> 1) + (i & 1u), base = q & ~capm, mine = meta[q], row = __umul24(q >> cl2, R);
          uint32_t s = q & capm;  // the slots looked at next lie below this one (a ring of two has none)
          for (uint32_t left = (s - sVF[(q >> cl2) & 15u].y) & capm; left != 0u;) {
            s = s ? s : cap;
            const uint32_t lo = (s - 1u) & ~3u, n = s - lo, four = *reinterpret_cast<const uint32_t*>(meta + base + lo);
            // bit 7 of each byte that names the region; bytes from the n-th on and those older than the oldest record do not count
            const uint32_t other = (four ^ (mine * 0x01010101u)) & 0x3F3F3F3Fu;
            uint32_t same = ~(other + 0x7F7F7F7Fu) & (0x80808080u >> (32u - 8u * n));
            if (left < n) same &= 0xFFFFFFFFu << (8u * (n - left));
            if (same != 0u) {
              const uint32_t b = (31u - (uint32_t)__builtin_clz(same)) >> 3, at = base + lo + b, mm = (four >> (8u * b)) & 0xFFu;
              if (!(mm & kEnd)) {
                meta[at] = (uint8_t)(mm | kPaired);
                account_row(row, mine & kRegion, clk[clk_word(q)] - clk[clk_word(at)]);
                found |= 1u << i;
              }
              break;
            }
            left = left > n ? left - n : 0u;
            s = lo;
          }
        }
#pragma unroll
        for (int i = 0; i < NR; ++i) set_paired(i, (found >> i) & 1u);
        if (found) atomicAdd(&tmp[T_PAIRS], (uint32_t)__popc(found));
        if (shortest == 0u) tmp[T_ZERO] = 1u;
        team_sync<BLOCK>();
        read_marks();
      }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) asm volatile("" : "+v"(t[i]));  // (opaque across the barrier, see below)
#pragma unroll
    for (int i = 0; i < NR / 4; ++i) asm volatile("" : "+v"(mq[i]));
    eligible = !misc[0] && wg_invalid == 0u && tmp[T_NONMONO] == 0u;

    if (eligible && stop_after != kStepPaired) {
      // ---- C: order the paired records of all waves by clock ---------------------------------------
      // A pair of length 0 overlaps nothing, and records of one clock come out of the counting sort in any order: its END
      // could open the region, in the general sweep, to every record of the same clock until its START.  Neither is an
      // event.  (The record a START is paired with is the next one of its region; the clocks of a wave do not fall here,
      // so that every record between the two has their clock: another one ends the search.  256 workgroups of 2 x 2048
      // records of 17 regions, half of them in any order: 295 us going to the partner every time, 244 this way.)
      if (rare(tmp[T_ZERO] != 0u)) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          const uint32_t m = meta_of(i);
          if (m & kPaired) {
            const uint32_t step = m & kEnd ? ~0u : 1u, q0 = qe + 128u * (i >> 1) + (i & 1), base = q0 & ~capm;
            uint32_t q = base + ((q0 + step) & capm);
            while (clk[clk_word(q)] == t[i] && ((meta[q] ^ m) & kRegion) != 0u) q = base + ((q + step) & capm);
            if (clk[clk_word(q)] == t[i]) mq[i >> 2] ^= kPaired << (8 * (i & 3));
          }
        }
      }
      const float scale = __builtin_bit_cast(float, misc[1]);
      // Straight-line code from here to the sorted sequence: the LDS operations of a lane's 16 records
      // are issued together and no array is assigned inside a branch.
      uint32_t ca[NR];  // 16 * cell + a fraction, below 16 * NCELL | arrival slot << kSlotShift
      static_assert(NCELL * 16u == 1u << kSlotShift && L::npos <= 1u << (32u - kSlotShift), "cell and slot in one word");
      uint32_t t_max = 0;
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const uint32_t te = meta_of(i) & kPaired ? t[i] : 0u;  // (a record that is no event adds nothing, so that all atomics are in flight together)
        t_max = te > t_max ? te : t_max;
        // (a conversion, a product and a conversion that never fall: the cells follow one another in time)
        const float at = (float)te * scale;
        const uint32_t y = (uint32_t)(at < (float)(NCELL * 16u - 1u) ? at : (float)(NCELL * 16u - 1u));
        const uint32_t sh = y & 16u;  // cell c: half (c & 1) of word c >> 1
        const uint32_t old = atomicAdd(&cells[y >> 5], ((mq[i >> 2] >> (8 * (i & 3) + 6)) & 1u) << sh);
        ca[i] = y | (((old >> sh) & 0xFFFFu) << kSlotShift);
      }
      if (__builtin_amdgcn_ballot_w64(t_max > misc[2]) && lane == 0u) tmp[T_WIDE] = 1u;  // a clock past the span
      team_sync<BLOCK>();
      if (stop_after == kStepCounted) break;
      // (the registers that cross this barrier are made opaque: values derived from them for the next
      // phase would otherwise be computed before it and held in registers across it)
#pragma unroll
      for (int i = 0; i < NR; ++i) asm volatile("" : "+v"(t[i]), "+v"(ca[i]));
#pragma unroll
      for (int i = 0; i < NR / 4; ++i) asm volatile("" : "+v"(mq[i]));
      {  // exclusive prefix sum over the cell counters, 16 cells (8 words) per thread
        u32x4 a = reinterpret_cast<u32x4*>(cells)[2 * tid], b = reinterpret_cast<u32x4*>(cells)[2 * tid + 1];
        uint32_t wv[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        uint32_t run = 0, fullest = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t lo = wv[i] & 0xFFFFu, hi = wv[i] >> 16;
          fullest = lo > fullest ? lo : fullest;
          fullest = hi > fullest ? hi : fullest;
          wv[i] = run | ((run + lo) << 16);
          run += lo + hi;
        }
        const uint32_t incl = wave_scan_add(run);
        if (lane == 63) wtot[hw] = incl;
        {  // fullest cell of the workgroup
          uint32_t f = fullest, o;
          o = scan_src<0>(f); f = o > f ? o : f; o = scan_src<1>(f); f = o > f ? o : f;
          o = scan_src<2>(f); f = o > f ? o : f; o = scan_src<3>(f); f = o > f ? o : f;
          o = scan_src<4>(f); f = o > f ? o : f; o = scan_src<5>(f); f = o > f ? o : f;
          if (lane == 63) atomicMax(&tmp[T_MAXCELL], f);
        }
        team_sync<BLOCK>();
        uint32_t base = incl - run;
        {  // + the totals of the waves below: lane h of the first row takes wave h's
          uint32_t below = (lane & 15u) < hw ? wtot[lane & 15u] : 0u;
          below += scan_src<0>(below); below += scan_src<1>(below); below += scan_src<2>(below); below += scan_src<3>(below);
          base += (uint32_t)__builtin_amdgcn_readlane((int)below, 15);
        }
        const uint32_t both = base * 0x00010001u;
        a = u32x4{wv[0] + both, wv[1] + both, wv[2] + both, wv[3] + both};
        b = u32x4{wv[4] + both, wv[5] + both, wv[6] + both, wv[7] + both};
        reinterpret_cast<u32x4*>(cells)[2 * tid] = a;
        reinterpret_cast<u32x4*>(cells)[2 * tid + 1] = b;
        if (tid == BLOCK - 1) { cells[NCELL / 2] = base + run; tmp[T_EVENTS] = base + run; }
      }
      team_sync<BLOCK>();
      if (stop_after == kStepCellSums) break;
      // (the registers that cross this barrier are made opaque: values derived from them for the next
      // phase would otherwise be computed before it and held in registers across it)
#pragma unroll
      for (int i = 0; i < NR; ++i) asm volatile("" : "+v"(t[i]), "+v"(ca[i]));
#pragma unroll
      for (int i = 0; i < NR / 4; ++i) asm volatile("" : "+v"(mq[i]));
      auto cell_start = [&](uint32_t c) -> uint32_t { return (cells[c >> 1] >> ((c & 1u) << 4)) & 0xFFFFu; };
      // sorted sequence entry besides the clock: START << 5 | region (four at a time)
      uint32_t info[NR / 4];
#pragma unroll
      for (int x = 0; x < NR / 4; ++x) info[x] = (mq[x] & 0x1F1F1F1Fu) | ((~mq[x] >> 2) & 0x20202020u);
      auto info_of = [&](int i) -> uint32_t { return (info[i >> 2] >> (8 * (i & 3))) & 0x3Fu; };
      // When clock and region fit one word and no cell holds more than kMaxCellWindow records, the records stay
      // in arrival order inside their cell here and every lane of the sweep sorts a window of the sequence
      // in registers; otherwise the records are ranked inside their cell first.
      const bool window_sort = !MANY && R <= 16u && misc[2] < (1u << 26) && !tmp[T_WIDE] && tmp[T_MAXCELL] <= kMaxCellWindow;
      if (MANY ? false : !rare(!window_sort)) {
        // the word the sweep sorts: clock << 6 | START << 5 | region (no branch: what is no event writes one unused word)
        // (opaque here: what both ways compute from these would otherwise be computed ahead of the choice between them)
#pragma unroll
        for (int i = 0; i < NR; ++i) asm volatile("" : "+v"(ca[i]));
#pragma unroll
        for (int i = 0; i < NR / 4; ++i) asm volatile("" : "+v"(mq[i]), "+v"(info[i]));
        constexpr int kTogether = NR < 16 ? NR : 16;
#pragma unroll
        for (int i0 = 0; i0 < NR; i0 += kTogether) {
          uint32_t to[kTogether];
#pragma unroll
          for (int i = 0; i < kTogether; ++i) {
            const uint32_t y = ca[i0 + i] & ((1u << kSlotShift) - 1u);
            to[i] = clk_word(((cells[y >> 5] >> (y & 16u)) & 0xFFFFu) + (ca[i0 + i] >> kSlotShift));
          }
#pragma unroll
          for (int i = 0; i < kTogether; ++i) {
            asm volatile("" : "+v"(to[i]));  // (ahead of the choice: the compiler would make a branch of it)
            clk[meta_of(i0 + i) & kPaired ? to[i] : kSpareWord] = (t[i0 + i] << 6) | info_of(i0 + i);
          }
        }
        team_sync<BLOCK>();
        if (stop_after >= kStepPlaced && stop_after <= kStepSorted) break;
      } else {
      // provisional place: cell start + arrival slot (plain index here, the padded layout comes with the
      // final places)
      uint32_t nm[NR];  // records in the cell (0: this record is no event) | arrival slot << 16
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const uint32_t ev = 0u - ((meta_of(i) >> 6) & 1u);  // all ones for an event
        const uint32_t c = (ca[i] & ((1u << kSlotShift) - 1u)) >> 4, mine = ca[i] >> kSlotShift;
        const uint32_t s0 = cell_start(c), s1 = cell_start(c + 1);
        clk[ev ? s0 + mine : kSpareWord] = t[i];  // no branch: the others all write one unused word
        ca[i] = s0;
        nm[i] = ((s1 - s0) | (mine << 16)) & ev;
      }
      team_sync<BLOCK>();
      if (stop_after == kStepPlaced) break;
      // rank among the records of the same cell: by clock, then by arrival slot
      // (the reads of all of a lane's records together: 4094 workgroups of 8 x 512, 32 regions 252.6 -> 246.0 us, 31 of 8 x 128, 24 regions
      // 19.0 -> 18.2; one-wave teams, whose cells are emptier, are better off record by record: 65534 of 1 x 512 926 / 987)
      // (so are two workgroups of 512 threads per CU, which have 128 registers for it: 4000 of 8 x 1024, 24 regions 304 / 326)
      if constexpr (MANY && TEAMS == 1 && (BLOCK != 512 || PERWAVE > 256)) {
        uint32_t most = 0, before[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) { const uint32_t n = nm[i] & 0xFFFFu; most = n > most ? n : most; before[i] = 0u; }
        for (uint32_t it = 0; __builtin_amdgcn_ballot_w64(it < most); ++it) {
          uint32_t tm[NR];
#pragma unroll
          for (int i = 0; i < NR; ++i) tm[i] = clk[it < (nm[i] & 0xFFFFu) ? ca[i] + it : kSpareWord];
#pragma unroll
          for (int i = 0; i < NR; ++i) {
            const bool lower = tm[i] < t[i] || (tm[i] == t[i] && it < (nm[i] >> 16));  // the record's own entry gives none
            before[i] += it < (nm[i] & 0xFFFFu) && lower ? 1u : 0u;
          }
        }
#pragma unroll
        for (int i = 0; i < NR; ++i) ca[i] += before[i];
      } else {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          const uint32_t n = nm[i] & 0xFFFFu, s0 = ca[i], mine = nm[i] >> 16, t0 = t[i];
          uint32_t before = 0;
          for (uint32_t it = 0; __builtin_amdgcn_ballot_w64(it < n); ++it) {
            if (it < n) {
              const uint32_t tm = clk[s0 + it];
              before += (uint32_t)(tm < t0) | ((uint32_t)(tm == t0) & (uint32_t)(it < mine));  // the record's own entry gives 0
            }
          }
          ca[i] = s0 + before;
        }
      }
      team_sync<BLOCK>();
      if (stop_after == kStepRanked) break;
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const bool ev = (meta_of(i) & kPaired) != 0u;
        clk[ev ? clk_word(ca[i]) : kSpareWord] = t[i];
        meta[ev ? ca[i] : NPOS] = (uint8_t)info_of(i);
      }
      team_sync<BLOCK>();
      if (stop_after == kStepSorted) break;
      }

      // ---- D: region-pair overlap, 16 consecutive records of the sorted sequence per lane ----------
      {
        const uint32_t n_events = tmp[T_EVENTS];
        const uint32_t g0 = tid * NR;
        const uint32_t region_bits = 0xFFFFFFFFu >> (32u - R);  // places past the end carry a bit above the regions
        uint32_t pl[PLANES], inc[PLANES];
#pragma unroll
        for (int k = 0; k < PLANES; ++k) pl[k] = 0u;
        // From each lane's net change (pl) to the state before its stretch (pl again): an inclusive scan
        // over the lanes, the waves' totals through LDS and one barrier, a scan over those.  `first_clock`
        // is the clock of the lane's first record, left for the last lane of the wave below.
        auto state_before = [&](uint32_t first_clock) {
#pragma unroll
          for (int k = 0; k < PLANES; ++k) inc[k] = pl[k];
          {
            uint32_t o[PLANES];
#pragma unroll
            for (int k = 0; k < PLANES; ++k) o[k] = scan_src<0>(inc[k]);
            planes_add<PLANES>(inc, o);
#pragma unroll
            for (int k = 0; k < PLANES; ++k) o[k] = scan_src<1>(inc[k]);
            planes_add<PLANES>(inc, o);
#pragma unroll
            for (int k = 0; k < PLANES; ++k) o[k] = scan_src<2>(inc[k]);
            planes_add<PLANES>(inc, o);
#pragma unroll
            for (int k = 0; k < PLANES; ++k) o[k] = scan_src<3>(inc[k]);
            planes_add<PLANES>(inc, o);
#pragma unroll
            for (int k = 0; k < PLANES; ++k) o[k] = scan_src<4>(inc[k]);
            planes_add<PLANES>(inc, o);
#pragma unroll
            for (int k = 0; k < PLANES; ++k) o[k] = scan_src<5>(inc[k]);
            planes_add<PLANES>(inc, o);
          }
          if (lane == 63) {
#pragma unroll
            for (int k = 0; k < PLANES; ++k) ptot[hw * 8 + k] = inc[k];
          }
          if (lane == 0) wtot[hw] = first_clock;
          team_sync<BLOCK>();
#pragma unroll
          for (int k = 0; k < PLANES; ++k) pl[k] = wave_shr1(inc[k], 0u);
          if (hw > 0) {  // lane h of a row takes wave h's net change; a scan over the row, then the entry of wave hw - 1
            uint32_t wsum[PLANES], o[PLANES];
#pragma unroll
            for (int k = 0; k < PLANES; ++k) wsum[k] = ptot[(lane & 15u) * 8 + k];
#pragma unroll
            for (int k = 0; k < PLANES; ++k) o[k] = scan_src<0>(wsum[k]);
            planes_add<PLANES>(wsum, o);
#pragma unroll
            for (int k = 0; k < PLANES; ++k) o[k] = scan_src<1>(wsum[k]);
            planes_add<PLANES>(wsum, o);
#pragma unroll
            for (int k = 0; k < PLANES; ++k) o[k] = scan_src<2>(wsum[k]);
            planes_add<PLANES>(wsum, o);
#pragma unroll
            for (int k = 0; k < PLANES; ++k) o[k] = scan_src<3>(wsum[k]);
            planes_add<PLANES>(wsum, o);
#pragma unroll
            for (int k = 0; k < PLANES; ++k) o[k] = (uint32_t)__builtin_amdgcn_readlane((int)wsum[k], (int)(hw - 1u));
            planes_add<PLANES>(pl, o);
          }
        };
        // One record of the sequence for the general way of adding up: a region that switches on or off
        // adds -t / +t to its sums with every region open at that instant (LDS atomics).  Here the records of one clock come in
        // any order: where waves end a region and start it again, its count may run past the last one that the planes hold
        // and the region is off for a moment.  It counts as switched whenever it changes, on whichever record, so that what
        // is added on one clock for such a moment cancels.
        auto switch_record = [&](uint32_t x, uint32_t up, uint32_t tt) {
          uint32_t act_before = pl[0];
#pragma unroll
          for (int k = 1; k < PLANES; ++k) act_before |= pl[k];
          planes_step<PLANES>(pl, x, up);
          uint32_t act_after = pl[0];
#pragma unroll
          for (int k = 1; k < PLANES; ++k) act_after |= pl[k];
          if (act_before != act_after) {  // (in the bit of this region)
            // modulo 2^32: the totals of one workgroup lie below its span, which is below 2^32
            const uint32_t a = __ffs(x) - 1;
            uint32_t* row = oacc32 + a * (R | 1u);
            const uint32_t val = act_after & x ? 0u - tt : tt;
            atomicAdd(&row[a], val);
            uint32_t set = act_before & act_after & region_bits;  // the others
            while (set) {
              const uint32_t bb = __ffs(set) - 1;
              set &= set - 1;
              atomicAdd(&row[bb], val);
            }
          }
        };
        if (MANY ? false : !rare(!window_sort)) {
          // ---- the order is finished in registers; one word per record from here on ------------------
          uint32_t key[NR];
          const uint32_t fake = (misc[2] << 6) | 0x3Fu;
          if (!rare(tmp[T_MAXCELL] > NR / 2 + 1u)) sorted_own<BLOCK, NR>(clk, tid, n_events, fake, key);
          else sorted_pairs<BLOCK, NR>(clk, tid, n_events, fake, key);
          if constexpr (PLANES == 4) {
            // Counts up to 15 of 16 regions are one number of 64 bits, four to each.  A sum of such numbers is right in every
            // digit as long as the counts it stands for are (from 0 to the number of waves behind every record: see the
            // words' order), whatever it took and gave on the way: so the state before a
            // lane's stretch is a prefix sum of integers, and becomes planes at the end.
            uint64_t ended = 0;  // ENDs less STARTs
#pragma unroll
            for (int i = 0; i < NR; ++i) ended += (uint64_t)((int64_t)(int32_t)(key_start_mask(key[i]) | 1u) << ((4u * key[i]) & 63u));
            if (__builtin_amdgcn_ballot_w64(g0 + NR > n_events)) {  // a place past the end counted as a START of region 15
              const uint32_t past = g0 + NR > n_events ? (g0 > n_events ? (uint32_t)NR : g0 + NR - n_events) : 0u;
              ended += (uint64_t)past << 60;
            }
            const uint64_t net = 0ull - ended;
            uint64_t incl = net;
            incl += scan_src64<0>(incl); incl += scan_src64<1>(incl); incl += scan_src64<2>(incl);
            incl += scan_src64<3>(incl); incl += scan_src64<4>(incl); incl += scan_src64<5>(incl);
            uint64_t* wave_net = reinterpret_cast<uint64_t*>(ptot);
            if (lane == 63u) wave_net[hw] = incl;
            if (lane == 0u) wtot[hw] = key_clock(key[0]);
            team_sync<BLOCK>();
            uint64_t state = incl - net;
            if (hw > 0u) {  // lane h of a row takes wave h's net change; a scan over the row, then the entry of wave hw - 1
              uint64_t sum = wave_net[lane & 15u];
              sum += scan_src64<0>(sum); sum += scan_src64<1>(sum); sum += scan_src64<2>(sum); sum += scan_src64<3>(sum);
              state += (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)sum, (int)(hw - 1u)) |
                       ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(sum >> 32), (int)(hw - 1u)) << 32);
            }
            const uint32_t lo = planes_of_nibbles((uint32_t)state), hi = planes_of_nibbles((uint32_t)(state >> 32));
#pragma unroll
            for (int k = 0; k < 4; ++k) pl[k] = __builtin_amdgcn_perm(hi, lo, 0x0C0C0400u + 0x0101u * k);
          } else {
#pragma unroll
            for (int i = 0; i < NR; ++i) planes_step<PLANES>(pl, key_region_bit(key[i]), key_start_mask(key[i]));
            state_before(key_clock(key[0]));
          }
#pragma unroll
          for (int i = 0; i < NR; ++i) asm volatile("" : "+v"(key[i]));  // (opaque across the barrier, as above)
          // ---- the sorted sequence as segments: the set of active regions after record k and the ticks
          // until record k + 1.  O[a][b] = sum over segments of ticks * active(a) * active(b) is a 16 x K by
          // K x 16 matrix product: the matrix cores take it 64 segments at a time (i8 operands: the ticks in
          // signed digits of base 256, one product per digit), and no accumulator atomics are left in the sweep.
          // clock of the record after the lane's 16: the first one of the lane above
          const uint32_t t_above = hw + 1 < BLOCK / 64 ? wtot[hw + 1 < BLOCK / 64 ? hw + 1 : hw] : misc[2];
          const uint32_t t_next = (uint32_t)__builtin_amdgcn_update_dpp((int)t_above, (int)key_clock(key[0]), 0x130, 0xF, 0xF, false);  // wave_shl:1
          // (places past the end of the sequence carry the workgroup's last clock: stretches of length 0
          // behind a last one in which no region is open)
          uint32_t len[NR];
          uint32_t any_len = 0;
#pragma unroll
          for (int i = 0; i < NR; ++i) {
            len[i] = (i + 1 < NR ? key_clock(key[i + 1]) : t_next) - key_clock(key[i]);
            any_len |= len[i];
          }
          {  // OR over the wave
            uint32_t f = any_len;
            f |= scan_src<0>(f); f |= scan_src<1>(f); f |= scan_src<2>(f);
            f |= scan_src<3>(f); f |= scan_src<4>(f); f |= scan_src<5>(f);
            any_len = (uint32_t)__builtin_amdgcn_readlane((int)f, 63);
          }
          if (!rare(any_len >= 0x7F7F80u)) {  // else: a gap of more than three digits, the general way takes this wave
            const uint32_t n_digits = any_len < 0x80u ? 1u : (any_len < 0x7F80u ? 2u : 3u);
            // The lane's own places of the sequence are free now (every neighbour read them before the last
            // barrier): they take the active sets (16 bits each) and two digits, its metadata bytes the third one.
            uint32_t* own = clk + clk_word(g0);
            // (digit k of a length, from -128 to 127: byte k of length + 0x808080, less 0x80)
#pragma unroll
            for (int i = 0; i < NR; ++i) len[i] += 0x808080u;
            auto digit_words = [&](uint32_t k, uint32_t (&l)[NR / 4]) __attribute__((always_inline)) {
#pragma unroll
              for (int i = 0; i < NR / 4; ++i) {
                const uint32_t a = __builtin_amdgcn_perm(len[4 * i + 1], len[4 * i], 0x0C0C0400u + 0x0101u * k);
                const uint32_t b = __builtin_amdgcn_perm(len[4 * i + 3], len[4 * i + 2], 0x0C0C0400u + 0x0101u * k);
                l[i] = __builtin_amdgcn_perm(b, a, 0x05040100u) ^ 0x80808080u;
              }
            };
            uint32_t l0[NR / 4], l1[NR / 4];
            digit_words(0, l0);
            if constexpr (NR == 16) {
              reinterpret_cast<u32x4*>(own)[2] = u32x4{l0[0], l0[1], l0[2], l0[3]};
              if (n_digits > 1u) {
                digit_words(1, l1);
                reinterpret_cast<u32x4*>(own)[3] = u32x4{l1[0], l1[1], l1[2], l1[3]};
              }
            } else {
              digit_words(1, l1);
            }
            if (n_digits > 2u) {
              uint32_t l2[NR / 4];
              digit_words(2, l2);
#pragma unroll
              for (int i = 0; i < NR / 4; ++i) reinterpret_cast<uint32_t*>(meta)[tid * (NR / 4) + i] = l2[i];
            }
            uint32_t mk[NR / 2];  // active sets after records 2x and 2x + 1, 16 bits each
            uint32_t act_even = 0u;
#pragma unroll
            for (int i = 0; i < NR; ++i) {
              planes_step<PLANES>(pl, key_region_bit(key[i]), key_start_mask(key[i]));
              uint32_t act = pl[0];
#pragma unroll
              for (int k = 1; k < PLANES; ++k) act |= pl[k];
              if (i & 1) mk[i >> 1] = __builtin_amdgcn_perm(act, act_even, 0x05040100u);  // the low halves of the two
              else act_even = act;
            }
            if constexpr (NR == 16) {
              reinterpret_cast<u32x4*>(own)[0] = u32x4{mk[0], mk[1], mk[2], mk[3]};
              reinterpret_cast<u32x4*>(own)[1] = u32x4{mk[4], mk[5], mk[6], mk[7]};
            } else {
              *reinterpret_cast<u32x4*>(own) = u32x4{mk[0], mk[1], l0[0], l1[0]};
            }
            products = (tid & ~63u) * NR < n_events ? n_digits : 0u;  // this wave holds records
          } else {
            // Its neighbours may add up their own stretches only: what is open where this wave's begin counts as
            // switched on there, what is open where they end as switched off.
            auto add_open = [&](uint32_t val) {
              uint32_t act = pl[0];
#pragma unroll
              for (int k = 1; k < PLANES; ++k) act |= pl[k];
              for (uint32_t rows = act & region_bits; rows; rows &= rows - 1)
                for (uint32_t set = rows; set; set &= set - 1)  // (from the diagonal on)
                  atomicAdd(&oacc32[(__ffs(rows) - 1u) * (R | 1u) + __ffs(set) - 1u], val);
            };
            if (lane == 0) add_open(0u - key_clock(key[0]));
#pragma unroll
            for (int i = 0; i < NR; ++i)
              switch_record(key_region_bit(key[i]) & region_bits, key_start_mask(key[i]), key_clock(key[i]));
            if (lane == 63) add_open(t_next);
          }
        } else {
          // ---- the general way: the sequence is already in order, clocks up to 32 bits, up to 32 regions --
          uint32_t st[NR], sx[NR];  // clock, region bit (0: no record)
          uint32_t starts = 0;         // bit i: record i is a START
          uint32_t mw[NR / 4];
          load_meta(tid, mw);
          load_run<NR>(clk, tid, st);
#pragma unroll
          for (int i = 0; i < NR; ++i) {
            const uint32_t info = (mw[i >> 2] >> (8 * (i & 3))) & 0xFFu;
            sx[i] = g0 + i < n_events ? 1u << (info & 31u) : 0u;
            starts |= ((info >> 5) & 1u) << i;
          }
          auto start_mask = [&](int i) -> uint32_t { return (uint32_t)((int32_t)(starts << (31 - i)) >> 31); };  // all ones for a START
#pragma unroll
          for (int i = 0; i < NR; ++i) planes_step<PLANES>(pl, sx[i], start_mask(i));
          state_before(st[0]);
#pragma unroll
          for (int i = 0; i < NR; ++i) switch_record(sx[i], start_mask(i), st[i]);
        }
      }
    }
    } while (0);
    // The first records of the next workgroup travel while the matrix cores work.
    request_units(wg_ahead, tid, std::integral_constant<int, 0>{}, std::integral_constant<int, kEarly>{});
    // (Wave-uniform, and in a scalar register: matrix instructions do not heed the execution mask, and a short branch on a
    // vector register is taken by masking alone.)
    const uint32_t n_digits = (uint32_t)__builtin_amdgcn_readfirstlane((int)products);
    if (n_digits) {
      __builtin_amdgcn_wave_barrier();
      typedef int i32x4 __attribute__((ext_vector_type(4)));
      i32x4 acc[3];
#pragma unroll
      for (int l = 0; l < 3; ++l) acc[l] = i32x4{0, 0, 0, 0};
      const uint32_t j = lane & 15u;  // operand row / column: region j
      const uint32_t up = 15u - j;      // shift that takes bit j of a 16-bit set to its top
      // (a wave that is not full has no segments past its share of the records; with 16 waves one register is too many)
      const uint32_t sets = BLOCK == 1024 && NR == 16 ? 16u : (uint32_t)__builtin_amdgcn_readfirstlane((int)(tmp[T_EVENTS] - (tid & ~63u) * NR + 63u)) >> 6;
      // this lane reads the places from 64 n + 16 (lane / 16) of the wave's on
      const uint32_t place0 = (tid & ~63u) * NR + 16u * (lane >> 4);
      const u32x4* from0 = reinterpret_cast<const u32x4*>(clk + clk_word(place0));
      for (uint32_t n = 0; n < NR && n < sets; ++n) {  // 64 segments: those of 64 / NR lanes
        const u32x4* from = from0 + 17u * n;  // (68 words: 64 and their padding)
        uint32_t w8[8];  // sets of 16 segments
        u32x4 l0, l1{0u, 0u, 0u, 0u};
        if constexpr (NR == 16) {
          const u32x4 s0 = from[0], s1 = from[1];
          w8[0] = s0.x; w8[1] = s0.y; w8[2] = s0.z; w8[3] = s0.w; w8[4] = s1.x; w8[5] = s1.y; w8[6] = s1.z; w8[7] = s1.w;
          l0 = from[2];
          if (n_digits > 1u) l1 = from[3];
        } else {  // four lanes' places side by side
          const u32x4 a = from[0], b = from[1], c = from[2], d = from[3];
          w8[0] = a.x; w8[1] = a.y; w8[2] = b.x; w8[3] = b.y; w8[4] = c.x; w8[5] = c.y; w8[6] = d.x; w8[7] = d.y;
          l0 = u32x4{a.z, b.z, c.z, d.z};
          l1 = u32x4{a.w, b.w, c.w, d.w};
        }
        // One byte per segment, all ones if region j is open in it: the byte permute's selectors 8..11
        // replicate the top bits of the four halves of its two operands.  As an i8 operand such a byte
        // is -1, so the products below come out negated.
        i32x4 ones;
#pragma unroll
        for (int y = 0; y < 4; ++y)
          ones[y] = (int)__builtin_amdgcn_perm(w8[2 * y + 1] << up, w8[2 * y] << up, 0x0B0A0908u);
        const i32x4 bits = ones;
        acc[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones & i32x4{(int)l0.x, (int)l0.y, (int)l0.z, (int)l0.w}, bits,
                                                       acc[0], 0, 0, 0);
        if (n_digits > 1u) {
          acc[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones & i32x4{(int)l1.x, (int)l1.y, (int)l1.z, (int)l1.w}, bits,
                                                         acc[1], 0, 0, 0);
        }
        if (n_digits > 2u) {
          const u32x4 l2 = *reinterpret_cast<const u32x4*>(meta + place0 + 64u * n);
          acc[2] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones & i32x4{(int)l2.x, (int)l2.y, (int)l2.z, (int)l2.w}, bits,
                                                         acc[2], 0, 0, 0);
        }
      }
      // element v of a lane: row 4 * (lane / 16) + v, column lane % 16.  The product is symmetric and the
      // fold below adds the two halves of a pair: the upper triangle takes the whole sum.
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const uint32_t a = 4u * (lane >> 4) + v, b = j;
        const uint32_t total = 0u - ((uint32_t)acc[0][v] + ((uint32_t)acc[1][v] << 8) + ((uint32_t)acc[2][v] << 16));
        if (a <= b && b < R && total) atomicAdd(&oacc32[a * (R | 1u) + b], total);
      }
    }
    team_sync<BLOCK>();
    request_header(wg_ahead, tid);
    if (stop_after) continue;

    // ---- E: per-(workgroup, wave, region) output, fold into running totals ------------------------
    for (uint32_t e = tid; e < W * R; e += BLOCK) {
      unsigned long long pk = 0;
      uint32_t mx = 0, mn = 0xFFFFFFFFu;
      for (uint32_t c = 0; c < n_copies; ++c) {
        const uint32_t ec = e * n_copies + c;
        pk += pw_pack[ec];
        mx = pw_max[ec] > mx ? pw_max[ec] : mx;
        mn = pw_min[ec] < mn ? pw_min[ec] : mn;
        pw_pack[ec] = 0; pw_max[ec] = 0; pw_min[ec] = 0xFFFFFFFFu;
      }
      const uint32_t n = (uint32_t)(pk >> 46);
      const unsigned long long s = pk & ((1ull << 46) - 1);
      uint64_t* dst = p.out + SL.per + ((size_t)wg * W * R + e) * 2;
      dst[0] = s;
      dst[1] = (uint64_t)n | ((uint64_t)mx << 32);
      if (n) {
        const uint32_t r = e % R;
        atomicAdd(&reg_sum[r], s);
        atomicMax(&reg_max[r], mx);
        atomicMin(&reg_min[r], mn);
      }
    }
    // region-pair sums of this workgroup: the two one-sided sums of a pair add up, modulo 2^32, to the
    // time both regions were open (below the span, hence exact); the upper triangle keeps the totals
    for (uint32_t i = tid; i < R * R; i += BLOCK) {
      const uint32_t a = i / R, b = i - a * R;
      if (a > b) continue;
      uint32_t* ab = oacc32 + a * (R | 1u) + b;
      uint32_t* ba = oacc32 + b * (R | 1u) + a;
      const uint32_t v = a == b ? *ab : *ab + *ba;
      *ab = 0u; *ba = 0u;
      if constexpr (TEAMS == 1) oacc[i] += v;
      else if (v) atomicAdd(&oacc[i], (unsigned long long)v);
    }
    if (tid == 0) {
      auto count = [&](int which, uint32_t n) {
        if constexpr (TEAMS == 1) ctr[which] += n;
        else if (n) atomicAdd(&ctr[which], (unsigned long long)n);
      };
      count(H_INVALID, wg_invalid);
      count(H_DISORDER, tmp[T_DISORDER]);
      count(H_NONMONO, tmp[T_NONMONO]);
      count(H_PAIRS, tmp[T_PAIRS]);
      count(H_ORPHAN_START, tmp[T_STARTS] - tmp[T_ENDS] - tmp[T_PAIRS]);  // T_STARTS counts the records
      count(H_ORPHAN_END, tmp[T_ENDS] - tmp[T_PAIRS]);
      count(H_SPAN_OVF, misc[0]);
      count(H_OVERLAP_WGS, eligible ? 1u : 0u);
    }
    // No barrier here: the arrays this tail reads and resets are next written in B, two barriers on, and
    // what the head of the next workgroup writes first (temporaries, header words) is touched here only by
    // thread 0, whose own wave writes them there.
  }
  __syncthreads();

  // ---- flush this decoder workgroup's totals --------------------------------------------------
  unsigned long long* out = reinterpret_cast<unsigned long long*>(p.out);
  for (uint32_t i = threadIdx.x; i < R * kBins; i += n_threads) {
    const uint32_t r = i / kBins, bin = i % kBins, h = hist[r * kHistStride + bin];
    if (h) atomicAdd(&out[SL.hist + r * 64u + bin], (unsigned long long)h);
  }
  for (uint32_t i = threadIdx.x; i < R * R; i += n_threads)
    if (oacc[i]) atomicAdd(&out[SL.F + i], oacc[i]);  // (the upper triangle)
  for (uint32_t r = threadIdx.x; r < R; r += n_threads) {
    if (reg_min[r] != 0xFFFFFFFFu || reg_max[r] || reg_sum[r]) {
      atomicAdd(&out[SL.sum + r], reg_sum[r]);
      atomicMax(&out[SL.max + r], (unsigned long long)reg_max[r]);
      atomicMin(&out[SL.min + r], (unsigned long long)reg_min[r]);
    }
  }
  if (threadIdx.x < H_STATUS && ctr[threadIdx.x]) atomicAdd(&out[threadIdx.x], ctr[threadIdx.x]);
}

// Launch shape of one kernel instantiation for one LDS size, queried once per device.
struct LaunchCache { int dev = -1; uint32_t max_grid = 0; };

template <int BLOCK, int NR, int TEAMS, int PLANES, int RMAX, int PERWAVE, int RINGS, bool MANY>
kp_status launch_main(const DecodeParams& p, hipStream_t s) {
  auto kern = kp_reduce_main<BLOCK, NR, TEAMS, PLANES, RMAX, PERWAVE, RINGS, MANY>;
  static thread_local LaunchCache cache;
  int dev = 0;
  KP_HIP_TRY(hipGetDevice(&dev));
  if (cache.dev != dev) {
    int per_cu = 0, cus = 0;
    KP_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, BLOCK * TEAMS, 0));
    if (per_cu < 1) return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "decoder kernel does not fit one CU (LDS %u B)", Lds<BLOCK, NR, TEAMS, RMAX, PERWAVE>::total);
    KP_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    cache.dev = dev; cache.max_grid = (uint32_t)per_cu * (uint32_t)cus;
  }
  uint32_t grid = cache.max_grid;
  if (grid > p.n_wg) grid = p.n_wg;
  uint32_t teams = (p.n_wg + grid - 1u) / grid;  // (every CU has a decoder workgroup before one gets a second team)
  if (teams > (uint32_t)TEAMS) teams = TEAMS;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(BLOCK * teams), 0, s, p);
  KP_HIP_TRY(hipGetLastError());
  return KP_OK;
}

template <int BLOCK, int NR, int TEAMS, int RMAX, int PERWAVE, int RINGS, bool MANY>
kp_status launch_rings(const DecodeParams& p, hipStream_t s) {
  // counters of open waves per region run up to the number of waves
  constexpr int kShortest = RINGS == kSmall ? 2 : RINGS == kWhole ? 64 * NR : 128;
  if constexpr (16 * kShortest <= BLOCK * NR && (!MANY || 16 * 17 <= PERWAVE)) {  // (else 16 waves have more records or sums than this form takes)
    if (p.W == 16) return launch_main<BLOCK, NR, TEAMS, 5, RMAX, PERWAVE, RINGS, MANY>(p, s);
  }
  return launch_main<BLOCK, NR, TEAMS, 4, RMAX, PERWAVE, RINGS, MANY>(p, s);
}

template <int BLOCK, int NR, int TEAMS, int RMAX, int PERWAVE, bool MANY = false>
kp_status launch_planes(DecodeParams& p, hipStream_t s) {
  p.ncopy = 4;  // as many copies of the per-(wave, region) sums as their LDS array has room for
  while (p.ncopy > 1 && p.ncopy * p.W * p.R > (uint32_t)PERWAVE) p.ncopy >>= 1;
  if constexpr (BLOCK * NR <= 1024) {  // (16 waves with rings of 64 slots have 1024 in all)
    if (p.cap < 128u) return launch_rings<BLOCK, NR, TEAMS, RMAX, PERWAVE, kSmall, MANY>(p, s);
  }
  if constexpr (BLOCK == 1024 && NR == 16) {  // (more than 8192 slots in at most 16 rings)
    return launch_rings<BLOCK, NR, TEAMS, RMAX, PERWAVE, kWhole, MANY>(p, s);
  } else if constexpr (BLOCK == 512 && MANY && PERWAVE == 512) {  // (more than 256 sums: nine rings or more in 8192 slots)
    return launch_rings<BLOCK, NR, TEAMS, RMAX, PERWAVE, kPart, MANY>(p, s);
  } else if constexpr ((TEAMS == 1 && BLOCK > 64) || (NR == 16 && !MANY)) {
    return p.cap < 64u * NR ? launch_rings<BLOCK, NR, TEAMS, RMAX, PERWAVE, kPart, MANY>(p, s) : launch_rings<BLOCK, NR, TEAMS, RMAX, PERWAVE, kWhole, MANY>(p, s);
  } else {
    return launch_rings<BLOCK, NR, TEAMS, RMAX, PERWAVE, kAny, MANY>(p, s);
  }
}

kp_status reduce_impl(const void* raw, size_t n, const kp_trace_hdr& h, void* out_stats, uint32_t stop_after,
                      hipStream_t s, hipEvent_t main_begin = nullptr, hipEvent_t main_end = nullptr) {
  if (h.magic != KP_TRACE_MAGIC || h.version != KP_TRACE_VERSION)
    return kp::fail(KP_ERR_BAD_TRACE, "trace header: bad magic/version (%08x, %u)", h.magic, h.version);
  if (h.waves_per_wg < 1 || h.waves_per_wg > KP_MAX_WAVES || h.n_regions < 1 || !kp::is_pow2(h.cap_wave))
    return kp::fail(KP_ERR_BAD_TRACE, "trace header: waves=%u regions=%u cap_wave=%u", h.waves_per_wg, h.n_regions, h.cap_wave);
  if ((size_t)h.n_wg * h.waves_per_wg * h.cap_wave != n)
    return kp::fail(KP_ERR_BAD_TRACE, "trace header describes %zu record slots, caller passed %zu",
                    (size_t)h.n_wg * h.waves_per_wg * h.cap_wave, n);
  if ((h.flags & ~(KP_FLAG_FLUSH | KP_FLAG_REALTIME | KP_FLAG_HW_IDS)) != 0) return kp::fail(KP_ERR_BAD_TRACE, "trace header: unknown flags %x", h.flags);
  if (h.n_regions > KP_MAX_TAG_REGIONS)
    return kp::fail(KP_ERR_BAD_TRACE, "trace header: n_regions=%u, the tag holds %d", h.n_regions, KP_MAX_TAG_REGIONS);
  if (h.cap_wave < 2) return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "cap_wave must be at least 2");
  if (h.cap_wave > (1u << 20)) return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "cap_wave=%u exceeds the range of seq", h.cap_wave);
  const uint32_t nrec = h.waves_per_wg * h.cap_wave;
  // geometries the LDS-resident kernel is not built for go to the multi-pass kernel
  const bool wide = h.n_regions > KP_MAX_REGIONS || nrec > kMaxRecPerWg;
  if (wide) {
    const kp_status st = wide_supported(h);
    if (st != KP_OK) return st;
  }
  if (wide && stop_after)
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "single steps exist for the LDS-resident decoder only (n_regions <= %d, %u records per workgroup)",
                    KP_MAX_REGIONS, kMaxRecPerWg);
  if (((uintptr_t)raw & 15u) || ((uintptr_t)out_stats & 15u))
    return kp::fail(KP_ERR_INVALID_ARG, "raw and out_stats must be 16-byte aligned");

  const uint32_t W = h.waves_per_wg, R = h.n_regions, cap = h.cap_wave;

  uint64_t* out = static_cast<uint64_t*>(out_stats);
  const uint8_t* base = static_cast<const uint8_t*>(raw);
  const StatsLayout SL = stats_layout(h.n_wg, W, R);
  int init_blocks = (int)((SL.per + 255) / 256);
  if (init_blocks > 64) init_blocks = 64;
  hipLaunchKernelGGL(kp_reduce_init, dim3(init_blocks), dim3(256), 0, s,
                     reinterpret_cast<const uint32_t*>(base), out, h.n_wg, W, R, cap, h.flags);
  KP_HIP_TRY(hipGetLastError());

  if (main_begin) KP_HIP_TRY(hipEventRecord(main_begin, s));
  if (h.n_wg > 0 && wide) {
    const kp_status st = launch_wide(reinterpret_cast<const uint32_t*>(base + sizeof(kp_trace_hdr)),
                                     base + sizeof(kp_trace_hdr) + sizeof(kp_wg_hdr) * (size_t)h.n_wg, out, h, s);
    if (st != KP_OK) return st;
  } else if (h.n_wg > 0) {
    DecodeParams p;
    p.wg_hdrs = reinterpret_cast<const uint32_t*>(base + sizeof(kp_trace_hdr));
    p.records = reinterpret_cast<const u32x4*>(base + sizeof(kp_trace_hdr) + sizeof(kp_wg_hdr) * (size_t)h.n_wg);
    p.out = out;
    p.n_wg = h.n_wg; p.W = W; p.R = R; p.cap = cap;
    p.cap_log2 = 0; while ((1u << p.cap_log2) < cap) ++p.cap_log2;
    p.rec_cost = h.rec_cost; p.flush = h.flags & KP_FLAG_FLUSH;
    p.nrec = nrec; p.ncopy = 1; p.stop_after = stop_after;
    uint32_t wgs = 0;
    kp_status st = wgs_of_256_cus(h.n_wg, &wgs);
    if (st != KP_OK) return st;
    // How many threads take a recorded workgroup, with how many records each (numbers of workgroups are those on 256 CUs).  Up to 16384 records: 1024
    // threads, 16 each, which is all that fits one CU.  Fewer records leave a choice.  With no more recorded workgroups than CUs the
    // time is one workgroup's chain of steps, and four records per lane make it shorter: 64 workgroups of 4 x 128 records
    // 20.6 us with 16 each (one wave), 16.7 with four (four waves); 256 of 8 x 512 32.3 and 30.1; 100 of 1 x 4096 26.7 and
    // 24.0.  With more of them it is the work, most of which a wave does for all its places whether they hold records or
    // not: as few places as the records need, and as many waves on a CU as LDS allows, whose arrays are sized for at most
    // 8, 16 or 32 regions.  Up to 1024 records one wave decodes a workgroup, and the waves of a decoder workgroup share
    // the running totals, which reach HBM once: every address of them takes about 20 ns per decoder workgroup.  Against
    // one wave per decoder workgroup, 16 records per lane, arrays for 32 regions: 20000 workgroups of 1 x 16 records 361 ->
    // 76 us (16 records per lane in teams 168), 60000 of 1 x 64, 16 regions 1084 -> 219 (490), 8192 of 4 x 128 172 -> 73, 3000
    // of 16 x 64 90 -> 42; 256 threads, arrays for 8 regions: 16000 of 2 x 1024 693 -> 487.
    // Of 257 to 1024 records some more of them are few in that sense: three decoder workgroups of 256 threads fit a CU, and until
    // their totals queue up on the way to HBM they beat waves that take 16 records a lane (257 to 1024 records: with four records
    // a lane / 16, us): 300 of 2 x 256, 5 regions 24.2 / 27.9, 600 35.9 / 29.2; 300 of 8 x 128, 16 regions 20.5 / 27.2, 600 27.5 /
    // 27.4, 768 31.2 / 27.7.  With more than 16 regions those waves take longer and are six to a CU, so that the line is where a fourth
    // decoder workgroup of 256 threads would have to wait for its CU: 400, 768 and 1100 of 2 x 256, 24 regions 25 / 31, 35 / 31, 39 / 33, of 4 x 256, 17
    // regions 28 / 40, 38 / 40, 46 / 41, of 7 x 64, 32 regions 28 / 37, 38 / 39, 45 / 40; and where nearly all lanes of such a wave have records of many
    // rings it is as late as their last turn begins: 700, 1100 and 1400 of 16 x 64, 20 regions 38 / 47, 48 / 48, 49 / 53, of 8 x 128, 24 regions 33 / 42,
    // 40 / 44, 41 / 44.
    // From 1024 records up the threads are as many as the records need, to the next power of two: with half of the places empty the
    // other half's waves come along to every barrier and every step, and two workgroups fit where one did.  512 threads against 1024:
    // 16384 of 8 x 1024, 16 regions 1622 -> 757 us, 510 of 16 x 512 72.4 -> 41.9, 100 of 8 x 1024 35.9 -> 27.1, 4000 of 8 x 1024, 24
    // regions 593 -> 324 (with more than 256 sums per workgroup one to a CU: 510 of 16 x 512, 32 regions 102.5 -> 80.5); 128 against
    // 256: 16000 of 2 x 1024 418 -> 215, 2000 of 8 x 256, 24 regions 127 -> 85, 300 of 2 x 1024 31.6 -> 30.2.  Four workgroups of 256
    // threads or eight of 128 fit a CU, so that with more than 1024 recorded ones the smaller form hands over more totals, one decoder workgroup after
    // the other at each address, until from 2048 on the larger one has to take several turns more.  What that comes to depends on how often the lanes
    // of a wave name the same region (128 / 256 threads, us): 1000, 1600, 2000, 2600 and 4000 of 2 x 1024, 5 regions 56 / 61, 78 / 72, 94 / 80, 98 / 99,
    // 108 / 120; of 8 x 256, 5 regions 58 / 62, 79 / 72, 95 / 79, 99 / 95, 110 / 122; of 3 x 512, 8 regions 44 / 49, 58 / 61, 67 / 67, 71 / 84, 82 / 121;
    // of 16 x 128, 3 regions 47 / 50, 63 / 64, 73 / 71, 76 / 88, 90 / 132; with more than 8 regions within 4 % up to 1600 (12 regions, 8 x 256 67 / 65), then
    // the smaller one.
    const uint32_t few = nrec <= 256 || nrec > 1024 ? 256u : R <= 16 ? 400u : W >= 8 && nrec > 768 ? 1400u : 768u;
    if (wgs <= few && nrec <= 4096) {
      if (R <= 16)
        st = nrec > 1024 ? launch_planes<1024, 4, 1, KP_MAX_REGIONS, kMaxPerWave>(p, s)
           : nrec > 256  ? launch_planes<256, 4, 1, KP_MAX_REGIONS, 512>(p, s)
                         : launch_planes<64, 4, 1, KP_MAX_REGIONS, 512>(p, s);
      else
        st = nrec > 1024 ? launch_planes<1024, 4, 1, KP_MAX_REGIONS, kMaxPerWave, true>(p, s)
           : nrec > 256  ? launch_planes<256, 4, 1, KP_MAX_REGIONS, 512, true>(p, s)
                         : launch_planes<64, 4, 1, KP_MAX_REGIONS, 512, true>(p, s);
    } else if (nrec > 4096 && nrec <= 8192) {
      st = R <= 16 ? launch_planes<512, 16, 1, 16, 512>(p, s) : W * R <= 256 ? launch_planes<512, 16, 1, KP_MAX_REGIONS, 256, true>(p, s)
                                                              : launch_planes<512, 16, 1, KP_MAX_REGIONS, 512, true>(p, s);
    } else if (nrec > 1024 && nrec <= 2048 && (R > 8 || wgs < 1500 || wgs >= 2500)) {
      st = R <= 8 ? launch_planes<128, 16, 1, 8, 128>(p, s) : R <= 16 ? launch_planes<128, 16, 1, 16, 256>(p, s)
                                                           : launch_planes<128, 16, 1, KP_MAX_REGIONS, 512, true>(p, s);
    } else if (nrec > 4096) {
      st = launch_planes<1024, 16, 1, KP_MAX_REGIONS, kMaxPerWave>(p, s);
    } else if (nrec > 1024) {
      st = R <= 8 ? launch_planes<256, 16, 1, 8, 128>(p, s) : R <= 16 ? launch_planes<256, 16, 1, 16, 256>(p, s)
                                                           : launch_planes<256, 16, 1, KP_MAX_REGIONS, 512, true>(p, s);
    } else if (nrec > 256) {
      st = R <= 8 ? launch_planes<64, 16, 12, 8, 128>(p, s) : R <= 16 ? launch_planes<64, 16, 12, 16, 256>(p, s)
                                                           : launch_planes<64, 16, 6, KP_MAX_REGIONS, 512, true>(p, s);
    } else {
      st = R <= 8 ? launch_planes<64, 4, 16, 8, 128>(p, s) : R <= 16 ? launch_planes<64, 4, 12, 16, 256>(p, s)
                                                           : launch_planes<64, 4, 8, KP_MAX_REGIONS, 512, true>(p, s);
    }
    if (st != KP_OK) return st;
  }
  if (main_end) KP_HIP_TRY(hipEventRecord(main_end, s));
  hipLaunchKernelGGL(kp_reduce_derive, dim3(1), dim3(1024), 0, s, out, h.n_wg, W, R);
  KP_HIP_TRY(hipGetLastError());
  return KP_OK;
}

}  // namespace

extern "C" kp_status kp_trace_reduce_hdr(const void* raw, size_t n, const kp_trace_hdr* hdr_host,
                                         void* out_stats, void* stream) {
  kp::clear_error();
  if (!raw || !hdr_host || !out_stats) return kp::fail(KP_ERR_INVALID_ARG, "NULL argument");
  return reduce_impl(raw, n, *hdr_host, out_stats, 0u, static_cast<hipStream_t>(stream));
}

extern "C" kp_status kp_trace_reduce_hdr_events(const void* raw, size_t n, const kp_trace_hdr* hdr_host,
                                                void* out_stats, void* stream, void* main_begin, void* main_end) {
  kp::clear_error();
  if (!raw || !hdr_host || !out_stats) return kp::fail(KP_ERR_INVALID_ARG, "NULL argument");
  return reduce_impl(raw, n, *hdr_host, out_stats, 0u, static_cast<hipStream_t>(stream),
                     static_cast<hipEvent_t>(main_begin), static_cast<hipEvent_t>(main_end));
}

extern "C" kp_status kp_trace_reduce_steps(const void* raw, size_t n, const kp_trace_hdr* hdr_host,
                                           void* out_stats, int last_step, void* stream) {
  kp::clear_error();
  if (!raw || !hdr_host || !out_stats) return kp::fail(KP_ERR_INVALID_ARG, "NULL argument");
  if (last_step < kStepOrdered || last_step > kStepSwept)
    return kp::fail(KP_ERR_INVALID_ARG, "last_step must be %d..%d", kStepOrdered, kStepSwept);
  return reduce_impl(raw, n, *hdr_host, out_stats, (uint32_t)last_step, static_cast<hipStream_t>(stream));
}

extern "C" kp_status kp_trace_reduce(const void* raw, size_t n, void* out_stats, void* stream) {
  kp::clear_error();
  if (!raw || !out_stats) return kp::fail(KP_ERR_INVALID_ARG, "NULL argument");
  kp_trace_hdr h;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const kp_status st = kp::read_header(raw, &h, s);
  if (st != KP_OK) return st;
  return reduce_impl(raw, n, h, out_stats, 0u, s);
}
