// Instrumented bf16 GEMM targets (kp_gemm_instrumented): C[M,N] = A[M,K] * B[K,N], fp32 accumulate,
// bf16 (round-to-nearest-even) output, all row-major.
//
// The paper profiles software-pipelined Triton GEMMs by inserting region records around the
// stages of the K loop (Sec. 5.3, GEMM-SWP-2/3; Sec. 2.3 software pipelining).  These kernels
// are this library's own MFMA GEMMs with hand-placed record sites.  Each exists twice from one
// template: INSTR=0 compiles every record site away (the uninstrumented baseline), INSTR=1 and 2
// record into the LDS ring.  Record sites contain no floating point, so all variants produce
// bit-identical C.
//
//   tile 64x64x32, 4 waves  : per K step regions 0 global load (issue), 1 LDS store (of a later K step, behind
//                              the operand reads of this one), 2 MFMA
//   tile 256x256x64, 8 waves: regions 0 / 1 first / second half of a K step's MFMAs with the
//                              staging of the next K step threaded in, 2 barrier wait, 3 epilogue (once);
//                              or (KP_MASK_PHASES) a K step whose stages follow one another, each its own
//                              region: 2 LDS write, 0 global load issue, 3 MFMA, 1 wait; 4 epilogue (once)
#include <type_traits>

#include "kp_common.h"
#include "kp_record.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct GemmArgs {
  const uint16_t* A;
  const uint16_t* B;
  uint16_t* C;
  uint32_t M, N, K;
  uint32_t region_mask;
  void* trace;
  uint32_t cap_lds, cap_hbm, flush, n_wg;
  uint32_t rec_cost;  // ticks the decoder takes off every duration (kp_set_rec_cost)
  uint32_t group_log2;  // 2^group_log2 waves share one record stream
  uint32_t collab;      // 1: all lanes store a record, hardware ids go to the workgroup header
  uint32_t flags;       // kp_trace_hdr.flags of the trace
};

// two fp32 -> packed bf16 pair (lo in bits 15:0), round to nearest even: one v_cvt_pk_bf16_f32
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pack_rne(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// LDS tiles hold rows of 64 bf16 (K contiguous) in 16-byte chunks; chunk c of row r lives at chunk position
// c ^ (r / 2) % 8, so that the 16-byte reads of 16 neighbouring rows spread over all banks: two neighbouring rows
// already differ in the upper half of the 16 chunk positions of a 256-byte bank line, the XOR takes the next three
// row bits (with row bits 0..2, rows r and r + 8 shared a position, and every operand read took twice as long).
template <int BK>
__device__ __forceinline__ uint32_t tile_off(uint32_t row, uint32_t chunk) {
  static_assert(BK == 64, "128-byte rows");
  return row * 128u + ((chunk ^ ((row >> 1) & 7u)) << 4);  // byte offset
}

// END of one region and START of the next with a single clock sample.  INSTR: 0 no record sites,
// 1 generic sites (region mask, either buffer strategy, either store), 3 the same on the constant-rate
// clock, 2 chained sites (circular, one lane stores; the region mask and wave-group records included), 5 chained
// sites on the constant-rate clock.  SITE is the form of the sites a kernel uses for INSTR (kp::site<>; 6: chained).
// Chained, the loop keeps only the clock of site K of the batch (kp::site_chain) and KP_COMMIT, which stands
// right after a wait for all LDS traffic, stores the batch's clocks; the records are made when the trace is
// copied out (the sites of both kernels are a fixed sequence).
#define KP_SITE_K(ring, K, end_r, start_r) do { if constexpr (INSTR != 0) { \
    if constexpr (SITE == 6) kp::site_chain<K, (INSTR == 5), kMayCross>(ring); else kp::site<SITE>(ring, end_r, start_r); } } while (0)
#define KP_COMMIT(ring, N) do { if constexpr (INSTR != 0 && SITE == 6) kp::chain_commit<N>(ring); } while (0)

// The sequence of the large kernel's record sites (n sites in all).  Default schedule: regions 0, 1, 2 in turn,
// three sites per K step; sites 0 and 1 write no record, they only fill the first two places of the first
// batch, so that every batch of the loop is "the site in the middle of the K step before, the one in front of
// its barrier and the one behind it" and is committed once the first MFMAs of the next K step have been
// issued: no commit waits for a clock it has just asked for, and none stands between a wave and the barrier,
// where its instructions and the latency of its LDS write would be time on the critical path of every K step.  Stages apart: regions 2, 0, 3, 1 in turn, four sites per K step, committed
// behind the barrier (every wave waits there in region 1 anyway); no leading site.  The last site of the loop
// opens the epilogue region instead (3, or 4 with the stages apart), the very last closes it.
template <bool PHASED>
struct GemmChain {
  static constexpr uint32_t kEpilogue = PHASED ? 4u : 3u, kRegions = kEpilogue + 1u, kLead = PHASED ? 0u : 2u;
  static constexpr bool kDense = true;
  // n = kLead + (3 or 4) K steps + 2: every enabled region of the loop leaves two records per K step, the epilogue two
  __device__ uint32_t total(uint32_t n, uint32_t mask) const {
    const uint32_t steps = (n - 2u - kLead) / (PHASED ? 4u : 3u);
    return 2u * steps * (uint32_t)__builtin_popcount(mask & ((1u << kEpilogue) - 1u)) + 2u * ((mask >> kEpilogue) & 1u);
  }
  __device__ static uint32_t in_turn(uint32_t i) {
    if constexpr (PHASED) return (0x1302u >> ((i & 3u) * 4u)) & 0xFu;  // 2, 0, 3, 1
    else return i % 3u;
  }
  __device__ uint32_t end_region(uint32_t site, uint32_t n) const {
    return site <= kLead ? kp::kNoRegion : site + 1u == n ? kEpilogue : in_turn(site - 1u - kLead);
  }
  __device__ uint32_t start_region(uint32_t site, uint32_t n) const {
    return (site < kLead || site + 1u == n) ? kp::kNoRegion : site + 2u == n ? kEpilogue : in_turn(site - kLead);
  }
};

// ------------------------------------------------------------------------------------------
// 64x64x32 tile, 4 waves as 2x2, each wave one 32x32 accumulator tile.
//
// What bounds it: with few workgroups the latency of a K step, with many the way of the tiles through registers into LDS:
// of the 36 us that 2112x1984x2080 took when this was looked at the loads were 8 (16 KiB per workgroup and pair of K steps: 545
// MB of 128-byte lines, none of which hits in L1), the LDS stores 9 more, half of the operand reads 1; what was left, 19 us, are
// the MFMAs (14 at the rate of a large product) and the barriers.  So the global loads run two pairs of K steps ahead in registers, the two LDS stages hold a pair each (one barrier
// per pair), B is stored as it comes and transposed by the operand read, and up to five workgroups share a CU.  The
// loop is one block without exits, in which the loads stand where they are written (with an exit behind every K step the
// compiler put them behind it, and waited for all of them once in two pairs), a lane's addresses move by one 64-bit
// addition per pair, and what needs to look at the end of K comes behind the loop.  Against the form with exits (median of
// passes in a row): 2112x1984x2080 32.8 -> 31.1 us (560 TFLOP/s), all regions recorded 42.5 -> 36.5; 4032x3968x4000 223
// -> 217, recorded 249 -> 228; 128x128x3776 (4 workgroups) 18.3 -> 16.3, recorded 29.3 -> 21.2.  Three pairs ahead: 3 %
// slower where many workgroups share a CU (registers), nothing gained with few.  Plain order of the tiles instead of bands
// per XCD: 39 us; four neighbouring tiles on one CU, to share panels in L1: no hits, 3 % slower.
//
// The sequence of its record sites (n in all): the first opens region 0, then three per K step close regions
// 0, 1 and 2 and open the next, the last only closes.
struct SmallGemmChain {
  static constexpr uint32_t kRegions = 3u, kLead = 0u;
  static constexpr bool kDense = true;
  __device__ uint32_t total(uint32_t n, uint32_t mask) const { return 2u * ((n - 1u) / 3u) * (uint32_t)__builtin_popcount(mask & 7u); }
  __device__ uint32_t end_region(uint32_t site, uint32_t) const { return site == 0u ? kp::kNoRegion : (site - 1u) % 3u; }
  __device__ uint32_t start_region(uint32_t site, uint32_t n) const { return site + 1u == n ? kp::kNoRegion : site % 3u; }
};

// A wave's 32x32 of C, transposed (register v of lane l is C[m, n] with m = l%32 and n = 8*(v/4) + 4*(l/32) + v%4), through
// 2 KiB of LDS of its own to memory: a lane holds four columns of a row, 32 rows with 16 bytes each per store instruction;
// this way there are two instead of four, with 64 bytes of 16 rows.  A row is four chunks of 16 bytes; chunk c of row r at
// position c ^ (r / 2) % 4, its halves swapped where r / 8 is odd: 16 lanes of an 8-byte write hit all banks once.
__device__ __forceinline__ void c_tile_to_lds(const f32x16& acc, unsigned char* lds) {
  const uint32_t lane = threadIdx.x & 63u, r = lane & 31u, half = (lane >> 5) ^ ((r >> 3) & 1u);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    u32x2 pk;
    pk.x = bf16_pack_rne(acc[4 * q + 0], acc[4 * q + 1]);
    pk.y = bf16_pack_rne(acc[4 * q + 2], acc[4 * q + 3]);
    *reinterpret_cast<u32x2*>(lds + r * 64u + (((uint32_t)q ^ ((r >> 1) & 3u)) << 4) + 8u * half) = pk;
  }
}
__device__ __forceinline__ void c_tile_to_memory(const unsigned char* lds, uint16_t* c, uint32_t ldc) {
  const uint32_t lane = threadIdx.x & 63u, r = lane >> 2, chunk = (lane & 3u) ^ ((r >> 1) & 3u);  // (the same chunk in row r + 16)
  uint16_t* at = c + (size_t)r * ldc + 8u * chunk;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(lds + 1024u * (uint32_t)i + 16u * lane);
    *reinterpret_cast<u32x4*>(at + (size_t)(16 * i) * ldc) = (r & 8u) ? u32x4{v.z, v.w, v.x, v.y} : v;
  }
}

template <int INSTR>
__global__ __launch_bounds__(256) void kp_gemm_small(GemmArgs g) {
  constexpr int SITE = (INSTR == 2 || INSTR == 5) ? 6 : INSTR;
  constexpr bool REALTIME = INSTR == 3 || INSTR == 5;
  constexpr int kMayCross = 0;
  constexpr int BM = 64, BN = 64, BK = 32;
  constexpr uint32_t A_BYTES = BM * 2 * BK * 2, STAGE = A_BYTES + BN * 2 * BK * 2;
  constexpr int AHEAD = 2;  // pairs of K steps between the request of a tile and its use
  __shared__ __align__(16) unsigned char tiles[2 * STAGE];  // [stage][A rows of 64 k | B rows of 64 n], two K steps each
  extern __shared__ __align__(16) uint32_t ring_lds[];

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t tiles_m = g.M / BM, tiles_n = g.N / BN;
  // Workgroups are dealt round-robin to the 8 XCDs: every XCD gets a run of consecutive tiles in an order that
  // goes down bands of eight tile rows, so that the panels it streams stay in its own L2.
  uint32_t tile_r, tile_c;
  {
    const uint32_t n = tiles_m * tiles_n, xcd = blockIdx.x & 7u, rest = n & 7u;
    const uint32_t t = xcd * (n >> 3) + (xcd < rest ? xcd : rest) + (blockIdx.x >> 3);
    const uint32_t band = t / (8u * tiles_n), first = band * 8u, in = t - band * (8u * tiles_n);
    const uint32_t rows = tiles_m - first < 8u ? tiles_m - first : 8u;
    tile_c = in / rows;
    tile_r = first + in - tile_c * rows;
  }
  const uint32_t wg = tile_r * tiles_n + tile_c;  // recorded workgroup id = tile index
  const uint32_t m0 = tile_r * BM, n0 = tile_c * BN;

  // Global -> registers -> LDS, two K steps at a time, so that a row of the A tile is a whole 128-byte line (one
  // K step of it is half a line, and every line went through the L1 twice): A in the even step of a pair, B in the
  // odd one, two 16-byte chunks per thread each.  Chunk c of A row r sits at position c ^ (r / 2) % 8 (16 rows of
  // an operand read cover all banks).  B stays as it lies in memory and is transposed by the operand read (see the
  // large kernel); chunk c of row k at position c ^ 4 (k / 2 % 2), which spreads the four rows of a read.
  const uint32_t KT = g.K / BK;
  const uint32_t row = tid >> 3, chunk = tid & 7u;
  const uint32_t a_dst = row * 128u + ((chunk ^ ((row >> 1) & 7u)) << 4);              // (row + 32: + 4096)
  const uint32_t b_dst = A_BYTES + row * 128u + ((chunk ^ (((row >> 1) & 1u) << 2)) << 4);
  const uint32_t PAIRS = (KT + 1u) / 2u;
  u32x4 ra[AHEAD][2], rb[AHEAD][2];
  // This lane's addresses in the pair requested last; every request moves them on (behind the site that opens its region:
  // the distance is opaque), up to the last pair, which is then asked for again (nobody uses it: a K step without loads
  // would have an empty region 0).  LAST: the pair may be the first or the last one, and of one K step only; what would
  // lie behind it is asked for as the same of the first step.
  const uint16_t* a_src = g.A + (size_t)(m0 + row) * g.K + chunk * 8u;
  const uint16_t* b_src = g.B + (size_t)row * g.N + n0 + chunk * 8u;
  const size_t a_down = (size_t)32u * g.K, b_down = (size_t)32u * g.N;
  auto request_a = [&](uint32_t pair, int set, auto last_c) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last_c)::value;
    size_t on = !LAST || (pair > 0u && pair < PAIRS) ? 2u * BK : 0u;
    asm volatile("" : "+s"(on) : : "memory");
    a_src += on;
    const uint16_t* at = a_src;
    if (LAST && pair + 1u >= PAIRS && (KT & 1u) && chunk >= 4u) at -= BK;
    ra[set][0] = *reinterpret_cast<const u32x4*>(at);
    ra[set][1] = *reinterpret_cast<const u32x4*>(at + a_down);
  };
  auto request_b = [&](uint32_t pair, int set, auto last_c) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last_c)::value;
    size_t on = !LAST || (pair > 0u && pair < PAIRS) ? 2u * b_down : 0u;
    asm volatile("" : "+s"(on) : : "memory");
    b_src += on;
    rb[set][0] = *reinterpret_cast<const u32x4*>(b_src);
    rb[set][1] = *reinterpret_cast<const u32x4*>(b_src + (LAST && pair + 1u >= PAIRS && (KT & 1u) ? 0u : b_down));
  };
  auto store_a = [&](uint32_t stage, int set) __attribute__((always_inline)) {
    *reinterpret_cast<u32x4*>(tiles + stage * STAGE + a_dst) = ra[set][0];
    *reinterpret_cast<u32x4*>(tiles + stage * STAGE + a_dst + 4096u) = ra[set][1];
  };
  auto store_b = [&](uint32_t stage, int set) __attribute__((always_inline)) {
    *reinterpret_cast<u32x4*>(tiles + stage * STAGE + b_dst) = rb[set][0];
    *reinterpret_cast<u32x4*>(tiles + stage * STAGE + b_dst + 4096u) = rb[set][1];
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) { request_a((uint32_t)i, i, yes); request_b((uint32_t)i, i, yes); }

  kp::Ring ring{};
  if constexpr (INSTR != 0)
    ring = kp::ring_init<true>(ring_lds, reinterpret_cast<uint64_t*>(tiles), g.cap_lds, g.region_mask, g.flush, g.cap_hbm, g.trace,
                         g.n_wg, 4u >> g.group_log2, wg, g.group_log2);
  ring.collab = g.collab;
  if constexpr (REALTIME) kp::ring_use_realtime(ring);
  // (with wave groups the host adds 16 bytes behind the ring for the waves that do not record)
  if constexpr (SITE == 6) kp::chain_begin(ring, (uint32_t)(uintptr_t)ring_lds + (4u >> g.group_log2) * g.cap_lds * 8u);
  else kp::sites_begin<SITE>(ring);

  const uint32_t wr = wave >> 1, wc = wave & 1u;  // wave position in the 2x2 grid
  // operand layout of v_mfma_f32_32x32x16_bf16: lane l supplies row/column l%32, k = 8*(l/32)..+7
  uint32_t a_rd[4], b_rd;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const uint32_t r = wr * 32u + (lane & 31u), c = 2u * (uint32_t)ks + (lane >> 5);
    a_rd[ks] = r * 128u + ((c ^ ((r >> 1) & 7u)) << 4);
  }
  {
    const uint32_t bi = lane & 15u, bg = lane >> 4;
    const uint32_t k = 8u * (bg >> 1) + (bi >> 2), n = wc * 32u + 16u * (bg & 1u) + 4u * (bi & 3u);
    b_rd = A_BYTES + k * 128u + (((n >> 3) ^ (((k >> 1) & 1u) << 2)) << 4) + 8u * ((n >> 2) & 1u);
  }
  auto read_b = [&](const unsigned char* stage, int ks) -> bf16x8 {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
    const unsigned char* at = stage + b_rd + (uint32_t)(16 * ks) * 128u;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(at));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(at + 4u * 128u));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };
  f32x16 acc = {0};  // transposed tile (B^T as the first operand): a lane holds four consecutive columns of a C row
  store_a(0, 0);
  store_b(0, 0);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  KP_SITE_K(ring, 0, kp::kNoRegion, 0);
  // The site that closes a K step and opens the next one, if there is one.  (A chained site keeps its clock either way.)
  auto close = [&](bool last) __attribute__((always_inline)) {
    if constexpr (SITE == 6) KP_SITE_K(ring, 0, 2, 0);
    else if (last) KP_SITE_K(ring, 0, 2, kp::kNoRegion);
    else KP_SITE_K(ring, 0, 2, 0);
  };
  // One pair of K steps; the registers of pair p are set p % AHEAD.  TAIL: the pair or one requested here may be the last.
  auto pair_of_steps = [&](uint32_t pair, int set, auto tail_c) __attribute__((always_inline)) {
    constexpr bool TAIL = decltype(tail_c)::value;
    const uint32_t s = (uint32_t)set;  // LDS stage
    const unsigned char* stage = tiles + s * STAGE;
    bf16x8 af[4], bf[4];
    auto operands = [&](int first) __attribute__((always_inline)) {
#pragma unroll
      for (int i = first; i < first + 2; ++i) {
        af[i] = *reinterpret_cast<const bf16x8*>(stage + a_rd[i]);
        bf[i] = read_b(stage, i);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    // ---- region 0: the global loads of pair + AHEAD are issued -----------------------------------
    request_a(pair + AHEAD, set, tail_c);
    __builtin_amdgcn_sched_barrier(0);
    KP_SITE_K(ring, 1, 0, 1);
    // ---- region 1: the operands of this K step are requested from LDS, pair + 1 goes to the other stage
    // (if there is one).  The requests come first and stay on this side of the site: behind
    // it they would be waited for together with its clock (29 against 33 us with four workgroups, recorded).
    operands(0);
    if (!TAIL || pair + 1u < PAIRS) store_a(s ^ 1u, set ^ 1);
    KP_SITE_K(ring, 2, 1, 2);
    // ---- region 2: MFMA
#pragma unroll
    for (int i = 0; i < 2; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[i], af[i], acc, 0, 0, 0);
    KP_COMMIT(ring, 3);
    close(TAIL && 2u * pair + 1u >= KT);
    if (TAIL && 2u * pair + 1u >= KT) return;
    __builtin_amdgcn_sched_barrier(0);
    // ---- the same for the second K step; behind it the barrier after which the other stage may be read and this one
    // written
    request_b(pair + AHEAD, set, tail_c);
    __builtin_amdgcn_sched_barrier(0);
    KP_SITE_K(ring, 1, 0, 1);
    operands(2);
    if (!TAIL || pair + 1u < PAIRS) store_b(s ^ 1u, set ^ 1);
    KP_SITE_K(ring, 2, 1, 2);
#pragma unroll
    for (int i = 2; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[i], af[i], acc, 0, 0, 0);
    KP_COMMIT(ring, 3);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    close(TAIL && 2u * pair + 2u >= KT);
  };
  static_assert(AHEAD == 2, "the K loop is unrolled by two pairs");
  uint32_t pair = 0;
  for (; 2u * (pair + 5u) <= KT; pair += 2u) {  // (both pairs requested in an iteration have two K steps, and eight steps are not worth one)
    pair_of_steps(pair, 0, no);
    pair_of_steps(pair + 1u, 1, no);
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {  // at most five pairs are left; written out, so that the compiler waits for the loads it has to
    if (pair >= PAIRS) break;
    pair_of_steps(pair, 0, yes);
    if (pair + 1u >= PAIRS) break;
    pair_of_steps(pair + 1u, 1, yes);
    pair += 2u;
  }

  // (through the stage that the last pair does not read: with an odd number of K steps there is no barrier behind it)
  unsigned char* c_lds = tiles + (PAIRS & 1u) * STAGE + 2048u * wave;
  c_tile_to_lds(acc, c_lds);
  KP_COMMIT(ring, 1);  // the site that closed the last K step
  c_tile_to_memory(c_lds, g.C + (size_t)(m0 + wr * 32u) * g.N + n0 + wc * 32u, g.N);
  if constexpr (INSTR != 0) {
    kp::TraceGeom tg{g.n_wg, 4u >> g.group_log2, 3, g.cap_hbm, g.flags};
    if constexpr (SITE == 6) {
      kp::ring_finish<REALTIME>(ring, g.cap_lds, g.trace, tg, wg, g.rec_cost, SmallGemmChain{});
    } else {
      kp::sites_end<SITE>(ring);
      kp::ring_finish<REALTIME>(ring, g.cap_lds, g.trace, tg, wg, g.rec_cost);
    }
  }
}

// The same tile for a short K and many workgroups: one K step at a time, 8 KiB of LDS.  A workgroup is then over
// before a pipeline has filled, its time is latency and the C tile, and what counts is how many of them share a CU:
// eight or more here, five of the pipelined kernel's, three of those with a ring of 16 KiB.  Measured, this kernel /
// the pipelined one, us: 3906 workgroups K = 32 8.0 / 12.3, 160 16.7 / 18.6, 256 22.0 / 22.3, 288 23.3 / 24.1, 320 24.6 /
// 24.3; 8010 K = 288 46.6 / 45.6, 320 50.9 / 46.5; 2205 K = 192 12.0 / 11.7, 224 13.0 / 12.5; 1155 K = 32 4.9 / 5.5, 224
// 7.7 / 7.7; 1023 K = 160 5.9 / 5.9; 930 K = 160 6.0 / 6.0, 192 6.4 / 6.1; 675 K = 96 4.8 / 4.9, 128 5.1 / 4.9; 272 K = 96
// 4.8 / 4.8.  With all regions recorded: 3906 K = 32 11.8 / 17.5, 288 28.2 / 31.7, 320 29.4 / 31.2; 1155 K = 224 10.5 /
// 11.3; 1023 K = 32 5.7 / 6.7, 160 8.0 / 8.3, 224 9.1 / 9.2; 812 K = 32 5.3 / 6.3, 160 7.5 / 7.8; 506 K = 64 5.2 / 5.3, 128
// 5.6 / 5.7; 255 K = 32 4.9 / 4.9.  Where the pipelined kernel has come to be the faster one without sites it is not with them
// (without / all regions / 64-lane store): 2205 K = 192 11.7, 15.0, 19.6 against 11.0, 15.1, 22.9, K = 224 12.8, 16.2, 21.8 against 12.0,
// 16.2, 25.4; 8010 K = 256 38.9, 47.7, 69.1 against 37.8, 48.3, 80.7, K = 288 44.4, 53.3, 75.2 against 41.7, 55.8, 89.2.  (B in four-byte loads by half of the threads, transposed on its way to LDS, and C in
// two-byte stores: 3906 K = 32 9.2, 288 27.3.)  Hence short_k(): a line for one, three, four and
// twelve workgroups per CU, the same with and without sites, so that a recorded kernel and its baseline are one. Its
// sites follow one another as the pipelined kernel's do.
//
// LDS rows of 32 bf16: chunk c of row r at position c ^ (r / 2) % 4.
__device__ __forceinline__ uint32_t short_off(uint32_t row, uint32_t chunk) {
  return row * 64u + ((chunk ^ ((row >> 1) & 3u)) << 4);
}

template <int INSTR>
__global__ __launch_bounds__(256) void kp_gemm_short(GemmArgs g) {
  constexpr int SITE = (INSTR == 2 || INSTR == 5) ? 6 : INSTR;
  constexpr bool REALTIME = INSTR == 3 || INSTR == 5;
  constexpr int kMayCross = 0;
  constexpr int BM = 64, BN = 64, BK = 32;
  __shared__ __align__(16) unsigned char sA[BM * BK * 2];
  __shared__ __align__(16) unsigned char sB[BN * BK * 2];
  extern __shared__ __align__(16) uint32_t ring_lds[];
  __shared__ uint64_t t_begin[2];

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t tiles_n = g.N / BN;
  const uint32_t wg = blockIdx.x;
  const uint32_t m0 = (wg / tiles_n) * BM, n0 = (wg % tiles_n) * BN;
  kp::Ring ring{};
  if constexpr (INSTR != 0)
    ring = kp::ring_init<true>(ring_lds, t_begin, g.cap_lds, g.region_mask, g.flush, g.cap_hbm, g.trace, g.n_wg, 4u >> g.group_log2, wg,
                         g.group_log2);
  ring.collab = g.collab;
  if constexpr (REALTIME) kp::ring_use_realtime(ring);
  if constexpr (SITE == 6) kp::chain_begin(ring, (uint32_t)(uintptr_t)ring_lds + (4u >> g.group_log2) * g.cap_lds * 8u);
  else kp::sites_begin<SITE>(ring);

  // global -> register mapping
  // A: 64 rows x 4 chunks of 16 bytes, B: 32 rows x 8 chunks as they lie in memory, one of each per thread
  const uint32_t a_row = tid >> 2, a_chunk = tid & 3u, b_row = tid >> 3, b_chunk = tid & 7u;
  const uint16_t* a_src = g.A + (size_t)(m0 + a_row) * g.K + a_chunk * 8;
  const uint16_t* b_src = g.B + (size_t)b_row * g.N + n0 + b_chunk * 8;

  const uint32_t wr = wave >> 1, wc = wave & 1u;  // wave position in the 2x2 grid
  // B is transposed by the operand read, as in the pipelined kernel; chunk c of row k at position c ^ 4 (k / 2 % 2)
  const unsigned char* b_rd;
  {
    const uint32_t bi = lane & 15u, bg = lane >> 4;
    const uint32_t k = 8u * (bg >> 1) + (bi >> 2), n = wc * 32u + 16u * (bg & 1u) + 4u * (bi & 3u);
    b_rd = sB + k * 128u + (((n >> 3) ^ (((k >> 1) & 1u) << 2)) << 4) + 8u * ((n >> 2) & 1u);
  }
  f32x16 acc = {0};

  for (uint32_t kt = 0; kt < g.K / BK; ++kt) {
    // ---- region 0: global load ---------------------------------------------------------------
    if (kt == 0) KP_SITE_K(ring, 0, kp::kNoRegion, 0); else KP_SITE_K(ring, 0, 2, 0);
    const u32x4 av = *reinterpret_cast<const u32x4*>(a_src + (size_t)kt * BK);
    const u32x4 bv = *reinterpret_cast<const u32x4*>(b_src + (size_t)kt * BK * g.N);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    KP_SITE_K(ring, 1, 0, 1);
    // ---- region 1: LDS store -----------------------------------------------------------------
    __syncthreads();  // previous step's MFMA reads are done
    *reinterpret_cast<u32x4*>(sA + short_off(a_row, a_chunk)) = av;
    *reinterpret_cast<u32x4*>(sB + b_row * 128u + ((b_chunk ^ (((b_row >> 1) & 1u) << 2)) << 4)) = bv;
    __syncthreads();
    KP_SITE_K(ring, 2, 1, 2);
    // ---- region 2: MFMA ------------------------------------------------------------------------
    bf16x8 af[BK / 16], bf[BK / 16];
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      // operand layout of v_mfma_f32_32x32x16_bf16: lane l supplies row/column l%32, k = 8*(l/32)..+7
      typedef short s16x4 __attribute__((ext_vector_type(4)));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
      af[ks] = *reinterpret_cast<const bf16x8*>(sA + short_off(wr * 32 + (lane & 31u), (uint32_t)ks * 2u + (lane >> 5)));
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(b_rd + 16 * ks * 128));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(b_rd + (16 * ks + 4) * 128));
      const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      bf[ks] = __builtin_bit_cast(bf16x8, v);
    }
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[ks], af[ks], acc, 0, 0, 0);  // (transposed)
    asm volatile("s_nop 0" ::: "memory");
    KP_COMMIT(ring, 3);
  }
  KP_SITE_K(ring, 0, 2, kp::kNoRegion);

  __syncthreads();  // every wave is past its last operand read
  unsigned char* c_lds = (wave & 2u ? sB : sA) + 2048u * (wave & 1u);
  c_tile_to_lds(acc, c_lds);
  KP_COMMIT(ring, 1);  // the site that closed the last K step
  c_tile_to_memory(c_lds, g.C + (size_t)(m0 + wr * 32u) * g.N + n0 + wc * 32u, g.N);
  if constexpr (INSTR != 0) {
    kp::TraceGeom tg{g.n_wg, 4u >> g.group_log2, 3, g.cap_hbm, g.flags};
    if constexpr (SITE == 6) {
      kp::ring_finish<REALTIME>(ring, g.cap_lds, g.trace, tg, wg, g.rec_cost, SmallGemmChain{});
    } else {
      kp::sites_end<SITE>(ring);
      kp::ring_finish<REALTIME>(ring, g.cap_lds, g.trace, tg, wg, g.rec_cost);
    }
  }
}


// ------------------------------------------------------------------------------------------
// 256x256x64 tile, 8 waves as 2 (M) x 4 (N); each wave owns 128x64 of C as 4x2 MFMA tiles.
// LDS holds two stages of the A tile [256][64] and of the B tile (128 KiB); the K loop is software-pipelined
// over the two stages.  Default schedule: while the MFMAs consume stage s, the tiles of K step +1 travel from
// global memory straight to stage s^1 (no staging registers; B stays row-major and is transposed by the LDS
// read).  Stage-by-stage schedule: K step +1 moves from staging registers to the same places of stage s^1 and the global
// loads of K step +2 are in flight.
// MFMA operands are swapped (B^T rows as the first operand) so that a lane ends up with four
// consecutive columns of one C row per accumulator quad and puts them into LDS as 8 bytes, on their way to memory.
// (With 4 waves as 2 x 2, 128x128 of C each, accumulators in AGPRs and one wave per SIMD, an earlier form was no faster: a third
// less LDS read traffic and a short barrier, but a single wave per SIMD hides less.)
constexpr int kBigBM = 256, kBigBN = 256, kBigBK = 64, kBigWaves = 8;
constexpr uint32_t kBigTileBytes = 2u * (kBigBM + kBigBN) * kBigBK * 2u;  // both stages

template <int INSTR, int SCHEDULE>
__global__ __launch_bounds__(kBigWaves * 64) void kp_gemm_big(GemmArgs g) {
  // default schedule: vector, scalar and LDS-read instructions may be scheduled across a chained site; the
  // regions are halves of the K step's MFMAs, which stay on their side (stages apart: nothing crosses)
  constexpr int kMayCross = SCHEDULE == 0 ? 0x106 : 0;
  // SCHEDULE 0: staging threaded through the MFMAs; 1: the stages of a K step one after the other; 2: the
  // same source without the scheduling fences between the stages and behind the MFMAs (uninstrumented only)
  constexpr bool PHASED = SCHEDULE != 0;
  static_assert(SCHEDULE != 2 || INSTR == 0, "the unfenced stage-by-stage form has no record sites");
  // INSTR 2 and 5 (constant-rate clock): chained sites; 1 and 3 are the generic sites, which the flush
  // strategy and the 64-lane store need
  static_assert(INSTR != 4, "no such form");
  constexpr int SITE = (INSTR == 2 || INSTR == 5) ? 6 : INSTR;
  constexpr bool REALTIME = INSTR == 3 || INSTR == 5;
  constexpr int BM = kBigBM, BN = kBigBN, BK = kBigBK;
  constexpr int TN = 2;                    // 32-column MFMA tiles per wave (wave tile 128 x 64)
  constexpr int T = kBigWaves * 64;         // threads
  constexpr int NA = 2048 / T;              // A chunks per thread and K step
  constexpr uint32_t A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
  extern __shared__ __align__(16) unsigned char smem[];  // [stage0 A|B][stage1 A|B][ring]
  uint32_t* ring_lds = reinterpret_cast<uint32_t*>(smem + 2 * STAGE);

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t tiles_m = g.M / BM, tiles_n = g.N / BN;
  // Workgroups are dealt round-robin to the 8 XCDs; give every XCD a compact block of tiles
  // so that the A and B panels it streams stay in its own L2.
  uint32_t tile_r, tile_c;
  if ((tiles_m % 4u) == 0u && (tiles_n % 2u) == 0u) {
    const uint32_t xcd = blockIdx.x & 7u, j = blockIdx.x >> 3;
    const uint32_t br = tiles_m / 4u, bc = tiles_n / 2u;  // block of tiles per XCD
    tile_r = (xcd >> 1) * br + j / bc;
    tile_c = (xcd & 1u) * bc + j % bc;
  } else {
    tile_r = blockIdx.x / tiles_n;
    tile_c = blockIdx.x % tiles_n;
  }
  const uint32_t wg = tile_r * tiles_n + tile_c;  // recorded workgroup id = tile index
  const uint32_t m0 = tile_r * BM, n0 = tile_c * BN;

  kp::Ring ring{};
  if constexpr (INSTR != 0)
    ring = kp::ring_init<true>(ring_lds, reinterpret_cast<uint64_t*>(smem), g.cap_lds, g.region_mask, g.flush,
                         g.cap_hbm, g.trace, g.n_wg, (uint32_t)kBigWaves >> g.group_log2, wg, g.group_log2);
  ring.collab = g.collab;
  if constexpr (REALTIME) kp::ring_use_realtime(ring);
  // (with wave groups the host adds 16 bytes behind the ring for the waves that do not record)
  if constexpr (SITE == 6) kp::chain_begin(ring, (uint32_t)(uintptr_t)ring_lds + ((uint32_t)kBigWaves >> g.group_log2) * g.cap_lds * 8u);
  else kp::sites_begin<SITE>(ring);

  // ---- global -> register -> LDS mapping (stage-by-stage schedule) ---------------------------
  // Every thread stages the same share of a K step, so all waves reach the barrier together:
  //   A: 256 rows x 8 chunks of 16 bytes; thread t takes chunk (t & 7) of rows (t >> 3) + (T/8)*i;
  //   B: blocks of 4 k x 8 n, 16 x 32 of them; thread t takes block t (k quad t >> 5, n block
  //      t & 31) and stores its four rows (16 bytes) as they come; the operand reads transpose.
  //      (Transposed in registers, 16 v_perm_b32 and eight 8-byte stores of which every pass took two cycles,
  //      the LDS write stage took 911 ticks per K step of a 2048x4096x4096 launch instead of 775, and the launch 4 us more.)
  // Eight 16-byte global loads per thread and K step: vector-memory instructions are
  // issued at a fixed rate per CU whatever their width, so wide loads keep the issue time short.
  const uint32_t a_row = tid >> 3, a_chunk = tid & 7u;
  const uint16_t* src_a = g.A + (size_t)(m0 + a_row) * g.K + a_chunk * 8;
  uint32_t a_dst[NA];  // LDS byte offsets inside a stage
#pragma unroll
  for (int i = 0; i < NA; ++i) a_dst[i] = tile_off<BK>(a_row + (T / 8) * i, a_chunk);
  const uint32_t b_nb = tid & 31u;
  uint32_t b_dst[4];  // row i of the block: k = 4 (k quad) + i, chunk nb at position nb ^ 4 (k % 4)
#pragma unroll
  for (int i = 0; i < 4; ++i) b_dst[i] = A_BYTES + (4u * (tid >> 5) + (uint32_t)i) * 512u + ((b_nb ^ (4u * (uint32_t)i)) << 4);
  const uint16_t* src_b = g.B + (size_t)((tid >> 5) * 4) * g.N + n0 + b_nb * 8;

  u32x4 la[NA], lb[4];  // staging registers: A chunks, B rows
  auto load_a = [&](uint32_t kt, int i) {
    la[i] = *reinterpret_cast<const u32x4*>(src_a + (size_t)kt * BK + (size_t)((T / 8) * i) * g.K);
  };
  auto load_b = [&](uint32_t kt, int i) {
    lb[i] = *reinterpret_cast<const u32x4*>(src_b + ((size_t)kt * BK + (size_t)i) * g.N);
  };
  auto store_a = [&](uint32_t stage, int i) {
    *reinterpret_cast<u32x4*>(smem + stage * STAGE + a_dst[i]) = la[i];
  };
  auto store_b = [&](uint32_t stage, int i) {
    *reinterpret_cast<u32x4*>(smem + stage * STAGE + b_dst[i]) = lb[i];
  };

  // ---- global -> LDS (default schedule) ------------------------------------------------------
  // The A tile goes from global memory straight to LDS (global_load_lds_dwordx4: lane l of
  // a wave lands at byte 16 l of a 1 KiB block whose base M0 holds), without staging registers and LDS write
  // instructions.  Wave w fills blocks 4 w .. 4 w + 3 of a stage's A tile, 8 rows each: lane l is row l / 8 of
  // the block and chunk position l % 8, and fetches the chunk that the tile's swizzle puts there.  The loads
  // are issued from inline assembly: the compiler would make the next LDS access of any kind wait for such a
  // load (it cannot tell the load's destination from the tile being read).  They are therefore not in its
  // count of outstanding vector-memory operations; they complete in order with the others, so its own waits
  // stay sufficient (they may wait for more), and the kernel waits for them itself before the barrier.
  constexpr bool DIRECT = !PHASED;
  const uint32_t d_lds0 = kp::wave_uniform((uint32_t)(uintptr_t)smem + 4096u * wave);
  uint32_t d_off[4];  // byte offsets from the tile's first element (the base stays in scalar registers)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t row = 32u * wave + 8u * (uint32_t)i + (lane >> 3);
    const uint32_t chunk = (lane & 7u) ^ ((row >> 1) & 7u);  // tile_off<64>: position = chunk ^ (row / 2) % 8
    d_off[i] = (row * g.K + chunk * 8u) * 2u;
  }
  const uint16_t* a_base = g.A + (size_t)m0 * g.K;
  // The B tile likewise, as it lies in memory: 64 rows (k) of 256 n, 512 bytes each; chunk c (8 n) of row k at
  // chunk position c ^ 4 (k % 4).  Wave w fills blocks 4 w .. 4 w + 3 of 1 KiB, two rows each.
  uint32_t db_off[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t row = 8u * wave + 2u * (uint32_t)i + (lane >> 5);
    const uint32_t chunk = (lane & 31u) ^ (4u * (row & 3u));
    db_off[i] = (row * g.N + chunk * 8u) * 2u;
  }
  const uint16_t* b_base = g.B + n0;
  // One load, its global address a scalar base (the tile's first element in this K step) plus the lane's 32-bit
  // byte offset, which never changes: no vector arithmetic per load (with a 64-bit pointer per lane and load
  // the kernel was 3.5 % slower).  M0 (the LDS base) is put back afterwards, the compiler does not expect
  // inline assembly to change it; one wait state between the write of M0 and the load that uses it.  The eight loads of a K step stay
  // separate statements: issued back to back from one block of assembly they made the uninstrumented kernel 4 %
  // slower (the address arithmetic of the next load no longer sits between two loads).
  auto direct_load = [&](const uint16_t* base, uint32_t off, uint32_t dst) {
    uint32_t saved_m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved_m0) : "v"(off), "s"(dst), "s"(base) : "memory");
  };
  auto direct_one = [&](uint32_t kt, uint32_t stage, int idx) {
    const uint32_t dst = d_lds0 + stage * STAGE;
    if (idx < 4) direct_load(a_base + (size_t)kt * BK, d_off[idx], dst + (uint32_t)idx * 1024u);
    else direct_load(b_base + (size_t)kt * BK * g.N, db_off[idx - 4], dst + A_BYTES + (uint32_t)(idx - 4) * 1024u);
  };
  auto direct_tiles = [&](uint32_t kt, uint32_t stage) {
    const uint32_t dst = d_lds0 + stage * STAGE;
#pragma unroll
    for (int i = 0; i < 4; ++i) direct_load(a_base + (size_t)kt * BK, d_off[i], dst + (uint32_t)i * 1024u);
#pragma unroll
    for (int i = 0; i < 4; ++i) direct_load(b_base + (size_t)kt * BK * g.N, db_off[i], dst + A_BYTES + (uint32_t)i * 1024u);
  };

  const uint32_t wm = wave >> 2, wn = wave & 3u;  // wave position: 2 x 4
  // Operand reads of the row-major B tile: ds_read_b64_tr_b16 hands lane j of a group of 16 lanes the elements
  // j, 16 + j, 32 + j, 48 + j of the 64 that the group's lanes address (4 each, lane after lane).  With lane i
  // of a group addressing B[k0 + i / 4][n0 + 4 (i % 4) ..+3], lane j receives B[k0 .. k0 + 3][n0 + j]: four
  // consecutive k of one column; two such reads make the eight k of the lane's MFMA operand.  Groups 0 and 1 are
  // columns 0-15 and 16-31 of the k octet 0, groups 2 and 3 the same columns of octet 1.
  uint32_t b_rd[TN];
  {
    const uint32_t bi = lane & 15u, bg = lane >> 4;
    const uint32_t k = 8u * (bg >> 1) + (bi >> 2);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      const uint32_t n = wn * (32 * TN) + (uint32_t)tn * 32u + 16u * (bg & 1u) + 4u * (bi & 3u);
      b_rd[tn] = k * 512u + ((((n >> 3) ^ (4u * (bi >> 2)))) << 4) + 8u * ((n >> 2) & 1u);
    }
  }
  auto read_b = [&](const unsigned char* sBt, int ks, int tn) -> bf16x8 {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
    const unsigned char* at = sBt + b_rd[tn] + (uint32_t)(16 * ks) * 512u;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(at));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(at + 4u * 512u));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };

  f32x16 acc[TN][4];                               // [tn][tm], transposed tiles (rows = n, cols = m)
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f32x16{0};

  // prologue: K step 0 into stage 0 (and, stage by stage, K step 1 into the staging registers)
  const uint32_t KT = g.K / BK;
  if constexpr (DIRECT) {
    static_assert(kBigWaves == 8 && BK == 64, "four 1 KiB blocks of either tile per wave");
    direct_tiles(0, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the tiles of K step 0 have landed
  } else {
#pragma unroll
    for (int i = 0; i < NA; ++i) load_a(0, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_b(0, i);
#pragma unroll
    for (int i = 0; i < NA; ++i) store_a(0, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) store_b(0, i);
    if (KT > 1) {
#pragma unroll
      for (int i = 0; i < NA; ++i) load_a(1, i);
#pragma unroll
      for (int i = 0; i < 4; ++i) load_b(1, i);
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

  // Default schedule.  Iteration kt runs the MFMAs of K step kt on LDS stage kt & 1.  It starts by sending
  // both tiles of K step kt+1 from global memory to the other stage, eight loads per wave that have the whole
  // iteration to land; the wave waits for them, and for its LDS reads, right before the barrier.  The operands
  // of MFMA step ks+1 are requested before the MFMAs of step ks are issued, and the MFMAs of a K step's last
  // step are issued behind the barrier, after the loads and the first operand reads of the next iteration:
  // a wave comes back from the barrier with matrix work at hand while the first operands of the new stage
  // are on their way.
  // MORE (K step kt+1 exists) is compile-time so that the steady-state body is one basic block.
  // operands of the last MFMA step of a K step: its MFMAs are issued behind the barrier, in the next iteration
  bf16x8 af_p[4], bf_p[TN];
#pragma unroll
  for (int i = 0; i < 4; ++i) af_p[i] = bf16x8{0};
#pragma unroll
  for (int i = 0; i < TN; ++i) bf_p[i] = bf16x8{0};
  constexpr int kLoadEvery = 2;  // (measured: 1 and 3 are 3 to 7 % slower)
  auto mfma_pending = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < 4; ++tm)
        acc[tn][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf_p[tn], af_p[tm], acc[tn][tm], 0, 0, 0);
  };
  auto iteration = [&](uint32_t kt, auto more_c, auto more2_c) {
    constexpr bool MORE = decltype(more_c)::value;
    const uint32_t stage = kt & 1u;
    const unsigned char* sA = smem + stage * STAGE;
    const unsigned char* sB = sA + A_BYTES;
    // operands of MFMA step ks + 1 are requested before the MFMAs of step ks are issued
    bf16x8 af[2][4], bfr[2][TN];
    auto read_step = [&](int ks, int buf) __attribute__((always_inline)) {
      const uint32_t chunk = (uint32_t)ks * 2u + (lane >> 5);
#pragma unroll
      for (int tm = 0; tm < 4; ++tm)
        af[buf][tm] = *reinterpret_cast<const bf16x8*>(sA + tile_off<BK>(wm * 128 + tm * 32 + (lane & 31u), chunk));
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) bfr[buf][tn] = read_b(sB, ks, tn);
    };
    // load d of the next K step's tiles goes behind MFMA kLoadEvery * d + kLoadEvery - 1 of the iteration's 32
    auto load_behind = [&](uint32_t kt_, uint32_t stage_, int mfma) __attribute__((always_inline)) {
      if (mfma % kLoadEvery == kLoadEvery - 1 && mfma / kLoadEvery < 8) {
        __builtin_amdgcn_sched_barrier(0);
        direct_one(kt_ + 1, stage_ ^ 1u, mfma / kLoadEvery);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    read_step(0, 0);
    // the last MFMA step of the K step before (zeros the first time).  The loads of the next K step's tiles go
    // behind every second MFMA of the first sixteen: the loads of all waves queue up in one unit of the CU, and a
    // wave that issues its eight in a row waits there with no matrix work in flight; spread further, the last
    // ones land too late
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < 4; ++tm) {
        acc[tn][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf_p[tn], af_p[tm], acc[tn][tm], 0, 0, 0);
        if constexpr (MORE) load_behind(kt, stage, tn * 4 + tm);
      }
    KP_COMMIT(ring, 3);  // the sites of the K step before: in its middle, in front of its barrier and behind it
#pragma unroll
    for (int ks = 0; ks + 1 < BK / 16; ++ks) {
      // ---- region 0: first half of the K step; region 1: second half
      if (ks == 1) KP_SITE_K(ring, 0, 0, 1);  // 16 MFMAs on either side
      read_step(ks + 1, (ks + 1) & 1);
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < 4; ++tm) {
          acc[tn][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ks & 1][tn], af[ks & 1][tm], acc[tn][tm], 0, 0, 0);
          if constexpr (MORE) load_behind(kt, stage, 8 * (ks + 1) + tn * 4 + tm);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) af_p[i] = af[(BK / 16 - 1) & 1][i];
#pragma unroll
    for (int i = 0; i < TN; ++i) bf_p[i] = bfr[(BK / 16 - 1) & 1][i];
    // the tiles of the next K step have landed (no other vector-memory operation is in flight in the loop)
    if constexpr (MORE) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    KP_SITE_K(ring, 1, 1, 2);
    // ---- region 2: every wave is done with the stage ----------------------------------------------
    // (chained sites: nothing behind the barrier uses the clock just asked for, so nothing waits for it there)
    if constexpr (SITE == 1 || SITE == 3) asm volatile("s_barrier\n\ts_waitcnt lgkmcnt(0)" ::: "memory");
    else asm volatile("s_barrier" ::: "memory");
    if constexpr (MORE) KP_SITE_K(ring, 2, 2, 0); else KP_SITE_K(ring, 2, 2, 3);
  };
  // The same K step with its stages one after the other, each a region of its own (the stage-by-stage
  // instrumentation of a software-pipelined GEMM, Sec. 5.3): 2 the staging registers (K step kt+1) go to
  // the other LDS stage, 0 the global loads of K step kt+2 are issued, 3 the MFMAs of K step kt, 1 the
  // wait for this wave's LDS traffic and for the other waves.  Four sites and eight records per K step.
  // With all waves behind one barrier in one order the LDS writes (800 cycles of the CU), the loads (1024 of its one unit) and
  // the MFMAs (2112 of a SIMD) of a K step add up to 3380 ticks.  Waves 4 to 7 half a K step behind (write, load, barrier, MFMAs)
  // take 2048x4096x4096 recorded from 101.4 to 93.3 us, without sites 117.8 -> 116.8 at 4096x4096x4096; but their barrier then
  // stands where region 0 meets region 3, and a wave's wait would count to its loads.
  // A record site pins its place in the instruction stream (it is a scheduling fence: nothing moves across
  // the clock read).  Without sites the compiler would be free to thread the stages through one another
  // again, and "the same schedule without record sites" would be another schedule: so the uninstrumented form has
  // a bare scheduling fence wherever the instrumented one has a site, and both have one behind every MFMA, which keeps
  // the operand requests where they are written.  SCHEDULE 2 leaves all of them out, for that comparison: at
  // 4096x4096x4096 128 us, 123 with the fences, 130 with the sites.
  auto stage_fence = [] { if constexpr (INSTR == 0 && SCHEDULE == 1) __builtin_amdgcn_sched_barrier(0); };
  auto iteration_phased = [&](uint32_t kt, auto more_c, auto more2_c) {
    constexpr bool MORE = decltype(more_c)::value, MORE2 = decltype(more2_c)::value;
    const uint32_t stage = kt & 1u;
    const unsigned char* sA = smem + stage * STAGE;
    const unsigned char* sB = sA + A_BYTES;
    if constexpr (MORE) {
#pragma unroll
      for (int i = 0; i < NA; ++i) store_a(stage ^ 1u, i);
#pragma unroll
      for (int i = 0; i < 4; ++i) store_b(stage ^ 1u, i);
    }
    KP_SITE_K(ring, 1, 2, 0);
    stage_fence();
    if constexpr (MORE2) {
#pragma unroll
      for (int i = 0; i < NA; ++i) load_a(kt + 2, i);
#pragma unroll
      for (int i = 0; i < 4; ++i) load_b(kt + 2, i);
    }
    KP_SITE_K(ring, 2, 0, 3);
    stage_fence();
    // The operands of MFMA step ks + 1 are requested between the MFMAs of step ks, in the order of their use: the stage
    // takes 1227 ticks of a wave (32 MFMAs alone: 1056).  All of a step's ahead of the step before's MFMAs 1456, ahead of
    // its own MFMAs 1313; 2048x4096x4096 recorded 106, 117.5 and 117 us.
    bf16x8 af[2][4], bfr[2][TN];
    auto read_operand = [&](int ks, int which) __attribute__((always_inline)) {
      if (which < TN) bfr[ks & 1][which] = read_b(sB, ks, which);
      else if (which < TN + 4)
        af[ks & 1][which - TN] = *reinterpret_cast<const bf16x8*>(
            sA + tile_off<BK>(wm * 128 + (which - TN) * 32 + (lane & 31u), (uint32_t)ks * 2u + (lane >> 5)));
    };
#pragma unroll
    for (int which = 0; which < TN + 4; ++which) read_operand(0, which);
    if constexpr (SCHEDULE == 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
#pragma unroll
      for (int tm = 0; tm < 4; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
          acc[tn][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ks & 1][tn], af[ks & 1][tm], acc[tn][tm], 0, 0, 0);
          if (ks + 1 < BK / 16) read_operand(ks + 1, TN * tm + tn);
          if constexpr (SCHEDULE == 1) __builtin_amdgcn_sched_barrier(0);
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (nothing of this wave's is in flight any more: see above)
    KP_SITE_K(ring, 3, 3, 1);
    stage_fence();
    asm volatile("s_barrier\n\ts_waitcnt lgkmcnt(0)" ::: "memory");
    KP_COMMIT(ring, 4);
    if constexpr (MORE) KP_SITE_K(ring, 0, 1, 2); else KP_SITE_K(ring, 0, 1, 4);
    stage_fence();
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  if constexpr (PHASED) {
    KP_SITE_K(ring, 0, kp::kNoRegion, 2);
    for (uint32_t kt = 0; kt + 2 < KT; ++kt) iteration_phased(kt, yes, yes);
    if (KT >= 2) iteration_phased(KT - 2, yes, no);
    iteration_phased(KT - 1, no, no);
  } else {
    if constexpr (SITE == 6) {  // (they fill the first two places of the first batch)
      kp::site_chain<0, REALTIME>(ring);
      kp::site_chain<1, REALTIME>(ring);
    }
    KP_SITE_K(ring, 2, kp::kNoRegion, 0);
    for (uint32_t kt = 0; kt + 2 < KT; ++kt) iteration(kt, yes, yes);
    if (KT >= 2) iteration(KT - 2, yes, no);
    iteration(KT - 1, no, no);
    mfma_pending();
    KP_COMMIT(ring, 3);
  }

  // ---- region 3 (4 with the stages apart): epilogue ---------------------------------------------------
  // transposed tile: register v of lane l is C[m, n] with m = l%32 and n = 8*(v/4) + 4*(l/32) + v%4.  The lanes of a
  // wave hold 16 bytes of 32 rows side by side, so the wave's 128 x 64 of C go through 16 KiB of LDS (every wave is past
  // its last operand read) and leave as whole 128-byte lines.  A row is eight chunks of 16 bytes; chunk c of row r at
  // position c ^ r % 8, its halves swapped where r / 8 is odd: 16 lanes of an 8-byte write hit all banks once.  Stored from the registers, the
  // epilogue took 13500 ticks of a 4096x4096x4096 launch, all regions recorded (118 us); it takes 3900 (111 us).
  {
    unsigned char* sC = smem + 16384u * wave;
    const uint32_t r = lane & 31u, half = (lane >> 5) ^ ((r >> 3) & 1u);
#pragma unroll
    for (int tm = 0; tm < 4; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          u32x2 pk;
          pk.x = bf16_pack_rne(acc[tn][tm][4 * q + 0], acc[tn][tm][4 * q + 1]);
          pk.y = bf16_pack_rne(acc[tn][tm][4 * q + 2], acc[tn][tm][4 * q + 3]);
          *reinterpret_cast<u32x2*>(sC + (32u * (uint32_t)tm + r) * 128u + ((((uint32_t)(4 * tn + q)) ^ (r & 7u)) << 4) + 8u * half) = pk;
        }
    // lane l of store i: row 8 i + l / 8, chunk position l % 8
    const uint32_t rr = lane >> 3, chunk = (lane & 7u) ^ rr;
    uint16_t* c_at = g.C + (size_t)(m0 + wm * 128 + rr) * g.N + n0 + wn * (32 * TN) + 8u * chunk;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(sC + 1024u * (uint32_t)i + 16u * lane);
      *reinterpret_cast<u32x4*>(c_at + (size_t)(8 * i) * g.N) = (i & 1) ? u32x4{v.z, v.w, v.x, v.y} : v;
    }
  }
  KP_SITE_K(ring, PHASED ? 1 : 0, PHASED ? 4 : 3, kp::kNoRegion);
  if constexpr (INSTR != 0) {
    kp::TraceGeom tg{g.n_wg, (uint32_t)kBigWaves >> g.group_log2, PHASED ? 5u : 4u, g.cap_hbm, g.flags};
    if constexpr (SITE == 6) {
      // the site that closed the epilogue and, with the stages apart, the one that opened it
      kp::chain_commit<PHASED ? 2 : 1>(ring);
      kp::ring_finish<REALTIME>(ring, g.cap_lds, g.trace, tg, wg, g.rec_cost, GemmChain<PHASED>{});
    } else {
      kp::sites_end<SITE>(ring);
      kp::ring_finish<REALTIME>(ring, g.cap_lds, g.trace, tg, wg, g.rec_cost);
    }
  }
}

}  // namespace

// ------------------------------------------------------------------------------------------
namespace {

struct GemmShape { int bm, bn, bk, waves, regions; };

bool pick_shape(int M, int N, int K, GemmShape* s) {
  if (M <= 0 || N <= 0 || K <= 0) return false;
  // the large tile only pays off once there are enough tiles to spread over the chip
  if (M % 256 == 0 && N % 256 == 0 && K % 64 == 0 && (M / 256) * (N / 256) >= 16) { *s = GemmShape{256, 256, 64, kBigWaves, 4}; return true; }
  if (M % 64 == 0 && N % 64 == 0 && K % 32 == 0) { *s = GemmShape{64, 64, 32, 4, 3}; return true; }
  return false;
}

// see kp_gemm_short
bool short_k(int K, int n_wg) { return K <= (n_wg >= 3072 ? 288 : n_wg >= 1024 ? 224 : n_wg > 768 ? 160 : n_wg > 256 ? 96 : 0); }

template <int INSTR, int SCHEDULE>
kp_status launch_big(const GemmArgs& g, int n_wg, size_t ring_bytes, hipStream_t st) {
  static thread_local int attr_dev = -1;  // the attribute is kept per device
  int dev = 0;
  KP_HIP_TRY(hipGetDevice(&dev));
  if (attr_dev != dev) {
    KP_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kp_gemm_big<INSTR, SCHEDULE>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    attr_dev = dev;
  }
  hipLaunchKernelGGL((kp_gemm_big<INSTR, SCHEDULE>), dim3(n_wg), dim3(kBigWaves * 64), kBigTileBytes + ring_bytes, st, g);
  KP_HIP_TRY(hipGetLastError());
  return KP_OK;
}

template <int INSTR>
kp_status launch_big_w(bool phased, const GemmArgs& g, int n_wg, size_t ring_bytes, hipStream_t st) {
  return phased ? launch_big<INSTR, 1>(g, n_wg, ring_bytes, st)
                : launch_big<INSTR, 0>(g, n_wg, ring_bytes, st);
}

}  // namespace

extern "C" kp_status kp_gemm_launch_shape(int M, int N, int K, int* n_wg, int* waves_per_wg, int* n_regions) {
  kp::clear_error();
  GemmShape s;
  if (!pick_shape(M, N, K, &s))
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "GEMM %dx%dx%d: M,N must be multiples of 64 and K of 32", M, N, K);
  if (n_wg) *n_wg = (M / s.bm) * (N / s.bn);
  if (waves_per_wg) *waves_per_wg = s.waves;
  if (n_regions) *n_regions = s.regions;
  return KP_OK;
}

extern "C" kp_status kp_gemm_instrumented(const void* A, const void* B, void* C, int M, int N, int K,
                                          uint32_t region_mask, void* trace_buf, size_t trace_cap,
                                          void* stream) {
  kp::clear_error();
  if (!A || !B || !C) return kp::fail(KP_ERR_INVALID_ARG, "NULL matrix pointer");
  GemmShape s;
  if (!pick_shape(M, N, K, &s))
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "GEMM %dx%dx%d: M,N must be multiples of 64 and K of 32", M, N, K);
  if (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) & 15u) return kp::fail(KP_ERR_INVALID_ARG, "A, B, C must be 16-byte aligned");
  const uint32_t regions = region_mask & ~(KP_MASK_FLUSH | KP_MASK_WAVE_GROUP | KP_MASK_PHASES | KP_MASK_REALTIME | KP_MASK_COLLAB | KP_MASK_UNFENCED);
  const bool unfenced = (region_mask & KP_MASK_UNFENCED) != 0u;
  const bool realtime = (region_mask & KP_MASK_REALTIME) != 0u, collab = (region_mask & KP_MASK_COLLAB) != 0u;
  const bool phased = (region_mask & KP_MASK_PHASES) != 0u;
  if (phased) {
    if (s.bm != 256) return kp::fail(KP_ERR_INVALID_ARG, "KP_MASK_PHASES: only the 256x256x64 kernel has the stage-by-stage K step");
    s.regions = 5;
  }
  if (unfenced && (!phased || regions != 0u))
    return kp::fail(KP_ERR_INVALID_ARG, "KP_MASK_UNFENCED goes with KP_MASK_PHASES and no region");
  const uint32_t flush = region_mask >> 31;
  const uint32_t group_log2 = (region_mask & KP_MASK_WAVE_GROUP) ? 2u : 0u;
  const int streams = s.waves >> group_log2;
  const int n_wg = (M / s.bm) * (N / s.bn);
  hipStream_t st = static_cast<hipStream_t>(stream);
  GemmArgs g{};
  g.A = static_cast<const uint16_t*>(A); g.B = static_cast<const uint16_t*>(B); g.C = static_cast<uint16_t*>(C);
  g.M = (uint32_t)M; g.N = (uint32_t)N; g.K = (uint32_t)K;
  g.region_mask = regions; g.trace = trace_buf; g.n_wg = (uint32_t)n_wg; g.flush = flush;
  g.group_log2 = group_log2;
  g.collab = collab ? 1u : 0u;
  g.flags = (flush ? KP_FLAG_FLUSH : 0u) | (realtime ? KP_FLAG_REALTIME : 0u) | (collab ? KP_FLAG_HW_IDS : 0u);
  const bool big = s.bm == 256;
  if (regions == 0) {  // uninstrumented baseline: no ring, no record sites
    if (big && unfenced) return launch_big<0, 2>(g, n_wg, 0, st);
    if (big) return launch_big_w<0>(phased, g, n_wg, 0, st);
    if (short_k(K, n_wg)) hipLaunchKernelGGL(kp_gemm_short<0>, dim3(n_wg), dim3(256), 0, st, g);
    else hipLaunchKernelGGL(kp_gemm_small<0>, dim3(n_wg), dim3(256), 0, st, g);
    KP_HIP_TRY(hipGetLastError());
    return KP_OK;
  }
  if (!trace_buf) return kp::fail(KP_ERR_INVALID_ARG, "trace_buf is NULL but region_mask enables regions");
  if (regions >> s.regions) return kp::fail(KP_ERR_INVALID_ARG, "region_mask enables regions this kernel does not have (%d regions)", s.regions);
  if (((uintptr_t)trace_buf) & 15u) return kp::fail(KP_ERR_INVALID_ARG, "trace_buf must be 16-byte aligned");
  if (trace_cap % (size_t)streams) return kp::fail(KP_ERR_TRACE_TOO_SMALL, "trace_cap must be a multiple of %d record streams", streams);
  const size_t cap_wave = trace_cap / (size_t)streams;
  if (!kp::is_pow2(cap_wave) || cap_wave < 2 || cap_wave > (1u << 19))
    return kp::fail(KP_ERR_TRACE_TOO_SMALL, "trace_cap/streams = %zu must be a power of two >= 2", cap_wave);
  uint32_t cap_lds = (uint32_t)cap_wave;
  if (flush && cap_lds > 64) cap_lds = 64;
  const size_t ring_bytes = (size_t)cap_lds * 8 * streams + (group_log2 ? 16 : 0);  // (16: see chain_begin)
  if (ring_bytes > 32 * 1024) return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "LDS ring of %zu bytes exceeds the 32 KiB budget", ring_bytes);
  g.cap_lds = cap_lds; g.cap_hbm = (uint32_t)cap_wave; g.rec_cost = kp::rec_cost();
  // The sites are chained whenever the strategy is circular and one lane stores: the region mask, wave-group records
  // and the constant-rate clock all keep that form.
  const bool chained = !flush && !collab;
  if (big) return chained ? (realtime ? launch_big_w<5>(phased, g, n_wg, ring_bytes, st) : launch_big_w<2>(phased, g, n_wg, ring_bytes, st))
                          : (realtime ? launch_big_w<3>(phased, g, n_wg, ring_bytes, st) : launch_big_w<1>(phased, g, n_wg, ring_bytes, st));
  const bool short_kernel = short_k(K, n_wg);
  auto kern = chained ? (realtime ? (short_kernel ? kp_gemm_short<5> : kp_gemm_small<5>) : (short_kernel ? kp_gemm_short<2> : kp_gemm_small<2>))
                      : (realtime ? (short_kernel ? kp_gemm_short<3> : kp_gemm_small<3>) : (short_kernel ? kp_gemm_short<1> : kp_gemm_small<1>));
  hipLaunchKernelGGL(kern, dim3(n_wg), dim3(256), ring_bytes, st, g);
  KP_HIP_TRY(hipGetLastError());
  return KP_OK;
}
