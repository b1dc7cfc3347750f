// Instrumented bf16 attention forward (kp_attn_instrumented): O = softmax(scale * Q K^T + mask) V,
// fp32 softmax and accumulation, head dimension 128, optional causal mask.
//
// The paper's case study profiles a flash-attention kernel whose regions are the two GEMMs and
// the softmax of every KV iteration (Sec. 5.2, Table 3: GEMM0 = Q K^T, softmax, GEMM1 = P V).
// This is the library's own MFMA kernel with the same three regions per KV tile of 64:
//   region 0  S^T = K Q^T     (MFMA), with the eight loads that send this wave's share of the next V and the next K
//             tile from global memory straight to LDS threaded in, and mask and maximum of the tile's lower 32 keys
//   region 1  online softmax   (VALU, fp32): what is left of it
//   region 2  O^T += V^T P^T   (MFMA; V is transposed by the LDS read); closes behind the barrier that follows it
// One workgroup = 4 waves = 128 query rows of one (batch, head); each wave owns 32 rows.  The
// products are formed transposed so that a lane holds all scores of ONE query row: the row
// maximum and sum are then in-lane reductions plus one exchange with the lane 32 away, and the
// rescaling of the output accumulators is a per-lane multiply.
//
// What bounds it: with two workgroups per CU the chip's power (0.97-1.03 PFLOP/s at some 1.5 GHz; the matrix pipes want
// 1056 cycles per wave and KV tile, the vector ALU about 800, and the two overlap only in part: a probe with an MFMA, four
// FMAs and two exponentials per step and two waves per SIMD takes 43 cycles a step where either kind alone takes 33 and
// 31).  With one, the rate at which a single wave issues: 6 cycles per vector instruction, 14 per exponential, some 330
// instructions per KV tile.  So every instruction counts, and every operand is requested eight (K) or four (V) MFMAs ahead
// in an order that the scheduling fences hold: left to itself the compiler reads the operands of one step, waits for them,
// multiplies.  4 x 32 x 4096, causal, all regions recorded 639 -> 550 us (541 with O as below); 1 x 12 x 1152, 108 workgroups 27.4 -> 24.3 us (21.8);
// 2 x 9 x 1920, causal 52 -> 38 us (half of which is the order of the workgroups).  Exponentials threaded between the
// MFMAs of either product, all or a part of them: within 1 % of this form, and region 1 no longer the softmax.  O goes
// through LDS and leaves as whole rows: 4 x 32 x 384 16.6 -> 14.6 us, 1 x 12 x 1152 24.2 -> 23.1, 4 x 32 x 4096 1-2 %.
#include <type_traits>

#include "kp_common.h"
#include "kp_record.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct AttnArgs {
  const uint16_t* Q;
  const uint16_t* K;
  const uint16_t* V;
  uint16_t* O;
  uint32_t B, H, S;
  uint32_t causal;
  float scale_log2;  // scale * log2(e)
  uint32_t region_mask;
  void* trace;
  uint32_t cap_lds, cap_hbm, flush, n_wg;
  uint32_t rec_cost;  // ticks the decoder takes off every duration (kp_set_rec_cost)
  uint32_t group_log2;  // 2^group_log2 waves share one record stream
  uint32_t collab;      // 1: all lanes store a record, hardware ids go to the workgroup header
  uint32_t flags;       // kp_trace_hdr.flags of the trace
};

constexpr int kD = 128, kBq = 128, kBkv = 64, kAttnThreads = 256;
constexpr uint32_t kRow = kD * 2;             // a row of either tile: one kv, 128 d, 256 bytes in 16 chunks of 16
constexpr uint32_t kKBytes = kBkv * kRow;     // K tile [64 kv][128 d]
constexpr uint32_t kVBytes = kBkv * kRow;     // V tile [64 kv][128 d], as it lies in memory
constexpr int kNoLoads = 0x0F70;              // s_waitcnt vmcnt(0), the other counters as they are
constexpr float kSlack = 8.0f;                // log2 of how far a score may exceed the softmax reference

// two fp32 -> packed bf16 pair (lo in bits 15:0), round to nearest even: one v_cvt_pk_bf16_f32
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pack_rne(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// The larger of a lane's value and that of the lane 32 away.
__device__ __forceinline__ float either_half_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x), false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}

// Both tiles go from global memory straight to LDS (global_load_lds_dwordx4: lane l of a wave lands at byte
// 16 l of a 1 KiB block, i.e. of four rows), so a tile's layout is a permutation of the 16 chunks inside each
// row, which the loading lane applies by fetching the chunk that belongs at its place.
// K tile: chunk c of row kv at position c ^ (kv % 16): the 16-byte operand reads of 16 neighbouring rows (one
// pass of a 16-byte LDS read) cover all banks.
// V tile: chunk c of row kv at position c ^ 4 (kv % 4).  Its operand reads transpose: ds_read_b64_tr_b16 hands
// lane j of a group of 16 lanes the elements j, 16 + j, 32 + j, 48 + j of the 64 that the group's lanes address
// (4 each), so with lane i addressing V[kv0 + i / 4][d0 + 4 (i % 4) ..+3] lane j receives V[kv0 .. kv0 + 3][d0 + j];
// the XOR spreads the four rows and two column groups of a pass over all banks.

// END of one region and/or START of the next with a single clock sample.  INSTR: 0 no record sites,
// 1 generic sites (region mask, either buffer strategy, either store), 3 the same on the constant-rate clock,
// 4 chained sites (circular strategy, one lane stores; region mask and wave-group records included: the loop
// keeps only the clocks and the records are made when the trace is copied out), 5 chained, constant-rate clock.
#define KP_BOUNDARY(ring, end_r, start_r) do { if constexpr (INSTR == 1 || INSTR == 3) kp::site<INSTR>(ring, end_r, start_r); } while (0)
#define KP_CHAIN(K, ring) do { if constexpr (INSTR >= 4) kp::site_chain<K, (INSTR == 5)>(ring); } while (0)

// The sequence of record sites: two that write no record (they fill the first batch), one ahead of the loop
// (opens region 0), three per KV tile, the last only closes.  A tile's three sites are committed as one batch
// inside region 0 of the next tile, once its first MFMAs have been issued: nothing but the clock reads stands
// behind a barrier, where every wave of the workgroup would pay for it at the same time.
struct AttnChain {
  static constexpr uint32_t kRegions = 3u, kLead = 2u;
  static constexpr bool kDense = true;
  // n = 2 + 1 + 3 tiles: every enabled region leaves two records per tile
  __device__ uint32_t total(uint32_t n, uint32_t mask) const { return 2u * ((n - 3u) / 3u) * (uint32_t)__builtin_popcount(mask & 7u); }
  __device__ uint32_t end_region(uint32_t site, uint32_t) const { return site <= kLead ? kp::kNoRegion : (site - 1u - kLead) % 3u; }
  __device__ uint32_t start_region(uint32_t site, uint32_t n) const {
    return (site < kLead || site + 1u == n) ? kp::kNoRegion : (site - kLead) % 3u;
  }
};

template <int INSTR>
__global__ __launch_bounds__(kAttnThreads, 2) void kp_attn_fwd(AttnArgs g) {
  extern __shared__ __align__(16) unsigned char smem[];  // [K tile][V tile, two buffers][ring]
  uint32_t* ring_lds = reinterpret_cast<uint32_t*>(smem + kKBytes + 2 * kVBytes);

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t h32 = lane >> 5, l32 = lane & 31u;
  const uint32_t q_blocks = g.S / kBq;
  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.  `wg` is the recorded workgroup:
  // head-major, the last query block of a head first.
  uint32_t wg = blockIdx.x;
  if (g.causal == 0u) {
    // every XCD takes a run of consecutive workgroups, so that it reads the K and V of few heads
    const uint32_t xcd = blockIdx.x & 7u, rest = g.n_wg & 7u;
    wg = xcd * (g.n_wg >> 3) + (xcd < rest ? xcd : rest) + (blockIdx.x >> 3);
  } else {
    // Causal work per block grows with its index.  All blocks of a (batch, head) go to one XCD where the heads can be
    // dealt out evenly, so that its K and V (2 MiB at 4096 keys) are fetched into one L2 (1.3 times, as those of two heads
    // fill it) instead of into all eight; as many heads as the XCD (the chip) has places for at a time (two per CU of the whole chip) are taken together, the longest blocks of
    // all of them first.  One head after the other, its long blocks start late and the last ones run on alone: 32
    // blocks and 16 heads per XCD take 292 times as long as one KV tile on 64 places, 264 with two heads together.
    const uint32_t heads = g.n_wg / q_blocks, per_xcd = (heads & 7u) == 0u ? 1u : 0u;
    const uint32_t xcd = per_xcd ? blockIdx.x & 7u : 0u, j = per_xcd ? blockIdx.x >> 3 : blockIdx.x;
    const uint32_t mine = per_xcd ? heads >> 3 : heads, places = per_xcd ? 64u : 512u;
    const uint32_t together = places > q_blocks ? places / q_blocks : 1u;
    const uint32_t group = j / (together * q_blocks), in = j - group * (together * q_blocks);
    const uint32_t left = mine - group * together, n = left < together ? left : together;
    const uint32_t block = in / n, h = group * together + in - block * n;
    wg = (per_xcd ? h * 8u + xcd : h) * q_blocks + block;
  }
  const uint32_t qb = q_blocks - 1u - (wg % q_blocks);
  const uint32_t bh = wg / q_blocks;
  const size_t head = (size_t)bh * g.S * kD;
  const uint32_t q0 = qb * kBq;

  kp::Ring ring{};
  if constexpr (INSTR != 0)
    ring = kp::ring_init<true>(ring_lds, reinterpret_cast<uint64_t*>(smem), g.cap_lds, g.region_mask, g.flush,
                         g.cap_hbm, g.trace, g.n_wg, 4u >> g.group_log2, wg, g.group_log2);
  ring.collab = g.collab;
  if constexpr (INSTR == 3 || INSTR == 5) kp::ring_use_realtime(ring);
  // (with wave groups the host adds 16 bytes behind the ring for the waves that do not record)
  if constexpr (INSTR >= 4) kp::chain_begin(ring, (uint32_t)(uintptr_t)ring_lds + (4u >> g.group_log2) * g.cap_lds * 8u);

  // Q fragments of this wave's 32 rows stay in registers: step s covers d = 16s .. 16s+15
  const uint32_t qrow = q0 + wave * 32 + l32;
  bf16x8 qf[8];
#pragma unroll
  for (int s = 0; s < 8; ++s)
    qf[s] = *reinterpret_cast<const bf16x8*>(g.Q + head + (size_t)qrow * kD + 16 * s + 8 * h32);

  // global -> LDS: either tile is 16 blocks of 1 KiB (four rows); wave w loads blocks w, w + 4, w + 8 and w + 12 of it.
  // Lane i of block j is row 4 j + i / 16, chunk position i % 16: rows 16 apart have the same swizzle, so that the
  // four loads of a tile share one lane offset and their scalar bases are 16 rows apart.
  const uint32_t lds0 = kp::wave_uniform((uint32_t)(uintptr_t)smem + 1024u * wave);
  uint32_t k_ofs, v_ofs;  // bytes
  {
    const uint32_t row = 4u * wave + (lane >> 4), pos = lane & 15u;
    k_ofs = row * kRow + ((pos ^ row) << 4);
    v_ofs = row * kRow + ((pos ^ (4u * (row & 3u))) << 4);
  }
  // One load: M0 (the LDS base) is put back afterwards, the compiler does not expect inline assembly to change
  // it.  From inline assembly because the compiler would make the next LDS access of any kind wait for such a
  // load; hidden from its count of outstanding vector-memory operations the loads still complete in order, and
  // the kernel waits for them itself in front of the barrier that precedes the tile's use.
  auto load_block = [&](const uint16_t* base, uint32_t ofs, uint32_t dst) __attribute__((always_inline)) {
    uint32_t saved_m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved_m0) : "v"(ofs), "s"(base), "s"(dst) : "memory");
  };
  const uint16_t* k_next = g.K + head;  // the K and V tile requested next
  const uint16_t* v_next = g.V + head;
  uint32_t v_into = kKBytes;   // LDS offset of the V buffer that the next tile goes to
  uint32_t v_other = kVBytes;  // from the V buffer in use to the other one
  auto load_k = [&](int i) __attribute__((always_inline)) { load_block(k_next + i * 16 * kD, k_ofs, lds0 + 4096u * (uint32_t)i); };
  auto load_v = [&](int i) __attribute__((always_inline)) { load_block(v_next + i * 16 * kD, v_ofs, lds0 + v_into + 4096u * (uint32_t)i); };
  auto tiles_requested = [&]() __attribute__((always_inline)) {
    k_next += kBkv * kD;
    v_next += kBkv * kD;
    v_into ^= kKBytes ^ (kKBytes + kVBytes);
  };
  // operand reads: K row 32 tk + l32, chunk 2 s + h32; V for the kv of MFMA step (tk, s) and the d of tile dt
  uint32_t k_rd[8], v_rd[4];
#pragma unroll
  for (int sx = 0; sx < 8; ++sx) k_rd[sx] = (uint32_t)(uintptr_t)smem + l32 * kRow + (((2u * (uint32_t)sx + h32) ^ (l32 & 15u)) << 4);
  {
    const uint32_t i = lane & 15u, grp = lane >> 4;  // groups 0, 1: d 0-15, 16-31 of the tile; 2, 3 the same for h = 1
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      const uint32_t d = 32u * (uint32_t)dt + 16u * (grp & 1u) + 4u * (i & 3u);
      v_rd[dt] = (uint32_t)(uintptr_t)smem + kKBytes + (4u * (grp >> 1) + (i >> 2)) * kRow + (((d >> 3) ^ (4u * (i >> 2))) << 4) + 8u * ((d >> 2) & 1u);
    }
  }
  auto read_k = [&](int s, int tk) -> bf16x8 {
    typedef const __attribute__((address_space(3))) bf16x8* lds_bf16x8;
    return *(lds_bf16x8)(uintptr_t)(k_rd[s] + (uint32_t)tk * 32u * kRow);
  };
  auto read_v = [&](uint32_t kv_step, int dt) -> bf16x8 {  // kv_step: first kv of the MFMA step (a multiple of 16)
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
    const uint32_t at = v_rd[dt] + kv_step * kRow;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)(at));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)(at + 8u * kRow));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };

  f32x16 oacc[4];  // O^T tiles: rows d = 32*dt + 8j + 4h + i, column q = lane % 32
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) oacc[dt] = f32x16{0};
  float m_run = -INFINITY, l_run = 0.f;

  const uint32_t n_tiles = g.causal ? (q0 + kBq) / kBkv : g.S / kBkv;
  // Staging overlaps arithmetic.  V tile t+1 goes to the other V buffer and is requested under the first MFMAs of region
  // 0 of tile t; every wave was done with that buffer before the barrier that ends tile t-1.  K has one buffer, whose
  // operands are all in registers half-way through region 0: behind a barrier there K tile t+1 is requested, under the
  // MFMAs that are left.  One wait covers both tiles, in front of the barrier that ends tile t.  The loads are spread over
  // the MFMAs because all loads of a CU queue up in one unit.
#pragma unroll
  for (int i = 0; i < 4; ++i) load_k(i);
#pragma unroll
  for (int i = 0; i < 4; ++i) load_v(i);
  tiles_requested();
  __builtin_amdgcn_s_waitcnt(kNoLoads);  // (the compiler's own count of outstanding loads: without it the loop would wait for the Q fragments)
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  // One KV tile.  MORE (tile t+1 exists) and MASK (the tile may reach past the diagonal) are compile-time: the
  // steady-state body has no branch but the one that moves the softmax reference.
  bf16x8 kf[8];  // operands of K Q^T, eight MFMAs ahead
  auto request_k_operands = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < 8; ++n) kf[n] = read_k(n, 0);
  };
  auto tile = [&](uint32_t t, auto more_c, auto mask_c) __attribute__((always_inline)) {
    constexpr bool MORE = decltype(more_c)::value, MASK = decltype(mask_c)::value;
    const uint32_t kv0 = t * kBkv;
    const bool diag = MASK && g.causal && (kv0 + kBkv > q0 + wave * 32);  // tile reaches past this wave's first row
    f32x16 sacc[2];  // raw scores of kv0 .. kv0 + 31 and of the 32 behind them
    sacc[0] = f32x16{0}; sacc[1] = f32x16{0};
    float mx = -INFINITY;  // maximum of the raw scores; the positive scale is applied afterwards
    float psum = 0.f;
    u32x4 pw[4];  // P as packed bf16 pairs, in accumulator order: one entry per MFMA step of V^T P^T (16 kv)
    auto mask = [&](int tk) __attribute__((always_inline)) {
      if (!diag) return;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t kv = kv0 + 32 * tk + 8 * (v >> 2) + 4 * h32 + (v & 3);
        if (kv > qrow) sacc[tk][v] = -INFINITY;
      }
    };
    auto exps = [&](int pair) __attribute__((always_inline)) {  // probabilities 2 pair and 2 pair + 1 of this lane's 32
      const int tk = pair >> 3, v = 2 * (pair & 7);
      const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[tk][v], g.scale_log2, -m_run));
      const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[tk][v + 1], g.scale_log2, -m_run));
      psum += p0 + p1;  // fp32 sum of the unrounded probabilities
      pw[pair >> 2][pair & 3] = bf16_pack_rne(p0, p1);
    };

    // ---- region 0: S^T = K Q^T --------------------------------------------------------------------
    // (opened by the site that closed region 2 of the tile before, or by the one ahead of the loop)
    // The two workgroups of a CU drift apart, so a SIMD usually holds one wave in a matrix region and
    // one in the softmax.  The matrix regions run at a higher wave priority: when both want to issue,
    // the MFMA goes first and the matrix pipe stays fed, while the softmax fills the gaps (equal priorities are
    // 3-6 % slower; this order of the two products or the other: 1 % apart).
    __builtin_amdgcn_s_setprio(2);
#pragma unroll
    for (int n = 0; n < 16; ++n) {  // the lower 32 kv, then the upper ones, whose operands are requested meanwhile
      const int s = n & 7, tk = n >> 3;
      sacc[tk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[s], sacc[tk], 0, 0, 0);
      if (tk == 0) kf[s] = read_k(s, 1);
      if (MORE && tk == 0 && (s & 1)) load_v(s >> 1);
      if (MORE && n >= 11 && n < 15) load_k(n - 11);
      if (tk == 1) {  // the maximum of the lower half
        if (s == 0) mask(0);
        mx = fmaxf(fmaxf(mx, sacc[0][2 * s]), sacc[0][2 * s + 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
      // the three sites of the tile before (ahead of the first tile: the one that opened region 0)
      if constexpr (INSTR >= 4) if (n == 10) kp::chain_commit<3>(ring);
      // every wave has read K tile t
      if (MORE && n == 9) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    __builtin_amdgcn_s_setprio(0);
    if constexpr (MORE) tiles_requested();
    KP_BOUNDARY(ring, 0, 1);
    KP_CHAIN(0, ring);

    // ---- region 1: online softmax (this lane: query row qrow, 32 of the tile's 64 kv) -------------
    bf16x8 vf[4];  // operands of one step of V^T P^T
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) vf[dt] = read_v(0, dt);
    mask(1);
#pragma unroll
    for (int v = 0; v < 16; v += 2) mx = fmaxf(fmaxf(mx, sacc[1][v]), sacc[1][v + 1]);
    mx = either_half_max(mx);
    // The value the exponentials are taken against only has to keep them in range; it need not be the
    // running maximum.  It moves (and O and l are rescaled) only when some row of the wave exceeds it
    // by more than 2^kSlack, which after the first few tiles practically never happens; until then a
    // probability may be as large as 2^kSlack, which fp32 sums and bf16 operands hold without loss.
    const float mx_s = mx * g.scale_log2;
    if (__builtin_amdgcn_ballot_w64(mx_s > m_run + kSlack) != 0ull) {  // always on the first tile (m_run = -inf)
      const float m_new = fmaxf(m_run, mx_s);  // finite from the first tile on: kv = 0 is visible to every row
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[dt][v] *= alpha;
      m_run = m_new;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) exps(i);
    l_run += psum;
    KP_BOUNDARY(ring, 1, 2);
    KP_CHAIN(1, ring);
    __builtin_amdgcn_s_setprio(1);

    // ---- region 2: O^T += V^T P^T ---------------------------------------------------------------------
    // The kv order inside an MFMA step follows the accumulator layout of S^T (kv = 16s + 4h + e for
    // e < 4, 16s + 8 + 4h + e - 4 otherwise), so P needs no cross-lane movement; V^T is read to match.
    auto pv = [&](int step, int dt) __attribute__((always_inline)) {
      oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[dt], __builtin_bit_cast(bf16x8, pw[step]), oacc[dt], 0, 0, 0);
    };
#pragma unroll
    for (int n = 0; n < 12; ++n) {
      pv(n >> 2, n & 3);
      vf[n & 3] = read_v(16u * (uint32_t)((n >> 2) + 1), n & 3);
      __builtin_amdgcn_sched_barrier(0);
    }

    // Every wave has read V tile t, and K and V tile t+1 have landed.  The last four MFMAs come behind the barrier, under
    // the first operand reads of the next tile.
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if constexpr (MORE) request_k_operands();
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) pv(3, dt);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) v_rd[dt] += v_other;
    v_other = 0u - v_other;
    __builtin_amdgcn_s_setprio(0);
    // One site closes region 2 and opens region 0 of the next tile: a tile costs three sites, not four.  It sits behind
    // the barrier: in front, the barrier's wait for LDS traffic would also wait for the two record stores that a generic
    // site has just issued, every tile (1.5 points of overhead).
    if constexpr (MORE) KP_BOUNDARY(ring, 2, 0); else KP_BOUNDARY(ring, 2, kp::kNoRegion);
    KP_CHAIN(2, ring);
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  KP_BOUNDARY(ring, kp::kNoRegion, 0);
  KP_CHAIN(0, ring);  // (the first two fill the first batch and write no record)
  KP_CHAIN(1, ring);
  KP_CHAIN(2, ring);
  request_k_operands();
  // only the last two tiles of a causal block can reach past the diagonal
  for (uint32_t t = 0; t + 2 < n_tiles; ++t) tile(t, yes, no);
  tile(n_tiles - 2, yes, yes);
  tile(n_tiles - 1, no, yes);

  // epilogue: O[q][d] = O^T[d][q] / l.  A lane holds four d of a row at a time; through LDS (8 KiB per wave: every wave is
  // past its last operand read) they leave as whole rows.  A row is 16 chunks of 16 bytes; chunk c of row r at position
  // c ^ r % 8, its halves swapped where r / 8 is odd: 16 lanes of an 8-byte write hit all banks once.
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  const float inv = 1.0f / l_tot;
  unsigned char* sO = smem + 8192u * wave;
  {
    const uint32_t half = h32 ^ ((l32 >> 3) & 1u);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        u32x2 pk2;
        pk2.x = bf16_pack_rne(oacc[dt][4 * q + 0] * inv, oacc[dt][4 * q + 1] * inv);
        pk2.y = bf16_pack_rne(oacc[dt][4 * q + 2] * inv, oacc[dt][4 * q + 3] * inv);
        *reinterpret_cast<u32x2*>(sO + l32 * 256u + (((uint32_t)(4 * dt + q) ^ (l32 & 7u)) << 4) + 8u * half) = pk2;
      }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {  // four rows: lane l takes row 4 i + l / 16, position l % 16
    const uint32_t r = 4u * (uint32_t)i + (lane >> 4), chunk = (lane & 15u) ^ (r & 7u);
    const u32x4 v = *reinterpret_cast<const u32x4*>(sO + 1024u * (uint32_t)i + 16u * lane);
    *reinterpret_cast<u32x4*>(g.O + head + (size_t)(q0 + wave * 32u + r) * kD + 8u * chunk) = (i & 2) ? u32x4{v.z, v.w, v.x, v.y} : v;
  }
  if constexpr (INSTR != 0) {
    kp::TraceGeom tg{g.n_wg, 4u >> g.group_log2, 3, g.cap_hbm, g.flags};
    if constexpr (INSTR >= 4) {
      kp::chain_commit<3>(ring);  // the sites of the last tile
      kp::ring_finish<INSTR == 5>(ring, g.cap_lds, g.trace, tg, wg, g.rec_cost, AttnChain{});
    } else {
      kp::ring_finish<INSTR == 3>(ring, g.cap_lds, g.trace, tg, wg, g.rec_cost);
    }
  }
}

bool attn_shape_ok(int B, int H, int S, int D) {
  return B > 0 && H > 0 && S > 0 && D == kD && S % kBq == 0 && (long long)B * H * (S / kBq) < (1ll << 31);
}

}  // namespace

extern "C" kp_status kp_attn_launch_shape(int B, int H, int S, int D, int* n_wg, int* waves_per_wg, int* n_regions) {
  kp::clear_error();
  if (!attn_shape_ok(B, H, S, D))
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "attention B=%d H=%d S=%d D=%d: D must be 128 and S a multiple of 128", B, H, S, D);
  if (n_wg) *n_wg = B * H * (S / kBq);
  if (waves_per_wg) *waves_per_wg = 4;
  if (n_regions) *n_regions = 3;
  return KP_OK;
}

extern "C" kp_status kp_attn_instrumented(const void* Q, const void* K, const void* V, void* O, int B, int H,
                                          int S, int D, int causal, float scale, uint32_t region_mask,
                                          void* trace_buf, size_t trace_cap, void* stream) {
  kp::clear_error();
  if (!Q || !K || !V || !O) return kp::fail(KP_ERR_INVALID_ARG, "NULL tensor pointer");
  if (!attn_shape_ok(B, H, S, D))
    return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "attention B=%d H=%d S=%d D=%d: D must be 128 and S a multiple of 128", B, H, S, D);
  if (((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V | (uintptr_t)O) & 15u)
    return kp::fail(KP_ERR_INVALID_ARG, "Q, K, V, O must be 16-byte aligned");
  if (!(scale > 0.f) || scale > 1e30f) return kp::fail(KP_ERR_INVALID_ARG, "scale must be positive and finite");
  if (region_mask & KP_MASK_PHASES) return kp::fail(KP_ERR_INVALID_ARG, "KP_MASK_PHASES belongs to the GEMM");
  const uint32_t regions = region_mask & ~(KP_MASK_FLUSH | KP_MASK_WAVE_GROUP | KP_MASK_REALTIME | KP_MASK_COLLAB), flush = region_mask >> 31;
  const bool realtime = (region_mask & KP_MASK_REALTIME) != 0u, collab = (region_mask & KP_MASK_COLLAB) != 0u;
  const uint32_t group_log2 = (region_mask & KP_MASK_WAVE_GROUP) ? 2u : 0u;
  const size_t streams = 4u >> group_log2;
  const int n_wg = B * H * (S / kBq);
  hipStream_t st = static_cast<hipStream_t>(stream);
  AttnArgs g{};
  g.Q = static_cast<const uint16_t*>(Q); g.K = static_cast<const uint16_t*>(K);
  g.V = static_cast<const uint16_t*>(V); g.O = static_cast<uint16_t*>(O);
  g.B = (uint32_t)B; g.H = (uint32_t)H; g.S = (uint32_t)S; g.causal = causal ? 1u : 0u;
  g.scale_log2 = scale * 1.4426950408889634f;
  g.region_mask = regions; g.trace = trace_buf; g.flush = flush; g.n_wg = (uint32_t)n_wg;
  g.group_log2 = group_log2;
  g.collab = collab ? 1u : 0u;
  g.flags = (flush ? KP_FLAG_FLUSH : 0u) | (realtime ? KP_FLAG_REALTIME : 0u) | (collab ? KP_FLAG_HW_IDS : 0u);
  const uint32_t tile_bytes = kKBytes + 2 * kVBytes;
  if (regions == 0) {
    hipLaunchKernelGGL(kp_attn_fwd<0>, dim3(n_wg), dim3(kAttnThreads), tile_bytes, st, g);
    KP_HIP_TRY(hipGetLastError());
    return KP_OK;
  }
  if (!trace_buf) return kp::fail(KP_ERR_INVALID_ARG, "trace_buf is NULL but region_mask enables regions");
  if (regions >> 3) return kp::fail(KP_ERR_INVALID_ARG, "region_mask enables regions this kernel does not have (3 regions)");
  if (((uintptr_t)trace_buf) & 15u) return kp::fail(KP_ERR_INVALID_ARG, "trace_buf must be 16-byte aligned");
  if (trace_cap % streams) return kp::fail(KP_ERR_TRACE_TOO_SMALL, "trace_cap must be a multiple of %zu record streams", streams);
  const size_t cap_wave = trace_cap / streams;
  if (!kp::is_pow2(cap_wave) || cap_wave < 2 || cap_wave > (1u << 19))
    return kp::fail(KP_ERR_TRACE_TOO_SMALL, "trace_cap/streams = %zu must be a power of two >= 2", cap_wave);
  uint32_t cap_lds = (uint32_t)cap_wave;
  if (flush && cap_lds > 64) cap_lds = 64;
  const size_t ring_bytes = (size_t)cap_lds * 8 * streams + (group_log2 ? 16 : 0);  // (16: see chain_begin)
  if (ring_bytes > 32 * 1024) return kp::fail(KP_ERR_UNSUPPORTED_SHAPE, "LDS ring of %zu bytes exceeds the 32 KiB budget", ring_bytes);
  g.cap_lds = cap_lds; g.cap_hbm = (uint32_t)cap_wave; g.rec_cost = kp::rec_cost();
  static thread_local int attr_dev = -1;  // the attribute is kept per device
  int dev = 0;
  KP_HIP_TRY(hipGetDevice(&dev));
  if (attr_dev != dev) {
    KP_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kp_attn_fwd<1>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024));
    KP_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kp_attn_fwd<5>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024));
    KP_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kp_attn_fwd<3>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024));
    KP_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kp_attn_fwd<4>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024));
    attr_dev = dev;
  }
  // circular strategy and one lane stores: chained record sites
  if (!flush && !collab) {
    if (realtime) hipLaunchKernelGGL(kp_attn_fwd<5>, dim3(n_wg), dim3(kAttnThreads), tile_bytes + ring_bytes, st, g);
    else hipLaunchKernelGGL(kp_attn_fwd<4>, dim3(n_wg), dim3(kAttnThreads), tile_bytes + ring_bytes, st, g);
  } else if (realtime) {
    hipLaunchKernelGGL(kp_attn_fwd<3>, dim3(n_wg), dim3(kAttnThreads), tile_bytes + ring_bytes, st, g);
  } else {
    hipLaunchKernelGGL(kp_attn_fwd<1>, dim3(n_wg), dim3(kAttnThreads), tile_bytes + ring_bytes, st, g);
  }
  KP_HIP_TRY(hipGetLastError());
  return KP_OK;
}
