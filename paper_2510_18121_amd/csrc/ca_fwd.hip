// Forward kernel: O = softmax(scale * Q K^T, causal) V and LSE over tiles of query rows
// (core attention, Section 2.1; one fused launch over all CA-tasks, Section 4.1).
//
// A forward unit is 256 query slots of one document x one query head, or, for the slots a document has left over after its full
// tiles, 256/hp slots x hp query heads of one KV group (same K/V tiles, same loads; only the (wave, row group) -> (slots, head)
// mapping differs).  A workgroup of four waves takes a unit, 64 rows per wave, or half of one, 32 rows per wave (the planner
// chooses per list; see there).  A K or V fragment that a wave reads from LDS feeds four MFMAs, or two.
//
// The wave computes the TRANSPOSED score block S^T = K Q^T with v_mfma_f32_16x16x32_bf16, in tiles of 16 keys x 16 rows: a lane
// owns one row (column l%16 of the MFMA result) of each of its row groups, and its 4 registers per tile are 4 keys.  The bf16
// probabilities of two such tiles, still in those registers, are exactly the B operand of O^T += V^T P^T (the key index is the
// contraction index; its order inside 32 keys is the same permutation on both operands).  V^T comes out of the natural-layout V
// tile in LDS through ds_read_b64_tr_b16.
//
// K and V tiles of 64 keys go from global memory straight into swizzled LDS tiles (global_load_lds).  Q fragments (64 registers at
// head_dim 128, 64 rows) and accumulators (128) stay in registers, one block of scores takes 32 more: within 256 two workgroups
// share a CU (three at head_dim 64), drift apart and fill each other's waits.  What bounds the kernel is the power limit: on N(0,1)
// data the 16x16 shape costs less energy per flop than 32x32 (alone 1928 against 1741 TFLOP/s), at twice the issue slots.
// One wave per SIMD with 384 registers, 32x32 MFMAs and a software pipeline across blocks written out slot by slot, against this
// (32/8 heads, head_dim 128): 52.0 -> 47.9 ms (128K tokens of long and short documents), 2.55 -> 2.29 ms (64K tokens of documents
// of about 2K), 9.54 -> 8.78 ms (64/8 heads); with halves 45 -> 24 us (32 units of 16 tiles), 16.2 -> 10.9 us (1.5K tokens, 4/2
// heads, head_dim 64).  Slower, by up to 4 %: lists short enough that the clock stays up (256 pieces of 32 tiles, 66 -> 67 to 69 us at
// 2.2 GHz).  It is not the fetches, for which a wave waits 1 % of a tile: units of eight waves with four stages took the same time, as
// did fragments further ahead and the exponentials spread over both blocks' MFMAs; K and V prefetched to L2 cost 9 %.
//
// The fast path exponentiates against the maximum of the first keys (see there) and masks on the diagonal; tile 0 of a document's
// first rows and units in which that maximum was outgrown take a general path with lazy rescaling of the accumulators.  The
// softmax runs in base 2 with scale*log2(e) folded into one FMA.
#include <atomic>
#include <type_traits>

#include "ca_device.h"
#include "ca_internal.h"

namespace ca {

template <int D>
struct FwdSmem {
  static constexpr int NST = D == 128 ? 2 : 3;  // stages of a K and a V tile
  static constexpr int TILE = FWD_BN * 2 * D;   // one K or V tile
  static constexpr int K_OFF = 0;
  static constexpr int V_OFF = TILE;
  static constexpr int STAGE = 2 * TILE;
  static constexpr int POS_OFF = NST * STAGE;   // positions of the unit's rows, as [wave][row group][16]
  static constexpr int TOTAL = POS_OFF + FWD_BM * 4;
};

template <int D, bool HALVES>
__global__ __launch_bounds__(256, D == 64 ? 3 : 2) void ca_fwd_kernel(const FwdUnit *__restrict__ units, int n_units, int turns,
                                                                   const int32_t *__restrict__ slot_row,
                                                                   const int32_t *__restrict__ slot_pos,
                                                                   const bf16_t *__restrict__ Q,
                                                                   const bf16_t *__restrict__ K,
                                                                   const bf16_t *__restrict__ V, bf16_t *__restrict__ O,
                                                                   float *__restrict__ LSE, float *__restrict__ parts,
                                                                   float *__restrict__ stats, int Hq, int Hkv,
                                                                   int64_t total_q, float c /* scale * log2(e) */) {
  using S = FwdSmem<D>;
  constexpr int W = 4;             // waves
  constexpr int NK = D / 32;       // MFMA k-steps over head_dim
  constexpr int ND = D / 16;       // 16-row blocks of O^T
  constexpr int CH = D / 8;        // 16-byte chunks per row
  constexpr int RPI = 64 / CH;     // rows covered by one wave-wide direct load (1 KB)
  constexpr int NLD = FWD_BN / (W * RPI);  // direct loads per wave per tile
  constexpr int NST = S::NST;
  constexpr int ROWB = 2 * D, HALF = 16 * ROWB;
  constexpr float RESCALE_LOG2 = 8.0f;
  constexpr float M_NONE = -3.402823466e38f;  // running maximum of a row that has seen no key: finite, so that -inf - m is -inf
  constexpr int NR = HALVES ? 2 : 4;  // groups of 16 rows per wave
  constexpr int TURN_LG = 13;         // a turn in clock cycles: two to three tiles
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(CA_LDS char *)smem;  // LDS byte address of the dynamic segment

  int at_unit = int(blockIdx.x), half = 0;
  if (HALVES) half_of_unit(at_unit, n_units, half);
  const FwdUnit u = units[at_unit];
  // A half of padding has nothing to store.  (Of one to a few rows per document it is every second one: 111 -> 92 us for 2 rows with 84K keys,
  // 32/8 heads, 109 -> 92 for 13 rows with 43K, 16/16, 1280 -> 918 for five times 4 rows with 126K, 16/16.)
  if (HALVES && ((W * half) >> __builtin_ctz(u.hp)) * 32 >= u.rows) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hk = __builtin_amdgcn_readfirstlane(u.head / (Hq / Hkv));  // (uniform, for scalar K/V addresses)
  // (wave, group of 32) -> 32-slot group and query head inside the unit: pair 2 wave + x takes slots 32 (pair / hp) ..
  // of head  head + pair % hp  (hp = 1 for a full tile, > 1 for a head-packed unit).  Row group rg of 16 is half rg % 2 of
  // group rg / 2; a lane's row in it is lane % 16.
  const int hp_lg = __builtin_ctz(u.hp), pair0 = HALVES ? W * half + wave : 2 * wave;
  auto head_of = [&](int rg) __attribute__((always_inline)) { return u.head + ((pair0 + (rg >> 1)) & (u.hp - 1)); };
  auto slot_of = [&](int rg, int li) __attribute__((always_inline)) {
    return u.slot0 + ((pair0 + (rg >> 1)) >> hp_lg) * 32 + 16 * (rg & 1) + li;
  };
  int n_tiles = (u.n_keys + FWD_BN - 1) / FWD_BN;
  if (HALVES) {  // tiles some row of the half sees (positions are sorted; at least one, which then is masked)
    const int last = slot_pos[u.slot0 + ((W * half + W - 1) >> hp_lg) * 32 + 31] - u.key0;
    n_tiles = max(1, min(n_tiles, last / FWD_BN + 1));
  }

  // ---- direct global -> LDS tile loads.  Load n of this wave covers tile rows RPI*(wave + 4n) .. +RPI-1;
  // lane i fills physical chunk i % CH of row i / CH, so it fetches logical chunk (i % CH) ^ sw(row).
  // The address is (scalar tile base) + (per-lane 32-bit offset): advancing to the next tile costs no
  // vector instruction.
  const uint32_t kv_row_bytes = uint32_t(Hkv) * D * 2;
  static_assert(W * RPI % 16 == 0);  // the swizzle repeats every 16 rows
  const int last_tile = n_tiles - 1, last_key_in_tile = min(FWD_BN, u.n_keys - last_tile * FWD_BN) - 1;
  const char *kg = reinterpret_cast<const char *>(K + (size_t(u.kv_row0) * Hkv + hk) * D);
  const char *vg = reinterpret_cast<const char *>(V + (size_t(u.kv_row0) * Hkv + hk) * D);
  const size_t tile_bytes = size_t(FWD_BN) * kv_row_bytes;
  uint32_t ld_off;
  {
    const int lane = lane_id_here(), ld_row0 = RPI * wave + lane / CH;
    ld_off = uint32_t(ld_row0) * kv_row_bytes + uint32_t((lane % CH) ^ tile_sw<D>(ld_row0)) * 16;
  }
  // tile j into its stage; rows beyond the last key are fetched as the last key, tiles beyond the last as the last
  auto issue_kv = [&](int tile) __attribute__((always_inline)) {
    const size_t at = size_t(min(tile, last_tile)) * tile_bytes;
    const uint32_t dst = lds0 + uint32_t((tile % NST) * S::STAGE + 1024 * wave);
    if (tile < last_tile) {
#pragma unroll
      for (int n = 0; n < NLD; ++n) {
        load_lds16_sbase(kg + at + n * W * RPI * kv_row_bytes, ld_off, dst + S::K_OFF + 1024 * W * n);
        load_lds16_sbase(vg + at + n * W * RPI * kv_row_bytes, ld_off, dst + S::V_OFF + 1024 * W * n);
      }
    } else {
      const int lane = lane_id_here(), ld_row0 = RPI * wave + lane / CH;
      const uint32_t cbytes = uint32_t((lane % CH) ^ tile_sw<D>(ld_row0)) * 16;
#pragma unroll
      for (int n = 0; n < NLD; ++n) {
        const uint32_t off = uint32_t(min(ld_row0 + W * RPI * n, last_key_in_tile)) * kv_row_bytes + cbytes;
        load_lds16_sbase(kg + at, off, dst + S::K_OFF + 1024 * W * n);
        load_lds16_sbase(vg + at, off, dst + S::V_OFF + 1024 * W * n);
      }
    }
  };
  auto issue_first = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NST - 1; ++t) issue_kv(t);
  };
  issue_first();

  // Q fragments: B operand of S^T = K Q^T; lane holds Q[row][32 s + 8 (lane / 16) .. +7]
  bf16x8 qf[NK][NR];
  // The last key that every row of the wave sees (positions are sorted), and that every row, that any row of the 64 sees that share a
  // wave in whole units: which blocks are multiplied, so whom a non-finite value of V reaches, does not depend on the form either.
  const int wmin = slot_pos[u.slot0 + (pair0 >> hp_lg) * 32] - u.key0;
  const int wmin64 = slot_pos[u.slot0 + ((pair0 & ~1) >> hp_lg) * 32] - u.key0;
  // (a wave without a row, which padding is behind all rows, multiplies nothing)
  const bool has_rows = ((pair0 & ~1) >> hp_lg) * 32 < u.rows;
  const int wmax64 = has_rows ? slot_pos[u.slot0 + ((pair0 | 1) >> hp_lg) * 32 + 31] - u.key0 : -1;
  uint32_t koff, voff;  // per-lane LDS read addresses into the current stage: natural reads of K, transposing reads of V
  {
    const int lane = lane_id_here(), j4 = lane >> 4, li = lane & 15;
    int pos[NR];
#pragma unroll
    for (int rg = 0; rg < NR; ++rg) {
      const int slot = slot_of(rg, li), row = slot_row[slot];
      pos[rg] = slot_pos[slot] - u.key0;  // counted from the first key of a piece's window (below 0: sees none of it)
      const bf16_t *qp = Q + (size_t(row < 0 ? 0 : row) * Hq + head_of(rg)) * D + 8 * j4;
#pragma unroll
      for (int s = 0; s < NK; ++s) qf[s][rg] = *reinterpret_cast<const bf16x8 *>(qp + 32 * s);
    }
    // (only masked blocks need the positions: they wait in LDS)
    if (lane < 16) {
#pragma unroll
      for (int rg = 0; rg < NR; ++rg) *(CA_LDS int *)(lds0 + S::POS_OFF + 64 * (NR * wave + rg) + 4 * li) = pos[rg];
    }
  }
  auto first_stage = [&]() __attribute__((always_inline)) {
    const int lane = lane_id_here(), j4 = lane >> 4, li = lane & 15;
    koff = lds0 + S::K_OFF + li * ROWB + 16 * (j4 ^ tile_sw<D>(li));
    voff = lds0 + S::V_OFF + (4 * j4 + (li >> 2)) * ROWB + 16 * (((li >> 1) & 1) ^ tile_sw<D>(4 * j4 + (li >> 2))) + 8 * (li & 1);
  };
  first_stage();
  // tiles j < n_fast are entirely visible to every row of this wave, tiles from n_seen on are seen by none of the 64
  // (rows may see past the window of a piece; one that is not the unit's last has whole tiles only)
  const int n_fast = min(wmin + 1, u.n_keys) / FWD_BN;
  const int n_seen = wmax64 < 0 ? 0 : min(wmax64 / FWD_BN + 1, n_tiles);

  f32x4 acc[ND][NR];
  float m[NR], lsum[NR];
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int rg = 0; rg < NR; ++rg) {
      m[rg] = M_NONE, lsum[rg] = 0.f;
#pragma unroll
      for (int b = 0; b < ND; ++b) acc[b][rg] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  clear();

  // Everything issued so far has landed, including the Q fragments: from here on the compiler places no
  // vector-memory waits inside the loop (they would drain the direct-load queue every iteration).
  wait_vmcnt<0>();
#pragma unroll
  for (int rg = 0; rg < NR; ++rg)
#pragma unroll
    for (int s = 0; s < NK; ++s) pin(qf[s][rg]);

  // this wave's parts of tile j have landed
  auto top = [&](int j) __attribute__((always_inline)) {
    wait_vmcnt<2 * (NST - 2) * NLD>();
    barrier_nofence();  // ... and everybody else's; everybody is done with tile j-1
    // Two workgroups of equal length that share a CU take turns at having priority (workgroups i and i + 256 share one).  Left to
    // itself the hardware serves the older one first: it runs nearly as fast as alone, and its neighbour ends up alone on the CU
    // (cycles per tile of the faster and the slower one, 4512 and 6701 of 506 tiles each; taking turns 5714 and 6263).
    if (D == 128 && turns) {
      if ((uint32_t(__builtin_amdgcn_s_memtime() >> TURN_LG) ^ (blockIdx.x / N_CU)) & 1) __builtin_amdgcn_s_setprio(1);
      else __builtin_amdgcn_s_setprio(0);
    }
    if (NST > 2 || j < last_tile) issue_kv(j + NST - 1);  // (with three stages always: the wait counts loads)
  };
  auto advance = [&](int j) __attribute__((always_inline)) {
    const int adv = (j % NST) == NST - 1 ? -(NST - 1) * S::STAGE : S::STAGE;
    koff += adv, voff += adv;
  };
  // K fragment (kt, s) and V^T fragment b of a 32-key block
  auto read_k = [&](int kb, int kt, int s) __attribute__((always_inline)) {
    return lds_read8_at((HALVES ? koff ^ (64 * s) : s == 0 ? koff : xor_here(koff, 64 * s)) + (32 * kb + 16 * kt) * ROWB);
  };
  auto read_v = [&](int kb, int b) __attribute__((always_inline)) {
    const uint32_t a = (HALVES ? voff ^ (32 * b) : b == 0 ? voff : xor_here(voff, 32 * b)) + 32 * kb * ROWB;
    return join(lds_read_tr4_at(a), lds_read_tr4_at(a + HALF));
  };
  // scores beyond a row's position become -infinity: register e holds key key0 + 4 (lane / 16) + e
  auto mask = [&](int r0, auto &s, int key0) __attribute__((always_inline)) {  // (s: of row groups r0 ..)
    const int lane = lane_id_here();
#pragma unroll
    for (int i = 0; i < int(sizeof(s) / sizeof(s[0])); ++i) {
      const int vis = lds_ld<int>(lds0 + S::POS_OFF + 64 * (NR * wave + r0 + i) + 4 * (lane & 15)) - key0 - 4 * (lane >> 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[i][e] = e <= vis ? s[i][e] : -INFINITY;
    }
  };
  // scores of the 32 keys at koff and row groups r0 .. (as x has), not interleaved with anything
  auto scores_plain = [&](int r0, auto &x) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < NK; ++s) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const bf16x8 a = read_k(0, kt, s);
#pragma unroll
        for (int i = 0; i < int(sizeof(x[0]) / sizeof(x[0][0])); ++i) x[kt][i] = mfma16(a, qf[s][r0 + i], s == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : x[kt][i]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto largest = [&](const f32x4 &a, const f32x4 &b) __attribute__((always_inline)) {
    return fmaxf(fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])), fmaxf(fmaxf(b[0], b[1]), fmaxf(b[2], b[3])));
  };

  // ------------------------------------------------------------------------------------------ general path
  // the first tile of a document's first rows (below) and, after an overflow, all tiles of the rows concerned, 32 keys at a time (at
  // koff and voff): mask, row maximum, lazy rescaling, nothing interleaved
  auto general_block = [&](int k0, auto residue) __attribute__((always_inline)) {
    constexpr bool RESIDUE = decltype(residue)::value;
    constexpr int GS = D == 64 && !RESIDUE ? NR : 2;  // row groups at a time: with more the registers do not hold all of it
    if (k0 > wmax64) return;
    // Lazy rescaling: the running reference m only moves when some row's maximum has grown by more than
    // 2^RESCALE_LOG2; until then probabilities are taken relative to the stale m (they stay below
    // 2^RESCALE_LOG2, harmless in fp32 and bf16) and the accumulators need no multiply.
    // (a row that sees none of these keys, having seen none before (in a piece that lies beyond its position), keeps
    // m = M_NONE and gets probabilities 0)
    // The first rows of a document see a handful of keys, their output is as large as a single V row, and the 2^-9 relative
    // rounding of P to bf16 would show up at the 1e-2 level next to the output's own bf16 rounding.  So the rounding residue of
    // P goes through the matrix pipe too (P = hi + lo), which makes P V as good as fp32.  Later tiles go without: with it, and 16 keys
    // at a time, a forward that repeats all of its 16K tokens took 700 us instead of 493 (16/16 heads, head_dim 64) and 1600
    // instead of 1310 (32/8, 128).
#pragma unroll
    for (int r0 = 0; r0 < NR; r0 += GS) {
      f32x4 x[2][GS];
      scores_plain(r0, x);
      if (k0 + 31 > wmin) mask(r0, x[0], k0), mask(r0, x[1], k0 + 16);  // some (row, key) may be above the diagonal
      bf16x8 hi[GS], lo[GS];
#pragma unroll
      for (int i = 0; i < GS; ++i) {
        const int rg = r0 + i;
        const float top = largest(x[0][i], x[1][i]);
        if (__any(top * c > m[rg] + RESCALE_LOG2)) {
          const float m_cand = fmaxf(m[rg], quad_max(top) * c);
          const float alpha = m[rg] == M_NONE ? 0.f : fast_exp2(m[rg] - m_cand);
          m[rg] = m_cand;
          lsum[rg] *= alpha;
#pragma unroll
          for (int b = 0; b < ND; ++b) acc[b][rg] *= alpha;
        }
        uint32_t h[4], l[4];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
          float v[4], r[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = fast_exp2(fmaf(x[kt][i][e], c, -m[rg])), r[e] = v[e] - float(bf16_t(v[e]));
          lsum[rg] += (v[0] + v[1]) + (v[2] + v[3]);
          h[2 * kt] = pack_bf16(v[0], v[1]), h[2 * kt + 1] = pack_bf16(v[2], v[3]);
          l[2 * kt] = pack_bf16(r[0], r[1]), l[2 * kt + 1] = pack_bf16(r[2], r[3]);
        }
        hi[i] = __builtin_bit_cast(bf16x8, u32x4{h[0], h[1], h[2], h[3]});
        lo[i] = __builtin_bit_cast(bf16x8, u32x4{l[0], l[1], l[2], l[3]});
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int b = 0; b < ND; ++b) {
        const bf16x8 a = read_v(0, b);
#pragma unroll
        for (int i = 0; i < GS; ++i) acc[b][r0 + i] = mfma16(a, hi[i], acc[b][r0 + i]);
        if (RESIDUE) {
#pragma unroll
          for (int i = 0; i < GS; ++i) acc[b][r0 + i] = mfma16(a, lo[i], acc[b][r0 + i]);
        }
        if (b & 1) __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  auto general_tile = [&](int jt, auto residue) __attribute__((always_inline)) {
#pragma unroll 1
    for (int kb = 0; kb < 2; ++kb) {
      general_block(jt * FWD_BN + 32 * kb, residue);
      koff += 32 * ROWB, voff += 32 * ROWB;
    }
    koff -= FWD_BN * ROWB, voff -= FWD_BN * ROWB;
    advance(jt);
  };

  int j = 0;
  if (wmin64 < FWD_BN) {  // rows that see less than a tile: hi + lo P on tile 0
    top(0);
    general_tile(0, std::true_type{});
    j = 1;
  }
  // ------------------------------------------------------------------------------------------ fast path
  // All other tiles the wave sees: without a mask as long as every row sees the whole tile (j < n_fast), with a mask up
  // to its last one.
  // Exponentials are taken against the running maximum m as it stood when this path was entered (the maximum of the first keys, or
  // of tile 0): no rescaling, no row maximum, no exit.  Probabilities relative to a stale m are merely larger numbers - bf16 and
  // fp32 carry the same exponent range, so neither P nor the accumulators lose accuracy - until one of them overflows;
  // that shows in the row sum.  If the row sum of any row of a workgroup has left the finite range, everything computed
  // here is thrown away and the workgroup computes its rows again by the general path alone (below), which rescales as it goes.
  // A later score would have to exceed that maximum by about 2^100 in probability for that (the row sum is
  // checked against 1e30, which leaves the accumulators, |V| times larger at most, well inside fp32).
  bool outgrown = false;
  if (j < n_seen) {
    // Blocks [KB0, KB1) of a tile.  Fragments come from LDS AHEAD fragments before the MFMAs that use them: per block 2 NK of K
    // and ND of V transposed.  The exponentials of the first 16 keys go between the score MFMAs of the other 16; fences keep that
    // order.  (Whole units have no registers for more than 2 ahead without spilling, and gain nothing from 3.)
    constexpr int NF = 2 * NK + ND, AHEAD = HALVES ? 4 : 2;
    auto blocks = [&](const int KB0, const int KB1, const bool MASK, int key0, const bool FIRST = false) __attribute__((always_inline)) {
      bf16x8 fr[AHEAD];
      auto fetch = [&](int i) __attribute__((always_inline)) -> bf16x8 {
        const int kb = KB0 + i / NF, f = i % NF;
        return f < 2 * NK ? read_k(kb, f / NK, f % NK) : read_v(kb, f - 2 * NK);
      };
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) fr[i] = fetch(i);
      int at = 0;  // the fragment in use
      auto next = [&]() __attribute__((always_inline)) {  // it has been used: its registers take the one AHEAD later
        if (at + AHEAD < NF * (KB1 - KB0)) fr[at % AHEAD] = fetch(at + AHEAD);
        ++at;
        __builtin_amdgcn_sched_barrier(0);
      };
#pragma unroll
      for (int kb = KB0; kb < KB1; ++kb) {
        f32x4 s[2][NR];
        uint32_t pw[NR][4];
        // the probabilities of tile kt and row group rg: exponentials, row sum, packing
        auto expo = [&](int kt, int rg) __attribute__((always_inline)) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = fast_exp2(fmaf(s[kt][rg][e], c, -m[rg]));
          lsum[rg] += (v[0] + v[1]) + (v[2] + v[3]);
          pw[rg][2 * kt] = pack_bf16(v[0], v[1]), pw[rg][2 * kt + 1] = pack_bf16(v[2], v[3]);
        };
#pragma unroll
        for (int f = 0; f < 2 * NK; ++f) {
          const int kt = f / NK;
#pragma unroll
          for (int rg = 0; rg < NR; ++rg) s[kt][rg] = mfma16(fr[at % AHEAD], qf[f % NK][rg], f % NK == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[kt][rg]);
          if (!MASK && !(FIRST && kb == 0) && kt == 1) {
#pragma unroll
            for (int rg = NR * (f - NK) / NK; rg < NR * (f - NK + 1) / NK; ++rg) expo(0, rg);
          }
          next();
        }
        if (FIRST && kb == 0) {
#pragma unroll
          for (int rg = 0; rg < NR; ++rg) m[rg] = quad_max(largest(s[0][rg], s[1][rg])) * c;
        }
        if (MASK) mask(0, s[0], key0), mask(0, s[1], key0 + 16);
        if (MASK || (FIRST && kb == 0)) {
#pragma unroll
          for (int rg = 0; rg < NR; ++rg) expo(0, rg);
        }
#pragma unroll
        for (int rg = 0; rg < NR; ++rg) {
          expo(1, rg);
          __builtin_amdgcn_sched_barrier(0);
        }
        bf16x8 pb[NR];
#pragma unroll
        for (int rg = 0; rg < NR; ++rg) pb[rg] = __builtin_bit_cast(bf16x8, u32x4{pw[rg][0], pw[rg][1], pw[rg][2], pw[rg][3]});
#pragma unroll
        for (int b = 0; b < ND; ++b) {
#pragma unroll
          for (int rg = 0; rg < NR; ++rg) acc[b][rg] = mfma16(fr[at % AHEAD], pb[rg], acc[b][rg]);
          next();
        }
      }
    };
    const int entry = j;
    top(j);
    if (j == 0) {  // the maximum over the first 32 keys, which every row sees, becomes the reference
      blocks(0, 2, false, 0, true);
      advance(0);
      j = 1;
    }
    for (; j < n_fast; ++j) {
      if (j > entry) top(j);
      blocks(0, 2, false, 0);
      advance(j);
    }
    for (; j < n_seen; ++j) {  // the same with the mask: the diagonal
      if (j > entry) top(j);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        if (FWD_BN * j + 32 * kb <= wmax64) blocks(kb, kb + 1, true, FWD_BN * j + 32 * kb);
      advance(j);
    }
    bool inside = true;  // (false for NaN)
#pragma unroll
    for (int rg = 0; rg < NR; ++rg) inside = inside && lsum[rg] < 1.0e30f;
    outgrown = __any(!inside);
  }
  for (; j < n_tiles; ++j) top(j);  // tiles only other waves see: this wave's part of the loads
  wait_vmcnt<0>();  // nothing may still be writing LDS
  // Did the fast path of any wave meet a maximum beyond its window?  Then the rows of its half of the unit (128 rows) are computed
  // again.  The tiles are shared, so all waves of the workgroup go along; those of the other half of a whole unit only fetch.
  // Flags go through the first bytes of LDS: every tile read and every direct load of the workgroup is complete after the
  // first barrier.
  barrier_nofence();
  if (lane_id_here() == 0) *reinterpret_cast<volatile int *>(smem + 4 * wave) = outgrown ? 1 : 0;
  __syncthreads();
  int flags = 0, mine = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const int f = *reinterpret_cast<volatile int *>(smem + 4 * w);
    flags |= f;
    if (HALVES || w / 2 == wave / 2) mine |= f;
  }
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(flags) != 0) {
    const bool again = __builtin_amdgcn_readfirstlane(mine) != 0;
    if (again) clear();
    first_stage();
    issue_first();
    top(0);  // every tile through the general path
    if (again) general_tile(0, std::true_type{});
    for (j = 1; j < n_tiles; ++j) {
      top(j);
      if (again) general_tile(j, std::false_type{});
    }
    wait_vmcnt<0>();
    __syncthreads();  // the epilogue writes into the stages
  }

  const int lane = lane_id_here();
  float l[NR];
#pragma unroll
  for (int rg = 0; rg < NR; ++rg) l[rg] = quad_sum(lsum[rg]);
  auto store = [&](auto x) __attribute__((always_inline)) {  // the groups of 32 rows
    constexpr int X = decltype(x)::value;
    if (u.part >= 0) {  // a piece: the accumulators as they stand
      const size_t at = size_t(u.part) * 8 + pair0 + X;
      store_tile16_as_part<2 * X>(parts + at * (32 * D), acc, lane);
      // (running maximum and sum of row lane % 32; the combine kernel adds the sums of both lane halves)
      const bool hi = (lane >> 4) & 1;
      *reinterpret_cast<f32x2 *>(stats + (at * 64 + lane) * 2) =
          f32x2{hi ? m[2 * X + 1] : m[2 * X], lane >= 32 ? 0.f : hi ? l[2 * X + 1] : l[2 * X]};
      return;
    }
    // O = acc / l (bf16), as whole lines through a patch of LDS (the stages are free: every wave is past its last tile);
    // LSE = ln 2 * (m + log2 l)
    static_assert(W * PATCH_BYTES <= S::POS_OFF, "patches fit in the stages");
    const int h = head_of(2 * X);
    const int32_t *const rows = slot_row + slot_of(2 * X, 0);
    store_tile16_as_lines<2 * X>(lds0 + wave * PATCH_BYTES, acc, 1.0f / l[2 * X], 1.0f / l[2 * X + 1], lane,
                                 [&](int p) __attribute__((always_inline)) -> bf16_t * {
      const int rw = rows[p];
      return rw >= 0 ? O + (size_t(rw) * Hq + h) * D : nullptr;
    });
    if (lane < 32) {
      const int rw = rows[lane];
      const float mm = lane < 16 ? m[2 * X] : m[2 * X + 1], ll = lane < 16 ? l[2 * X] : l[2 * X + 1];
      if (rw >= 0) LSE[size_t(h) * total_q + rw] = 0.6931471805599453f * (mm + fast_log2(ll));
    }
  };
  store(std::integral_constant<int, 0>{});
  if constexpr (NR == 4) store(std::integral_constant<int, 1>{});
}

// Adds up the pieces of the cut units: O = sum_i 2^(m_i - M) acc_i / sum_i 2^(m_i - M) l_i with M = max_i m_i, and LSE.
// One workgroup per (unit, group of 32 rows, 64 columns); see combine_parts.
template <int D>
__global__ __launch_bounds__(256) void ca_combine_fwd_kernel(const CombineUnit *__restrict__ units,
                                                             const int32_t *__restrict__ slot_row,
                                                             const float *__restrict__ parts,
                                                             const float *__restrict__ stats, bf16_t *__restrict__ O,
                                                             float *__restrict__ LSE, int Hq, int64_t total_q) {
  constexpr int NH = D / 64;  // 64-column halves
  __shared__ __attribute__((aligned(16))) float lds[COMBINE_LDS];
  __shared__ float ml[4][64][2];
  const CombineUnit u = units[blockIdx.x / (8 * NH)];
  const int h = blockIdx.x % NH, pair = (blockIdx.x / NH) % 8;
  const int head = u.b + (pair & (u.c - 1));
  const int32_t *const rows = slot_row + u.a + (pair >> __builtin_ctz(u.c)) * 32;
  const int row = rows[threadIdx.x & 31], orow = rows[threadIdx.x >> 3];  // of the lane's row, and of the row it stores
  float m = 0.f, l = 0.f;
  combine_parts<true>(parts + size_t(u.part0) * (FWD_BM * D) + pair * (32 * D) + h * (8 * 256), FWD_BM * D,
                      stats + (size_t(u.part0) * 8 + pair) * 128, 8 * 128, u.n_parts, 1.f, lds, ml, m, l,
                      [&](int) __attribute__((always_inline)) -> bf16_t * {
                        return orow >= 0 ? O + (size_t(orow) * Hq + head) * D + 64 * h : nullptr;
                      });
  if (h == 0 && threadIdx.x < 32 && row >= 0) LSE[size_t(head) * total_q + row] = 0.6931471805599453f * (m + fast_log2(l));
}

template <int D>
static hipError_t launch_fwd_t(const ca_plan_t *p, const void *q, const void *k, const void *v, void *o, float *lse,
                               void *parts, hipStream_t st) {
  if (p->fwd_units.empty()) return hipSuccess;
  const float c = p->scale * 1.4426950408889634f;
  float *const pp = static_cast<float *>(parts);
  float *const stats = pp ? pp + size_t(p->n_fwd_parts) * (FWD_BM * D) : nullptr;
  const size_t n = pp ? p->fwd_pieces.size() : p->fwd_units.size();
  const FwdForm form = pp ? p->fwd_piece_form : p->fwd_form;
  auto launch = [&](auto halves) {
    constexpr bool HALVES = decltype(halves)::value;
    auto kern = ca_fwd_kernel<D, HALVES>;
    constexpr int SMEM = FwdSmem<D>::TOTAL;
    static std::atomic<bool> attr_done[16];  // once per device; a second thread repeating the call is harmless
    if (!attr_done[p->device & 15].load(std::memory_order_acquire)) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
      if (e != hipSuccess) return e;
      attr_done[p->device & 15].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3(unsigned(HALVES ? 2 * n : n)), dim3(256), SMEM, st, pp ? p->d_fwd_pieces : p->d_fwd_units, int(n),
                       int(form.turns), p->d_slot_row, p->d_slot_pos, static_cast<const bf16_t *>(q), static_cast<const bf16_t *>(k),
                       static_cast<const bf16_t *>(v), static_cast<bf16_t *>(o), lse, pp, stats, p->hq, p->hkv, p->total_q, c);
    return hipSuccess;
  };
  const hipError_t launched = form.halves ? launch(std::true_type{}) : launch(std::false_type{});
  if (launched != hipSuccess) return launched;
  if (pp) {
    hipLaunchKernelGGL(ca_combine_fwd_kernel<D>, dim3(unsigned(p->fwd_combine.size() * 8 * (D / 64))), dim3(256), 0, st,
                       p->d_fwd_combine, p->d_slot_row, pp, stats, static_cast<bf16_t *>(o), lse, p->hq, p->total_q);
  }
  return hipGetLastError();
}

hipError_t launch_fwd(const ca_plan_t *p, const void *q, const void *k, const void *v, void *o, float *lse, void *parts,
                      hipStream_t st) {
  return p->d == 128 ? launch_fwd_t<128>(p, q, k, v, o, lse, parts, st) : launch_fwd_t<64>(p, q, k, v, o, lse, parts, st);
}

}  // namespace ca
