// The backward in one pass: dK, dV and dQ from one recomputation of S and dP (five contractions; the dK/dV and dQ kernels of
// ca_bwd.hip take seven between them).  For batches of some hundred microseconds and more (OnePass in ca_plan.cpp has the rule).
//
// A workgroup owns a tile of keys of one document and KV head (256 keys and eight waves at head_dim 128, 128 keys and four waves
// at 64), keeps dK and dV in registers like the dK/dV kernel and walks the document's query rows backwards, 32 rows of one query
// head per step.  Lane <-> key:
//   S = Q K^T, dP = dO V^T, P = exp2(c S - L2), dS = P (dP - Delta), dV^T += dO^T P, dK^T += Q^T dS       (as in ca_bwd.hip)
// What is new is dQ^T[16 columns per wave] += K^T dS^T over all keys of the tile: dS of the step before, which every wave has left
// in LDS, comes back through transposing reads, K transposed stays in registers (its natural fragments come from LDS instead).
// The sums of dQ so far are fp32 in memory.  They are added to in the order of the tiles: tile j + 1 waits until tile j has added
// to the 32-row tile of dQ (a counter per wave and tile), loads the sums as the MFMAs' C operand, and stores them back; the
// last tile that a row sees writes bf16 dQ.  So dQ is the sum the dQ kernel forms, in its order: all results are
// the same bit for bit as those of whole units in the other kernels, and from run to run.  (Where those are finite: what a NaN or Inf
// in one row of Q, K, V or dO reaches here is part of what it reaches there.)
//
// Why plain loads and stores: all tiles of one (document, KV head) run on one XCD, so the sums live in its L2, the point of
// coherence of its CUs.  There an ordered load-add-store of 16 KiB tiles by 64 workgroups per XCD runs at 15 to 18 TB/s read + written over the
// chip; fp32 atomic adds retire at 1.36 TB/s.  A load has to bypass the CU's own vector L1 (sc1); a store has arrived in L2
// when vmcnt says so.  A workgroup asks which XCD it is on and takes units from that XCD's queue; a queue that no XCD has claimed
// yet is claimed by whoever gets to it, so every unit is run on any partition of the chip.  A unit only waits for units that were
// taken before it from the same queue, so the first unit that is not finished never waits for one that nobody runs.
//
// Why 256 keys at head_dim 128: the sums move once per tile, 16 KiB read and written per 32 rows of a head, half of what 128 keys
// cost (without waiting for, loading and storing them the kernel would take 141 of 157 ms).  One workgroup fills a CU, and its waves leave every barrier together; a wave's priority falls
// from phase to phase, so the one that is behind goes first (163.0 -> 161.5 ms).  LDS fragments come through a ring of registers
// across the phases (S alone 1100 -> 480 cycles of a step), addresses are made with few scalar instructions (605 -> 503 instructions per
// step, 174 -> 163 ms), the turn at dQ is taken early in dV (159 -> 157 ms).  128K tokens in shuffled shards, 32/8 heads, head_dim 128:
// 177 ms in two kernels, 157 in this one (64K tokens of documents of about 2K: 8.3 -> 7.5 ms; last 1000 rows of 130K: 5.8 -> 5.2 ms).
// Waves whose keys a block below the diagonal does not see only add dQ there (7.50 -> 7.35 ms on the 64K tokens).  That what a row does
// not see may hold Inf or NaN costs 0.4 % on the 128K tokens, 0.9 % on the 64K, up to 2 % on shards in contexts of 1K.
// Matrix pipe busy 53 % of the time at 1.9 GHz, 56 % while two waves are there (dK/dV kernel 76 %, dQ kernel 66 %): what is left is
// barriers, LDS latency after them, waits for turns.
// Tried and not kept: workgroups of 128 keys, two to a CU (188 ms: the sums move twice as often); half the waves adding dQ at the
// start of a step and half at its end (+3 %); dK of a step after the next barrier (+4 %: nothing is left to cover the sums' loads), dQ
// before dK (+3 %); polls by direct loads to LDS at the start of a step (+2 %: older values); every other run of 32 tiles walked
// forwards (+2.5 %); the next unit's ticket and first tiles on their way before dK and dV are stored (+0.5 %; level on short units).
// The pause between polls must stay: without it they take the L2 from everybody (5 to 40 times slower); longer ones change nothing.
#include <algorithm>
#include <atomic>
#include <type_traits>
#include <utility>

#include "ca_device.h"
#include "ca_fused.h"

namespace ca {

constexpr float LOG2E = 1.4426950408889634f;

template <class F, int... I>
__device__ __forceinline__ void static_for(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
// f(0) .. f(N - 1), each with a constant
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
  static_for(f, std::make_integer_sequence<int, N>{});
}

// The order in which a wave uses the fragments of a step: 4 NK of K and Q (S; two of 16 keys and two of 16 rows for 32 columns at a
// time), 2 NK of dO (dP), ND of dO transposed (dV), ND of Q transposed (dK), 2 W of dS (dQ).  They come from LDS through a ring of
// R fragments' registers, as far ahead as there is room beside what else is alive.
template <int D>
struct FusedRing {
  static constexpr int NK = D / 32, ND = D / 16;
  static constexpr int DO = 4 * NK, DV = DO + 2 * NK, DK = DV + ND, DQ = DK + ND, N = DQ + 2 * fused_waves(D);
  static constexpr int R = 7, AHEAD_DP = 2, AHEAD = 4;
  // how many are there or on their way once `used` of them have been used
  static constexpr int fetched(int used) {
    if (used <= DO) return used + R < DO + AHEAD_DP ? used + R : DO + AHEAD_DP;
    if (used < DV) return used + AHEAD_DP;
    return used + AHEAD < N ? used + AHEAD : N;
  }
};

template <int D>
struct FusedSmem {
  static constexpr int W = fused_waves(D), KEYS = 32 * W;
  static constexpr int NST = 2;
  static constexpr int TILE = FUSED_BQ * 2 * D;  // one Q or dO tile of 32 slots
  static constexpr int Q_OFF = 0;
  static constexpr int DO_OFF = TILE;
  static constexpr int L2_OFF = 2 * TILE;       // 32 floats of log2e * LSE
  static constexpr int DL_OFF = L2_OFF + 128;   // 32 floats of -Delta
  static constexpr int POS_OFF = L2_OFF + 256;  // 64 positions, those of the block
  static constexpr int SPARE_OFF = POS_OFF + 256;
  static constexpr int STAGE = 2 * TILE + 1024;
  static constexpr int K_OFF = NST * STAGE;          // the unit's K tile
  static constexpr int DS_OFF = K_OFF + KEYS * 2 * D;  // dS of two steps, [KEYS][32 rows] each
  static constexpr int DS_BYTES = KEYS * 64;
  static constexpr int TICKET_OFF = DS_OFF + 2 * DS_BYTES;
  static constexpr int TOTAL = TICKET_OFF + 16;
  static_assert(W * PATCH_BYTES <= TICKET_OFF, "patches fit in the rest");
  static_assert(K_OFF % 1024 == 0 && DS_OFF % 1024 == 0);
};

constexpr int SC1 = 16;  // cache policy of a load of what other CUs of the XCD have written: not from this CU's vector L1
// Polls (of about a microsecond) that a wave makes in all while it runs a unit.  By the order in which units are taken every turn comes
// long before.  If one does not, the wave marks its additions as LOST from there on, whoever waits for them does the same, and
// the last of them writes NaN to dQ: nobody goes on from a sum that lacks some.
constexpr int MAX_POLLS = 1 << 22, LOST = -1;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void *base_uniform, uint32_t bytes) {
  const uint64_t b = (uint64_t)(uintptr_t)base_uniform;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void *)(uintptr_t)(((uint64_t)hi << 32) | lo), 0, int(bytes), 0x00027000);
}
// Direct loads global -> LDS through a buffer descriptor: lane i's 16 (or 4) bytes from base + lane_off + tile_off land at lds_off +
// 16 i (or 4 i).  Assembly for the same reason as load_lds16_sbase.  (The compiler does not see a vector-memory instruction here:
// with the nop there are five wait states behind a restored spill of one of its scalar operands.)
__device__ __forceinline__ void load_lds16_buf(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t tile_off, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 3\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" : : "v"(lane_off), "s"(r), "s"(tile_off), "s"(lds_off) : "memory", "m0");
}
__device__ __forceinline__ void load_lds4_buf(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t tile_off, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 3\n\tbuffer_load_dword %0, %1, %2 offen lds" : : "v"(lane_off), "s"(r), "s"(tile_off), "s"(lds_off) : "memory", "m0");
}
// Keeps what is computed from an address from being computed ahead of this point, and kept or spilled
__device__ __forceinline__ void fresh(int &a) { asm volatile("" : "+v"(a)); }
__device__ __forceinline__ float uniform(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}

template <int D>
__device__ __forceinline__ void fused_unit(const BwdUnit u, const FusedArgs &a, const int wave) {
  using S = FusedSmem<D>;
  constexpr int W = S::W, KEYS = S::KEYS;
  constexpr int NK = D / 32, ND = D / 16, CH = D / 8, RPI = 64 / CH, NST = S::NST;
  static_assert(FUSED_BQ == W * RPI, "one direct load per wave per Q (or dO) tile");
  constexpr int ROWB = 2 * D, HALF = 16 * ROWB;
  constexpr int LPI = 3;                     // direct loads per wave per step
  constexpr int NDW = ND / W, NQ = 2 * NDW;  // 16-column tiles of dQ that a wave computes; its accumulators
  static_assert(NDW >= 1);
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(CA_LDS char *)smem;
  const int G = a.hq / a.hkv;
  const float c = uniform(a.scale * LOG2E);
  const int lane = lane_id_here(), j = lane >> 4, li = lane & 15;
  const int kw0 = 32 * wave;
  const int hk = u.kv_head;
  const int n_blocks = (u.slot_end - u.slot_begin) / BWD_BQ;
  const int run_len = 2 * u.heads;  // steps per block: two halves of 32 rows for each tile
  const int n_it = n_blocks * run_len;
  const int n_full = (u.slot_end - u.slot_full) / BWD_BQ * run_len;
  const int order = u.key_pos0 / KEYS;  // the tile's place in the order of additions to dQ

  // Tiles of 32 rows are counted as [block][head][half]; a step's follows the one before, but for the first of a block.
  const int block0 = u.slot_begin / BWD_BQ + n_blocks - 1;
  const int tile0 = (block0 * a.hq + hk * G) * 2, jump = 2 * a.hq + run_len;
  int ld_left = n_it, ld_tile = tile0, ld_run = run_len, ld_block = block0, ld_stage = 0;
  const __amdgpu_buffer_rsrc_t rq = rsrc_of(a.q_sorted, a.copy_bytes), rdo = rsrc_of(a.do_sorted, a.copy_bytes),
                               raux = wave == 0 ? rsrc_of(a.stats_kv, ~0u) : rsrc_of(a.pos_kv, ~0u);
  const uint32_t aux_lds = wave == 0 ? S::L2_OFF : wave == 1 ? S::POS_OFF : S::SPARE_OFF;
  // the loads of the next step, in three parts; after the last step, its loads once more (into the other stage, which nobody reads)
  auto issue_q = [&](uint32_t &off) __attribute__((always_inline)) {
    const int il = lane_id_here(), trow = RPI * wave + il / CH;
    off = uint32_t(trow * ROWB + 16 * ((il % CH) ^ tile_sw<D>(trow)));
    load_lds16_buf(rq, off, uint32_t(ld_tile) * (FUSED_BQ * ROWB), lds0 + ld_stage * S::STAGE + S::Q_OFF + RPI * wave * ROWB);
  };
  auto issue_do = [&](uint32_t off) __attribute__((always_inline)) {
    load_lds16_buf(rdo, off, uint32_t(ld_tile) * (FUSED_BQ * ROWB), lds0 + ld_stage * S::STAGE + S::DO_OFF + RPI * wave * ROWB);
  };
  auto issue_aux = [&]() __attribute__((always_inline)) {
    load_lds4_buf(raux, uint32_t(lane_id_here()) * 4, uint32_t(wave == 0 ? ld_tile : ld_block) * 256, lds0 + ld_stage * S::STAGE + aux_lds);
    ld_stage = ld_stage + 1 == NST ? 0 : ld_stage + 1;
    if (--ld_left > 0) {
      ++ld_tile;
      if (--ld_run == 0) ld_run = run_len, ld_tile -= jump, --ld_block;
    }
  };
  // K tile -> LDS, 32 rows per wave
  {
    const uint32_t kv_row_bytes = uint32_t(a.hkv) * ROWB;
    const char *kg = reinterpret_cast<const char *>(a.k + (size_t(u.kv_row) * a.hkv + hk) * D);
#pragma unroll
    for (int n = 0; n < 32 / RPI; ++n) {
      const int r = kw0 + RPI * n + lane / CH;
      const uint32_t off = uint32_t(min(r, u.n_valid - 1)) * kv_row_bytes + 16 * ((lane % CH) ^ tile_sw<D>(r));
      load_lds16_sbase(kg, off, lds0 + S::K_OFF + (kw0 + RPI * n) * ROWB);
    }
  }
  if (n_it > 0) {
    uint32_t off;
    issue_q(off), issue_do(off), issue_aux();
  }
  // steps until the blocks, walked backwards, no longer see the wave's first key (looked up for the first 64 blocks)
  const int unseen = lane < n_blocks && a.pos_kv[u.slot_begin + lane * BWD_BQ + BWD_BQ - 1] < u.key_pos0 + kw0;
  const int n_seen = __builtin_amdgcn_readfirstlane(max(n_full, n_it - run_len * __builtin_popcountll(__ballot(unseen))));
  bf16x8 vf[NK][2];
#pragma unroll
  for (int kg = 0; kg < 2; ++kg) {
    const int key = min(kw0 + 16 * kg + li, u.n_valid - 1);
    const size_t off = (size_t(u.kv_row + key) * a.hkv + hk) * D + 8 * j;
#pragma unroll
    for (int s = 0; s < NK; ++s) {
      vf[s][kg] = *reinterpret_cast<const bf16x8 *>(a.v + off + 32 * s);
    }
  }
  wait_vmcnt<0>();
#pragma unroll
  for (int s = 0; s < NK; ++s) pin(vf[s][0]), pin(vf[s][1]);
  barrier_nofence();  // K is there
  bf16x8 kt[W][NDW];  // K transposed: the wave's columns of dQ, all keys
  const auto kt_address = [&]() __attribute__((always_inline)) {
    const int l = lane_id_here();
    return int(lds0 + S::K_OFF + (l >> 2) * ROWB + 16 * (((l >> 1) & 1) ^ tile_sw<D>(l >> 2)) + 8 * (l & 1)) ^ (32 * NDW * wave);
  };
  auto fetch_kt = [&](int t0, int key, int i) __attribute__((always_inline)) -> bf16x8 {  // of keys `key` (a multiple of 32) .. + 31
    const int t = (t0 ^ (32 * i)) + key * ROWB;
    return join(lds_read_tr4_at(t), lds_read_tr4_at(t + HALF));
  };
  {
    const int t0 = kt_address();
#pragma unroll
    for (int ks = 0; ks < W; ++ks)
#pragma unroll
      for (int i = 0; i < NDW; ++i) kt[ks][i] = fetch_kt(t0, 32 * ks, i), pin(kt[ks][i]);
  }
  // A zero masks a product only if the other factor is finite, and what a row does not see may hold Inf or NaN.  So a unit with a
  // diagonal multiplies the wave's part of K transposed, and V of its keys, by zeros once.  Where that does not give zeros, masked steps
  // leave out the keys that their rows do not see (last_dq, rest_of_dq), and dS is zero where P is.  (Leaving them out always: shards in
  // contexts of up to 1K to 3K keys 1.7 % slower.)
  bool k_finite = true, v_finite = true;
  if (n_full < n_it) {
    const bf16x8 zero = __builtin_bit_cast(bf16x8, u32x4{0, 0, 0, 0});
    f32x4 x[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int ks = 0; ks < W; ++ks)
#pragma unroll
      for (int i = 0; i < NDW; ++i) x[0] = mfma16(kt[ks][i], zero, x[0]);
#pragma unroll
    for (int s = 0; s < NK; ++s) x[1] = mfma16(zero, vf[s][1], mfma16(zero, vf[s][0], x[1]));
    auto finite = [&](const f32x4 &y) __attribute__((always_inline)) { return __ballot(y[0] + y[1] + y[2] + y[3] != 0.f) == 0; };
    k_finite = finite(x[0]), v_finite = finite(x[1]);
  }
  int kb = lds0 + S::K_OFF + (kw0 + li) * ROWB + 16 * (j ^ tile_sw<D>(li));
  int nb = lds0 + li * ROWB + 16 * (j ^ tile_sw<D>(li));
  int tb = lds0 + (4 * j + (li >> 2)) * ROWB + 16 * (((li >> 1) & 1) ^ tile_sw<D>(4 * j + (li >> 2))) + 8 * (li & 1);
  int auxo = lds0 + 16 * j, stage = 0;

  f32x4 acc_dk[ND][2], acc_dv[ND][2];
#pragma unroll
  for (int b = 0; b < ND; ++b)
#pragma unroll
    for (int kg = 0; kg < 2; ++kg) acc_dk[b][kg] = acc_dv[b][kg] = f32x4{0.f, 0.f, 0.f, 0.f};

  const __amdgpu_buffer_rsrc_t rf = rsrc_of(a.flags, a.flag_bytes);
  // sums of dQ so far (a descriptor of no bytes: the loads of the first tile in the order return zeros), and with this unit's part
  const __amdgpu_buffer_rsrc_t rsum = rsrc_of(a.dq_sums, order > 0 ? a.dq_bytes : 0), rout = rsrc_of(a.dq_sums, a.dq_bytes);
  constexpr int DQ_TILE = FUSED_BQ * D * 4;
  auto dq_at = [&](int t) __attribute__((always_inline)) { return uint32_t(t) * DQ_TILE + wave * (NQ * 1024); };
  int tile = tile0, run = run_len;  // of the step
  // dQ of the step before: its tile (-1: none), and the last of this unit's keys that its rows see (ALL_KEYS: some row sees a later
  // one too; otherwise this unit is the last to add to the tile)
  constexpr int ALL_KEYS = KEYS + 31;
  int prev = -1, prev_run = 0, prev_seen = -1;
  int pending = -1;   // the tile whose additions are on their way, and not yet made known
  int polls_left = MAX_POLLS;  // 0: a turn has not come
  int dsb = 0;        // which of the two dS buffers the step writes
  auto flag_at = [&](int t) __attribute__((always_inline)) { return (t * W + wave) * 4; };
  auto publish = [&]() __attribute__((always_inline)) {
    // (the stores have arrived in L2)
    if (pending >= 0) {
      __builtin_amdgcn_raw_buffer_store_b32(opaque(polls_left > 0 ? order + 1 : LOST), rf, 0, flag_at(pending), 0);  // (all lanes the same)
      pending = -1;
    }
  };
  f32x4 dq[NDW][2];
#pragma unroll
  for (int i = 0; i < NQ; ++i) dq[i / 2][i & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
  // this wave's turn at the tile of dQ: wait for the tile before in the order, then fetch the sums so far
  auto take_turn = [&](int seen) __attribute__((always_inline)) {
    if (order > 0 && prev >= 0 && __builtin_amdgcn_readfirstlane(seen) < order) {
      for (; polls_left > 0; --polls_left) {
        asm volatile("" ::: "memory");  // every poll is a load of its own
        const int at = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_raw_buffer_load_b32(rf, 0, flag_at(prev), SC1));
        if (at >= order) break;
        if (at == LOST) {
          polls_left = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
      asm volatile("" ::: "memory");
    }
    const int il = lane_id_here() * 16;
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      dq[i / 2][i & 1] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsum, il + 1024 * i, dq_at(max(prev, 0)), SC1));
  };
  // fragments of dS of the step before: of k-step f / 2 (32 keys), 16 rows
  auto ds_address = [&]() __attribute__((always_inline)) {
    const int rl = lane_id_here(), rj = rl >> 4;
    return int(lds0) + S::DS_OFF + (dsb ^ 1) * S::DS_BYTES + (rl >> 2) * 64 + 8 * ((rl & 3) ^ ((rj & 1) << 2) ^ (rj & 2));
  };
  auto fetch_ds = [&](int ds_rd, int f) __attribute__((always_inline)) -> bf16x8 {
    const int t = (f % 2 == 0 ? ds_rd : ds_rd ^ 32) + 2048 * (f / 2);
    return join(lds_read_tr4_at(t), lds_read_tr4_at(t + 1024));
  };
  // dQ of the step before from the 32 keys of which its rows see some, without the others
  auto rest_of_dq = [&]() __attribute__((always_inline)) {
    const int begin = (prev_seen + 1) & ~31;
    if (k_finite || begin > prev_seen) return;
    const int at = ds_address() + 64 * begin;
    const bf16x8 g[2] = {fetch_ds(at, 0), fetch_ds(at, 1)};
    const int last = prev_seen - begin - 4 * (lane_id_here() >> 4);  // the lane holds keys 0 .. 3 and 16 .. 19 from here on
#pragma unroll
    for (int i = 0; i < NDW; ++i) {
      u32x4 w = __builtin_bit_cast(u32x4, fetch_kt(kt_address(), begin, i));
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const int first = 16 * (n >> 1) + 2 * (n & 1);
        w[n] = last > first ? w[n] : last == first ? w[n] & 0xffffu : 0u;
      }
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) dq[i][rt] = mfma16(__builtin_bit_cast(bf16x8, w), g[rt], dq[i][rt]);
    }
  };
  // dQ of the step before where nothing else is to be done
  auto last_dq = [&]() __attribute__((always_inline)) {
    const int ds_rd = ds_address();
    bf16x8 g[4];
    static_for<4>([&](auto f) __attribute__((always_inline)) { g[f] = fetch_ds(ds_rd, f); });
    static_for<W>([&](auto ks) __attribute__((always_inline)) {
      constexpr int at = 2 * ks % 4;
      __builtin_amdgcn_sched_barrier(0);
      if (k_finite || 32 * ks + 31 <= prev_seen) {
#pragma unroll
        for (int i = 0; i < NDW; ++i) dq[i][0] = mfma16(kt[ks][i], g[at], dq[i][0]), dq[i][1] = mfma16(kt[ks][i], g[at + 1], dq[i][1]);
      }
      if constexpr (ks + 2 < W) g[at] = fetch_ds(ds_rd, 2 * ks + 4), g[at + 1] = fetch_ds(ds_rd, 2 * ks + 5);
    });
    rest_of_dq();
  };
  auto store_dq = [&](const bool MAY_END) __attribute__((always_inline)) {
    if (!MAY_END || prev_seen == ALL_KEYS || prev < 0) {
      if (prev >= 0) {
        const int il = lane_id_here() * 16;
#pragma unroll
        for (int i = 0; i < NQ; ++i) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, dq[i / 2][i & 1]), rout, il + 1024 * i, dq_at(prev), 0);
      }
      pending = prev;
    } else {
      const int ol = lane_id_here(), rpk = BWD_BQ * u.heads / G;  // rows of a head in the tile: 64, or fewer where heads share it
      const int blk = prev / (2 * a.hq), at = run_len - prev_run;  // the step in its block
      const float f = polls_left > 0 ? a.scale : __builtin_nanf("");
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        const int tr = 32 * (at & 1) + 16 * rt + (ol & 15);
        const int row = a.slot_row[int64_t(blk) * BWD_BQ + tr % rpk];
        const int head = hk * G + (at >> 1) * (BWD_BQ / rpk) + tr / rpk;
        if (row >= 0) {
          bf16_t *dst = a.dq + (size_t(row) * a.hq + head) * D + 16 * NDW * wave + 4 * (ol >> 4);
#pragma unroll
          for (int i = 0; i < NDW; ++i)
            *reinterpret_cast<u32x2 *>(dst + 16 * i) = u32x2{pack_bf16(dq[i][rt][0] * f, dq[i][rt][1] * f), pack_bf16(dq[i][rt][2] * f, dq[i][rt][3] * f)};
        }
      }
    }
  };

  // S, P, dP, dV, dS and dK of a step for the wave's keys (sees: some row sees some of them), and dQ of the step before for its columns
  auto compute = [&](const bool MASK, const bool sees) __attribute__((always_inline)) {
    using F = FusedRing<D>;
    constexpr int R = F::R;
    bf16x8 fr[R];
    int ds_rd = 0;
    auto fetch = [&](int f) __attribute__((always_inline)) -> bf16x8 {
      if (f < F::DO) {
        const int s = f / 4, i = f % 4;  // K0, Q1, K1, Q0
        const int base = i % 2 == 0 ? kb : nb;
        return lds_read8_at((i % 2 == 0 ? HALF * (i / 2) : S::Q_OFF + HALF * (1 - i / 2)) + (base ^ (64 * s)));
      }
      if (f < F::DV) {
        const int g = f - F::DO;
        return lds_read8_at(S::DO_OFF + HALF * (g / NK) + (nb ^ (64 * (g % NK))));
      }
      if (f < F::DQ) {
        const int b = (f - F::DV) % ND, t = (f < F::DK ? S::DO_OFF : S::Q_OFF) + (tb ^ (32 * b));
        return join(lds_read_tr4_at(t), lds_read_tr4_at(HALF + t));
      }
      if (f == F::DQ) ds_rd = ds_address();
      return fetch_ds(ds_rd, f - F::DQ);
    };
    auto fetch_range = [&](auto from, auto to) __attribute__((always_inline)) {
      static_for<to - from>([&](auto i) __attribute__((always_inline)) { fr[(from + i) % R] = fetch(from + i); });
      __builtin_amdgcn_sched_barrier(0);
    };
    // a fragment of Q or dO transposed, or zeros: rows that see none of the wave's keys may hold Inf or NaN as well
    auto rows_seen = [&](const bf16x8 &x) __attribute__((always_inline)) {
      u32x4 w = __builtin_bit_cast(u32x4, x);
#pragma unroll
      for (int n = 0; n < 4; ++n) w[n] = !MASK || sees ? w[n] : 0u;
      return __builtin_bit_cast(bf16x8, w);
    };
    // fragments at .. at + n - 1 have been used
    auto used = [&](auto at, auto n) __attribute__((always_inline)) {
      fetch_range(std::integral_constant<int, F::fetched(at)>{}, std::integral_constant<int, F::fetched(at + n)>{});
    };
    constexpr std::integral_constant<int, 0> none{};
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    f32x4 sa[2][2], pa[2][2];  // [16 rows][16 keys]: S, then P; dP - Delta
    f32x4 nd, l2v;
    fetch_range(none, std::integral_constant<int, F::fetched(0)>{});
    __builtin_amdgcn_s_setprio(3);  // (see the top)
    uint32_t ld_off = 0;
    static_for<NK>([&](auto s) __attribute__((always_inline)) {
      constexpr int at = 4 * s, k0 = at % R, q1 = (at + 1) % R, k1 = (at + 2) % R, q0 = (at + 3) % R;
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      sa[0][0] = mfma16(fr[q0], fr[k0], s == 0 ? zero : sa[0][0]);
      sa[1][0] = mfma16(fr[q1], fr[k0], s == 0 ? zero : sa[1][0]);
      used(std::integral_constant<int, at>{}, one);
      if (s == 0) issue_q(ld_off);
      if (s == 1) issue_do(ld_off);
      sa[1][1] = mfma16(fr[q1], fr[k1], s == 0 ? zero : sa[1][1]);
      used(std::integral_constant<int, at + 1>{}, one);
      if (s == NK - 1) nd = lds_ld<f32x4>(S::DL_OFF + auxo), l2v = lds_ld<f32x4>(S::L2_OFF + auxo);
      sa[0][1] = mfma16(fr[q0], fr[k1], s == 0 ? zero : sa[0][1]);
      used(std::integral_constant<int, at + 2>{}, two);
      fresh(nb), fresh(kb);
      if (s == 1) issue_aux();
    });
    fresh(tb);
    __builtin_amdgcn_s_setprio(2);
    const int seen = __builtin_amdgcn_raw_buffer_load_b32(rf, 0, flag_at(max(prev, 0)), SC1);
    // dP in two halves of 16 rows: P, and dS of the first half, are ready when the second half's MFMAs are
    uint32_t pw[2][4], dw[2][4];
    auto pack_pair = [&](int rt, int i) __attribute__((always_inline)) {
      const int e = 2 * (i & 1), kg = i >> 1;
      pw[kg][2 * rt + e / 2] = pack_bf16(sa[rt][kg][e], sa[rt][kg][e + 1]);
      dw[kg][2 * rt + e / 2] = pack_bf16(sa[rt][kg][e] * pa[rt][kg][e], sa[rt][kg][e + 1] * pa[rt][kg][e + 1]);
      asm volatile("" : "+v"(dw[kg][2 * rt + e / 2]));  // (here: not sunk to where dS is used, with S and dP alive until then)
    };
    static_for<2>([&](auto rt) __attribute__((always_inline)) {
      static_for<NK>([&](auto f) __attribute__((always_inline)) {
        constexpr int at = F::DO + rt * NK + f;
#pragma unroll
        for (int kg = 0; kg < 2; ++kg) pa[rt][kg] = mfma16(fr[at % R], vf[f][kg], f == 0 ? nd : pa[rt][kg]);
#pragma unroll
        for (int i = 8 * f / NK; i < 8 * (f + 1) / NK; ++i) {
          const int e = i & 3, kg = i >> 2;
          sa[rt][kg][e] = fast_exp2(fmaf(sa[rt][kg][e], c, -l2v[e]));
        }
        if (rt == 0 && f == NK - 1) nd = lds_ld<f32x4>(S::DL_OFF + 64 + auxo), l2v = lds_ld<f32x4>(S::L2_OFF + 64 + auxo);
        if (rt == 1) {
#pragma unroll
          for (int i = 4 * f / NK; i < 4 * (f + 1) / NK; ++i) pack_pair(0, i);
        }
        used(std::integral_constant<int, at>{}, one);
        fresh(nb);
      });
      if (MASK) {
        const int key_pos = u.key_pos0 + kw0 + (lane_id_here() & 15);
        const u32x4 pv = lds_ld<u32x4>(S::POS_OFF + 128 * ((run_len - run) & 1) + 64 * rt + auxo);
#pragma unroll
        for (int kg = 0; kg < 2; ++kg)
#pragma unroll
          for (int e = 0; e < 4; ++e) sa[rt][kg][e] = key_pos + 16 * kg <= int(pv[e]) ? sa[rt][kg][e] : 0.f;
      }
    });
    __builtin_amdgcn_s_setprio(1);
    bf16x8 pb[2], db[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) pack_pair(1, i);
    if (MASK && !(v_finite && sees)) {  // dS is zero where P is, whatever V and dO hold
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t p = pw[i >> 2][i & 3];
        dw[i >> 2][i & 3] &= (p & 0xffffu ? 0xffffu : 0u) | (p >> 16 ? 0xffff0000u : 0u);
      }
    }
#pragma unroll
    for (int kg = 0; kg < 2; ++kg) pb[kg] = __builtin_bit_cast(bf16x8, u32x4{pw[kg][0], pw[kg][1], pw[kg][2], pw[kg][3]});
    __builtin_amdgcn_sched_barrier(0);
    static_for<ND>([&](auto b) __attribute__((always_inline)) {
      constexpr int at = F::DV + b;
#pragma unroll
      for (int kg = 0; kg < 2; ++kg) acc_dv[b][kg] = mfma16(rows_seen(fr[at % R]), pb[kg], acc_dv[b][kg]);
      used(std::integral_constant<int, at>{}, one);
      if (b == 0) {
        wait_vmcnt<0>();
        publish();
        take_turn(seen);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int kg = 0; kg < 2; ++kg) db[kg] = __builtin_bit_cast(bf16x8, u32x4{dw[kg][0], dw[kg][1], dw[kg][2], dw[kg][3]});
    static_for<ND>([&](auto b) __attribute__((always_inline)) {
      constexpr int at = F::DK + b;
#pragma unroll
      for (int kg = 0; kg < 2; ++kg) acc_dk[b][kg] = mfma16(rows_seen(fr[at % R]), db[kg], acc_dk[b][kg]);
      if (b == 0) {
        const int wl = lane_id_here();
        const uint32_t ds_wr = lds0 + S::DS_OFF + dsb * S::DS_BYTES + (kw0 + (wl & 15)) * 64 + 8 * ((wl >> 4) ^ (wl & 4) ^ ((wl >> 2) & 2));
#pragma unroll
        for (int kg = 0; kg < 2; ++kg) {
          *(CA_LDS u32x2 *)(uintptr_t)(ds_wr + 1024 * kg) = u32x2{dw[kg][0], dw[kg][1]};
          *(CA_LDS u32x2 *)(uintptr_t)((ds_wr ^ 32) + 1024 * kg) = u32x2{dw[kg][2], dw[kg][3]};
        }
      }
      used(std::integral_constant<int, at>{}, one);
    });
    if (MASK && !k_finite) return;  // (to last_dq)
    static_for<2 * W>([&](auto f) __attribute__((always_inline)) {
      constexpr int at = F::DQ + f;
#pragma unroll
      for (int i = 0; i < NDW; ++i) dq[i][f % 2] = mfma16(kt[f / 2][i], fr[at % R], dq[i][f % 2]);
      used(std::integral_constant<int, at>{}, one);
    });
  };

  // ... of a step in which no row sees any of the wave's keys: dS is zero
  auto idle = [&]() __attribute__((always_inline)) {
    uint32_t off;
    issue_q(off), issue_do(off), issue_aux();
    wait_vmcnt<0>();
    publish();
    take_turn(-1);
    const uint32_t ds_wr = lds0 + S::DS_OFF + dsb * S::DS_BYTES + kw0 * 64 + 16 * lane_id_here(), zero = opaque(0);
#pragma unroll
    for (int n = 0; n < 2; ++n) *(CA_LDS u32x4 *)(uintptr_t)(ds_wr + 1024 * n) = u32x4{zero, zero, zero, zero};
  };

  int it = 0;
  auto step = [&](const bool MASK, const bool IDLE) __attribute__((always_inline)) {
    // the step's tiles have landed (this wave's part): younger are at most the stores of dQ of the step before the last
    if (!MASK && it > 1) wait_vmcnt<NQ>();
    else wait_vmcnt<0>();
    barrier_nofence();  // ... and everybody else's; everybody is done with the step before, whose dS is complete
    int seen = ALL_KEYS;  // the last key of the tile that some row sees
    if (MASK) {
      seen = __builtin_amdgcn_readfirstlane(lds_ld<int>(lds0 + stage * S::STAGE + S::POS_OFF + (32 * ((run_len - run) & 1) + 31) * 4)) - u.key_pos0;
      if (seen >= KEYS) seen = ALL_KEYS;
    }
    if (IDLE) idle();
    else compute(MASK, seen >= kw0);
    if (MASK && (IDLE || !k_finite)) last_dq();
    store_dq(MASK);
    prev = seen >= 0 ? tile : -1, prev_run = run, prev_seen = seen;
    dsb ^= 1;
    ++tile;
    if (--run == 0) run = run_len, tile -= jump;
    const int adv = stage == NST - 1 ? -(NST - 1) * S::STAGE : S::STAGE;
    stage = stage == NST - 1 ? 0 : stage + 1;
    nb += adv, tb += adv, auxo += adv;
  };
  for (; it < n_full; ++it) step(false, false);
  for (; it < n_seen; ++it) step(true, false);
  for (; it < n_it; ++it) step(true, true);
  wait_vmcnt<0>();
  publish();
  barrier_nofence();  // dS of the last step
  take_turn(-1);
  last_dq();
  store_dq(true);
  wait_vmcnt<0>();
  publish();
  const int ol = lane_id_here();
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 2; ++t)
    store_tile16_as_lines<0>(lds0 + wave * PATCH_BYTES, t == 0 ? acc_dk : acc_dv, t == 0 ? a.scale : 1.0f, t == 0 ? a.scale : 1.0f, ol,
                             [&](int p) __attribute__((always_inline)) -> bf16_t * {
      const int key = kw0 + p;
      return key < u.n_valid ? (t == 0 ? a.dk : a.dv) + (size_t(u.kv_row + key) * a.hkv + hk) * D : nullptr;
    });
}

template <int D>
__global__ __launch_bounds__(64 * fused_waves(D), fused_waves(D) == 8 ? 2 : 3) void ca_bwd_fused_kernel(const FusedArgs a) {
  using S = FusedSmem<D>;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(CA_LDS char *)smem;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int xcc = __builtin_amdgcn_s_getreg(20 | (31 << 11)) & (N_XCD - 1);
  for (int i = 0; i < N_XCD; ++i) {
    const int qi = (xcc + i) & (N_XCD - 1);
    const int begin = a.queue[qi], end = a.queue[qi + 1];
    for (;;) {
      __syncthreads();
      if (wave == 0 && lane_id_here() == 0) {
        int *const ctrl = a.ctrl + 64 * qi;
        int t = end - begin;
        int was = 0;
        if (__hip_atomic_compare_exchange_strong(ctrl, &was, xcc + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) || was == xcc + 1)
          t = __hip_atomic_fetch_add(ctrl + 32, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *(CA_LDS int *)(uintptr_t)(lds0 + opaque(S::TICKET_OFF)) = t;
      }
      __syncthreads();
      const int t = __builtin_amdgcn_readfirstlane(lds_ld<int>(lds0 + opaque(S::TICKET_OFF)));
      if (t >= end - begin) break;
      fused_unit<D>(a.units[begin + t], a, wave);
    }
  }
}

template <int D>
static hipError_t launch_t(const FusedArgs &a, int device, hipStream_t st) {
  auto kern = ca_bwd_fused_kernel<D>;
  constexpr int SMEM = FusedSmem<D>::TOTAL, PER_CU = fused_waves(D) == 8 ? 1 : 3;
  static std::atomic<bool> done[16];
  if (!done[device & 15].load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return e;
    done[device & 15].store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(kern, dim3(unsigned(PER_CU * N_CU)), dim3(64 * fused_waves(D)), SMEM, st, a);
  return hipSuccess;
}
hipError_t launch_bwd_fused(const FusedArgs &a, int d, int device, hipStream_t st) {
  return d == 128 ? launch_t<128>(a, device, st) : launch_t<64>(a, device, st);
}

}  // namespace ca
