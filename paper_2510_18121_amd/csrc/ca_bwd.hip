// Backward kernels: dQ, dK, dV of L = sum(dO * O) with P recomputed from the saved log-sum-exp
// (Section 2.1: P is not stored in forward, it is recomputed during backward).
//
//   prep : per (slot, head): -Delta = -<dO, O> and L2 = log2(e) * LSE, stored in SLOT order (the order of the
//          planner's per-document sorted query rows), so that both main kernels read them contiguously.
//          Padding slots get L2 = +huge, which makes their recomputed probabilities exactly 0.
//   dq   : one workgroup = one of the forward's work units (256 query slots x one query head, or 256/hp slots x hp
//          heads of one KV group), walking over the document's keys like the forward does.  Lane <-> query row:
//            S^T = K Q^T, dP^T = V dO^T, P^T = exp2(c S^T - L2), dS^T = P^T (dP^T - Delta),
//            dQ^T += K^T dS^T   (K^T through transposing LDS reads of the same K tile)
//   dkv  : one workgroup = 128 keys of one document x one KV head, walking over every block of 64 query
//          slots that can see them, for each query head of the group.  Lane <-> key:
//            S = Q K^T, dP = dO V^T (K, V fragments of the wave's 32 keys stay in registers),
//            dV^T += dO^T P, dK^T += Q^T dS   (Q^T, dO^T through transposing LDS reads)
//          dK and dV are written once, already summed over the group's heads and all tasks of the document.
//   joint: both kinds of workgroup in one launch, for batches that fill the chip with neither.
//   combine: adds up the fp32 partial results of units that the planner cut into pieces, in order, and stores them.
// All products are v_mfma_f32_16x16x32_bf16.  On N(0,1) operands the chip's power limit, not the matrix pipe, sets the rate, and
// this shape costs less energy per flop than 32x32x16 (alone 1928 against 1741 TFLOP/s).  Its price is twice the MFMA
// instructions, each about 9 cycles of the vector issue port (probe; an exponential 9, other vector instructions 4): 870 port
// cycles per 1024 matrix cycles in the dK/dV kernel, 726 per 768 in the dQ kernel.  32x32x16 -> 16x16x32 with everything else
// alike, 128K tokens of long and short documents in shuffled shards (32/8 heads, head_dim 128): dK/dV kernel 108.0 -> 104.2 ms,
// dQ kernel 82.2 -> 77.4 ms.
// No atomics and no fp32 dQ accumulation: the price is that S and dP are computed in both kernels (7 contractions
// instead of the minimal 5).  Results are deterministic.  All but small batches take five, in ca_bwd_fused.hip, with the same
// results.
#include <algorithm>
#include <atomic>

#include "ca_device.h"
#include "ca_fused.h"
#include "ca_internal.h"

namespace ca {

constexpr float LOG2E = 1.4426950408889634f;
constexpr float L2_PADDING = 1.0e30f;  // exp2(x - 1e30) == 0 for every finite score

__global__ void ca_bwd_prep_kernel(const int32_t *__restrict__ slot_row, const int32_t *__restrict__ block_rpk,
                                   const bf16_t *__restrict__ Q, const bf16_t *__restrict__ O,
                                   const bf16_t *__restrict__ dO, const float *__restrict__ LSE,
                                   float *__restrict__ delta_slot, float *__restrict__ l2_slot,
                                   float *__restrict__ stats_kv,
                                   bf16_t *__restrict__ q_sorted, bf16_t *__restrict__ do_sorted,
                                   u32x4 *__restrict__ zero, int64_t zero16, int64_t padded, int64_t total_q, int Hq, int G,
                                   int D) {
  // D/8 lanes per (slot, head): -Delta = -<dO, O> and log2(e)*LSE in slot order (for the dQ kernel), and for the
  // dK/dV kernel the slot-ordered copies of Q and dO as [block of 64 slots][head][64][D] - the 64-row tile of a
  // (block, head) is one contiguous run, and the tiles of the heads of a block follow each other - with the same two
  // statistics in the row order of those tiles (padding rows: zeros, with an LSE that makes every probability 0).
  // In a packed block (a document of at most rpk = 16 or 32 rows) tile t of a KV group holds the rows of the group's
  // heads 64/rpk t .. 64/rpk (t + 1) - 1, rpk rows each; the group's remaining tiles are neither written nor read.
  const int lanes = D / 8;
  const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx < zero16) zero[idx] = u32x4{0, 0, 0, 0};
  const int64_t pair = idx / lanes;
  const int c = int(idx % lanes);
  const bool ok = pair < padded * Hq;
  const int64_t slot = ok ? pair / Hq : 0;
  const int h = int(pair % Hq);
  const int row = ok ? slot_row[slot] : -1;
  float s = 0.f;
  u32x4 qv = {0, 0, 0, 0}, dv = {0, 0, 0, 0};
  if (row >= 0) {
    const size_t off = (size_t(row) * Hq + h) * D + 8 * c;
    const bf16x8 a = *reinterpret_cast<const bf16x8 *>(O + off);
    const bf16x8 b = *reinterpret_cast<const bf16x8 *>(dO + off);
    qv = *reinterpret_cast<const u32x4 *>(Q + off);
    dv = __builtin_bit_cast(u32x4, b);
#pragma unroll
    for (int i = 0; i < 8; ++i) s += float(a[i]) * float(b[i]);
  }
  for (int o = lanes / 2; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (ok) {
    const float nd = row >= 0 ? -s : 0.f;  // stored negated: both kernels add it
    const float l2 = row >= 0 && c == 0 ? LSE[int64_t(h) * total_q + row] * LOG2E : L2_PADDING;
    const int64_t blk = slot / BWD_BQ;
    const int rpk = block_rpk[blk];
    int th = h, tr = int(slot % BWD_BQ);  // tile (as a head index) and row of this (slot, head) in the dK/dV tiles
    bool in_tile = true;
    if (rpk != 0) {
      const int hpk = BWD_BQ / rpk, hg = h % G;
      in_tile = tr < rpk;  // the slots beyond are padding of the document
      th = h - hg + hg / hpk;
      tr += (hg % hpk) * rpk;
    }
    if (in_tile) {
      const size_t so = ((size_t(blk) * Hq + th) * BWD_BQ + tr) * D + 8 * c;
      *reinterpret_cast<u32x4 *>(q_sorted + so) = qv;
      *reinterpret_cast<u32x4 *>(do_sorted + so) = dv;
    }
    if (c == 0) {
      delta_slot[int64_t(h) * padded + slot] = nd;
      l2_slot[int64_t(h) * padded + slot] = l2;
      if (in_tile) {
        float *const st = stats_kv + ((blk * Hq + th) * 2 + tr / 32) * 64 + tr % 32;
        st[0] = l2, st[32] = nd;
      }
    }
  }
}

__global__ void ca_fill_zero_kernel(u32x4 *__restrict__ p, int64_t n16) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n16; i += stride) p[i] = u32x4{0, 0, 0, 0};
}

// ------------------------------------------------------------------------------------------------ dQ
// Eight waves on a CU of their own have four stages; workgroups of four, two to a CU, share its LDS.
template <int D, int W>
struct DqSmem {
  static constexpr int NST = D == 128 && W == 4 ? 2 : 4;
  static constexpr int TILE = FWD_BN * 2 * D;
  // a stage holds the K tile and then the V tile of one key block: both are reached from one address register
  // through the 16-bit offset field of the LDS instructions
  static constexpr int K_OFF = 0;
  static constexpr int V_OFF = TILE;
  static constexpr int STAGE = 2 * TILE;
  static constexpr int TOTAL = NST * STAGE;
};

// The workgroup of W waves: all eight 32-row groups of the unit (W = 8), or groups 4 half .. 4 half + 3 of them.  Both do the same
// arithmetic in the same order, so dQ does not depend on which of them computes it.
// The order of a 32-key block is written out: its fragments are fetched AHEAD of the MFMAs that use them through a ring of
// registers, the exponentials go between the MFMAs of dP, and fences keep the compiler from bunching either.  Left to the
// compiler, the same arithmetic waited for LDS in every pair of dQ's MFMAs: 77.3 -> 74.8 ms (128K tokens, 32/8 heads).
template <int D, int W>
__device__ __forceinline__ void dq_workgroup(const FwdUnit &u, const int half, const int32_t *__restrict__ slot_row,
                                             const int32_t *__restrict__ slot_pos, const bf16_t *__restrict__ Q,
                                             const bf16_t *__restrict__ K, const bf16_t *__restrict__ V,
                                             const bf16_t *__restrict__ dO, const float *__restrict__ l2_slot,
                                             const float *__restrict__ delta_slot, bf16_t *__restrict__ dQ,
                                             float *__restrict__ parts, int Hq, int Hkv, int64_t padded, float scale) {
  using S = DqSmem<D, W>;
  constexpr int NK = D / 32, ND = D / 16, CH = D / 8, RPI = 64 / CH, NLD = FWD_BN / (W * RPI), NST = S::NST;
  constexpr int ROWB = 2 * D, HALF = 16 * ROWB;
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const uint32_t lds0 = (uint32_t)(uintptr_t)(CA_LDS char *)smem;  // LDS byte address of the dynamic segment
  const int tid = threadIdx.x, lane = tid & 63, j4 = lane >> 4, li = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hk = __builtin_amdgcn_readfirstlane(u.head / (Hq / Hkv));  // (uniform, for scalar K/V addresses)
  // (group of the unit) -> (32-slot group, query head) inside the unit, as in the forward kernel
  const int hp_lg = __builtin_ctz(u.hp), pair = W * half + wave;
  const int head = u.head + (pair & (u.hp - 1));
  const int slot = u.slot0 + (pair >> hp_lg) * 32 + li;  // the lane's first query row (the other is 16 further on)
  int row[2], pos[2];
  float l2[2], dl[2];
#pragma unroll
  for (int rg = 0; rg < 2; ++rg) {
    row[rg] = slot_row[slot + 16 * rg];
    pos[rg] = slot_pos[slot + 16 * rg] - u.key0;  // counted from the first key of a piece's window (below 0: sees none of it)
    l2[rg] = l2_slot[int64_t(head) * padded + slot + 16 * rg];
    dl[rg] = delta_slot[int64_t(head) * padded + slot + 16 * rg];
  }
  const int wmax = wave_max(max(pos[0], pos[1])), wmin = wave_min(min(pos[0], pos[1]));
  // tiles some row of the workgroup sees (positions are sorted; at least one, which then is masked)
  int n_tiles = (u.n_keys + FWD_BN - 1) / FWD_BN;
  if (W < 8) {
    const int last = slot_pos[u.slot0 + ((W * half + W - 1) >> hp_lg) * 32 + 31] - u.key0;
    n_tiles = max(1, min(n_tiles, last / FWD_BN + 1));
  }
  const float c = scale * LOG2E;

  // direct loads addressed as (scalar tile base) + (per-lane 32-bit offset); rows past the last key are fetched as the last key,
  // and with more than two stages tiles past the end as the last tile (the wait at the top of a tile counts loads)
  const uint32_t kv_row_bytes = uint32_t(Hkv) * D * 2;
  const int ld_row0 = RPI * wave + lane / CH;  // + W*RPI*n
  const uint32_t ld_cbytes = uint32_t((lane % CH) ^ tile_sw<D>(ld_row0)) * 16;
  const int last_tile = n_tiles - 1, last_key_in_tile = min(FWD_BN, u.n_keys - last_tile * FWD_BN) - 1;
  const uint32_t ld_off = uint32_t(ld_row0) * kv_row_bytes + ld_cbytes;  // + W*RPI*n rows (the swizzle repeats every 16)
  static_assert(W * RPI % 16 == 0);
  const char *kg = reinterpret_cast<const char *>(K + (size_t(u.kv_row0) * Hkv + hk) * D);
  const char *vg = reinterpret_cast<const char *>(V + (size_t(u.kv_row0) * Hkv + hk) * D);
  const size_t tile_bytes = size_t(FWD_BN) * kv_row_bytes;
  auto issue_kv = [&](int tile) __attribute__((always_inline)) {
    const bool last = tile >= last_tile;
    const size_t at = size_t(last ? last_tile : tile) * tile_bytes;
    const uint32_t dst = lds0 + uint32_t((tile % NST) * S::STAGE + 1024 * wave);
    if (!last) {
#pragma unroll
      for (int n = 0; n < NLD; ++n) {
        load_lds16_sbase(kg + at + n * W * RPI * kv_row_bytes, ld_off, dst + S::K_OFF + 1024 * W * n);
        load_lds16_sbase(vg + at + n * W * RPI * kv_row_bytes, ld_off, dst + S::V_OFF + 1024 * W * n);
      }
    } else {
#pragma unroll
      for (int n = 0; n < NLD; ++n) {
        const uint32_t off = uint32_t(min(ld_row0 + W * RPI * n, last_key_in_tile)) * kv_row_bytes + ld_cbytes;
        load_lds16_sbase(kg + at, off, dst + S::K_OFF + 1024 * W * n);
        load_lds16_sbase(vg + at, off, dst + S::V_OFF + 1024 * W * n);
      }
    }
  };
#pragma unroll
  for (int t = 0; t < NST - 1; ++t) issue_kv(t);

  // Q and dO fragments (B operands); lane holds row's elements 32 s + 8 j4 .. +7
  bf16x8 qf[NK][2], dof[NK][2];
#pragma unroll
  for (int rg = 0; rg < 2; ++rg) {
    const size_t off = (size_t(row[rg] < 0 ? 0 : row[rg]) * Hq + head) * D + 8 * j4;
#pragma unroll
    for (int s = 0; s < NK; ++s) {
      qf[s][rg] = *reinterpret_cast<const bf16x8 *>(Q + off + 32 * s);
      dof[s][rg] = *reinterpret_cast<const bf16x8 *>(dO + off + 32 * s);
    }
  }
  int koff = lds0 + li * ROWB + 16 * (j4 ^ tile_sw<D>(li));
  int toff = lds0 + (4 * j4 + (li >> 2)) * ROWB + 16 * (((li >> 1) & 1) ^ tile_sw<D>(4 * j4 + (li >> 2))) + 8 * (li & 1);

  f32x4 acc[ND][2];
#pragma unroll
  for (int b = 0; b < ND; ++b) acc[b][0] = acc[b][1] = f32x4{0.f, 0.f, 0.f, 0.f};

  // All register loads above are complete from here on, so the compiler places no vector-memory waits
  // inside the loop (they would drain the direct-load queue every iteration).
  wait_vmcnt<0>();
  f32x4 nd[2];  // -Delta, from which the dP chains start
#pragma unroll
  for (int rg = 0; rg < 2; ++rg) {
#pragma unroll
    for (int s = 0; s < NK; ++s) pin(qf[s][rg]), pin(dof[s][rg]);
    pin(l2[rg]), pin(dl[rg]);
    nd[rg] = f32x4{dl[rg], dl[rg], dl[rg], dl[rg]};
  }

  for (int j = 0; j < n_tiles; ++j) {
    const int j0 = j * FWD_BN;
    wait_vmcnt<2 * (NST - 2) * NLD>();  // this wave's parts of K(j), V(j) have landed
    barrier_nofence();      // ... and everybody else's; everybody is done with tile j-1
    if (NST > 2 || j < last_tile) issue_kv(j + NST - 1);
    const bool seen = j0 <= wmax;  // some row of this wave sees the tile
    const bool masked = j0 + FWD_BN - 1 > wmin;
    // one 64-key tile; MASKED is a compile-time constant in each of the two instantiations below
    auto tile = [&](const bool MASKED) __attribute__((always_inline)) {
      // Fragments come from LDS AHEAD fragments before the MFMAs that use them: per 32-key block 2 NK of K (scores), 2 NK of V
      // (dP) and ND of K transposed (dQ).
      constexpr int NF = 2 * NK + 2 * NK + ND, AHEAD = 4;
      bf16x8 fr[AHEAD];
      auto fetch = [&](int i) __attribute__((always_inline)) -> bf16x8 {
        const int kb = i / NF, f = i % NF;
        const int KT = S::K_OFF + 32 * kb * ROWB, VT = S::V_OFF + 32 * kb * ROWB;
        if (f < 4 * NK) return lds_read8_at((f < 2 * NK ? KT : VT) + HALF * (f & 1) + (koff ^ (64 * (f % (2 * NK) / 2))));
        const int ta = toff ^ (32 * (f - 4 * NK));
        return join(lds_read_tr4_at(KT + ta), lds_read_tr4_at(KT + HALF + ta));
      };
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) fr[i] = fetch(i);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        auto next = [&](int f) __attribute__((always_inline)) {  // fragment f is used: its registers take the one AHEAD later
          if (NF * kb + f + AHEAD < 2 * NF) fr[f % AHEAD] = fetch(NF * kb + f + AHEAD);
        };
        static_assert(NF % AHEAD == 0);
        f32x4 sa[2][2], pa[2][2];  // [16 keys][16 rows]
#pragma unroll
        for (int f = 0; f < 2 * NK; ++f) {
#pragma unroll
          for (int rg = 0; rg < 2; ++rg) sa[f & 1][rg] = mfma16(fr[f % AHEAD], qf[f / 2][rg], f < 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : sa[f & 1][rg]);
          next(f);
          __builtin_amdgcn_sched_barrier(0);
        }
        float p[2][2][4];
#pragma unroll
        for (int f = 0; f < 2 * NK; ++f) {
          const int kt = f & 1;
#pragma unroll
          for (int rg = 0; rg < 2; ++rg) pa[kt][rg] = mfma16(fr[f % AHEAD], dof[f / 2][rg], f < 2 ? nd[rg] : pa[kt][rg]);
          next(2 * NK + f);
          // 16 probabilities over 2 NK slots
#pragma unroll
          for (int i = 16 * f / (2 * NK); i < 16 * (f + 1) / (2 * NK); ++i) {
            const int e = i & 3, ekt = (i >> 2) & 1, rg = i >> 3;
            p[ekt][rg][e] = fast_exp2(fmaf(sa[ekt][rg][e], c, -l2[rg]));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        uint32_t dw[2][4];
#pragma unroll
        for (int rg = 0; rg < 2; ++rg) {
          // register e of tile kt holds key j0 + 32 kb + 16 kt + 4 j4 + e: visible iff 16 kt + e <= vis
          const int vis = pos[rg] - (j0 + 32 * kb + 4 * j4);
#pragma unroll
          for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
              float p0 = p[kt][rg][e], p1 = p[kt][rg][e + 1];
              if (MASKED) {
                p0 = 16 * kt + e <= vis ? p0 : 0.f;
                p1 = 16 * kt + e + 1 <= vis ? p1 : 0.f;
              }
              dw[rg][2 * kt + e / 2] = pack_bf16(p0 * pa[kt][rg][e], p1 * pa[kt][rg][e + 1]);
            }
        }
        bf16x8 db[2];
#pragma unroll
        for (int rg = 0; rg < 2; ++rg) db[rg] = __builtin_bit_cast(bf16x8, u32x4{dw[rg][0], dw[rg][1], dw[rg][2], dw[rg][3]});
#pragma unroll
        for (int b = 0; b < ND; ++b) {
#pragma unroll
          for (int rg = 0; rg < 2; ++rg) acc[b][rg] = mfma16(fr[b % AHEAD], db[rg], acc[b][rg]);
          next(4 * NK + b);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    if (seen) {
      if (masked) tile(true);
      else tile(false);
    }
    // the offsets follow the stages round
    const int adv = (j % NST) == NST - 1 ? -(NST - 1) * S::STAGE : S::STAGE;
    koff += adv, toff += adv;
  }
  wait_vmcnt<0>();
  const int out_lane = lane_id_here();
  if (u.part >= 0) {  // a piece: the accumulators as they stand
    store_tile16_as_part<0>(parts + size_t(u.part) * (FWD_BM * D) + pair * (32 * D), acc, out_lane);
    return;
  }
  // dQ of the wave's 32 rows, as whole lines through a patch of LDS (the stages are free once every wave is past its
  // last tile)
  __syncthreads();
  static_assert(W * PATCH_BYTES <= S::TOTAL, "patches fit in the stages");
  store_tile16_as_lines<0>(lds0 + wave * PATCH_BYTES, acc, scale, scale, out_lane, [&](int p) __attribute__((always_inline)) -> bf16_t * {
    const int r0 = __shfl(row[0], p & 15), r1 = __shfl(row[1], p & 15);
    const int rw = p < 16 ? r0 : r1;
    return rw >= 0 ? dQ + (size_t(rw) * Hq + head) * D : nullptr;
  });
}

template <int D>
__global__ __launch_bounds__(512, 2) void ca_bwd_dq_kernel(const FwdUnit *__restrict__ units,
                                                           const int32_t *__restrict__ slot_row,
                                                           const int32_t *__restrict__ slot_pos,
                                                           const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K,
                                                           const bf16_t *__restrict__ V, const bf16_t *__restrict__ dO,
                                                           const float *__restrict__ l2_slot,
                                                           const float *__restrict__ delta_slot,
                                                           bf16_t *__restrict__ dQ, float *__restrict__ parts, int Hq,
                                                           int Hkv, int64_t padded, float scale) {
  dq_workgroup<D, 8>(units[blockIdx.x], 0, slot_row, slot_pos, Q, K, V, dO, l2_slot, delta_slot, dQ, parts, Hq, Hkv, padded,
                     scale);
}

// ------------------------------------------------------------------------------------------------ dK, dV
template <int D>
struct DkvSmem {
  static constexpr int NST = D == 128 ? 2 : 3;      // two workgroups share a CU's LDS at head_dim 128, three at 64
  static constexpr int TILE = BWD_BQ * 2 * D;       // one Q or dO tile of 64 slots
  static constexpr int Q_OFF = 0;
  static constexpr int DO_OFF = TILE;
  static constexpr int L2_OFF = 2 * TILE;           // 64 floats each: 32 L2 and 32 -Delta of either half of the rows, positions, spare
  static constexpr int DL_OFF = L2_OFF + 128;
  static constexpr int POS_OFF = L2_OFF + 512;
  static constexpr int SPARE_OFF = POS_OFF + 256;
  static constexpr int STAGE = 2 * TILE + 1024;
  static constexpr int TOTAL = NST * STAGE;
  static_assert(4 * PATCH_BYTES <= TOTAL, "patches fit in the stages");
};

// A unit, or a chain of short units one after the other, in a workgroup of four waves, each of which owns 32 keys: K and V
// fragments (64 registers at head_dim 128) and dK / dV accumulators (128) stay in registers, and what is left of 256 holds one
// 32 x 32 tile of S and of dP and a ring of LDS fragments, so that two waves share a SIMD.  The two are of different workgroups
// and drift apart: one's exponentials, LDS latencies, barriers, first fetches and stores run under the other's MFMAs.  One wave
// per SIMD with 472 registers, its stream software-pipelined by hand across sub-blocks and across the units of a chain, did that
// less well everywhere (both with 32x32 MFMAs; dK/dV kernel, 32/8 heads unless noted): 222 -> 181 us on 4K tokens of documents
// of about 1K, 5.04 -> 4.76 ms on 64K tokens of about 2K, 112.7 -> 107.9 ms on 128K tokens of long and short documents, 3.85 ->
// 3.50 ms on the last 1000 rows of 130K, 3.55 -> 3.05 ms on lone 64-row shards with contexts (8/2).  Workgroups no longer wait for
// each other to share Q/dO tiles in L2.
// To stay within the registers, LDS addresses are one register per kind of read, from which an exclusive or makes the address of
// each fragment (4 cycles per 2 MFMAs), and what the lane index gives is derived again where it is needed.
template <int D>
__device__ __forceinline__ void dkv_workgroup(const int me /* index of the first unit */, const BwdUnit *__restrict__ units,
                                              const int32_t *__restrict__ slot_pos, const bf16_t *__restrict__ Qs,
                                              const bf16_t *__restrict__ K, const bf16_t *__restrict__ V,
                                              const bf16_t *__restrict__ dOs, const float *__restrict__ stats_kv,
                                              bf16_t *__restrict__ dK,
                                              bf16_t *__restrict__ dV, float *__restrict__ parts, int Hq, int Hkv, float scale) {
  using S = DkvSmem<D>;
  constexpr int NK = D / 32, ND = D / 16, CH = D / 8, RPI = 64 / CH, NST = S::NST;
  constexpr int NLD = BWD_BQ / (4 * RPI);  // direct loads per wave per Q (or dO) tile
  constexpr int RPW = BWD_BQ / 4;          // tile rows fetched by one wave (contiguous)
  constexpr int ROWB = 2 * D;
  constexpr int LPI = 2 * NLD + 1;  // loads per wave per iteration
  constexpr int SUB = 32 * ROWB, HALF = 16 * ROWB;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(CA_LDS char *)smem;  // LDS byte address of the dynamic segment
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int G = Hq / Hkv;
  const float c = scale * LOG2E;
  const int64_t head_stride = BWD_BQ * D * 2;            // bytes between the tiles of consecutive heads of a block
  const int64_t block_stride = int64_t(Hq) * head_stride;  // ... of consecutive blocks, same head
  const BwdUnit *up = units + me;
  const int count = up->count, follow = up->follow;
  for (int done = 0;;) {
    const BwdUnit u = *up;
    const int lane = lane_id_here(), j = lane >> 4, li = lane & 15;
    const int kw0 = 32 * wave;
    const int hk = u.kv_head;
    const int n_blocks = (u.slot_end - u.slot_begin) / BWD_BQ;
    const int Gu = u.heads;  // tiles per block: the heads of the group, or fewer in a block of packed rows
    const int n_it = n_blocks * Gu;
    // Query blocks are walked from the document's LAST block backwards: the blocks that lie entirely below the diagonal of this KV
    // tile come first and need no mask, and workgroups that run side by side on an XCD (same KV head, neighbouring KV tiles)
    // start on the same Q/dO tiles.
    const int n_full = ((u.slot_end - u.slot_full) / BWD_BQ) * Gu;

    // Loads of one (block, head): this wave fetches tile rows RPW*wave .. of Q and of dO, RPI rows per load, plus one 64-float
    // auxiliary array: log2e*LSE and -Delta of 32 rows each (waves 0 and 1), slot positions (wave 2; wave 3 the same into a spare
    // area, so that every wave issues the same number of loads).  Q and dO come from their slot-ordered copies [block][head][64][D], in which
    // the tile of a (block, head) is one contiguous run: a load is (wave-uniform tile address) + (per-lane constant).
    const int trow = RPW * wave + lane / CH;
    const uint32_t ld_off = uint32_t(trow * ROWB + 16 * ((lane % CH) ^ tile_sw<D>(trow)));
    int left = n_it;  // tiles still to be fetched
    int ph = 0, pst = 0;
    const int64_t tile0 = (int64_t(u.slot_begin / BWD_BQ + n_blocks - 1) * Hq + hk * G) * head_stride;
    const char *q_tile = reinterpret_cast<const char *>(Qs) + tile0, *do_tile = reinterpret_cast<const char *>(dOs) + tile0;
    const int64_t aux_hstride = wave < 2 ? 128 : 0, aux_bstride = wave < 2 ? int64_t(Hq) * 128 : BWD_BQ;
    const float *aux_ptr = (wave < 2 ? stats_kv + hk * G * 128 + wave * 64 : reinterpret_cast<const float *>(slot_pos)) +
                           (u.slot_begin / BWD_BQ + n_blocks - 1) * aux_bstride;
    const uint32_t aux_lds = wave < 2 ? S::L2_OFF + 256 * wave : wave == 2 ? S::POS_OFF : S::SPARE_OFF;
    auto issue_next = [&]() __attribute__((always_inline)) {
      const uint32_t st = lds0 + pst * S::STAGE;
      uint32_t ld0 = ld_off;
      asm volatile("" : "+v"(ld0));
#pragma unroll
      for (int n = 0; n < NLD; ++n) {
        // (rows RPI n further down; the swizzle of the row changes by an exclusive or)
        const uint32_t off = (ld0 ^ (D == 128 ? 16 * (2 * ((n & 1) ^ (n >> 1)) + (n >> 1)) : 48 * n)) + RPI * n * ROWB;
        load_lds16_sbase(q_tile, off, st + S::Q_OFF + (RPW * wave + RPI * n) * ROWB);
        load_lds16_sbase(do_tile, off, st + S::DO_OFF + (RPW * wave + RPI * n) * ROWB);
      }
      load_lds4_sbase(aux_ptr, uint32_t(lane_id_here()) * 4, st + aux_lds);
      pst = pst + 1 == NST ? 0 : pst + 1;
      if (--left <= 0) return;
      if (ph + 1 < Gu) {  // next tile of the group, same block
        ++ph;
        q_tile += head_stride, do_tile += head_stride, aux_ptr += aux_hstride;
      } else {  // first head of the group, previous block
        ph = 0;
        q_tile -= (Gu - 1) * head_stride + block_stride, do_tile -= (Gu - 1) * head_stride + block_stride;
        aux_ptr -= (Gu - 1) * aux_hstride + aux_bstride;
      }
    };
    if (n_it > 0) {
#pragma unroll
      for (int i = 0; i < NST - 1; ++i) issue_next();
    }

    // K, V fragments of the wave's 32 keys (B operands of S = Q K^T and dP = dO V^T).  Keys past the document's last key are
    // clamped; their positions exceed every query position, so they are masked.
    bf16x8 kf[NK][2], vf[NK][2];
#pragma unroll
    for (int kg = 0; kg < 2; ++kg) {
      const int key = min(kw0 + 16 * kg + li, u.n_valid - 1);
      const size_t off = (size_t(u.kv_row + key) * Hkv + hk) * D + 8 * j;
#pragma unroll
      for (int s = 0; s < NK; ++s) {
        kf[s][kg] = *reinterpret_cast<const bf16x8 *>(K + off + 32 * s);
        vf[s][kg] = *reinterpret_cast<const bf16x8 *>(V + off + 32 * s);
      }
    }
    wait_vmcnt<0>();  // (from here on the compiler places no vector-memory waits: they would drain the direct loads)
#pragma unroll
    for (int s = 0; s < NK; ++s) pin(kf[s][0]), pin(kf[s][1]), pin(vf[s][0]), pin(vf[s][1]);
    // natural reads, transposing reads and row statistics in the current stage
    int nb = lds0 + li * ROWB + 16 * (j ^ tile_sw<D>(li));
    int tb = lds0 + (4 * j + (li >> 2)) * ROWB + 16 * (((li >> 1) & 1) ^ tile_sw<D>(4 * j + (li >> 2))) + 8 * (li & 1);
    int auxo = lds0 + 16 * j, stage = 0;

    f32x4 acc_dk[ND][2], acc_dv[ND][2];
#pragma unroll
    for (int b = 0; b < ND; ++b)
#pragma unroll
      for (int kg = 0; kg < 2; ++kg) acc_dk[b][kg] = acc_dv[b][kg] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Sub-blocks [QB0, QB1) of 32 rows each; MASK: some row of the block does not see some key of the tile.
    // Fragments come from LDS AHEAD fragments before the MFMAs that use them: per sub-block 2 NK of Q (scores), 2 NK of dO
    // (dP), ND of dO transposed (dV) and ND of Q transposed (dK).  The exponentials go between the MFMAs of dP, dS between those of
    // dV: 4.60 -> 4.31 ms on 64K tokens of documents of about 2K, 103.7 -> 99.9 ms on 128K tokens (32/8 heads), against
    // the compiler's order.  (3 ahead is within 0.5 %, and does not fit the registers.)
    constexpr int NF = 4 * NK + 2 * ND, AHEAD = 2;
    auto sub_blocks = [&](const int QB0, const int QB1, const bool MASK) __attribute__((always_inline)) {
      bf16x8 fr[AHEAD];
      auto fetch = [&](int i) __attribute__((always_inline)) -> bf16x8 {
        const int qb = i / NF, f = i % NF;
        const int QT = S::Q_OFF + qb * SUB, DOT = S::DO_OFF + qb * SUB;
        if (f < 4 * NK) return lds_read8_at((f < 2 * NK ? QT : DOT) + HALF * (f & 1) + (f % (2 * NK) < 2 ? nb : xor_here(nb, 64 * (f % (2 * NK) / 2))));
        const int t = (f < 4 * NK + ND ? DOT : QT) + ((f - 4 * NK) % ND == 0 ? tb : xor_here(tb, 32 * ((f - 4 * NK) % ND)));
        return join(lds_read_tr4_at(t), lds_read_tr4_at(HALF + t));
      };
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) fr[i] = fetch(NF * QB0 + i);
#pragma unroll
      for (int qb = QB0; qb < QB1; ++qb) {
        int at = NF * (qb - QB0);  // the fragment in use, counted from the first
        auto next = [&]() __attribute__((always_inline)) {  // it has been used: its registers take the one AHEAD later
          if (at + AHEAD < NF * (QB1 - QB0)) fr[at % AHEAD] = fetch(NF * QB0 + at + AHEAD);
          ++at;
          __builtin_amdgcn_sched_barrier(0);
        };
        f32x4 sa[2][2], pa[2][2];  // [16 rows][16 keys]: S, and dP - Delta: its chain starts from -Delta
        f32x4 nd[2], l2v[2];
#pragma unroll
        for (int f = 0; f < 2 * NK; ++f) {
          if (f == 2 * NK - 2) {
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) nd[rt] = lds_ld<f32x4>(S::DL_OFF + 256 * qb + 64 * rt + auxo);
          }
          if (f == 2 * NK - 1) {
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) l2v[rt] = lds_ld<f32x4>(S::L2_OFF + 256 * qb + 64 * rt + auxo);
          }
#pragma unroll
          for (int kg = 0; kg < 2; ++kg) sa[f & 1][kg] = mfma16(fr[at % AHEAD], kf[f / 2][kg], f < 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : sa[f & 1][kg]);
          next();
        }
#pragma unroll
        for (int f = 0; f < 2 * NK; ++f) {
#pragma unroll
          for (int kg = 0; kg < 2; ++kg) pa[f & 1][kg] = mfma16(fr[at % AHEAD], vf[f / 2][kg], f < 2 ? nd[f & 1] : pa[f & 1][kg]);
          // P, in place of S: 16 values over 2 NK slots
#pragma unroll
          for (int i = 16 * f / (2 * NK); i < 16 * (f + 1) / (2 * NK); ++i) {
            const int e = i & 3, kg = (i >> 2) & 1, rt = i >> 3;
            sa[rt][kg][e] = fast_exp2(fmaf(sa[rt][kg][e], c, -l2v[rt][e]));
          }
          next();
        }
        if (MASK) {
#pragma unroll
          for (int rt = 0; rt < 2; ++rt) {
            const int key_pos = u.key_pos0 + kw0 + (lane_id_here() & 15);  // position of this lane's first key (the other is 16 further on)
            const u32x4 pv = lds_ld<u32x4>(S::POS_OFF + (32 * qb + 16 * rt) * 4 + auxo);
#pragma unroll
            for (int kg = 0; kg < 2; ++kg)
#pragma unroll
              for (int e = 0; e < 4; ++e) sa[rt][kg][e] = key_pos + 16 * kg <= int(pv[e]) ? sa[rt][kg][e] : 0.f;
          }
        }
        bf16x8 pb[2], db[2];
        uint32_t dw[2][4];
#pragma unroll
        for (int kg = 0; kg < 2; ++kg)
          pb[kg] = __builtin_bit_cast(bf16x8, u32x4{pack_bf16(sa[0][kg][0], sa[0][kg][1]), pack_bf16(sa[0][kg][2], sa[0][kg][3]),
                                                    pack_bf16(sa[1][kg][0], sa[1][kg][1]), pack_bf16(sa[1][kg][2], sa[1][kg][3])});
#pragma unroll
        for (int b = 0; b < ND; ++b) {
#pragma unroll
          for (int kg = 0; kg < 2; ++kg) acc_dv[b][kg] = mfma16(fr[at % AHEAD], pb[kg], acc_dv[b][kg]);
          // dS: 8 pairs over ND slots
#pragma unroll
          for (int i = 8 * b / ND; i < 8 * (b + 1) / ND; ++i) {
            const int e = 2 * (i & 1), rt = (i >> 1) & 1, kg = i >> 2;
            dw[kg][2 * rt + e / 2] = pack_bf16(sa[rt][kg][e] * pa[rt][kg][e], sa[rt][kg][e + 1] * pa[rt][kg][e + 1]);
          }
          next();
        }
#pragma unroll
        for (int kg = 0; kg < 2; ++kg) db[kg] = __builtin_bit_cast(bf16x8, u32x4{dw[kg][0], dw[kg][1], dw[kg][2], dw[kg][3]});
#pragma unroll
        for (int b = 0; b < ND; ++b) {
#pragma unroll
          for (int kg = 0; kg < 2; ++kg) acc_dk[b][kg] = mfma16(fr[at % AHEAD], db[kg], acc_dk[b][kg]);
          next();
        }
      }
    };
    int it = 0;
    auto step = [&](const bool MASK) __attribute__((always_inline)) {
      wait_vmcnt<(NST - 2) * LPI>();  // block `it` has landed (this wave's part); block it+1 may be in flight
      barrier_nofence();              // ... and everybody else's; everybody is done with block it-1
      if (NST > 2 || left > 0) issue_next();
      if (!MASK) {
        sub_blocks(0, 2, false);
      } else {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {  // (a sub-block entirely above the diagonal for this wave's keys is left out: positions are sorted)
          const int sub_max_pos = lds_ld<int>(lds0 + stage * S::STAGE + S::POS_OFF + (32 * qb + 31) * 4);
          if (sub_max_pos >= u.key_pos0 + kw0) sub_blocks(qb, qb + 1, true);
        }
      }
      const int adv = stage == NST - 1 ? -(NST - 1) * S::STAGE : S::STAGE;
      stage = stage == NST - 1 ? 0 : stage + 1;
      nb += adv, tb += adv, auxo += adv;
    };
    for (; it < n_full; ++it) step(false);
    for (; it < n_it; ++it) step(true);
    wait_vmcnt<0>();  // nothing may still be writing LDS
    const int ol = lane_id_here();
    if (count <= 1 && follow < 0) {  // a piece of a unit's query blocks: the accumulators as they stand
      float *const dst = parts + size_t(-1 - follow) * (FWD_BM * D) + 2 * wave * (32 * D);
      store_tile16_as_part<0>(dst, acc_dk, ol);
      store_tile16_as_part<0>(dst + 32 * D, acc_dv, ol);
      return;
    }
    __syncthreads();  // every wave is done with the stages
#pragma unroll
    for (int t = 0; t < 2; ++t)
      store_tile16_as_lines<0>(lds0 + wave * PATCH_BYTES, t == 0 ? acc_dk : acc_dv, t == 0 ? scale : 1.0f, t == 0 ? scale : 1.0f, ol,
                                [&](int p) __attribute__((always_inline)) -> bf16_t * {
        const int key = kw0 + p;
        return key < u.n_valid ? (t == 0 ? dK : dV) + (size_t(u.kv_row + key) * Hkv + hk) * D : nullptr;
      });
    if (++done >= count) return;
    __syncthreads();  // ... and with its patch
    up = units + follow + done - 1;
  }
}

template <int D>
__global__ __launch_bounds__(256, 2) void ca_bwd_dkv_kernel(const BwdUnit *__restrict__ units,
                                                            const int32_t *__restrict__ slot_pos,
                                                            const bf16_t *__restrict__ Qs, const bf16_t *__restrict__ K,
                                                            const bf16_t *__restrict__ V, const bf16_t *__restrict__ dOs,
                                                            const float *__restrict__ stats_kv, bf16_t *__restrict__ dK,
                                                            bf16_t *__restrict__ dV, float *__restrict__ parts, int Hq, int Hkv,
                                                            float scale) {
  dkv_workgroup<D>(int(blockIdx.x), units, slot_pos, Qs, K, V, dOs, stats_kv, dK, dV, parts, Hq, Hkv, scale);
}

// dK/dV units and dQ half units (workgroups of 4 groups of 32 rows) in one launch, longest first.  For batches too small to
// fill the chip with either kernel: what a launch takes there is mostly its fixed part, and the dQ work finds CUs that the
// dK/dV units leave idle.  Measured, backward, two launches against one: 49 -> 30 us (384 rows, 8/1 heads, head_dim 128), 31 -> 22 us
// (1.5K tokens, 4/2 heads, head_dim 64), 356 -> 315 us (16K tokens of documents of about 2K, 8/2 heads, where the two kernels' last
// units leave CUs idle one after the other).  Batches that fill the chip gain 1 or 2 % or lose as much, 4 % at head_dim 64: the
// planner decides by a simulation of both and a limit (JOINT_MAX_US).
struct JointArgs {
  const int32_t *order;  // what each workgroup does (ca_plan::joint_order), or nullptr
  const BwdUnit *units;
  const FwdUnit *dq_units;
  const int32_t *slot_row, *slot_pos, *pos_kv;
  const bf16_t *q, *k, *v, *d_o, *q_sorted, *do_sorted;
  const float *l2_slot, *delta_slot, *stats_kv;
  bf16_t *dq, *dk, *dv;
  float *parts_dq, *parts_kv;
  int n_dkv, n_dq, hq, hkv;
  int64_t padded;
  float scale;
};
template <int D>
__global__ __launch_bounds__(256, 2) void ca_bwd_joint_kernel(const JointArgs a) {
  const int i = int(blockIdx.x) - a.n_dkv;
  int w = int(blockIdx.x);
  if (a.order) {
    w = a.order[blockIdx.x];
  } else if (i >= 0) {
    // (all second halves before all first ones: 4.50 against 4.27 ms on lone 64-row shards with contexts, 312 against 298 us on 4K
    // tokens of documents of about 1K)
    int unit = i, half;
    half_of_unit(unit, a.n_dq, half);
    w = -1 - (unit + half * a.n_dq);
  }
  if (w >= 0) {
    dkv_workgroup<D>(w, a.units, a.pos_kv, a.q_sorted, a.k, a.v, a.do_sorted, a.stats_kv, a.dk, a.dv, a.parts_kv, a.hq, a.hkv, a.scale);
  } else {
    const int half = -1 - w >= a.n_dq ? 1 : 0;
    dq_workgroup<D, 4>(a.dq_units[-1 - w - half * a.n_dq], half, a.slot_row, a.slot_pos, a.q, a.k, a.v, a.d_o, a.l2_slot,
                       a.delta_slot, a.dq, a.parts_dq, a.hq, a.hkv, a.padded, a.scale);
  }
}

// Adds up the pieces of the cut units: dQ of the forward / dQ units (from parts_dq; 8 groups of 32 rows), then dK and dV of
// the dK/dV units (from parts_kv; 4 groups of 32 keys, two tensors).  One workgroup per (unit, group, 64 columns); see
// combine_parts.
template <int D>
__global__ __launch_bounds__(256) void ca_combine_bwd_kernel(const CombineUnit *__restrict__ units_dq, int n_dq,
                                                             const CombineUnit *__restrict__ units_kv,
                                                             const int32_t *__restrict__ slot_row,
                                                             const float *__restrict__ parts_dq,
                                                             const float *__restrict__ parts_kv,
                                                             bf16_t *__restrict__ dQ, bf16_t *__restrict__ dK,
                                                             bf16_t *__restrict__ dV, int Hq, int Hkv, float scale) {
  constexpr int NH = D / 64;  // 64-column halves
  __shared__ __attribute__((aligned(16))) float lds[COMBINE_LDS];
  __shared__ float ml[4][64][2];
  const int un = blockIdx.x / (8 * NH), h = blockIdx.x % NH, pair = (blockIdx.x / NH) % 8;
  const bool kv = un >= n_dq;
  const CombineUnit u = kv ? units_kv[un - n_dq] : units_dq[un];
  const float *src = (kv ? parts_kv : parts_dq) + size_t(u.part0) * (FWD_BM * D) + pair * (32 * D) + h * (8 * 256);
  const int row = threadIdx.x >> 3;  // the row of the tile this lane stores
  bf16_t *dst;
  float f = scale;
  if (kv) {  // pair: (32 keys, dK or dV)
    const int key = 32 * (pair >> 1) + row;
    if (pair & 1) f = 1.f;
    dst = key < u.b ? ((pair & 1) ? dV : dK) + (size_t(u.a + key) * Hkv + u.c) * D + 64 * h : nullptr;
  } else {
    const int head = u.b + (pair & (u.c - 1));
    const int rw = slot_row[u.a + (pair >> __builtin_ctz(u.c)) * 32 + row];
    dst = rw >= 0 ? dQ + (size_t(rw) * Hq + head) * D + 64 * h : nullptr;
  }
  float m, l;
  combine_parts<false>(src, FWD_BM * D, nullptr, 0, u.n_parts, f, lds, ml, m, l,
                       [&](int) __attribute__((always_inline)) { return dst; });
}

static void launch_fill(void *p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return;
  const int64_t n16 = int64_t(bytes / 16);
  const unsigned blocks = unsigned(std::min<int64_t>((n16 + 255) / 256, 256 * 32));
  hipLaunchKernelGGL(ca_fill_zero_kernel, dim3(blocks), dim3(256), 0, st, static_cast<u32x4 *>(p), n16);
}

template <class F>
static hipError_t set_smem(F kern, int bytes, int device, std::atomic<bool> *done) {
  // once per device; two threads that meet here both set the same value, which is harmless
  if (!done[device & 15].load(std::memory_order_acquire)) {
    hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    done[device & 15].store(true, std::memory_order_release);
  }
  return hipSuccess;
}

template <int D>
static hipError_t launch_bwd_t(const ca_plan_t *p, const void *q, const void *k, const void *v, const void *o,
                               const void *d_o, const float *lse, void *dq, void *dk, void *dv, void *ws,
                               bool split, bool fused, hipStream_t st, hipEvent_t *ev) {
  if (ev) (void)hipEventRecord(ev[0], st);
  const size_t q_elems = size_t(p->total_q) * p->hq * D, kv_elems = size_t(p->total_kv) * p->hkv * D;
  const int64_t padded = int64_t(p->slot_row.size());
  float *delta_slot = static_cast<float *>(ws);
  float *l2_slot = reinterpret_cast<float *>(static_cast<char *>(ws) + p->ws_off_l2);
  float *stats_kv = reinterpret_cast<float *>(static_cast<char *>(ws) + p->ws_off_stats_kv);
  bf16_t *q_sorted = reinterpret_cast<bf16_t *>(static_cast<char *>(ws) + p->ws_off_qs);
  bf16_t *do_sorted = reinterpret_cast<bf16_t *>(static_cast<char *>(ws) + p->ws_off_dos);
  // partial results of cut units, where the caller's workspace has room for them
  float *const parts_kv = split && p->n_bwd_parts > 0 ? reinterpret_cast<float *>(static_cast<char *>(ws) + p->ws_off_parts_kv) : nullptr;
  float *const parts_dq = split && p->n_fwd_parts > 0 ? reinterpret_cast<float *>(static_cast<char *>(ws) + p->ws_off_parts_dq) : nullptr;
  const int32_t n_dkv = parts_kv ? p->bwd_piece_workgroups : p->bwd_workgroups;
  auto combine = [&](bool dq_units, bool kv_units) {
    const int c_dq = dq_units && parts_dq ? int(p->fwd_combine.size()) : 0, c_kv = kv_units && parts_kv ? int(p->bwd_combine.size()) : 0;
    if (c_dq + c_kv > 0)
      hipLaunchKernelGGL(ca_combine_bwd_kernel<D>, dim3(unsigned((c_dq + c_kv) * 8 * (D / 64))), dim3(256), 0, st,
                         p->d_fwd_combine, c_dq, p->d_bwd_combine, p->d_slot_row, parts_dq, parts_kv,
                         static_cast<bf16_t *>(dq), static_cast<bf16_t *>(dk), static_cast<bf16_t *>(dv), p->hq, p->hkv,
                         p->scale);
  };
  // rows that belong to no work unit (KV outside every scheduled document, Q rows outside every task)
  if (!p->kv_covered) {
    launch_fill(dk, kv_elems * 2, st);
    launch_fill(dv, kv_elems * 2, st);
  }
  if (!p->q_covered) launch_fill(dq, q_elems * 2, st);
  if (padded > 0) {
    const int64_t threads = padded * p->hq * (D / 8);
    hipLaunchKernelGGL(ca_bwd_prep_kernel, dim3(unsigned((threads + 255) / 256)), dim3(256), 0, st, p->d_slot_row,
                       p->d_block_rpk, static_cast<const bf16_t *>(q), static_cast<const bf16_t *>(o),
                       static_cast<const bf16_t *>(d_o), lse, delta_slot, l2_slot, stats_kv, q_sorted, do_sorted,
                       reinterpret_cast<u32x4 *>(static_cast<char *>(ws) + p->ws_off_flags), fused ? int64_t(p->ws_bwd_fused - p->ws_off_flags) / 16 : int64_t(0), padded, p->total_q, p->hq, p->hq / p->hkv, D);
  }
  if (ev) (void)hipEventRecord(ev[1], st);
  if (fused) {
    FusedArgs a = {};
    a.units = p->d_fused_units;
    std::copy(p->fused_queue, p->fused_queue + N_XCD + 1, a.queue);
    a.slot_row = p->d_slot_row, a.pos_kv = p->d_pos_kv;
    a.k = static_cast<const bf16_t *>(k), a.v = static_cast<const bf16_t *>(v), a.q_sorted = q_sorted, a.do_sorted = do_sorted;
    a.stats_kv = stats_kv, a.flag_bytes = uint32_t(p->ws_off_ctrl - p->ws_off_flags);
    a.copy_bytes = uint32_t(p->ws_off_dos - p->ws_off_qs), a.dq_bytes = uint32_t(p->ws_off_flags - p->ws_off_dq_sums);
    a.dq = static_cast<bf16_t *>(dq), a.dk = static_cast<bf16_t *>(dk), a.dv = static_cast<bf16_t *>(dv);
    a.dq_sums = reinterpret_cast<float *>(static_cast<char *>(ws) + p->ws_off_dq_sums);
    a.flags = reinterpret_cast<int *>(static_cast<char *>(ws) + p->ws_off_flags);
    a.ctrl = reinterpret_cast<int *>(static_cast<char *>(ws) + p->ws_off_ctrl);
    a.hq = p->hq, a.hkv = p->hkv, a.scale = p->scale;
    hipError_t e = launch_bwd_fused(a, D, p->device, st);
    if (e != hipSuccess) return e;
    if (ev) (void)hipEventRecord(ev[2], st), (void)hipEventRecord(ev[3], st);
    return hipGetLastError();
  }
  const FwdUnit *const dq_list = parts_dq ? p->d_fwd_pieces : p->d_fwd_units;
  const int n_dq = int(parts_dq ? p->fwd_pieces.size() : p->fwd_units.size());
  const bool joint = p->joint && (split || p->n_fwd_parts + p->n_bwd_parts == 0);
  JointArgs args = {};
  auto launch_joint = [&](int32_t workgroups) {
    constexpr int SMEM = std::max(DkvSmem<D>::TOTAL, DqSmem<D, 4>::TOTAL);
    hipLaunchKernelGGL(ca_bwd_joint_kernel<D>, dim3(unsigned(workgroups)), dim3(256), SMEM, st, args);
  };
  if (joint) {
    auto kern = ca_bwd_joint_kernel<D>;
    constexpr int SMEM = std::max(DkvSmem<D>::TOTAL, DqSmem<D, 4>::TOTAL);
    static std::atomic<bool> done[16];
    hipError_t e = set_smem(kern, SMEM, p->device, done);
    if (e != hipSuccess) return e;
    args = {p->joint_order.empty() || ev ? nullptr : p->d_joint_order, parts_kv ? p->d_bwd_pieces : p->d_bwd_units, dq_list,
            p->d_slot_row, p->d_slot_pos, p->d_pos_kv, static_cast<const bf16_t *>(q), static_cast<const bf16_t *>(k),
            static_cast<const bf16_t *>(v), static_cast<const bf16_t *>(d_o), q_sorted, do_sorted, l2_slot, delta_slot, stats_kv,
            static_cast<bf16_t *>(dq), static_cast<bf16_t *>(dk), static_cast<bf16_t *>(dv), parts_dq, parts_kv,
            n_dkv, n_dq, p->hq, p->hkv, padded, p->scale};
    // (with timing enabled the same workgroups run as two launches, so that each kind has a time)
    launch_joint(ev ? n_dkv : n_dkv + 2 * n_dq);
  } else if (!p->bwd_units.empty()) {
    auto kern = ca_bwd_dkv_kernel<D>;
    constexpr int SMEM = DkvSmem<D>::TOTAL;
    static std::atomic<bool> done[16];
    hipError_t e = set_smem(kern, SMEM, p->device, done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(unsigned(n_dkv)), dim3(256), SMEM, st,
                       parts_kv ? p->d_bwd_pieces : p->d_bwd_units, p->d_pos_kv, q_sorted, static_cast<const bf16_t *>(k), static_cast<const bf16_t *>(v), do_sorted,
                       stats_kv, static_cast<bf16_t *>(dk), static_cast<bf16_t *>(dv), parts_kv, p->hq, p->hkv, p->scale);
  }
  if (p->shared_parts) combine(false, true);  // before the dQ pieces write over them
  if (ev) (void)hipEventRecord(ev[2], st);
  if (joint) {
    args.n_dkv = 0;  // dQ halves only
    if (ev) launch_joint(2 * n_dq);
  } else if (n_dq > 0) {
    auto kern = ca_bwd_dq_kernel<D>;
    constexpr int SMEM = DqSmem<D, 8>::TOTAL;
    static std::atomic<bool> done[16];
    hipError_t e = set_smem(kern, SMEM, p->device, done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(unsigned(n_dq)), dim3(512), SMEM, st, dq_list, p->d_slot_row, p->d_slot_pos,
                       static_cast<const bf16_t *>(q), static_cast<const bf16_t *>(k), static_cast<const bf16_t *>(v),
                       static_cast<const bf16_t *>(d_o), l2_slot, delta_slot, static_cast<bf16_t *>(dq), parts_dq, p->hq,
                       p->hkv, padded, p->scale);
  }
  combine(true, !p->shared_parts);
  if (ev) (void)hipEventRecord(ev[3], st);
  return hipGetLastError();
}

hipError_t launch_bwd(const ca_plan_t *p, const void *q, const void *k, const void *v, const void *o, const void *d_o,
                      const float *lse, void *dq, void *dk, void *dv, void *ws, bool split, bool fused,
                      hipStream_t st, hipEvent_t *ev) {
  return p->d == 128 ? launch_bwd_t<128>(p, q, k, v, o, d_o, lse, dq, dk, dv, ws, split, fused, st, ev)
                     : launch_bwd_t<64>(p, q, k, v, o, d_o, lse, dq, dk, dv, ws, split, fused, st, ev);
}

}  // namespace ca

