// Device-side helpers for the gfx950 kernels: MFMA fragment types, LDS reads, bf16 packing.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace ca {

typedef __bf16 bf16_t;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

#define CA_LDS __attribute__((address_space(3)))

// v_mfma_f32_16x16x32_bf16: C[16x16] += A[16x32] * B[32x16].
//   A: lane l holds A[l%16][8*(l/16) .. +7];  B: lane l holds B[8*(l/16) .. +7][l%16];
//   C: lane l, register i holds C[4*(l/16) + i][l%16].
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ds_read_b64_tr_b16: inside each group of 16 lanes, lane i points at 4 consecutive bf16 and receives
// element (i%4) of the 4 values read by lanes 4j + i/4, j = 0..3.  With lane i pointing at
// tile[r0 + i/4][c0 + 4*(i%4)] the lane gets tile[r0 .. r0+3][c0 + i]: a 4x16 block, transposed.
// (LDS reads are addressed by a 32-bit LDS byte address: no generic-pointer arithmetic, and constant parts of the address fold
// into the instruction's offset field.)
__device__ __forceinline__ bf16x4 lds_read_tr4_at(uint32_t a) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((CA_LDS bf16x4 *)a);
}
// 16-byte LDS read of 8 consecutive bf16
__device__ __forceinline__ bf16x8 lds_read8_at(uint32_t a) { return *(const CA_LDS bf16x8 *)a; }
template <class T>
__device__ __forceinline__ T lds_ld(uint32_t a) {
  return *(const CA_LDS T *)a;
}

__device__ __forceinline__ bf16x8 join(bf16x4 lo, bf16x4 hi) {
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// two fp32 -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  f32x2 v = {a, b};
  bf16x2 r = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// max of a value with the one held by lane l ^ 32 (v_permlane32_swap: no LDS round trip)
__device__ __forceinline__ float xor32_max(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}

// max of, and sum with, the values held by the lanes that differ in bits 4 and 5 of their index
__device__ __forceinline__ float quad_max(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return xor32_max(fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1])));
}
__device__ __forceinline__ float quad_sum(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

// A constant that the compiler cannot see through: what is computed from it is computed where it stands, not kept in a register
// (or spilled) across a long loop.  The vector instruction itself stays the compiler's, which places the wait states that
// MFMAs in flight need around it.
__device__ __forceinline__ int opaque(int k) {
  asm volatile("" : "+s"(k));
  return k;
}
__device__ __forceinline__ int lane_id_here() {
  const uint32_t all = opaque(-1);
  return int(__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u)));
}
// a ^ b: of a loop-carried LDS address and the distance to one of its fragments
__device__ __forceinline__ int xor_here(int a, const int b) { return a ^ opaque(b); }

__device__ __forceinline__ int wave_max(int v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ int wave_min(int v) {
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  return v;
}

}  // namespace ca

// ---------------------------------------------------------------------------------------------
// LDS tiles of R rows x D bf16 in natural (row-major) layout, rows unpadded, with the 16-byte chunks of
// each row XOR-swizzled by a function of the row.  gfx950's LDS has 64 banks of 4 bytes (256 B/clk).
//   * A natural read is 16 rows x 64 bytes: lane l reads chunk 4 s + l / 16 of row l % 16, and the 16 lanes served together are 0-3,
//     12-15 of one run of 16 lanes and 4-11 of the next one's (a swizzle without conflicts inside each run has them in every
//     second read: 30 to 40 % of the LDS cycles of the backward kernels).  So with q = r / 4 % 4 the low bits f(q) of sw are
//     0, 2, 3, 1: f(1) = f(2) ^ 1 and f(0) = f(3) ^ 1 keep those apart; bits 2..3 follow the row's low bits.
//   * An 8-byte transposing read is served 8 consecutive rows x one 32-byte piece at a time: f(0), f(1) as well as f(2), f(3)
//     differ in bit 1.
// (At head_dim 64 two rows share a 256-byte line.)  So one tile can feed natural and transposed MFMA operands.
// Because rows are unpadded, a tile can be filled by global_load_lds_dwordx4, which writes
// lane i's 16 bytes at (wave-uniform LDS base) + 16 i: the swizzle is applied by choosing which global
// chunk each lane fetches.
namespace ca {

template <int D>
__device__ __forceinline__ int tile_sw(int r) {
  const int q0 = (r >> 2) & 1, q1 = (r >> 3) & 1;
  return (D == 128 ? (r & 3) << 2 : ((r >> 1) & 1) << 2) | (q0 ^ q1) << 1 | q1;
}

// One wave-wide direct load global -> LDS: lane i's 16 (or 4) bytes from `src` land at
// lds_base + 16 i (or 4 i); lds_base must be wave-uniform.  Written as inline assembly on purpose: the
// compiler's wait-count insertion treats every LDS read as possibly aliasing an in-flight direct load
// and would drain the whole prefetch queue (s_waitcnt vmcnt(0)) before it.  Here the kernels pace
// the queue themselves with wait_vmcnt<N>() and a barrier.  Loads the compiler does not know about can
// only make its own vmcnt waits stricter than needed, never weaker: vector loads retire in order.
// The address is (wave-uniform 64-bit base in SGPRs) + (per-lane unsigned 32-bit byte offset); the LDS destination is a
// wave-uniform LDS byte address.
__device__ __forceinline__ void load_lds16_sbase(const void *base_uniform, uint32_t lane_off, uint32_t lds_off_uniform) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds_off_uniform);
  const uint64_t b = (uint64_t)(uintptr_t)base_uniform;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  const uint64_t sb = ((uint64_t)hi << 32) | lo;
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(lane_off), "s"(sb), "s"(m0v)
               : "memory", "m0");
}
// the 4-byte form
__device__ __forceinline__ void load_lds4_sbase(const void *base_uniform, uint32_t lane_off, uint32_t lds_off_uniform) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds_off_uniform);
  const uint64_t b = (uint64_t)(uintptr_t)base_uniform;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  const uint64_t sb = ((uint64_t)hi << 32) | lo;
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
               :
               : "v"(lane_off), "s"(sb), "s"(m0v)
               : "memory", "m0");
}
// workgroup barrier without the memory fence of __syncthreads() (which would also drain the direct loads):
// the caller has waited for its own LDS reads (lgkmcnt) and for the direct loads that must be visible
__device__ __forceinline__ void barrier_nofence() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Pins a loaded register value: the load is issued and waited for before this point (the compiler would
// otherwise be free to sink loads from read-only memory to their first use inside a loop, together
// with a vector-memory wait that would drain the direct-load queue on every iteration).
__device__ __forceinline__ void pin(bf16x8 &v) {
  u32x4 w = __builtin_bit_cast(u32x4, v);
  asm volatile("" : "+v"(w));
  v = __builtin_bit_cast(bf16x8, w);
}
__device__ __forceinline__ void pin(float &v) { asm volatile("" : "+v"(v)); }

// wait until at most n of this wave's vector-memory loads are outstanding (n <= 63)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  // the empty asm statements keep the compiler from moving loads or stores across the wait
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}


// Workgroups that are halves of n units: which unit and which half workgroup i of 2 n is.  The halves of a unit are 8 workgroups
// apart, on one XCD: they read the same K and V.
__device__ __forceinline__ void half_of_unit(int &i, int n, int &half) {
  const int n8 = n & ~7, rest = n - n8, t = i - 2 * n8;  // (the last units have fewer than 8 neighbours)
  half = t < 0 ? !((i >> 3) & 1) : t < rest;
  i = t < 0 ? (i >> 4) * 8 + (i & 7) : n8 + t - (half ? 0 : rest);
}

// ---- a wave's 32 x D result tile, stored as whole lines.
// In the accumulator layout of Xt = A B (16x16 MFMAs, 16-row blocks b of the D values, tiles t of 16 rows of X) lane l holds, of row
// 16 t + l % 16 (a key, or a query row), the values 16 b + 4 (l / 16) .. + 3 in acc[b][t].  Stored from there, one instruction
// touches 16 rows with 32 bytes each, and a CU's address unit is busy with a tile's stores for microseconds.  Instead the wave
// passes 64 values per row at a time through an LDS patch of its own (PATCH_BYTES at `patch`, an LDS byte address; a wave's LDS
// instructions execute in order, so nothing synchronises) and stores 8 rows x 128 bytes per instruction.  dst_of_row(p)
// returns where row p (0..31) of the tile begins in memory, or nullptr for a row that is not stored.
constexpr int PATCH_ROW_BYTES = 128 + 16;  // 16 bytes off a power of two
constexpr int PATCH_BYTES = 32 * PATCH_ROW_BYTES;
// (tiles T0 and T0 + 1 of acc; f0 and f1 scale their values.)
template <int T0, int ND, int NT, class F>
__device__ __forceinline__ void store_tile16_as_lines(uint32_t patch, const f32x4 (&acc)[ND][NT], float f0, float f1, int lane,
                                                      F dst_of_row) {
  const int orow = lane >> 3, ocol = lane & 7;
  const uint32_t wr = patch + (lane & 15) * PATCH_ROW_BYTES + 8 * (lane >> 4);  // + 16 rows t + 32 b
  const uint32_t rd = patch + orow * PATCH_ROW_BYTES + 16 * ocol;               // the lane's row (+ 8 i) and 16-byte piece
  bf16_t *dst[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) dst[i] = dst_of_row(orow + 8 * i);
#pragma unroll
  for (int h = 0; h < ND / 4; ++h) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const f32x4 a = acc[4 * h + b][T0 + t];
        const float f = t == 0 ? f0 : f1;
        *(CA_LDS u32x2 *)(wr + 16 * t * PATCH_ROW_BYTES + 32 * b) = u32x2{pack_bf16(a[0] * f, a[1] * f), pack_bf16(a[2] * f, a[3] * f)};
      }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x4 x = *(const CA_LDS u32x4 *)(rd + 8 * i * PATCH_ROW_BYTES);
      if (dst[i]) *reinterpret_cast<u32x4 *>(dst[i] + 64 * h + 8 * ocol) = x;
    }
  }
}
// ... and as a partial result, in the order of 32x32 accumulators that the combine kernels read: quad k of lane (r, g) is
// columns 8 k + 4 g .. + 3 of row r (256-byte runs per 16 lanes)
template <int T0, int ND, int NT>
__device__ __forceinline__ void store_tile16_as_part(float *dst, const f32x4 (&acc)[ND][NT], int lane) {
  dst += 256 * (lane >> 5) + 128 * ((lane >> 4) & 1) + 4 * (lane & 15);
#pragma unroll
  for (int b = 0; b < ND; ++b)
#pragma unroll
    for (int t = 0; t < 2; ++t) *reinterpret_cast<f32x4 *>(dst + 512 * b + 64 * t) = acc[b][T0 + t];
}

// ---- sums of partial results (the combine kernels).  One workgroup of four waves adds up the n_parts blocks of 32 rows x
// 64 columns at `src` (fp32 in accumulator order: instruction k of the 8 of a block reads quad k, 1 KB), wave w taking
// blocks w, w + 4, ..; so a sum of up to 8 pieces waits for memory about once.  The waves' sums meet in LDS, and wave w
// stores rows 8 w .. 8 w + 7 of the tile as whole lines.  With STATS, `st` holds {m, l} per lane and block, and block i
// counts with weight 2^(m_i - M); then m (M, of the lane's row) and l (the row's whole sum, of both lane halves) are set in
// every wave.  Otherwise the blocks are added.  The order of additions is fixed.
constexpr int COMBINE_ROW = 64 + 4;  // floats between the rows of a wave's sum in LDS
constexpr int COMBINE_LDS = 4 * 32 * COMBINE_ROW;
template <bool STATS, class F>
__device__ __forceinline__ void combine_parts(const float *src, size_t src_stride, const float *st, size_t st_stride,
                                              int n_parts, float f, float (&lds)[COMBINE_LDS], float (&ml)[4][64][2],
                                              float &m, float &l, F dst_of_row) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, g = lane >> 5;
  f32x4 acc[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
  float mw = -3.402823466e38f, lw = 0.f;
#pragma unroll 2
  for (int i = wave; i < n_parts; i += 4) {
    float wgt = 1.f;
    if (STATS) {
      const f32x2 s = *reinterpret_cast<const f32x2 *>(st + size_t(i) * st_stride + 2 * lane);
      const float mn = fmaxf(mw, s[0]), old = fast_exp2(mw - mn);
      wgt = fast_exp2(s[0] - mn);
      mw = mn, lw = lw * old + wgt * s[1];
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] *= old;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const f32x4 x = *reinterpret_cast<const f32x4 *>(src + size_t(i) * src_stride + k * 256 + 4 * lane);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[k][e] = STATS ? fmaf(wgt, x[e], acc[k][e]) : acc[k][e] + x[e];
    }
  }
  // quad k of lane (r, g): columns 8 k + 4 g .. + 3 of row r
#pragma unroll
  for (int k = 0; k < 8; ++k) *reinterpret_cast<f32x4 *>(&lds[(wave * 32 + r) * COMBINE_ROW + 8 * k + 4 * g]) = acc[k];
  if (STATS) ml[wave][lane][0] = mw, ml[wave][lane][1] = lw;
  __syncthreads();
  const int orow = 8 * wave + (lane >> 3), ocol = 8 * (lane & 7);
  float wt[4] = {1.f, 1.f, 1.f, 1.f}, inv = f;
  if (STATS) {
    auto of_row = [&](int row, float &mm, float &ll, float (&w)[4]) __attribute__((always_inline)) {
      mm = fmaxf(fmaxf(ml[0][row][0], ml[1][row][0]), fmaxf(ml[2][row][0], ml[3][row][0]));
      ll = 0.f;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        w[v] = fast_exp2(ml[v][row][0] - mm);  // (both lanes of a row have the same m)
        ll += w[v] * (ml[v][row][1] + ml[v][row + 32][1]);
      }
    };
    float mo, lo, unused[4];
    of_row(orow, mo, lo, wt);
    inv = 1.0f / lo;
    of_row(r, m, l, unused);
  }
  float y[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) y[e] = 0.f;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const f32x4 a = *reinterpret_cast<const f32x4 *>(&lds[(v * 32 + orow) * COMBINE_ROW + ocol]);
    const f32x4 b = *reinterpret_cast<const f32x4 *>(&lds[(v * 32 + orow) * COMBINE_ROW + ocol + 4]);
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] += wt[v] * a[e], y[4 + e] += wt[v] * b[e];
  }
  bf16_t *const dst = dst_of_row(orow);
  if (dst)
    *reinterpret_cast<u32x4 *>(dst + ocol) = u32x4{pack_bf16(y[0] * inv, y[1] * inv), pack_bf16(y[2] * inv, y[3] * inv),
                                                   pack_bf16(y[4] * inv, y[5] * inv), pack_bf16(y[6] * inv, y[7] * inv)};
}

}  // namespace ca
