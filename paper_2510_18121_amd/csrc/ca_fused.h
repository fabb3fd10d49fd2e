// Arguments of the fused backward kernel.
#pragma once
#include <hip/hip_runtime.h>

#include "ca_internal.h"

namespace ca {
struct FusedArgs {
  const BwdUnit *units;
  int32_t queue[N_XCD + 1];
  const int32_t *slot_row, *pos_kv;
  const __bf16 *k, *v, *q_sorted, *do_sorted;
  const float *stats_kv;  // [block][head][half of 32 rows][log2e * LSE, -Delta][32]
  __bf16 *dq, *dk, *dv;
  float *dq_sums;
  int *flags, *ctrl;
  uint32_t flag_bytes, copy_bytes, dq_bytes;  // (all below 4 GiB: 32-bit offsets)
  int hq, hkv;
  float scale;
};
hipError_t launch_bwd_fused(const FusedArgs &a, int d, int device, hipStream_t st);
}  // namespace ca
