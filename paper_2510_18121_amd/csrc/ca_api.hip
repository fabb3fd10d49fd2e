// C-ABI entry points that touch the device: plan upload, forward and backward launches.
#include <hip/hip_runtime.h>

#include <cstring>
#include <mutex>
#include <new>
#include <sstream>
#include <type_traits>

#include "ca_internal.h"

namespace ca {
// parts / split: (there is) device memory for the partial results of the piece lists; otherwise the whole units are run
hipError_t launch_fwd(const ca_plan_t *p, const void *q, const void *k, const void *v, void *o, float *lse, void *parts,
                      hipStream_t st);
hipError_t launch_bwd(const ca_plan_t *p, const void *q, const void *k, const void *v, const void *o, const void *d_o,
                      const float *lse, void *dq, void *dk, void *dv, void *ws, bool split, bool fused, hipStream_t st,
                      hipEvent_t *ev);

static int hip_fail(const char *what, hipError_t e) {
  std::ostringstream os;
  os << what << ": " << hipGetErrorName(e) << " (" << hipGetErrorString(e) << ")";
  set_error(os.str());
  return CA_ERR_HIP;
}
#define CA_HIP(call)                                  \
  do {                                                \
    hipError_t e_ = (call);                           \
    if (e_ != hipSuccess) return hip_fail(#call, e_); \
  } while (0)

// Device-resident backward workspace for callers that cannot allocate (ca_backward_static_ws).  In host code the
// array's name is only a handle for hipGetSymbolAddress: the address each device holds its copy at is looked up once
// per device and kept in static_ws_ptr; only that pointer is ever handed to kernels.
static __device__ __align__(256) __attribute__((used)) unsigned char static_ws[CA_STATIC_WS_BYTES];
static void *static_ws_ptr[16];
static std::mutex static_ws_mutex;

static int static_ws_on_device(int device, void **out) {
  if (device < 0 || device >= 16) {
    set_error("ca_backward_static_ws supports device ordinals 0..15");
    return CA_ERR_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> lock(static_ws_mutex);
  if (!static_ws_ptr[device]) {  // the calling thread's current device is `device` (checked by the caller)
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(static_ws));
    if (e != hipSuccess) return hip_fail("hipGetSymbolAddress(static workspace)", e);
    if (!ptr || reinterpret_cast<uintptr_t>(ptr) % 256 != 0) {
      set_error("static workspace has no usable device address");
      return CA_ERR_HIP;
    }
    static_ws_ptr[device] = ptr;
  }
  *out = static_ws_ptr[device];
  return CA_OK;
}

// A transfer costs 10 to 15 us before it moves a byte, collecting an array in `blob` 0.25 ms per MiB (fresh pages, and the bytes
// twice through the caches).  ca_plan on the plan of 32K tokens in lone 20-row shards (16/16 heads, the two unit lists are
// megabytes): 12.6 ms with everything collected, 4.9 with arrays beyond 256 KiB by themselves; on 60 batches of all sizes
// 0.82 and 0.79 of what one allocation and one transfer per array took, 0.80 with the line at 64 or 128 KiB.
constexpr size_t SMALL_ARRAY = 256 << 10;

static void free_device(ca_plan_t *p) {
  if (p->within_static) free_device(p->within_static.get());
  if (p->device < 0) return;
  int cur = -1;
  if (hipGetDevice(&cur) == hipSuccess && cur != p->device) (void)hipSetDevice(p->device);
  if (p->d_blob) (void)hipFree(p->d_blob);
  p->d_blob = nullptr;
  p->d_slot_row = p->d_slot_pos = p->d_block_rpk = p->d_pos_kv = nullptr;
  p->d_joint_order = nullptr;
  p->d_fwd_units = p->d_fwd_pieces = nullptr;
  p->d_bwd_units = p->d_bwd_pieces = p->d_fused_units = nullptr;
  p->d_fwd_combine = p->d_bwd_combine = nullptr;
  if (cur >= 0 && cur != p->device) (void)hipSetDevice(cur);
  p->device = -1;
}

static int check_call(const ca_plan_t *p, void *ws, size_t ws_bytes, size_t need) {
  if (!p) {
    set_error("plan is null");
    return CA_ERR_INVALID_ARG;
  }
  if (p->device < 0) {
    set_error("plan was not uploaded (ca_plan_upload)");
    return CA_ERR_STATE;
  }
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return hip_fail("hipGetDevice", e);
  if (cur != p->device) {
    set_error("plan was uploaded to another device than the current one");
    return CA_ERR_STATE;
  }
  if (need > 0) {
    if (!ws || ws_bytes < need) {
      std::ostringstream os;
      os << "workspace of " << ws_bytes << " bytes given, " << need << " needed";
      set_error(os.str());
      return CA_ERR_WORKSPACE;
    }
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) {
      set_error("workspace is not 256-byte aligned");
      return CA_ERR_WORKSPACE;
    }
  }
  return CA_OK;
}
}  // namespace ca

extern "C" {

int ca_plan_upload(ca_plan_t *p, void *hip_stream) {
  using namespace ca;
  if (!p) {
    set_error("plan is null");
    return CA_ERR_INVALID_ARG;
  }
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  free_device(p);
  if (p->within_static) {
    const int rc = ca_plan_upload(p->within_static.get(), hip_stream);
    if (rc != CA_OK) return rc;
  }
  int dev = -1;
  CA_HIP(hipGetDevice(&dev));
  p->device = dev;
  // One allocation.  The small arrays come first, collected in `blob`, and go up in one transfer; a large one goes up by itself,
  // straight from the plan's vector (see SMALL_ARRAY).
  struct Array {
    const void *src;
    size_t bytes, at;
  };
  std::vector<Array> arrays;
  size_t bytes = 0, small = 0;
  try {
    auto add = [&](const auto &src) { arrays.push_back({src.data(), src.size() * sizeof(src[0]), 0}); };
    add(p->slot_row), add(p->slot_pos), add(p->block_rpk), add(p->pos_kv), add(p->fwd_units), add(p->bwd_units);
    add(p->fwd_pieces), add(p->bwd_pieces), add(p->fwd_combine), add(p->bwd_combine), add(p->joint_order), add(p->fused_units);
    for (const bool large : {false, true}) {
      for (Array &a : arrays)
        if ((a.bytes > SMALL_ARRAY) == large) a.at = bytes, bytes = (bytes + a.bytes + 255) / 256 * 256;
      if (!large) small = bytes;
    }
    if (bytes == 0) return CA_OK;
    p->blob.resize(small);
  } catch (const std::bad_alloc &) {
    free_device(p);
    set_error("out of host memory while uploading the plan");
    return CA_ERR_INVALID_ARG;
  }
  hipError_t e = hipMalloc(&p->d_blob, bytes);
  if (e != hipSuccess) {
    p->d_blob = nullptr;
    free_device(p);
    return hip_fail("plan upload", e);
  }
  char *const device = static_cast<char *>(p->d_blob);
  for (const Array &a : arrays) {
    if (a.bytes == 0 || e != hipSuccess) continue;
    if (a.bytes <= SMALL_ARRAY) std::memcpy(p->blob.data() + a.at, a.src, a.bytes);
    else e = hipMemcpyAsync(device + a.at, a.src, a.bytes, hipMemcpyHostToDevice, st);
  }
  if (e == hipSuccess && small > 0) e = hipMemcpyAsync(device, p->blob.data(), small, hipMemcpyHostToDevice, st);
  if (e != hipSuccess) {
    free_device(p);
    return hip_fail("plan upload", e);
  }
  auto place = [&](auto *&dst, int i) { dst = reinterpret_cast<std::remove_reference_t<decltype(dst)>>(device + arrays[size_t(i)].at); };
  place(p->d_slot_row, 0), place(p->d_slot_pos, 1), place(p->d_block_rpk, 2), place(p->d_pos_kv, 3);
  place(p->d_fwd_units, 4), place(p->d_bwd_units, 5), place(p->d_fwd_pieces, 6), place(p->d_bwd_pieces, 7);
  place(p->d_fwd_combine, 8), place(p->d_bwd_combine, 9), place(p->d_joint_order, 10), place(p->d_fused_units, 11);
  // the vectors and `blob` stay alive in the plan, so the asynchronous copies read valid memory
  return CA_OK;
}

int ca_plan(const ca_batch_desc *desc, ca_plan_t **out) {
  int rc = ca_plan_host(desc, out);
  if (rc != CA_OK) return rc;
  rc = ca_plan_upload(*out, nullptr);
  if (rc == CA_OK) {  // callers launch on streams of their own: the schedule must have landed before they do
    const hipError_t e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) rc = ca::hip_fail("plan upload", e);
  }
  if (rc != CA_OK) {
    ca_plan_destroy(*out);
    *out = nullptr;
  }
  return rc;
}

int ca_profile_enable(ca_plan_t *p, int on) {
  using namespace ca;
  if (!p) {
    set_error("plan is null");
    return CA_ERR_INVALID_ARG;
  }
  if (on && !p->profile) {
    for (int i = 0; i < 6; ++i) {
      hipEvent_t e;
      const hipError_t rc = hipEventCreate(&e);
      if (rc != hipSuccess) {  // leave nothing half-made behind
        for (int j = 0; j < i; ++j) (void)hipEventDestroy(static_cast<hipEvent_t>(p->ev[j])), p->ev[j] = nullptr;
        return hip_fail("hipEventCreate", rc);
      }
      p->ev[i] = e;
    }
    p->profile = true;
  } else if (!on && p->profile) {
    for (int i = 0; i < 6; ++i)
      if (p->ev[i]) (void)hipEventDestroy(static_cast<hipEvent_t>(p->ev[i])), p->ev[i] = nullptr;
    p->profile = false;
  }
  p->ev_fwd = p->ev_bwd = false;
  return CA_OK;
}

int ca_profile_read(ca_plan_t *p, float *out) {
  using namespace ca;
  if (!p || !out) {
    set_error("plan or output is null");
    return CA_ERR_INVALID_ARG;
  }
  for (int i = 0; i < 4; ++i) out[i] = 0.f;
  if (!p->profile) {
    set_error("profiling is not enabled on this plan");
    return CA_ERR_STATE;
  }
  auto E = [&](int i) { return static_cast<hipEvent_t>(p->ev[i]); };
  if (p->ev_fwd) {
    CA_HIP(hipEventSynchronize(E(1)));
    CA_HIP(hipEventElapsedTime(&out[0], E(0), E(1)));
  }
  if (p->ev_bwd) {
    CA_HIP(hipEventSynchronize(E(5)));
    CA_HIP(hipEventElapsedTime(&out[1], E(2), E(3)));
    CA_HIP(hipEventElapsedTime(&out[2], E(3), E(4)));
    CA_HIP(hipEventElapsedTime(&out[3], E(4), E(5)));
  }
  return CA_OK;
}

void ca_plan_destroy(ca_plan_t *p) {
  if (!p) return;
  if (p->profile) (void)ca_profile_enable(p, 0);
  ca::free_device(p);
  delete p;
}

int ca_forward(const ca_plan_t *p, const void *q, const void *k, const void *v, void *o, float *lse, void *ws,
               size_t ws_bytes, void *hip_stream) {
  using namespace ca;
  int rc = check_call(p, ws, ws_bytes, p ? p->ws_fwd : 0);
  if (rc != CA_OK) return rc;
  if (p->total_q > 0 && (!q || !o || !lse)) {
    set_error("q, o or lse is null");
    return CA_ERR_INVALID_ARG;
  }
  if (p->total_kv > 0 && (!k || !v)) {
    set_error("k or v is null");
    return CA_ERR_INVALID_ARG;
  }
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  ca_plan_t *mp = const_cast<ca_plan_t *>(p);  // timing state only
  if (p->profile) (void)hipEventRecord(static_cast<hipEvent_t>(mp->ev[0]), st);
  // with room for partial results (and only then) long units are cut into pieces
  auto fits = [&](const ca_plan_t *x) {
    return x->ws_fwd_split > 0 && ws && ws_bytes >= x->ws_fwd_split && reinterpret_cast<uintptr_t>(ws) % 256 == 0;
  };
  const ca_plan_t *const use = p->within_static && !fits(p) ? p->within_static.get() : p;
  hipError_t e = launch_fwd(use, q, k, v, o, lse, fits(use) ? ws : nullptr, st);
  if (e != hipSuccess) return hip_fail("forward launch", e);
  if (p->profile) {
    (void)hipEventRecord(static_cast<hipEvent_t>(mp->ev[1]), st);
    mp->ev_fwd = true;
  }
  return CA_OK;
}

int ca_backward(const ca_plan_t *p, const void *q, const void *k, const void *v, const void *o, const void *d_o,
                const float *lse, void *dq, void *dk, void *dv, void *ws, size_t ws_bytes, void *hip_stream) {
  using namespace ca;
  int rc = check_call(p, ws, ws_bytes, p ? p->ws_bwd : 0);
  if (rc != CA_OK) return rc;
  if (p->total_q > 0 && (!q || !o || !d_o || !lse || !dq)) {
    set_error("q, o, d_o, lse or dq is null");
    return CA_ERR_INVALID_ARG;
  }
  if (p->total_kv > 0 && (!k || !v || !dk || !dv)) {
    set_error("k, v, dk or dv is null");
    return CA_ERR_INVALID_ARG;
  }
  ca_plan_t *mp = const_cast<ca_plan_t *>(p);  // timing state only
  const ca_plan_t *const use = p->within_static && ws_bytes < p->ws_bwd_split ? p->within_static.get() : p;
  const bool split = use->ws_bwd_split > use->ws_bwd && ws_bytes >= use->ws_bwd_split;
  const bool fused = p->fused && ws_bytes >= p->ws_bwd_fused;
  hipError_t e = launch_bwd(fused ? p : use, q, k, v, o, d_o, lse, dq, dk, dv, ws, split, fused, static_cast<hipStream_t>(hip_stream),
                            p->profile ? reinterpret_cast<hipEvent_t *>(&mp->ev[2]) : nullptr);
  if (e != hipSuccess) return hip_fail("backward launch", e);
  if (p->profile) mp->ev_bwd = true;
  return CA_OK;
}

int ca_backward_static_ws(const ca_plan_t *p, const void *q, const void *k, const void *v, const void *o,
                          const void *d_o, const float *lse, void *dq, void *dk, void *dv, void *hip_stream) {
  using namespace ca;
  int rc = check_call(p, nullptr, 0, 0);  // plan present, uploaded, and on the current device
  if (rc != CA_OK) return rc;
  if (p->ws_bwd > size_t(CA_STATIC_WS_BYTES)) {
    std::ostringstream os;
    os << "this batch needs a backward workspace of " << p->ws_bwd << " bytes; the static workspace holds "
       << size_t(CA_STATIC_WS_BYTES) << " (use ca_backward with a caller-provided workspace)";
    set_error(os.str());
    return CA_ERR_WORKSPACE;
  }
  void *ws = nullptr;
  rc = static_ws_on_device(p->device, &ws);
  if (rc != CA_OK) return rc;
  return ca_backward(p, q, k, v, o, d_o, lse, dq, dk, dv, ws, size_t(CA_STATIC_WS_BYTES), hip_stream);
}

size_t ca_static_workspace_bytes(void) { return size_t(CA_STATIC_WS_BYTES); }

}  // extern "C"
