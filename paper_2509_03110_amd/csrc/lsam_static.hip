// lsam_step_grads_static: the raw-vector iteration of lsam_step_grads for callers that cannot
// allocate (code under HIP graph capture, tight serving loops, harnesses that forbid
// hipMalloc).  All state is the caller's; the only device memory beyond inputs and outputs --
// the partial sums of squares of the gradient-norm reduction, the norms and the perturbation
// scales -- lives in a file-scope device array of fixed size, one copy per GPU, resolved to a
// device address once per device.  No hipMalloc, hipFree or allocating library call is made.
#include <mutex>

#include "engine.h"

namespace lsam {
namespace {

constexpr int kMaxDevices = 64;
constexpr size_t kPartialBytes = (size_t)kMaxK * kMaxPartials * sizeof(double);   // 512 KiB
constexpr size_t kScratchBytes = kPartialBytes + 2 * kMaxK * sizeof(float);     // + norms, scales

// Host code never passes this name to a kernel: it is a stand-in on the host side.  The device
// address of each GPU's copy comes from hipGetSymbolAddress below.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

std::mutex g_lock;
void* g_scratch_ptr[kMaxDevices] = {nullptr};

thread_local char g_msg[256];

int report(int code) {
  set_last_error(g_msg);
  return code;
}

// Device address of the current device's copy of `scratch` (looked up on first use per device).
int scratch_for_current_device(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) {
    snprintf(g_msg, sizeof g_msg, "hipGetDevice: %s", hipGetErrorString(e));
    return report(LSAM_EHIP);
  }
  if (dev < 0 || dev >= kMaxDevices) {
    snprintf(g_msg, sizeof g_msg, "device index %d beyond the %d this entry point keeps track of", dev,
             kMaxDevices);
    return report(LSAM_EINVAL);
  }
  std::lock_guard<std::mutex> hold(g_lock);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr) {
      snprintf(g_msg, sizeof g_msg, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
      return report(LSAM_EHIP);
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return LSAM_OK;
}

// Whether x~ lies over any of the step's other arrays.
bool shares_memory(const lsam_update_desc* u, const float* x, const float* v, const float* S, const float* y,
                   const float* g1, const float* g2, const float* xt) {
  auto meets = [&](const float* p, int64_t rows, int64_t stride) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(xt), b = reinterpret_cast<uintptr_t>(p);
    const uintptr_t la = ((u->K - 1) * u->stride + u->d) * 4, lb = ((rows - 1) * stride + u->d) * 4;
    return a < b + lb && b < a + la;
  };
  return meets(x, u->K, u->stride) || meets(v, u->K, u->stride) || meets(S, u->K, u->stride) || meets(y, 1, u->stride) ||
         meets(g1, u->K, u->g_stride) || meets(g2, u->K, u->g_stride);
}

}  // namespace

}  // namespace lsam

using namespace lsam;

extern "C" int lsam_step_grads_static(const lsam_update_desc* u, float* x, float* v, float* S,
                                      const float* y, const float* g1, const float* g2, float* xt,
                                      float* norms_out, void* stream) {
  auto bad = [](const char* why) {
    set_last_error(why);
    return LSAM_EINVAL;
  };
  if (!u || !x || !v || !S || !y || !g1 || !g2) return bad("NULL argument");
  if (u->K < 1 || u->K > LSAM_MAX_REPLICAS) return bad("K outside 1..LSAM_MAX_REPLICAS");
  if (u->d < 1 || u->d > LSAM_STATIC_MAX_D) return bad("d outside 1..LSAM_STATIC_MAX_D");
  if (u->stride < u->d || u->g_stride < u->d) return bad("row strides must be >= d");
  if (!u->lambda) return bad("lambda is NULL");
  if (!(u->rho >= 0.f) || !(u->gamma >= 0.f) || !(u->lr >= 0.f) || !(u->momentum >= 0.f && u->momentum < 1.f))
    return bad("rho, gamma, lr must be >= 0 and momentum in [0, 1)");
  if (u->rho != 0.f && !xt) return bad("xt is NULL although rho > 0");
  const uintptr_t align = reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(v) |
                          reinterpret_cast<uintptr_t>(S) | reinterpret_cast<uintptr_t>(y) |
                          reinterpret_cast<uintptr_t>(xt);
  if ((align & 15) || (u->stride % 4)) return bad("x, v, S, y, xt must be 16-byte aligned with a row stride that is a multiple of 4");
  if ((reinterpret_cast<uintptr_t>(g1) & 3) || (reinterpret_cast<uintptr_t>(g2) & 3))
    return bad("gradients must be 4-byte aligned");

  void* base = nullptr;
  int rc = scratch_for_current_device(&base);
  if (rc != LSAM_OK) return rc;
  double* partials = static_cast<double*>(base);
  float* norms = reinterpret_cast<float*>(static_cast<char*>(base) + kPartialBytes);
  float* scale = norms + kMaxK;
  if (norms_out) norms = norms_out;       // the caller's array takes the norms directly

  hipStream_t s = static_cast<hipStream_t>(stream);
  const int K = u->K;
  const int64_t d = u->d;
  ReplicaScalars lam;
  for (int i = 0; i < K; ++i) lam.v[i] = u->lambda[i];
  // every slot that is read is written first, so nothing of an earlier call is seen
  AscentPass up;
  up.g1 = g1; up.g1_stride = u->g_stride;
  up.partials = partials; up.nblk = sumsq_blocks(d);
  up.rho = u->rho; up.gamma = u->gamma;
  up.norms = norms; up.scale = scale;
  if (u->rho != 0.f) up.xt = xt;
  if (up.xt && shares_memory(u, x, v, S, y, g1, g2, xt)) {
    // x~ takes the place of something that the descent reads: it has to be whole before that
    launch_sumsq_partials(g1, u->g_stride, d, K, partials, up.nblk, s);
    launch_norm_finish(partials, up.nblk, up.nblk, K, u->rho, u->gamma, norms, scale, nullptr, 0, nullptr, s);
    launch_perturb(x, g1, u->g_stride, scale, xt, nullptr, nullptr, 0, u->stride, d, K, s);
    launch_descent(x, g2, u->g_stride, v, S, y, nullptr, nullptr, 0, u->stride, d, K, lam, u->lr,
                   u->momentum, u->nesterov, nullptr, s);
  } else {
    launch_raw_norm(d, K, s, nullptr, up);
    launch_raw_descent(x, g2, u->g_stride, v, S, y, u->stride, d, K, lam, u->lr, u->momentum, u->nesterov, nullptr, s,
                       nullptr, up);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_last_error(hipGetErrorString(e));
    return LSAM_EHIP;
  }
  return LSAM_OK;
}
