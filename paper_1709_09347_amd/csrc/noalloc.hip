// Operator application without device allocation (cbs_apply_noalloc).
//
// cbs_apply keeps its projector coefficients in the system's grow-only workspace, which calls
// hipMalloc the first time a size is seen.  This variant runs the same kernels with them
// inside one fixed device array, `scratch`, so a call allocates nothing: callers
// that cannot allocate (code under graph capture, tight serving loops) use it.
//
// The array is a file-scope __device__ symbol: in host code its name is only a stand-in,
// so its device address is looked up once per device with hipGetSymbolAddress (at system
// creation, with that device current) and that address is what the kernels receive.
// Every call on one device shares the array and leaves its contents behind; calls that
// overlap on one device race.
#include <mutex>
#include <type_traits>
#include <vector>

#include "cbs_internal.hpp"

namespace cbs {

constexpr size_t kScratchBytes = (size_t)64 << 20;   // CBS_APPLY_NOALLOC_BYTES in cbs.h
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
static void* g_scratch[kMaxDevices] = {};
static std::mutex g_scratch_mu;

// Device address of the scratch array on `device` (which must be current); looked up once.
int32_t noalloc_scratch(int32_t device, void** out) {
  *out = nullptr;
  if (device < 0 || device >= kMaxDevices) {
    set_error("device %d beyond the %d devices the allocation-free entry points track", device, kMaxDevices);
    return CBS_EINVAL;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch[device] == nullptr) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      set_error("hipGetSymbolAddress of the scratch array failed: %s", hipGetErrorString(e));
      return CBS_EHIP;
    }
    g_scratch[device] = p;
  }
  *out = g_scratch[device];
  return CBS_OK;
}

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Bytes of scratch a call is admitted by (the limit that callers rely on): per pair of vectors its
// coefficients, two staging vectors and the projector coefficients, each 256-byte aligned.  The
// kernels use less of it: the projector coefficients, and a copy of x when y overlaps it.
static size_t need_bytes(const cbs_system* s, int32_t n_vec, size_t pair_bytes) {
  const size_t nr = (size_t)(n_vec + 1) / 2;
  size_t b = align256(nr * sizeof(RunCoef));
  b += 2 * align256(nr * (size_t)s->N * pair_bytes);
  if (s->proj.n_atoms > 0) b += align256(nr * (size_t)s->proj.n_atoms * 12 * pair_bytes);
  return b;
}

template <typename R>
static int32_t apply_noalloc(cbs_system* s, double E, int32_t n_vec, const double* z, const void* x, void* y,
                             unsigned char* base, hipStream_t st) {
  std::vector<double2> c0, cp, cm;
  apply_coefs(n_vec, z, c0, cp, cm);
  const size_t kt_bytes = align256(apply_kt_bytes(s, n_vec, sizeof(R)));
  const size_t bytes = (size_t)n_vec * s->N * sizeof(cplx<R>);
  if ((const char*)x < (const char*)y + bytes && (const char*)y < (const char*)x + bytes) {
    CBS_HIP(hipMemcpyAsync(base + kt_bytes, x, bytes, hipMemcpyDeviceToDevice, st));
    x = base + kt_bytes;
  }
  return launch_apply<R>(s, E, n_vec, c0.data(), cp.data(), cm.data(), x, y, base, nullptr, 0.0, st);
}

}  // namespace cbs

using namespace cbs;

extern "C" int32_t cbs_apply_noalloc(cbs_system* s, double E, int32_t n_vec, const double* z, int32_t dtype,
                                     const void* x, void* y, void* stream) {
  if (!s || n_vec < 0 || (n_vec > 0 && (!z || !x || !y)) || (dtype != CBS_C128 && dtype != CBS_C64)) {
    set_error("cbs_apply_noalloc: bad argument");
    return CBS_EINVAL;
  }
  for (int v = 0; v < n_vec; ++v) {
    if (z[2 * v] == 0.0 && z[2 * v + 1] == 0.0) {
      set_error("cbs_apply_noalloc: z must be nonzero");
      return CBS_EINVAL;
    }
  }
  if (n_vec == 0) return CBS_OK;
  const size_t pb = (dtype == CBS_C128) ? sizeof(Pair<double>) : sizeof(Pair<float>);
  const size_t need = need_bytes(s, n_vec, pb);
  if (need > kScratchBytes) {
    set_error("cbs_apply_noalloc: %d vectors of %lld points need %zu bytes of scratch, the fixed array holds %zu",
              n_vec, (long long)s->N, need, kScratchBytes);
    return CBS_EINVAL;
  }
  CBS_HIP(hipSetDevice(s->device));
  void* base = nullptr;
  CBS_TRY(noalloc_scratch(s->device, &base));
  hipStream_t st = (hipStream_t)stream;
  if (dtype == CBS_C128) return apply_noalloc<double>(s, E, n_vec, z, x, y, (unsigned char*)base, st);
  return apply_noalloc<float>(s, E, n_vec, z, x, y, (unsigned char*)base, st);
}
