// An entry point that allocates nothing: the starlet transform Phi^T (Eq. 6)
// without a plan, for callers that cannot allocate device memory (code under
// graph capture, tight loops, hosts that forbid allocation). Its working planes
// live in one fixed device array of this file, `scratch`, whose device address
// is looked up once per device; inputs and outputs are the caller's.
#include "starred.h"
#include "starred_internal.h"
#include "starred_scales.h"

#include <hip/hip_runtime.h>

#include <cstdio>
#include <mutex>
#include <string>

using namespace starred;

namespace {

// The planes between the transform's passes (two of N^2 floats, N <= kStaticMaxSide).
constexpr int kStaticMaxSide = 512;
constexpr int kStaticMaxScales = 16;
constexpr size_t kScratchFloats = 2 * (size_t)kStaticMaxSide * kStaticMaxSide + 16;

static __device__ __align__(256) float scratch[kScratchFloats];

constexpr int kMaxDevices = 64;
std::mutex g_mu;
float *g_ptr[kMaxDevices] = {};

}  // namespace

// defined with the plan (sets the calling thread's message)
int starred_set_error(int code, const char *msg);

extern "C" int starred_starlet_fwd_noalloc(int32_t N, int32_t J, const float *img, float *coeffs, void *stream)
{
    if (!img || !coeffs) return starred_set_error(STARRED_EINVAL, "NULL argument");
    if (N < 2 || J < 1) return starred_set_error(STARRED_EINVAL, "N must be >= 2 and J >= 1");
    if (J > 1 && (1 << (J - 1)) > N - 1) return starred_set_error(STARRED_EINVAL, "2^(J-1) must not exceed N-1");
    if (N > kStaticMaxSide || J > kStaticMaxScales)
        return starred_set_error(STARRED_EINVAL, "starred_starlet_fwd_noalloc: N above 512 or J above 16 "
                                                 "(the fixed working array holds two 512 x 512 planes)");
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return starred_set_error(STARRED_EHIP, hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return starred_set_error(STARRED_EUNSUPPORTED, "device index above 63");
    float *base = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (!g_ptr[dev]) {
            // the array's device address on this device (the host-side name is not one)
            void *ptr = nullptr;
            e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !ptr) {
                char buf[256];
                snprintf(buf, sizeof buf, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
                return starred_set_error(STARRED_EHIP, buf);
            }
            g_ptr[dev] = (float *)ptr;
        }
        base = g_ptr[dev];
    }
    hipStream_t st = (hipStream_t)stream;
    StarArgs a;
    a.N = N;
    a.J = J;
    a.B = 1;
    a.fp64 = false;  // the working planes are FP32
    a.img = img;
    a.coeffs = coeffs;
    a.ca = base;
    a.cb = base + (size_t)N * N;
    e = launch_star_forward(st, a);
    if (e != hipSuccess) return starred_set_error(STARRED_EHIP, hipGetErrorString(e));
    return STARRED_OK;
}
