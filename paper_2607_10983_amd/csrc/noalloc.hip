// mg_geometry_bwd_noalloc: the reverse mode of the moving-mesh geometry
// without any device allocation.  mg_geometry_bwd needs a temporary only where
// its result overlaps an input; this variant then uses a fixed, library-owned
// device array.
#include <hip/hip_runtime.h>

#include <mutex>

#include "geometry_bwd.h"
#include "kernels.h"
#include "mg.h"

using namespace mg;

namespace {

// 48 MiB of doubles per GPU, held until the process ends.
constexpr size_t kScratchDoubles = (size_t)48 * 1024 * 1024 / sizeof(double);
static_assert(kScratchDoubles == (size_t)MG_NOALLOC_SCRATCH_BYTES / sizeof(double), "header and library agree");

__device__ __align__(256) double scratch[kScratchDoubles];

// Device address of `scratch` per device, looked up once per device with that
// device current.  In host code the array's name is only a stand-in symbol.
constexpr int kMaxDevices = 64;
double* g_scratch[kMaxDevices] = {};
std::mutex g_scratch_mutex;

hipError_t scratch_of_current_device(double** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch[dev] = static_cast<double*>(p);
    }
    *out = g_scratch[dev];
    return hipSuccess;
}

}  // namespace

extern "C" mg_status mg_geometry_bwd_noalloc(int n, double h, const double* psi, const double* Cbar,
                                             const double* sqrtgbar, double* psibar, void* stream) {
    if (n < 4 || n > MG_NOALLOC_MAX_N || (n & (n - 1)) != 0 || !(h > 0) || !psi || !Cbar || !psibar)
        return MG_ERR_INVALID;
    const double ih2 = 1.0 / (h * h);
    const size_t N = (size_t)n * n * n;
    hipStream_t s = (hipStream_t)stream;
    if (!geometry_bwd_overlaps(N, psi, Cbar, sqrtgbar, psibar))
        return launch_geometry_bwd(n, ih2, psi, Cbar, sqrtgbar, psibar, s) == hipSuccess ? MG_OK : MG_ERR_HIP;
    if (N > kScratchDoubles) return MG_ERR_INVALID;  // it would overwrite what other blocks still read
    double* tmp = nullptr;
    if (scratch_of_current_device(&tmp) != hipSuccess) {
        (void)hipGetLastError();
        return MG_ERR_HIP;
    }
    hipError_t e = launch_geometry_bwd(n, ih2, psi, Cbar, sqrtgbar, tmp, s);
    if (e == hipSuccess) e = launch_shift(N, tmp, 0.0, psibar, s);
    return e == hipSuccess ? MG_OK : MG_ERR_HIP;
}
