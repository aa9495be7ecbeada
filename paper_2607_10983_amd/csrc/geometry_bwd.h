// Reverse mode of the moving-mesh geometry (geometry_bwd.hip).  Internal interface.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

namespace mg {

// psibar from the cotangents Cbar (6 n^3) and sbar (n^3, or null) at psi.
// psibar must not overlap the inputs (geometry_bwd_overlaps).
hipError_t launch_geometry_bwd(int n, double ih2, const double* psi, const double* Cbar, const double* sbar,
                               double* psibar, hipStream_t s);

inline bool geometry_bwd_overlaps(size_t N, const double* psi, const double* Cbar, const double* sbar,
                                  const double* psibar) {
    auto hit = [&](const double* p, size_t count) { return p && p < psibar + N && psibar < p + count; };
    return hit(psi, N) || hit(Cbar, 6 * N) || hit(sbar, N);
}

}  // namespace mg
