// Fused level visits of the 32^3 and 64^3 seven-point levels with Chebyshev
// smoothing (visit.hip).  Internal interface.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

namespace mg {

// Largest smoothing degree a fused visit handles (its halo must fit LDS).
constexpr int kVisitMaxDegree = 4;

// True when the pre (post) visit of the level (n^3 points of elem bytes,
// smoothing degree) can run fused.
bool visit_pre_applies(int n, int degree, size_t elem);
bool visit_post_applies(int n, int degree, size_t elem);

// Pre-smoothing from zero, residual and full weighting in one launch:
// xout (n^3) = `degree` steps from zero on b; coarse_b ((n/2)^3) = R(b - M xout).
// a[k], c[k]: the step coefficients of the level (x + a_k (x - x_prev) + c_k D^-1 (b - M x)).
template <typename T>
hipError_t launch_visit_pre(int n, double ih2, const T* b, T* xout, T* coarse_b, const double* a, const double* c,
                            int degree, hipStream_t s);

// Prolongation and post-smoothing in one launch: xout = `degree` steps on
// xin + P e (e on the (n/2)^3 grid); xout must differ from xin.
template <typename T>
hipError_t launch_visit_post(int n, double ih2, const T* xin, const T* e, const T* b, T* xout, const double* a,
                             const double* c, int degree, hipStream_t s);

}  // namespace mg
