// Fused visits of small variable-coefficient levels (var_visit.hip).
// Internal interface.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

namespace mg {

// Visits run on levels of 32^3 points, up to kVarVisitMaxSteps smoothing steps
// a pass where the tile and its halo fit LDS (float: 4, double: 3).
constexpr int kVarVisitMaxSteps = 4;
bool var_visit_applies(int n, int steps, size_t elem);

// Pre visit: from x1 (the first step from zero) the remaining steps - 1
// smoothing steps, the residual and its full weighting.  Writes the smoothed
// iterate to xout (another buffer than x1), the coarse right-hand side to cb
// and, where cx1 is given, the coarse level's first step cx1 = cc0 cb / D
// with the coarse coefficients cC.  a, c: the pass's coefficients; cheb: the
// steps read the previous iterate.
template <typename T>
hipError_t launch_var_visit_pre(int n, double ih2, const T* C, const T* x1, const T* b, T* xout, T* cb, const T* cC,
                                T* cx1, double cc0, const double* a, const double* c, int steps, bool cheb,
                                hipStream_t s);
// Post visit: x + P e, then the smoothing pass; xout is another buffer than x.
template <typename T>
hipError_t launch_var_visit_post(int n, double ih2, const T* C, const T* x, const T* e, const T* b, T* xout,
                                 const double* a, const double* c, int steps, bool cheb, hipStream_t s);

}  // namespace mg
