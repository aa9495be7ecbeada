// Passes of the conjugate-gradient solve for the seven-point operator on rows
// of 64 points and more (pcg_row.hip).  Internal interface.
#pragma once
#include <hip/hip_runtime.h>

#include "sums.h"

namespace mg {

// n = 64 ... 1024; smaller and larger grids and 19-point operators take the
// passes of pcg.hip, which store q = M p.
bool pcg_row_applies(int n);
// Each pass writes this many partial sums per sum.
int pcg_row_blocks(int n);

// TI: type of the hierarchy.  r_in (TI's copy of r) is written for float only;
// with a double hierarchy the caller lets r be its right-hand side.

// r = b - mean - M phi; sums (b - mean)^2, (r, r), phi.
template <typename TI>
hipError_t launch_pcg_row_residual(int n, double ih2, const double* phi, const double* b, Mean mean, double* r,
                                   TI* rin, double* partials, hipStream_t s);
// (r, z) and, with p_prev, (z, M p_prev).
template <typename TI>
hipError_t launch_pcg_row_dots(int n, double ih2, const double* r, const TI* z, const double* p_prev,
                               double* partials, hipStream_t s);
// p = z + beta p_prev (p_prev null: p = z); (p, M p).  p is not p_prev.
template <typename TI>
hipError_t launch_pcg_row_direction(int n, double ih2, const TI* z, const double* p_prev, double* p,
                                    const double* scal, double* partials, hipStream_t s);
// phi += alpha p, r -= alpha M p; (r, r).
template <typename TI>
hipError_t launch_pcg_row_update(int n, double ih2, double* phi, const double* p, double* r, TI* rin,
                                 const double* scal, double* partials, hipStream_t s);

}  // namespace mg
