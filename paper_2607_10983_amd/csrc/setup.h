// Setup of a variable-coefficient hierarchy on the device (setup.hip): level
// coefficients, their validity, the Gershgorin bounds and the dense inverse of
// the coarsest operator.  Internal interface; everything is stream-ordered and
// nothing waits for the host.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

namespace mg {

typedef unsigned long long u64;

// slots[i] = 0, i < count
hipError_t launch_clear_slots(u64* slots, int count, hipStream_t s);

// Six coefficient fields of n3 values each, src -> inner (type TI) and, where
// given, outer (double); the number of cells that are not finite or have a
// diagonal component <= 0 is added to *bad.
template <typename TS, typename TI>
hipError_t launch_coeff_copy(size_t n3, const TS* src, TI* inner, double* outer, u64* bad, hipStream_t s);

// *lmax = max(*lmax, Gershgorin bound of D^-1 M) as the bits of a double.
template <typename TC>
hipError_t launch_bound(int n, const TC* C, u64* lmax, hipStream_t s);

// Full weighting of ncomp fields (values of type TS, sums in double) into dst
// and, where given, a copy rounded to float.
template <typename TS>
hipError_t launch_restrict_fields(int n, const TS* src, double* dst, float* copy, int ncomp, hipStream_t s);

// Moving-mesh geometry of psi: C in double and / or float (six fields), det J
// where sqrtg is given; bad as for launch_coeff_copy where given.
hipError_t launch_geometry_fields(int n, double ih2, const double* psi, double* Cd, float* Cf, double* sqrtg, u64* bad,
                                  hipStream_t s);

// Zero-mean pseudo-inverse G of the 19-point operator on the coarsest level
// (n = 4 or 8, N = n^3), by an elimination without pivoting: right where the
// operator is negative semidefinite, as it is for positive definite C.  work:
// 2 N^2 + 2 N doubles.  Adds the number of values of G that are not finite to
// *bad, and to *indefinite the number of steps that met a pivot which is not
// negative; where either is not zero, G is to be formed with pivoting.
hipError_t launch_dense_inverse(int n, double ih2, const double* C, double* G, double* work, u64* bad,
                                u64* indefinite, hipStream_t s);
inline size_t dense_work(int n) {
    const size_t N = (size_t)n * n * n;
    return 2 * N * N + 2 * N;
}

}  // namespace mg
