// Single-workgroup V-cycle tail (tail.hip): the levels of at most 16^3 points
// of a seven-point hierarchy, down to a coarsest level of at most 8^3 points,
// in one kernel launch.  Internal interface.
#pragma once
#include <hip/hip_runtime.h>

#include "sums.h"

namespace mg {

constexpr int kTailMaxLevels = 4;
constexpr int kTailMaxSteps = 16;

struct TailSchedule {
    int steps;
    int cheb;  // 1: Chebyshev (uses the previous iterate), 0: Jacobi
    double a[kTailMaxLevels][kTailMaxSteps];
    double c[kTailMaxLevels][kTailMaxSteps];
};

template <typename T>
struct TailArgs {
    int nlev;                      // levels in the tail, the last one is the coarsest
    int n[kTailMaxLevels];
    double ih2[kTailMaxLevels];
    const T* b;                    // right-hand side of the first tail level
    T* x;                          // its V-cycle result
    TailSchedule sched;
    const double* Q;               // coarsest separable basis (nc x nc)
    const double* lam1;            // its 1-D eigenvalues
    SumsJob sums;                  // count > 0: outer sums finished by a second block
};

template <typename T>
hipError_t launch_tail(const TailArgs<T>& args, hipStream_t s);

}  // namespace mg
