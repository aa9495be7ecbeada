// Single-workgroup V-cycle tail of a variable-coefficient hierarchy
// (var_tail.hip): the levels of at most 16^3 points down to a coarsest level
// of 8^3 or 4^3, in one kernel launch.  Internal interface.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

#include "tail.h"

namespace mg {

template <typename T>
struct VarTailArgs {
    int nlev;                    // levels in the tail, the last one is the coarsest
    int n[kTailMaxLevels];
    double ih2[kTailMaxLevels];
    const T* C[kTailMaxLevels];  // six coefficient fields of each level
    const T* b;                  // right-hand side of the first tail level
    T* x;                        // its V-cycle result
    const double* G;             // dense pseudo-inverse of the coarsest operator
    TailSchedule sched;
    SumsJob sums;                // count > 0: outer sums finished by a second block
};

// Levels of 16^3 and 8^3 points (or one of them) above a coarsest level of
// 4^3, halving each time.
inline bool var_tail_dense4(int first_n, int nlev) { return (first_n == 16 && nlev == 3) || (first_n == 8 && nlev == 2); }
// 16^3 points above a coarsest level of 8^3: the workgroup reads a dense
// inverse of 2 MB by itself, which only passes of enough steps make up for, and
// more of them the more levels (`above`) run between two reads.  One cycle,
// tail against launches in us:
//   float   16^3  degree 3 50 and 49, 4 53 and 58; 32^3 3 66 and 64, 4 74 and 80
//           64^3  3 139 and 98, 8 265 and 264; 128^3 3 263 and 219, 8 532 and 517,
//           16 Jacobi sweeps 64^3 438 and 510, 128^3 908 and 956
//   double  16^3  4 64 and 60, 5 69 and 70; 64^3 3 119 and 111, 5 190 and 197;
//           128^3 5 525 and 520, 7 699 and 700
inline bool var_tail_dense8(int above, int steps, size_t elem) {
    return elem == sizeof(float) ? steps >= (above <= 1 ? 4 : 12) : steps >= (above <= 2 ? 5 : 7);
}
// The levels from `above` down to the coarsest (coarsest_n points per side) run in the tail.
inline bool var_tail_applies(int first_n, int coarsest_n, int nlev, int above, int steps, size_t elem) {
    if (coarsest_n == 4) return var_tail_dense4(first_n, nlev);
    return first_n == 16 && coarsest_n == 8 && nlev == 2 && var_tail_dense8(above, steps, elem);
}

template <typename T>
hipError_t launch_var_tail(const VarTailArgs<T>& args, hipStream_t s);

}  // namespace mg
