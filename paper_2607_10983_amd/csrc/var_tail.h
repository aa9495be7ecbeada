// Single-workgroup V-cycle tail of a variable-coefficient hierarchy
// (var_tail.hip): the levels of at most 16^3 points down to a coarsest level
// of 8^3 or 4^3, in one kernel launch.  Internal interface.
#pragma once
#include <hip/hip_runtime.h>

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
// 8^3 or 4^3, halving each time.  With a coarsest level of 8^3 the workgroup
// reads a dense inverse of 2 MB by itself, which only passes of many steps make
// up for.  One cycle, tail against launches in us, 64^3 mixed: degree 3 140
// and 102, 6 224 and 212, 8 265 and 272; 64^3 double: 121 and 114, 219 and 235,
// 272 and 298; 128^3 mixed: 264 and 223, 433 and 422, 533 and 538.
constexpr int kVarTailDense8Steps = 8;
inline bool var_tail_applies(int first_n, int coarsest_n, int nlev, int steps) {
    return (first_n == 16 && coarsest_n == 4 && nlev == 3) || (first_n == 8 && coarsest_n == 4 && nlev == 2) ||
           (first_n == 16 && coarsest_n == 8 && nlev == 2 && steps >= kVarTailDense8Steps);
}

template <typename T>
hipError_t launch_var_tail(const VarTailArgs<T>& args, hipStream_t s);

}  // namespace mg
