// Two smoothing steps in one pass on rows of 4 KB and more, in x tiles
// (pair_tile.hip).  Internal interface.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

#include "sums.h"

namespace mg {

bool pair_tile_applies(int n, size_t elem);

// How the pair gets its first iterate x and x_prev.
enum PairStart {
    PAIR_PLAIN = 0,   // x, and xp (null: x_prev = 0)
    PAIR_ZERO = 1,    // steps 1 and 2 of a pass from zero: x = cd0 b, x_prev = 0 (x, xp not read)
    PAIR_PREVB = 2,   // steps 2 and 3 of a pass from zero: x, x_prev = cd0 b
    PAIR_PRO = 3      // the start of a pass from x + P ec, x_prev = 0
};
// y2 (and y1 when not null) as launch_smooth_pair_row; y1 with PAIR_PLAIN,
// PAIR_ZERO and PAIR_PRO only.  sums: PAIR_ZERO and PAIR_PREVB only.
template <typename T>
hipError_t launch_pair_tile(int n, double ih2, PairStart start, const T* x, const T* xp, const T* b, T* y2, T* y1,
                            const T* ec, double a1, double cd1, double a2, double cd2, double cd0,
                            const SumsJob& sums, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);

}  // namespace mg
