// Index arithmetic of the one-launch LSTM recurrence (pf_lstm_persist.hip), for device and host.
#pragma once

#include "pf_lstm_persist.h"

namespace pf {

// Walks the elements first, first + step, ... of a list of rows of n elements each; row and o are the current element's row
// and place in it.  All steps' rows together have more elements than 32 bits count (three layers of rank 384, batch 32: from
// 34953 steps on), the rows alone do not, and no division is needed after the first element.
struct LpWalk {
    int row, o, n, rows_per_step, left_per_step;
    __host__ __device__ __forceinline__ LpWalk(int n_, int first, int step)
    {
        n = n_;
        row = first / n, o = first - row * n;
        rows_per_step = step / n, left_per_step = step - rows_per_step * n;
    }
    __host__ __device__ __forceinline__ void next()
    {
        row += rows_per_step;
        o += left_per_step;
        if (o >= n) o -= n, ++row;
    }
};

} // namespace pf
