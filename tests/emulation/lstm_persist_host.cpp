// The index arithmetic of the one-launch LSTM recurrence on the host (test infrastructure, CPU only).  Built by
// tests/test_host_lstm_persist.py; nothing in the product loads it.
#include "pf_lstm_persist_index.h"

using namespace pf;

extern "C" {
// What a walk visits before row `rows`: how many elements, the last of them; 0 if one of them is not first + i * step.
int emu_walk(int n, int first, int step, int rows, long long *count, long long *last)
{
    *count = 0, *last = -1;
    for (LpWalk at(n, first, step); at.row < rows; at.next()) {
        const long long e = (long long)at.row * n + at.o;
        if (at.o < 0 || at.o >= n || e != first + *count * step) return 0;
        *last = e;
        ++*count;
    }
    return 1;
}
}
