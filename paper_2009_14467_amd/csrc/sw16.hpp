// 16-bit lanes of Smith-Waterman (sw16.hip).
#pragma once

#include "sw_common.hpp"

namespace pastis {

int sw16_waves();       // waves per block
int sw16_step_words();  // most words of direction bits a step stores per wave

// Pass 1 (trace = false) or the traced statistics pass of the launch's bins.
// A.queue holds one counter per (bin, rows class).
hipError_t launch_sw16(bool trace, const Sw16Launch &P, const SwArgs &A, hipStream_t s);

// The windows of A.idx (A.bounds) for the launches of P: win, nwin (zeroed before).
hipError_t launch_sw16_windows(int64_t npairs, const Sw16Launch &P, const SwArgs &A, int *win, int *nwin,
                               hipStream_t s);
// The backward start bound of the A.queue[1] pairs listed in A.idx: rejected
// pairs get their final record, the others are listed for the traceback or
// binned for the statistics kernels (bin_of) and counted (counters[1], [2]).
hipError_t launch_sw16_bound(int64_t npairs, const SwArgs &A, const TraceRule &T, int8_t *bin_of,
                             unsigned long long *counters, hipStream_t s);

}  // namespace pastis
