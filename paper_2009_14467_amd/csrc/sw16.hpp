// 16-bit lanes of Smith-Waterman (sw16.hip).
#pragma once

#include "sw_common.hpp"

namespace pastis {

int sw16_waves();       // waves per block
int sw16_step_words();  // most words of direction bits a step stores per wave

// Pass 1 (trace = false) or the traced statistics pass of the launch's bins.
// A.queue holds one counter per (bin, rows class).
hipError_t launch_sw16(bool trace, const Sw16Launch &P, const SwArgs &A, hipStream_t s);

}  // namespace pastis
