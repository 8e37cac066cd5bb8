// 16-bit lanes of Smith-Waterman (sw16.hip).
#pragma once

#include "sw_common.hpp"

namespace pastis {

// Waves per block of a group's 16-bit kernel (groups as in sw.hip: one-strip
// bins of 1-4, 5-8, 9-12 and 13-16 rows per lane, multi-strip bins).
int sw16_waves(int group);
// Pass 1 of the group's bins of the mask; bins of at most `narrow` rows per
// lane (<= 4) run strips of 16 lanes.  A.queue holds one counter per (bin,
// rows class).
hipError_t launch_sw16(int group, int blocks, int narrow, const SwArgs &A, uint32_t bins, hipStream_t s);

}  // namespace pastis
