// Long pairs of Smith-Waterman, one workgroup each (sw_long.hip).
#pragma once

#include "sw_common.hpp"

namespace pastis {

// Scratch words of one block where no sequence is longer than max_len.
int64_t sw_long_slot_words(int max_len);

// Pass 1 (stats = false) or the statistics of the items of the given bins
// (A.idx, A.starts, a queue counter per bin).  A.scratch, A.scratch_per_wave:
// slots of sw_long_slot_words, one per block.
hipError_t launch_sw_long(bool stats, int blocks, uint32_t bins, const SwArgs &A, hipStream_t s);

}  // namespace pastis
