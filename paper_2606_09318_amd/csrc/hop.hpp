// When a pointer-doubling loop has to stop: host and device code, so that the
// loops' end can be tested on the CPU.
#pragma once
#include <stdint.h>

#if defined(__HIP__)
#define LR_HD __host__ __device__ __forceinline__
#else
#define LR_HD inline
#endif

namespace lr {

// An element composes its record, `before` links long, with the record it
// points to and gets one of `after` links (32-bit sum); ended: that one leads to
// a terminal. True where the element must stop because the records are not a
// forest's: more links than a list can have (climit: elements of the input), or
// an open record that added none. The second needs no valid record to hold: an
// input that is not a forest leaves records unwritten, and whatever the memory
// holds there (counts of zero, counts that wrap), an element that goes on has
// counted at least one link more, so it goes on less than climit times.
LR_HD bool hop_stuck(uint32_t before, uint32_t after, bool ended, uint32_t climit) {
    return after >= climit || (!ended && after <= before);
}

}  // namespace lr
