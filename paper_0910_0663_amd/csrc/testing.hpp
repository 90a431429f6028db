// Functions that the tests call in the built library; not part of the interface.
#pragma once

#include <cstdint>

#include "vtm.h"

extern "C" {

// Bounds every wait of h's resident runs to `ticks` of 10 ns (0: one try), to exercise the
// way back to a launch per sweep.  Returns whether h runs resident.
int vtm_testing_wait_ticks(vtm_handle h, uint64_t ticks);

// The number of sweep that h's next resident run starts from (as if that many had run).
// Returns the number it had.
uint32_t vtm_testing_epoch(vtm_handle h, uint32_t epoch);

// Bounds the device memory that handles set up or refreshed on the calling thread may take
// from now on (negative: no bound).  Returns the least that was left under the bound before,
// or -1 without one.
int64_t vtm_testing_memory(int64_t bytes);

}  // extern "C"
