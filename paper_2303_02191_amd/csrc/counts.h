// The counters behind rtoss_pattern_histogram, for the library's own callers (host_ext.cpp makes fresh ones).
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "rtoss.h"

namespace rtoss {

// Zeros the counters of a dictionary of at most 256 patterns (select.hip): fresh counters need no trip through the framework's fill.
rtoss_status clear_counts(uint32_t* hist, int P, hipStream_t s);

}  // namespace rtoss
