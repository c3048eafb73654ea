// The launch of the quantizer passes that take a large tensor in one trip (not installed; compiles without HIP).
#pragma once

#include <stdint.h>

namespace cdl {

// A wave's loads and stores share one counter that goes down in the order of their issue: in a loop that loads, computes and stores, the
// wait for a trip's loads is also a wait for the stores of the trip before it, which take microseconds to complete, and blocks that drift
// apart spread the accesses in flight over the whole tensor.  Tensors of more than kOneTripEntries therefore go through in one trip:
// a block of kOneTripThreads issues all its loads (kOneTripVectors of four entries a thread) before its first store, and blocks
// start in the order of the tensor.  us, as a loop of up to 2048 blocks / so (with the shorter arithmetic of cdl_quantizer_math.h), 31 levels, two on each side, from a
// cold cache: gradient without scalars (8 B read, 4 written an entry) 12.8 M entries 28.1 / 26.0, 25.6 M 52.6 / 49.3, 50.3 M 102 / 97, 115.6 M 239 / 224 (6.2 TB/s); with
// them 36.6 / 32.3, 62.7 / 56.4, 112 / 104, 256 / 235; index and soft value without PMF (4 B read, 5 written) 25.2 / 21.7, 43.4 / 37.8, 83.8 / 72.3,
// 198 / 167 (6.2 TB/s).  Blocks of 256 x 2 vectors against 512 x 3: 46 / 49 us (gradient of 25.6 M); one vector a thread 50.  (How many entries each pass
// needs for it: gradient_one_trip, entropy_one_trip and forward_one_trip in cdl_quantizer.hip.)
constexpr int kOneTripThreads = 256, kOneTripVectors = 2;

// Blocks.  The last one has at most the rest of the vectors, and the entries beyond them.
inline int64_t one_trip_grid(int64_t n) { return ((n >> 2) + (int64_t)kOneTripThreads * kOneTripVectors) / ((int64_t)kOneTripThreads * kOneTripVectors); }

// Whether a launch can have as many: fewer than 2^32 threads (2^35 entries, 137 GB of fp32; larger tensors go through in a loop).
inline bool one_trip_fits(int64_t n) { return one_trip_grid(n) * kOneTripThreads < (1ll << 32); }

}  // namespace cdl
