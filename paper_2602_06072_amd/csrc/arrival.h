// How the workgroups of a launch find out which of them is the last to finish: each counts itself in once, and the count
// wraps to zero with the last arrival.  One operation for both: were zero stored by a second one, an arrival of another launch
// between the two (launches that overlap on one workspace, which the caller must not let happen) would be lost, and every
// later launch would merge too early or not at all.
#pragma once
#include <cstdint>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define PK_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define PK_HOST_DEVICE inline
#endif

namespace pk {

// Count::next(limit): x -> x >= limit ? 0 : x + 1 in one atomic operation; returns x.
template <class Count>
PK_HOST_DEVICE bool arrives_last(Count&& count, const uint32_t arrivals) { return count.next(arrivals - 1) == arrivals - 1; }

}  // namespace pk
