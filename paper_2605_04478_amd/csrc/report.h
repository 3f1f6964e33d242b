// How a pass ends: its counters in pinned host memory, which the host watches (wait_report in api.hip).
#pragma once
#include "ccld_internal.h"
#include "device_utils.h"

namespace ccld {

// Each counter goes out with its ticket (ticket.h).  The host waits until every word carries the ticket, so the
// words need no order among themselves.  Called by the first wavefronts of one workgroup.
__device__ __forceinline__ void report_words(const u64* counters, u64* host, u64 ticket) {
  if (threadIdx.x < CNT_COUNT) {
    const u64 v = __hip_atomic_load(&counters[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&host[threadIdx.x], report_word(v, ticket), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}
static_assert(CNT_COUNT <= 64, "one wavefront copies the counters");

// The last workgroup to get here reports.  No cache is written back on the way: what the kernel wrote for later
// kernels is, at its end; what the caller reads has been written by earlier kernels, or with store_agent.
__device__ __forceinline__ void report_counters(u64* counters, u32* arrivals, u64* host, u64 ticket) {
  __shared__ u32 s_last;
  if (last_arrival(arrivals, gridDim.x, &s_last)) report_words(counters, host, ticket);
}

}  // namespace ccld
