// Hang alerts: what the list of a few (groups.hip) and of many (window.hip) share.
#pragma once
#include "ccld_internal.h"
#include "device_utils.h"

namespace ccld {

// Class of an alert by the first two questions of the hang decision tree.  Not entered: the members with no record for
// this operation counter are the candidates; else inconsistent: everyone entered, and the ranks that completed are; else all
// hung: needs the Send/Recv counters.
__device__ __forceinline__ int alert_class(u32 n, u32 n_inflight, u32 size) {
  return n < size ? CCLD_HANG_H1_NOT_ENTERED : n_inflight < n ? CCLD_HANG_H2_INCONSISTENT : CCLD_HANG_H3_HARDWARE;
}

}  // namespace ccld
