// The blame order: ranks by (flags descending, summed lag descending, rank ascending).  Ranks with any flag come first and
// only they need ranking: a wavefront per flagged rank counts the flagged ranks that precede it.  The ranks without a
// flag follow in ascending order.
#pragma once
#include "ccld_internal.h"
#include "device_utils.h"

namespace ccld {

// Number of flagged ranks that come before rank r, counted by one wavefront over a list of the flagged ranks.
template <class T>
__device__ __forceinline__ u32 blamed_before(const i64* __restrict__ blame, u32 n_ranks, const T* list, u32 nb, u32 r, u32 lane) {
  const i64* NE = blame + (u64)CCLD_BLM_N_LATE_ENTER * n_ranks;
  const i64* NX = blame + (u64)CCLD_BLM_N_LATE_EXIT * n_ranks;
  const i64* SE = blame + (u64)CCLD_BLM_SUM_LAG_ENTER * n_ranks;
  const i64* SX = blame + (u64)CCLD_BLM_SUM_LAG_EXIT * n_ranks;
  const i64 myn = NE[r] + NX[r];
  const i64 mys = (i64)((u64)SE[r] + (u64)SX[r]);
  u32 before = 0;
  for (u32 i = lane; i < nb; i += CCLD_WAVE) {
    const u32 o = list[i];
    const i64 on = NE[o] + NX[o];
    const i64 os = (i64)((u64)SE[o] + (u64)SX[o]);
    before += (on > myn) || (on == myn && (os > mys || (os == mys && o < r)));
  }
  return wave_sum(before);
}

}  // namespace ccld
