// Hang alerts: what the list of a few (groups.hip) and of many (window.hip) share.
#pragma once
#include "ccld_internal.h"
#include "device_utils.h"
#include "grid.h"
#include "rows.h"
#include "window_kernels.h"

namespace ccld {

// Where the records of a collective are found: by binary search among the sorted keys, or by cell on the grid.
// t_exit of member slot q's record in table row s, or false: no record
template <bool GRID>
__device__ __forceinline__ bool alert_record(const AlertArgs& a, u32 s, u32 comm, u32 first, u32 nn, u32 q, i64* t_exit) {
  if (GRID) {
    const CommLayout L = a.grid.lay[comm];
    const u32 k = s - L.seg_base, fr = k / L.rpb;
    const u32 li = a.grid.cell_row[L.cell_base + k * L.size + q];
    if (li == GRID_EMPTY) return false;
    *t_exit = unpack_row(a.grid.rows[L.cell_base + fr * L.rpb * L.size + li], a.grid.hdr->ref, a.grid.wide).t_exit;
    return true;
  }
  const u64 mmask = ((u64)1 << a.sf.mb) - 1;      // key slot = position among the members in ascending rank order
  u32 lo = first, hi = first + nn;
  while (lo < hi) { const u32 m = (lo + hi) / 2; if ((u32)(a.key[m] & mmask) < q) lo = m + 1; else hi = m; }
  if (lo >= first + nn || (u32)(a.key[lo] & mmask) != q) return false;
  *t_exit = load_rec(a.win, a.idx[lo]).t_exit;
  return true;
}
// Class of an alert by the first two questions of the hang decision tree.  Not entered: the members with no record for
// this operation counter are the candidates; else inconsistent: everyone entered, and the ranks that completed are; else all
// hung: needs the Send/Recv counters.
__device__ __forceinline__ int alert_class(u32 n, u32 n_inflight, u32 size) {
  return n < size ? CCLD_HANG_H1_NOT_ENTERED : n_inflight < n ? CCLD_HANG_H2_INCONSISTENT : CCLD_HANG_H3_HARDWARE;
}

}  // namespace ccld
