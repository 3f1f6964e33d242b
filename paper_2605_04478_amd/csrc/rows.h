// The window's payload rows: 16 bytes per record.
//
//   x        low 32 bits of t_enter
//   y        bits 0-11 t_enter 32..43 | 12-15 op | 16-26 number of the record in its round of the ingest where
//            batches are placed by bucket (the grid placement puts the record's cell here) | 27-31 bytes 32..36
//   z        t_exit - t_enter, ROW_INFLIGHT while the operation runs, ROW_WIDE for a row that does not fit
//   w        low 32 bits of bytes; the window slot for a row that does not fit
//
// t_enter is kept modulo 2^44 ns (4.9 hours) and read relative to the first record of a batch.  A record whose t_enter lies
// 2^42 ns or more from its batch's first one, that runs for 2^32 - 2 ns or more, or that moves 2^37 bytes or more
// keeps its three values at full width in a second array that is written for such records only.
#pragma once
#include "device_utils.h"
#include "ccld_internal.h"

namespace ccld {

constexpr u32 ROW_INFLIGHT = 0xFFFFFFFFu, ROW_WIDE = 0xFFFFFFFEu;
constexpr u32 ROW_SAME_MASK = 0xF800F000u;        // bits of y that hold op and the upper bytes
constexpr u32 ROW_CELL_SHIFT = 16, ROW_CELL_MASK = 2047u;

// A row in full: what every kernel but the grid statistics works on.
struct Rec { i64 t_enter, t_exit; u64 bytes; u32 op; };

// packs one record; false: it does not fit, and wide[3 slot ..] takes its values
__device__ __forceinline__ bool pack_row(i64 te, i64 tx, u64 nb, u32 op, i64 ref, u32 slot, uint4* out) {
  const u64 off = (u64)te - (u64)ref + ((u64)1 << 42);
  const bool open = tx == INT64_MAX;
  const u64 dur = (u64)tx - (u64)te;
  const bool fits = (off >> 43) == 0 && (open || dur < (u64)ROW_WIDE) && (nb >> 37) == 0;
  const u32 opb = (op & 15u) << 12;
  if (fits) *out = make_uint4((u32)(u64)te, ((u32)((u64)te >> 32) & 0xFFFu) | opb | ((u32)(nb >> 32) << 27), open ? ROW_INFLIGHT : (u32)dur, (u32)nb);
  else *out = make_uint4(0u, opb, ROW_WIDE, slot);
  return fits;
}
__device__ __forceinline__ u64 row_t44(const uint4& v) { return (u64)v.x | ((u64)(v.y & 0xFFFu) << 32); }
__device__ __forceinline__ u32 row_op(const uint4& v) { return (v.y >> 12) & 15u; }
__device__ __forceinline__ u64 row_bytes(const uint4& v) { return (u64)v.w | ((u64)(v.y >> 27) << 32); }
// signed difference of two times kept modulo 2^44
__device__ __forceinline__ i64 t44_diff(u64 a, u64 b) { return (i64)((a - b) << 20) >> 20; }
__device__ __forceinline__ Rec unpack_row(const uint4& v, i64 ref, const i64* __restrict__ wide) {
  Rec r;
  r.op = row_op(v);
  if (v.z == ROW_WIDE) {
    const i64* w = wide + 3ull * v.w;
    r.t_enter = w[0]; r.t_exit = w[1]; r.bytes = (u64)w[2];
  } else {
    r.t_enter = ref + t44_diff(row_t44(v), (u64)ref);
    r.t_exit = v.z == ROW_INFLIGHT ? INT64_MAX : r.t_enter + (i64)v.z;
    r.bytes = row_bytes(v);
  }
  return r;
}
// Time that the rows of the batch holding window slot `slot` are relative to: one time serves the whole window unless
// its batches lie hours apart (W.far), when the slot's batch is looked up.
__device__ __forceinline__ i64 ref_of_slot(const WindowRows& W, u32 slot) {
  if (!W.far) return W.ref;
  const u32 off = slot >= W.head ? slot - W.head : slot + W.cap - W.head;
  for (u32 m = 0; m < W.n_batch; ++m) {
    const BatchMeta& b = W.meta[(W.slot0 + m) % W.n_meta];
    const u32 t = (u32)b.tail;
    const u32 start = t >= W.head ? t - W.head : t + W.cap - W.head;
    if (b.n && off - start < (u32)b.n) return b.ref;
  }
  return W.ref;
}
// Position of a window slot in the window's order of arrival.  A batch that was placed by bucket has the record's number
// in its round in the row; the round follows from the slot, since every round has a stretch of its own in every bucket.
// (Two searches for the few callers that ask, instead of 4 bytes more per record at ingest: 82M records 3.69 -> 3.50 ms.)
__device__ __forceinline__ u32 arrival_of_slot(const WindowRows& W, u32 slot) {
  const u32 off = slot >= W.head ? slot - W.head : slot + W.cap - W.head;
  if (!W.rounds) return off;
  for (u32 m = 0; m < W.n_batch; ++m) {
    const u32 at = (W.slot0 + m) % W.n_meta;
    const BatchMeta& b = W.meta[at];
    const u32 t = (u32)b.tail, start = t >= W.head ? t - W.head : t + W.cap - W.head;
    if (!b.n || off - start >= (u32)b.n) continue;
    const u32 o = off - start;
    const u32* base = W.bucket_base + (u64)at * (W.n_buckets + 1);
    u32 lo = 0, hi = W.n_buckets;                       // the bucket: the last one that starts at or before o
    while (hi - lo > 1) { const u32 mid = (lo + hi) >> 1; if (base[mid] <= o) lo = mid; else hi = mid; }
    const u32* col = W.rounds + (u64)b.round0 * W.n_buckets + lo;
    u32 r = 0, end = b.n_rounds;                        // the round, likewise
    while (end - r > 1) { const u32 mid = (r + end) >> 1; if (col[(u64)mid * W.n_buckets] <= o) r = mid; else end = mid; }
    const u32 num = (W.row[slot].y >> ROW_CELL_SHIFT) & ROW_CELL_MASK;
    return start + (u32)(r / b.per_group * b.chunk) + r % b.per_group * INGEST_ROUND + num;
  }
  return off;
}
static_assert(INGEST_ROUND == ROW_CELL_MASK + 1, "a round's numbers fit the row's free bits");
__device__ __forceinline__ Rec load_rec(const WindowRows& W, u32 slot) {
  return unpack_row(W.row[slot], ref_of_slot(W, slot), W.wide);
}

}  // namespace ccld
