// Per-collective statistics for gfx950.  Collectives of up to 64 records are packed side by side
// into the lanes of a wavefront and sorted there with a bitonic network whose exchanges are DPP
// row operations wherever the lane pattern allows, which yields minimum, exact lower median
// (order statistic floor((n-1)/2)), maximum, and then the median absolute deviation.  Collectives
// of 65 to 512 records take a wavefront each with 2, 4 or 8 values per lane in registers, those of
// up to 16,384 records a workgroup each with a bitonic sort in LDS (k_seg_team, k_seg_large), and longer ones
// the counting selection of k_seg_big.  Windows on the grid placement (grid.h) have kernels of their own at the end.
#include <type_traits>

#include "window_kernels.h"
#include "grid.h"
#include "rows.h"

namespace ccld {

constexpr i64 T_INFLIGHT = INT64_MAX;
constexpr int SEG_WAVE_MAX = 64;     // longest collective handled inside one wavefront's registers
constexpr int SEG_MULTI_MAX = 512;   // longest collective one wavefront sorts in registers (eight values per lane)
constexpr int SEG_TEAM_MAX = 2048;   // longest collective a workgroup of 256 threads sorts in LDS (three arrays)
constexpr int SEG_LARGE_MAX = 16384; // longest collective a workgroup of 1,024 threads sorts in LDS (one array of 128 KB)

__device__ __forceinline__ u64 atomic_add_u64(u64* p, u64 v) {
  return atomicAdd((unsigned long long*)p, (unsigned long long)v);
}

__device__ __forceinline__ void seg_put(const SegArgs& a, int col, u32 srow, i64 v) {
  if (srow < a.seg_cap) a.seg[(u64)col * a.seg_cap + srow] = v;
}
// detection-group code (op, size class) and intra-round range T_max - T_min (Eq. 2) of one collective
__device__ __forceinline__ u32 seg_group_code(bool usable, u32 op, u64 nb) {
  return usable ? op * GROUP_CLS + (63 - (u32)__clzll((long long)(nb | 1))) : NO_GROUP;
}
__device__ __forceinline__ void seg_put_group(const SegArgs& a, u32 srow, bool usable, u32 op, u64 nb, i64 dmax, i64 dmin) {
  a.gcode[srow] = (uint16_t)seg_group_code(usable, op, nb);
  a.range_c[srow] = usable ? dmax - dmin : 0;
}
// counts a collective that raises a hang alert (an operation in flight longer than the threshold, barriers excepted);
// the first few leave their rows for the end of the analysis, which lists them; longer lists are built when they are known
__device__ __forceinline__ void seg_count_alert(const SegArgs& a, u32 srow, u32 ninfl, bool barrier, i64 imin) {
  if (!ninfl || barrier || a.now_ns - imin <= a.hang_threshold_ns || srow >= a.seg_cap) return;
  const u64 at = atomic_add_u64(&a.counters[CNT_NALERT], 1);
  if (at < END_ALERTS) a.alert_rows[at] = srow;
}
__device__ __forceinline__ i64 absdiff(i64 a, i64 b) { return a >= b ? a - b : b - a; }
// the j-th record in (communicator, counter, rank) order
__device__ __forceinline__ Rec load_row(const SegArgs& a, u32 j) { return load_rec(a.win, a.idx[j]); }
__device__ __forceinline__ bool is_late(i64 lag, i64 floor_ns, u32 knum, u32 kden, i64 mad) {
  return lag > floor_ns && (i128)lag * (i128)kden > (i128)knum * (i128)mad;
}
__device__ __forceinline__ void seg_put_empty_stats(const SegArgs& a, u32 srow) {
  for (int c = CCLD_SEG_ENTER_MIN; c <= CCLD_SEG_DUR_MAX; ++c) seg_put(a, c, srow, 0);
  seg_put(a, CCLD_SEG_ARGMIN_RANK, srow, CCLD_NO_RANK);
  seg_put(a, CCLD_SEG_ARGMAX_RANK, srow, CCLD_NO_RANK);
}


// ---- lane exchanges ------------------------------------------------------------------------
// value held by lane (lane ^ M)
template <int M>
__device__ __forceinline__ u32 xor_lane_u32(u32 v) {
  const int s = (int)v;
  // every lane of these patterns reads a valid lane, so no previous value has to be kept: the plain
  // DPP move needs no copy of the destination first
  if constexpr (M == 1) return (u32)__builtin_amdgcn_mov_dpp(s, 0xB1, 0xF, 0xF, true);        // quad_perm [1,0,3,2]
  else if constexpr (M == 2) return (u32)__builtin_amdgcn_mov_dpp(s, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
  else if constexpr (M == 3) return (u32)__builtin_amdgcn_mov_dpp(s, 0x1B, 0xF, 0xF, true);   // quad_perm [3,2,1,0]
  else if constexpr (M == 7) return (u32)__builtin_amdgcn_mov_dpp(s, 0x141, 0xF, 0xF, true);  // row_half_mirror
  else if constexpr (M == 15) return (u32)__builtin_amdgcn_mov_dpp(s, 0x140, 0xF, 0xF, true); // row_mirror
  else if constexpr (M == 8) return (u32)__builtin_amdgcn_mov_dpp(s, 0x128, 0xF, 0xF, true);  // row_ror:8
  else if constexpr (M == 4) {
    int t = __builtin_amdgcn_mov_dpp(s, 0x104, 0xF, 0x5, true);           // banks 0,2 read lane + 4 (row_shl:4)
    t = __builtin_amdgcn_update_dpp(t, s, 0x114, 0xF, 0xA, false);        // banks 1,3 read lane - 4 (row_shr:4)
    return (u32)t;
  } else
    return __shfl_xor(v, M, CCLD_WAVE);       // masks that cross a row of 16 lanes
}
template <int M>
__device__ __forceinline__ i64 xor_lane_i64(i64 v) {
  const u32 lo = xor_lane_u32<M>((u32)(u64)v), hi = xor_lane_u32<M>((u32)((u64)v >> 32));
  return (i64)(((u64)hi << 32) | lo);
}
__device__ __forceinline__ i64 shfl_i64(i64 v, int src) { return (i64)shfl_u64((u64)v, src); }

constexpr int high_bit(int m) { int b = 1; while (b * 2 <= m) b *= 2; return b; }

// compare-exchange with lane ^ M: the lane whose top bit of M is clear keeps the smaller value
template <int M>
__device__ __forceinline__ i64 cmpx(i64 v, u32 lane) {
  const i64 p = xor_lane_i64<M>(v);
  const bool upper = (lane & high_bit(M)) != 0;
  return ((p < v) != upper) ? p : v;
}

// ascending sort inside every aligned group of G lanes (bitonic merges: mirror, then halving strides)
template <int G>
__device__ __forceinline__ i64 sort_groups(i64 v, u32 lane) {
  if constexpr (G >= 2) { v = cmpx<1>(v, lane); }
  if constexpr (G >= 4) { v = cmpx<3>(v, lane); v = cmpx<1>(v, lane); }
  if constexpr (G >= 8) { v = cmpx<7>(v, lane); v = cmpx<2>(v, lane); v = cmpx<1>(v, lane); }
  if constexpr (G >= 16) { v = cmpx<15>(v, lane); v = cmpx<4>(v, lane); v = cmpx<2>(v, lane); v = cmpx<1>(v, lane); }
  if constexpr (G >= 32) {
    v = cmpx<31>(v, lane); v = cmpx<8>(v, lane); v = cmpx<4>(v, lane); v = cmpx<2>(v, lane); v = cmpx<1>(v, lane);
  }
  if constexpr (G >= 64) {
    v = cmpx<63>(v, lane); v = cmpx<16>(v, lane); v = cmpx<8>(v, lane); v = cmpx<4>(v, lane);
    v = cmpx<2>(v, lane); v = cmpx<1>(v, lane);
  }
  return v;
}

// ascending sort of a sequence that falls and then rises inside every aligned group of G lanes (one bitonic
// merge: halving strides).  The absolute deviations of sorted values from their median form such a sequence,
// with the empty lanes' largest value at its end.
template <int G>
__device__ __forceinline__ i64 merge_groups(i64 v, u32 lane) {
  if constexpr (G >= 64) v = cmpx<32>(v, lane);
  if constexpr (G >= 32) v = cmpx<16>(v, lane);
  if constexpr (G >= 16) v = cmpx<8>(v, lane);
  if constexpr (G >= 8) v = cmpx<4>(v, lane);
  if constexpr (G >= 4) v = cmpx<2>(v, lane);
  if constexpr (G >= 2) v = cmpx<1>(v, lane);
  return v;
}

// all-reduce inside a group: smallest (d, r) / largest d with the smallest r among equals
template <int G, bool MAXIMUM>
__device__ __forceinline__ void reduce_dur(i64& d, u32& r) {
#define CCLD_DUR_STEP(M)                                                        \
  if constexpr (G > M) {                                                        \
    const i64 od = xor_lane_i64<M>(d);                                          \
    const u32 orr = xor_lane_u32<M>(r);                                         \
    const bool better = MAXIMUM ? (od > d) : (od < d);                          \
    if (better || (od == d && orr < r)) { d = od; r = orr; }                    \
  }
  CCLD_DUR_STEP(1) CCLD_DUR_STEP(2) CCLD_DUR_STEP(4) CCLD_DUR_STEP(8) CCLD_DUR_STEP(16) CCLD_DUR_STEP(32)
#undef CCLD_DUR_STEP
}
template <int G>
__device__ __forceinline__ i64 reduce_min(i64 v) {
#define CCLD_MIN_STEP(M) if constexpr (G > M) { const i64 o = xor_lane_i64<M>(v); v = o < v ? o : v; }
  CCLD_MIN_STEP(1) CCLD_MIN_STEP(2) CCLD_MIN_STEP(4) CCLD_MIN_STEP(8) CCLD_MIN_STEP(16) CCLD_MIN_STEP(32)
#undef CCLD_MIN_STEP
  return v;
}

typedef __attribute__((address_space(3))) i64 lds_i64;      // an LDS word: 32-bit addresses, ds instructions

// What one lane knows about its record before the group-wide statistics.
struct DenseLane {
  i64 e, x;          // arrival, completion (T_INFLIGHT while the operation runs)
  u64 nb;            // bytes
  u32 op, rank;
  bool valid;        // the lane's member has a record in this collective
  u32 fl;            // first lane of this lane's collective that has a record
  u32 n, first, j;   // records of the collective, sorted position of its first record and of this record
  u32 srow;          // the collective's row of the table
  u32 comm;
  u64 seq;           // operation counter
  // LDS words that take the collective's table row (STAGE_COLS of them) when `staged`; otherwise the row goes
  // straight to the table.  A flag and not a null pointer: LDS address 0 is a valid address (the first staged row).
  lds_i64* stage;
  bool staged;
  // grid placement: the record's cell in its fine bucket, where the bucket's flags are collected, their number so far
  u32 cell, rec0;
  struct GridFlags* flags;
};
// A staged table row of k_seg_wave: the 21 columns, then the detection-group code and the range T_max - T_min; the
// rows are STAGE_COLS words apart (an odd stride).
constexpr u32 STAGE_COLS = CCLD_SEG_NCOL + 2;

// Table rows of the collectives of one wavefront pass (called by the first lane of every collective; the rows of a
// pass are consecutive).  A staged row goes to LDS and the workgroup writes it out later; a row that is not staged
// is written here: the columns are written from one wavefront-uniform pointer that steps from column to column,
// plus a 32-bit byte offset per lane: no 64-bit address arithmetic per lane and column, and the kernel arguments need
// not stay in scalar registers across the whole pass (212 spilled scalar registers become 20).  Storing G words of
// a row per instruction from the G lanes of its group (3 instead of 23 store instructions at G = 8) was measured
// too: the selects that bring each lane its word cost more than the stores save (2.18 -> 2.56 ms).
// PUT_SORTED: the sorted window's pass, rows staged where L.staged; PUT_GRID: the grid placement's, rows written directly
enum { PUT_SORTED = 0, PUT_GRID = 1 };
template <int MODE>
__device__ __forceinline__ void dense_put_row(const SegArgs& a, const DenseLane& L, u32 ninfl, bool complete, bool incons,
                                              bool barrier, bool usable, u32 hop, u64 hb, i64 imin, u32 nd, i64 min_e,
                                              i64 med_e, i64 max_e, i64 mad_e, i64 min_x, i64 med_x, i64 max_x, i64 mad_x,
                                              i64 dmin, i64 dmax, u32 rmin, u32 rmax) {
  const u32 srow = L.srow;
  const bool none = nd == 0;            // no completed record: the statistics columns are empty
  seg_count_alert(a, srow, ninfl, barrier, imin);
  if (MODE == PUT_SORTED && L.staged) {
    // the row waits in LDS until the workgroup writes the table column by column, whole lines at a time
    lds_i64* st = L.stage;
    auto put = [&](u32 c, i64 v) { st[c] = v; };
    put(CCLD_SEG_COMM, (i64)L.comm); put(CCLD_SEG_SEQ, (i64)L.seq); put(CCLD_SEG_N, (i64)L.n); put(CCLD_SEG_INFLIGHT, (i64)ninfl);
    put(CCLD_SEG_STATE, (complete ? CCLD_SEG_COMPLETE : 0) | (!incons ? CCLD_SEG_CONSISTENT : 0) |
                            (barrier ? CCLD_SEG_BARRIER : 0) | (usable ? CCLD_SEG_USABLE : 0));
    put(CCLD_SEG_OP, (i64)hop); put(CCLD_SEG_BYTES, (i64)hb);
    put(CCLD_SEG_ENTER_MIN, none ? 0 : min_e); put(CCLD_SEG_ENTER_MED, none ? 0 : med_e);
    put(CCLD_SEG_ENTER_MAX, none ? 0 : max_e); put(CCLD_SEG_ENTER_MAD, none ? 0 : mad_e);
    put(CCLD_SEG_EXIT_MIN, none ? 0 : min_x); put(CCLD_SEG_EXIT_MED, none ? 0 : med_x);
    put(CCLD_SEG_EXIT_MAX, none ? 0 : max_x); put(CCLD_SEG_EXIT_MAD, none ? 0 : mad_x);
    put(CCLD_SEG_DUR_MIN, none ? 0 : dmin); put(CCLD_SEG_DUR_MAX, none ? 0 : dmax);
    put(CCLD_SEG_ARGMIN_RANK, none ? (i64)CCLD_NO_RANK : (i64)rmin); put(CCLD_SEG_ARGMAX_RANK, none ? (i64)CCLD_NO_RANK : (i64)rmax);
    put(CCLD_SEG_INFLIGHT_ENTER_MIN, imin); put(CCLD_SEG_FIRST, (i64)L.first);
    put(CCLD_SEG_NCOL, (i64)seg_group_code(usable, hop, hb)); put(CCLD_SEG_NCOL + 1, usable ? dmax - dmin : 0);
    return;
  }
  seg_put_group(a, srow, usable, hop, hb, dmax, dmin);
  if (srow >= a.seg_cap) return;
  const u32 s0 = (u32)__builtin_amdgcn_readfirstlane((int)srow);      // the first of the pass's rows that fit the table
  const u32 off = (srow - s0) * 8u;
  const u64 stride = a.seg_cap * 8u;
  char* p = reinterpret_cast<char*>(a.seg + s0);
  auto put = [&](i64 v) { *reinterpret_cast<i64*>(p + off) = v; p += stride; };
  static_assert(CCLD_SEG_COMM == 0 && CCLD_SEG_SEQ == 1 && CCLD_SEG_N == 2 && CCLD_SEG_INFLIGHT == 3 && CCLD_SEG_STATE == 4 &&
                CCLD_SEG_OP == 5 && CCLD_SEG_BYTES == 6 && CCLD_SEG_ENTER_MIN == 7 && CCLD_SEG_ENTER_MAD == 10 &&
                CCLD_SEG_EXIT_MIN == 11 && CCLD_SEG_EXIT_MAD == 14 && CCLD_SEG_DUR_MIN == 15 && CCLD_SEG_DUR_MAX == 16 &&
                CCLD_SEG_ARGMIN_RANK == 17 && CCLD_SEG_ARGMAX_RANK == 18 && CCLD_SEG_INFLIGHT_ENTER_MIN == 19 &&
                CCLD_SEG_FIRST == 20 && CCLD_SEG_NCOL == 21, "the columns are written in this order");
  put((i64)L.comm);
  put((i64)L.seq);
  put((i64)L.n);
  put((i64)ninfl);
  put((complete ? CCLD_SEG_COMPLETE : 0) | (!incons ? CCLD_SEG_CONSISTENT : 0) | (barrier ? CCLD_SEG_BARRIER : 0) |
      (usable ? CCLD_SEG_USABLE : 0));
  put((i64)hop);
  put((i64)hb);
  put(none ? 0 : min_e); put(none ? 0 : med_e); put(none ? 0 : max_e); put(none ? 0 : mad_e);
  put(none ? 0 : min_x); put(none ? 0 : med_x); put(none ? 0 : max_x); put(none ? 0 : mad_x);
  put(none ? 0 : dmin); put(none ? 0 : dmax);
  put(none ? (i64)CCLD_NO_RANK : (i64)rmin); put(none ? (i64)CCLD_NO_RANK : (i64)rmax);
  put(imin);
  put((i64)L.first);
}
// One record's lags and flags.  Sorted windows mark every record's flag byte and leave the lags of flagged records at
// their sorted position; the grid placement collects the flagged records of a fine bucket from the bucket's first sorted
// position on (a.flag_pos takes cell | kind << 16), in any order: grid_order_flags orders them by cell.
struct GridFlags {
  u32 n;                     // flagged records so far
  u32 bits[GRID_B / 32];     // their cells
  u32 pre[GRID_B / 32];      // flagged cells before each word
};
__device__ __forceinline__ void grid_put_record(const SegArgs& a, u32 j, u32 cell, u32 rec0, GridFlags* F, u32 f, i64 le, i64 lx) {
  if (a.rec_flag) a.rec_flag[j] = (uint8_t)f;
  if (a.lag_e) a.lag_e[j] = le;
  if (a.lag_x) a.lag_x[j] = lx;
  if (f) {
    const u32 at = rec0 + atomicAdd(&F->n, 1u);
    atomicOr(&F->bits[cell >> 5], 1u << (cell & 31));
    a.flag_pos[at] = cell | (f << 16);
    a.flag_lag[at] = le; a.flag_lag[a.cap_n + at] = lx;
  }
}
template <int MODE>
__device__ __forceinline__ void dense_put_record(const SegArgs& a, const DenseLane& L, u32 f, i64 le, i64 lx) {
  if constexpr (MODE == PUT_GRID) {
    grid_put_record(a, L.j, L.cell, L.rec0, L.flags, f, le, lx);
  } else {
    a.rec_flag[L.j] = (uint8_t)f;
    if (a.lag_e) a.lag_e[L.j] = le;
    if (a.lag_x) a.lag_x[L.j] = lx;
    if (f) { a.flag_lag[L.j] = le; a.flag_lag[a.cap_n + L.j] = lx; }
  }
}

// Statistics of the collectives of one wavefront pass in 64-bit arithmetic (any spread of the times).
template <int G, int MODE>
__device__ __forceinline__ void dense_pass64(const SegArgs& a, const DenseLane& L, u32 size, u32 lane, u32 gbase, u64 gmask) {
  const i64 e = L.e, x = L.x;
  const bool valid = L.valid;
  const bool done = valid && x != T_INFLIGHT;
  const u64 m_infl = ballot64(valid && !done);
  const u32 nd = (u32)__popcll(ballot64(done) & gmask);
  const u32 ninfl = (u32)__popcll(m_infl & gmask);
  const u32 km = nd ? (nd - 1) / 2 : 0, kl = nd ? nd - 1 : 0;
  const i64 se = sort_groups<G>(done ? e : T_INFLIGHT, lane);
  const i64 sx = sort_groups<G>(done ? x : T_INFLIGHT, lane);
  const i64 med_e = shfl_i64(se, gbase + km), med_x = shfl_i64(sx, gbase + km);
  const i64 min_e = shfl_i64(se, gbase), max_e = shfl_i64(se, gbase + kl);
  const i64 min_x = shfl_i64(sx, gbase), max_x = shfl_i64(sx, gbase + kl);
  // deviations of the sorted values: the first nd lanes of a group hold its finished records
  const bool held = lane - gbase < nd;
  const i64 sde = merge_groups<G>(held ? absdiff(se, med_e) : T_INFLIGHT, lane);
  const i64 sdx = merge_groups<G>(held ? absdiff(sx, med_x) : T_INFLIGHT, lane);
  const i64 mad_e = shfl_i64(sde, gbase + km), mad_x = shfl_i64(sdx, gbase + km);
  i64 dmin = done ? x - e : INT64_MAX, dmax = done ? x - e : INT64_MIN;
  u32 rmin = done ? L.rank : 0xFFFFFFFFu, rmax = rmin;
  reduce_dur<G, false>(dmin, rmin);
  reduce_dur<G, true>(dmax, rmax);
  const u64 hb = shfl_u64(L.nb, (int)L.fl);
  const u32 hop = __shfl(L.op, (int)L.fl, CCLD_WAVE);
  const bool incons = (ballot64(valid && (L.nb != hb || L.op != hop)) & gmask) != 0;
  i64 imin = T_INFLIGHT;
  if (m_infl) imin = reduce_min<G>((valid && !done) ? e : T_INFLIGHT);
  if (!valid) return;
  const bool complete = L.n == size && ninfl == 0;
  const bool barrier = hop == CCLD_OP_ALLREDUCE && hb < (u64)a.barrier_bytes;
  const bool usable = complete && !incons && !barrier;
  if (lane == L.fl)
    dense_put_row<MODE>(a, L, ninfl, complete, incons, barrier, usable, hop, hb, imin, nd, min_e, med_e, max_e, mad_e, min_x,
                  med_x, max_x, mad_x, dmin, dmax, rmin, rmax);
  i64 le = 0, lx = 0;
  u32 f = 0;
  if (usable) {
    le = e - med_e; lx = x - med_x;
    if (is_late(le, a.lag_floor, a.kmad_num, a.kmad_den, mad_e)) f |= CCLD_FLAG_LATE_ENTER;
    if (is_late(lx, a.lag_floor, a.kmad_num, a.kmad_den, mad_x)) f |= CCLD_FLAG_LATE_EXIT;
  }
  dense_put_record<MODE>(a, L, f, le, lx);
}

// ---- the same statistics on 32-bit times relative to the collective's first record --------------------
// Inside one collective the arrivals and completions lie within a second or so of each other, so they
// are sorted, compared and subtracted as signed 32-bit offsets from the arrival of the collective's first
// present member (half the instructions of the 64-bit form); the results are turned back into absolute
// times where they are stored.  A pass in which some offset does not fit takes the 64-bit form.
constexpr i32 REL_NONE = 0x7FFFFFFF;         // sorts behind every real offset (those stay below 2^30 in magnitude)

//
// A compare-exchange is one exchange and one median of three: with the smallest or the largest integer as the third value
// the median is the minimum or the maximum, so each lane's side of an exchange is a word that is set up once per kernel
// (minimum, maximum and a select were three instructions).  The word is computed and not selected: a value known to be one
// of two would make the median a select again.  Distances of 16 and 32 lanes are swaps of rows and halves in registers;
// through the LDS crossbar they were the longest waits of the chain.
__device__ __forceinline__ i32 med3_i32(i32 x, i32 y, i32 bound) {
  const i32 lo = x < y ? x : y, hi = x < y ? y : x, c = hi < bound ? hi : bound;
  return lo < c ? c : lo;
}
// The mirrored exchanges beyond a row of 16 lanes meet the same pairs of values as cmpx<31> and cmpx<63>, but leave the
// larger ones in another order (the exchanges that follow sort either): 31 turns every second row round first, 63
// expects the complements of the upper half's values in rising order.
template <int M>
__device__ __forceinline__ i32 cmpx32(i32 v, u32 lane) {
  constexpr int B = M == 31 ? 16 : M == 63 ? 32 : high_bit(M);
  const i32 bound = 0x7FFFFFFF ^ (i32)(((lane & B) / B) - 1u);        // without the bit its complement, the smallest integer
  if constexpr (M == 31) v = __builtin_amdgcn_update_dpp(v, v, 0x140, 0xA, 0xF, false);       // rows 1 and 3: row_mirror
  if constexpr (M == 63) v ^= -(i32)(lane >> 5);
  if constexpr (B == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap((u32)v, (u32)v, false, false);
    return med3_i32((i32)r[0], (i32)r[1], bound);
  } else if constexpr (B == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap((u32)v, (u32)v, false, false);
    return med3_i32((i32)r[0], (i32)r[1], bound);
  } else {
    return med3_i32((i32)xor_lane_u32<M>((u32)v), v, bound);
  }
}
template <int G>
__device__ __forceinline__ i32 sort_groups32(i32 v, u32 lane) {
  if constexpr (G >= 64) v ^= -(i32)(lane >> 5);
  if constexpr (G >= 2) { v = cmpx32<1>(v, lane); }
  if constexpr (G >= 4) { v = cmpx32<3>(v, lane); v = cmpx32<1>(v, lane); }
  if constexpr (G >= 8) { v = cmpx32<7>(v, lane); v = cmpx32<2>(v, lane); v = cmpx32<1>(v, lane); }
  if constexpr (G >= 16) { v = cmpx32<15>(v, lane); v = cmpx32<4>(v, lane); v = cmpx32<2>(v, lane); v = cmpx32<1>(v, lane); }
  if constexpr (G >= 32) {
    v = cmpx32<31>(v, lane); v = cmpx32<8>(v, lane); v = cmpx32<4>(v, lane); v = cmpx32<2>(v, lane); v = cmpx32<1>(v, lane);
  }
  if constexpr (G >= 64) {
    v = cmpx32<63>(v, lane); v = cmpx32<16>(v, lane); v = cmpx32<8>(v, lane); v = cmpx32<4>(v, lane);
    v = cmpx32<2>(v, lane); v = cmpx32<1>(v, lane);
  }
  return v;
}
template <int G>
__device__ __forceinline__ i32 merge_groups32(i32 v, u32 lane) {
  if constexpr (G >= 64) v = cmpx32<32>(v, lane);
  if constexpr (G >= 32) v = cmpx32<16>(v, lane);
  if constexpr (G >= 16) v = cmpx32<8>(v, lane);
  if constexpr (G >= 8) v = cmpx32<4>(v, lane);
  if constexpr (G >= 4) v = cmpx32<2>(v, lane);
  if constexpr (G >= 2) v = cmpx32<1>(v, lane);
  return v;
}
// all-reduce of an unsigned 32-bit word inside a group
template <int G, bool MAXIMUM>
__device__ __forceinline__ u32 reduce_u32(u32 v) {
  auto take = [](u32 x, u32 y) { return MAXIMUM ? (x > y ? x : y) : (x < y ? x : y); };
  if constexpr (G > 1) v = take(v, xor_lane_u32<1>(v));
  if constexpr (G > 2) v = take(v, xor_lane_u32<2>(v));
  if constexpr (G > 4) v = take(v, xor_lane_u32<7>(v));       // four lanes hold the same word by now: the mirrors
  if constexpr (G > 8) v = take(v, xor_lane_u32<15>(v));      // reach the other half like the exchanges by 4 and by 8
  if constexpr (G > 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = take(r[0], r[1]);
  }
  if constexpr (G > 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = take(r[0], r[1]);
  }
  return v;
}
// all-reduce of an unsigned 64-bit word inside a group
template <int G, bool MAXIMUM>
__device__ __forceinline__ u64 reduce_u64(u64 v) {
#define CCLD_U64_STEP(M)                                                                         \
  if constexpr (G > M) {                                                                         \
    const u64 o = (u64)xor_lane_i64<M>((i64)v);                                                  \
    v = MAXIMUM ? (o > v ? o : v) : (o < v ? o : v);                                             \
  }
  CCLD_U64_STEP(1) CCLD_U64_STEP(2) CCLD_U64_STEP(4) CCLD_U64_STEP(8) CCLD_U64_STEP(16) CCLD_U64_STEP(32)
#undef CCLD_U64_STEP
  return v;
}
// late iff lag > floor and lag * kden > knum * mad, with a 32-bit lag and a non-negative 32-bit mad
__device__ __forceinline__ bool is_late32(i32 lag, i64 floor_ns, u32 knum, u32 kden, i32 mad) {
  if (lag <= 0 || (i64)lag <= floor_ns) return false;       // a lag that is not positive never exceeds knum * mad >= 0
  return (u64)(u32)lag * (u64)kden > (u64)knum * (u64)(u32)mad;
}

template <int G, int MODE>
__device__ __forceinline__ void dense_pass32(const SegArgs& a, const DenseLane& L, i64 ref, i32 er, i32 xr, u32 size,
                                             u32 lane, u32 gbase, u64 gmask) {
  const bool valid = L.valid;
  const bool done = valid && L.x != T_INFLIGHT;
  const u64 m_infl = ballot64(valid && !done);
  const u32 nd = (u32)__popcll(ballot64(done) & gmask);
  const u32 ninfl = (u32)__popcll(m_infl & gmask);
  const u32 km = nd ? (nd - 1) / 2 : 0, kl = nd ? nd - 1 : 0;
  const i32 se = sort_groups32<G>(done ? er : REL_NONE, lane);
  const i32 sx = sort_groups32<G>(done ? xr : REL_NONE, lane);
  const i32 med_e = __shfl(se, (int)(gbase + km), CCLD_WAVE), med_x = __shfl(sx, (int)(gbase + km), CCLD_WAVE);
  const i32 min_e = __shfl(se, (int)gbase, CCLD_WAVE), max_e = __shfl(se, (int)(gbase + kl), CCLD_WAVE);
  const i32 min_x = __shfl(sx, (int)gbase, CCLD_WAVE), max_x = __shfl(sx, (int)(gbase + kl), CCLD_WAVE);
  // deviations of the sorted offsets (the first nd lanes of a group hold its finished records): they fall to zero
  // at the median and rise again, so one merge sorts them
  const bool held = lane - gbase < nd;
  const i32 sde = merge_groups32<G>(held ? (se >= med_e ? se - med_e : med_e - se) : REL_NONE, lane);
  const i32 sdx = merge_groups32<G>(held ? (sx >= med_x ? sx - med_x : med_x - sx) : REL_NONE, lane);
  const i32 mad_e = __shfl(sde, (int)(gbase + km), CCLD_WAVE), mad_x = __shfl(sdx, (int)(gbase + km), CCLD_WAVE);
  // T_min / T_max of the Duration Time with the ranks attaining them (ties: smallest rank): duration and rank
  // travel as one 64-bit word
  const u32 dur = (u32)(xr - er);
  u64 wmin = done ? (((u64)dur << 32) | L.rank) : ~0ull;
  u64 wmax = done ? (((u64)dur << 32) | (u32)~L.rank) : 0ull;
  wmin = reduce_u64<G, false>(wmin);
  wmax = reduce_u64<G, true>(wmax);
  const u64 hb = shfl_u64(L.nb, (int)L.fl);
  const u32 hop = __shfl(L.op, (int)L.fl, CCLD_WAVE);
  const bool incons = (ballot64(valid && (L.nb != hb || L.op != hop)) & gmask) != 0;
  i64 imin = T_INFLIGHT;
  if (m_infl) imin = reduce_min<G>((valid && !done) ? L.e : T_INFLIGHT);
  if (!valid) return;
  const bool complete = L.n == size && ninfl == 0;
  const bool barrier = hop == CCLD_OP_ALLREDUCE && hb < (u64)a.barrier_bytes;
  const bool usable = complete && !incons && !barrier;
  if (lane == L.fl)
    dense_put_row<MODE>(a, L, ninfl, complete, incons, barrier, usable, hop, hb, imin, nd, ref + min_e, ref + med_e, ref + max_e,
                  (i64)mad_e, ref + min_x, ref + med_x, ref + max_x, (i64)mad_x, (i64)(wmin >> 32), (i64)(wmax >> 32),
                  (u32)wmin, ~(u32)wmax);
  i32 le = 0, lx = 0;
  u32 f = 0;
  if (usable) {
    le = er - med_e; lx = xr - med_x;
    if (is_late32(le, a.lag_floor, a.kmad_num, a.kmad_den, mad_e)) f |= CCLD_FLAG_LATE_ENTER;
    if (is_late32(lx, a.lag_floor, a.kmad_num, a.kmad_den, mad_x)) f |= CCLD_FLAG_LATE_EXIT;
  }
  dense_put_record<MODE>(a, L, f, (i64)le, (i64)lx);
}

// ---- collectives of up to 64 records, 64/G of them per wavefront pass --------------------------
constexpr u32 SEG_STAGE_ROWS = 144;      // table rows a tile stages in LDS (a tile of eight-member collectives has 128 or 129)
template <int G>
__device__ __forceinline__ void seg_wave_batches(const SegArgs& a, u32 base, u32 seg0, u32 nheads,
                                                 const unsigned short* s_head, i64* s_stage, u32 lane, u32 wave) {
  constexpr int SPW = CCLD_WAVE / G, NW = SEG_THREADS / CCLD_WAVE;
  const int mb = a.sf.mb;
  const u64 mmask = ((u64)1 << mb) - 1, smask = ((u64)1 << a.sf.ws) - 1;
  const u32 q = lane / G, l = lane % G, gbase = q * G;
  const u64 gmask = (G == 64 ? ~0ull : (((u64)1 << (G & 63)) - 1)) << gbase;
  for (u32 b = wave; b * SPW < nheads; b += NW) {
    const u32 sl = b * SPW + q;
    u32 a0 = 0, n = 0;
    if (sl < nheads) { a0 = s_head[sl]; n = (u32)s_head[sl + 1] - a0; }
    const bool small = n >= 1 && n <= (u32)SEG_WAVE_MAX;
    if (n > (u32)SEG_WAVE_MAX && l == 0) {            // too long for a wavefront: leave it to k_seg_big
      const u64 slot = atomic_add_u64(&a.counters[CNT_NBIG], 1);
      a.big_list[3 * slot] = seg0 + sl;
      a.big_list[3 * slot + 1] = base + a0;
    }
    DenseLane L;
    L.valid = small && l < n;
    L.e = 0; L.x = T_INFLIGHT; L.nb = 0; L.op = 0; L.rank = 0;
    L.first = base + a0; L.j = L.first + l; L.fl = gbase; L.n = n; L.srow = seg0 + sl;
    // rows beyond the staging area (a tile of many short collectives) go straight to the table
    L.staged = sl < SEG_STAGE_ROWS;
    L.stage = (lds_i64*)s_stage + sl * STAGE_COLS;
    u64 key = 0;
    u32 size = 0;
    if (L.valid) {
      key = a.key[L.j];
      const Rec rw = load_row(a, L.j);
      // first member and size of the communicator in one load; the slot -> rank lookup overlaps the row gather
      const uint2 ci = a.comm_info[(u32)(key >> (mb + a.sf.ws))];
      L.rank = a.members_sorted[ci.x + (u32)(key & mmask)];
      size = ci.y;
      L.e = rw.t_enter; L.x = rw.t_exit; L.nb = rw.bytes; L.op = rw.op;
    }
    L.comm = (u32)(key >> (mb + a.sf.ws));
    L.seq = ((key >> mb) & smask) + a.sf.seq_base;
    // offsets from the arrival of the collective's first record
    const i64 ref = shfl_i64(L.e, (int)gbase);
    const i64 oe = L.e - ref, ox = L.x - ref;
    constexpr i64 LIM = (i64)1 << 30;
    const bool wide = L.valid && (oe < -LIM || oe >= LIM || (L.x != T_INFLIGHT && (ox < -LIM || ox >= LIM)));
    if (ballot64(wide) == 0) dense_pass32<G, PUT_SORTED>(a, L, ref, (i32)oe, (i32)ox, size, lane, gbase, gmask);
    else dense_pass64<G, PUT_SORTED>(a, L, size, lane, gbase, gmask);
  }
}

// One workgroup per tile of SEG_TILE sorted records: finds the collectives that start in the
// tile, then its wavefronts take them 64/G at a time (G = the tile's widest short collective,
// rounded up to a power of two).
__global__ __launch_bounds__(SEG_THREADS) void k_seg_wave(SegArgs a) {
  constexpr int OWN = SEG_TILE / SEG_THREADS, NW = SEG_THREADS / CCLD_WAVE;
  __shared__ unsigned short s_head[SEG_TILE + 2];
  __shared__ u32 s_cnt[OWN * NW];
  __shared__ u32 s_halo_head, s_gmax;
  // Table rows of the tile's first SEG_STAGE_ROWS collectives wait here (STAGE_COLS words each: an odd stride, so
  // the lanes that read one column of consecutive rows spread over the banks) and leave column by column at the
  // end, consecutive lanes to consecutive rows: one store instruction per 64 rows and column instead of one per
  // wavefront pass and column.
  __shared__ i64 s_stage[SEG_STAGE_ROWS * STAGE_COLS];
  const u32 tid = threadIdx.x, lane = lane_id(), wave = tid / CCLD_WAVE;
  const u32 tile = blockIdx.x, base = tile * SEG_TILE;
  const u32 rem = a.n - base;                                     // records from the tile's start to the end
  const u32 own = rem < (u32)SEG_TILE ? rem : (u32)SEG_TILE;
  const int mb = a.sf.mb;
  if (tid == 0) { s_halo_head = rem <= (u32)(SEG_TILE + SEG_WAVE_MAX) ? rem : 0xFFFFu; s_gmax = 0; }
  // Heads of the tile.  Position r * SEG_THREADS + tid ascends with (r, wavefront, lane), so a head's index is
  // the number of heads in the (r, wavefront) blocks before its own (16 counts in LDS, one ballot each) plus
  // the heads below its lane: no scan over the workgroup, one barrier.
  bool head[OWN];
  u64 hm[OWN];
#pragma unroll
  for (int r = 0; r < OWN; ++r) {
    const u32 pos = r * SEG_THREADS + tid, j = base + pos;
    head[r] = pos < own && (j == 0 || (a.key[j - 1] >> mb) != (a.key[j] >> mb));
    hm[r] = ballot64(head[r]);
    if (lane == 0) s_cnt[r * NW + wave] = (u32)__popcll(hm[r]);
  }
  __syncthreads();
  u32 before[OWN], acc = 0;
#pragma unroll
  for (int r = 0; r < OWN; ++r) before[r] = 0;
#pragma unroll
  for (int bl = 0; bl < OWN * NW; ++bl) {
    if ((u32)(bl % NW) == wave) before[bl / NW] = acc;
    acc += s_cnt[bl];
  }
  const u32 nheads = acc;
#pragma unroll
  for (int r = 0; r < OWN; ++r)
    if (head[r]) s_head[before[r] + mbcnt64(hm[r])] = (unsigned short)(r * SEG_THREADS + tid);
  // where the tile's last collective ends: the first head within 64 records past the tile
  if (tid <= (u32)SEG_WAVE_MAX) {
    const u32 pos = SEG_TILE + tid;
    if (pos < rem) {
      const u32 j = base + pos;
      if ((a.key[j - 1] >> mb) != (a.key[j] >> mb)) atomicMin(&s_halo_head, pos);
    }
  }
  __syncthreads();
  const u32 halo = s_halo_head & 0xFFFFu;
  if (tid == 0) s_head[nheads] = (unsigned short)halo;
  for (u32 s = tid; s < nheads; s += SEG_THREADS) {
    const u32 n = (s + 1 < nheads ? (u32)s_head[s + 1] : halo) - (u32)s_head[s];
    if (n <= (u32)SEG_WAVE_MAX) atomicMax(&s_gmax, n);
  }
  __syncthreads();
  const u32 gmax = s_gmax, seg0 = a.tile_heads[tile];
  if (gmax <= 2) seg_wave_batches<2>(a, base, seg0, nheads, s_head, s_stage, lane, wave);
  else if (gmax <= 4) seg_wave_batches<4>(a, base, seg0, nheads, s_head, s_stage, lane, wave);
  else if (gmax <= 8) seg_wave_batches<8>(a, base, seg0, nheads, s_head, s_stage, lane, wave);
  else if (gmax <= 16) seg_wave_batches<16>(a, base, seg0, nheads, s_head, s_stage, lane, wave);
  else if (gmax <= 32) seg_wave_batches<32>(a, base, seg0, nheads, s_head, s_stage, lane, wave);
  else seg_wave_batches<64>(a, base, seg0, nheads, s_head, s_stage, lane, wave);
  __syncthreads();
  const u32 staged = nheads < SEG_STAGE_ROWS ? nheads : SEG_STAGE_ROWS;
  for (u32 col = wave; col < STAGE_COLS; col += NW) {
    for (u32 sl = lane; sl < staged; sl += CCLD_WAVE) {
      // a collective of more than 64 records is on the list of the kernels that take those: they write its row
      if ((u32)s_head[sl + 1] - (u32)s_head[sl] > (u32)SEG_WAVE_MAX) continue;
      const i64 v = s_stage[sl * STAGE_COLS + col];
      const u32 srow = seg0 + sl;
      if (col < (u32)CCLD_SEG_NCOL) { if (srow < a.seg_cap) a.seg[(u64)col * a.seg_cap + srow] = v; }
      else if (col == (u32)CCLD_SEG_NCOL) a.gcode[srow] = (uint16_t)v;
      else a.range_c[srow] = v;
    }
  }
}

// ---- collectives of 65 to 512 records: E values per lane, sorted in registers ---------------------
// Element i of the collective sits in register i / 64 of lane i % 64.  Every register is sorted by
// the 64-lane network, then runs of 2, 4, 8 registers are merged: the mirror step pairs register r
// with r ^ (run - 1) and lane l with 63 - l, strides of whole registers need no lane exchange, and
// strides below 64 are the lane exchanges of the 64-lane merge.
template <int E>
__device__ __forceinline__ void sort_multi(i64 (&v)[E], u32 lane) {
#pragma unroll
  for (int r = 0; r < E; ++r) v[r] = sort_groups<64>(v[r], lane);
#pragma unroll
  for (int kb = 2; kb <= E; kb <<= 1) {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      if ((r & (kb >> 1)) == 0) {
        const int q = r ^ (kb - 1);
        const i64 b = xor_lane_i64<63>(v[q]);
        const bool sw = b < v[r];
        const i64 lo = sw ? b : v[r], hi = sw ? v[r] : b;
        v[r] = lo;
        v[q] = xor_lane_i64<63>(hi);
      }
    }
#pragma unroll
    for (int jb = kb >> 2; jb >= 1; jb >>= 1) {
#pragma unroll
      for (int r = 0; r < E; ++r) {
        if ((r & jb) == 0) {
          const int q = r | jb;
          const bool sw = v[q] < v[r];
          const i64 lo = sw ? v[q] : v[r], hi = sw ? v[r] : v[q];
          v[r] = lo; v[q] = hi;
        }
      }
    }
#pragma unroll
    for (int r = 0; r < E; ++r) {
      v[r] = cmpx<32>(v[r], lane); v[r] = cmpx<16>(v[r], lane); v[r] = cmpx<8>(v[r], lane);
      v[r] = cmpx<4>(v[r], lane); v[r] = cmpx<2>(v[r], lane); v[r] = cmpx<1>(v[r], lane);
    }
  }
}
// k-th smallest after sort_multi (k uniform across the wavefront)
template <int E>
__device__ __forceinline__ i64 kth_multi(const i64 (&v)[E], u32 k) {
  i64 sel = v[0];
#pragma unroll
  for (int r = 1; r < E; ++r) if ((k >> 6) == (u32)r) sel = v[r];
  return shfl_i64(sel, (int)(k & 63));
}

// Lower median of |value - median| over the nd smallest values of a sorted collective (nd >= 1, km = (nd - 1) / 2,
// all uniform across the wavefront).  The deviations of the values up to the median, walked downwards, and of
// the values above it, walked upwards, are two ascending lists; the km-th smallest of their union is found by
// the split that takes km + 1 entries from the two lists in order, without sorting the deviations.
template <int E>
__device__ __forceinline__ i64 mad_of_sorted(const i64 (&v)[E], u32 nd, u32 km) {
  const i64 med = kth_multi<E>(v, km);
  const u32 nl = km + 1, nr = nd - nl, d = km + 1;
  auto below = [&](u32 j) { return med - kth_multi<E>(v, km - j); };          // j < nl, ascending, below(0) = 0
  auto above = [&](u32 j) { return kth_multi<E>(v, km + 1 + j) - med; };      // j < nr, ascending
  u32 lo = d > nr ? d - nr : 0u, hi = d < nl ? d : nl;
  while (lo < hi) {
    const u32 mid = (lo + hi) >> 1;
    if (below(mid) <= above(d - 1 - mid)) lo = mid + 1; else hi = mid;
  }
  // lo entries come from the lower list, d - lo from the upper one; the largest of them is the answer
  i64 r = lo > 0 ? below(lo - 1) : INT64_MIN;
  if (d - lo > 0) { const i64 u = above(d - lo - 1); r = u > r ? u : r; }
  return r;
}

// One wavefront per listed collective of 32 E + 1 .. 64 E records.
template <int E>
__global__ __launch_bounds__(SEG_THREADS) void k_seg_multi(SegArgs a) {
  constexpr u32 LO = 32 * E + 1, HI = 64 * E, NW = SEG_THREADS / CCLD_WAVE;
  const u32 lane = lane_id();
  const int mb = a.sf.mb;
  const u64 mmask = ((u64)1 << mb) - 1, smask = ((u64)1 << a.sf.ws) - 1;
  const u32 nbig = (u32)a.counters[CNT_NBIG];
  for (u32 ent = blockIdx.x * NW + threadIdx.x / CCLD_WAVE; ent < nbig; ent += gridDim.x * NW) {
    const u32 nn = a.big_list[3 * ent + 2];
    if (nn < LO || nn > HI) continue;
    const u32 srow = a.big_list[3 * ent], a0 = a.big_list[3 * ent + 1];
    const u64 k0 = a.key[a0];
    const u32 comm = (u32)(k0 >> (mb + a.sf.ws));
    const u32* ms = a.members_sorted + a.member_off[comm];
    i64 e[E], x[E];
    u32 ninfl = 0, nd = 0;
    bool inc = false;
    i64 imin = T_INFLIGHT, dmin = INT64_MAX, dmax = INT64_MIN;
    u32 rmin = 0xFFFFFFFFu, rmax = 0xFFFFFFFFu;
    u64 hb = 0;
    u32 hop = 0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const u32 i = r * CCLD_WAVE + lane;
      const bool valid = i < nn;
      e[r] = 0; x[r] = T_INFLIGHT;
      u64 nb = 0;
      u32 op = 0, rank = 0;
      if (valid) {
        const u32 j = a0 + i;
        const u64 key = a.key[j];
        const Rec rw = load_row(a, j);
        rank = ms[(u32)(key & mmask)];
        e[r] = rw.t_enter; x[r] = rw.t_exit; nb = rw.bytes; op = rw.op;
      }
      if (r == 0) { hb = shfl_u64(nb, 0); hop = __shfl(op, 0, CCLD_WAVE); }
      inc |= valid && (nb != hb || op != hop);
      const bool done = valid && x[r] != T_INFLIGHT;
      nd += (u32)__popcll(ballot64(done));
      ninfl += (u32)__popcll(ballot64(valid && !done));
      if (valid && !done) imin = e[r] < imin ? e[r] : imin;
      if (done) {
        const i64 d = x[r] - e[r];
        if (d < dmin || (d == dmin && rank < rmin)) { dmin = d; rmin = rank; }
        if (d > dmax || (d == dmax && rank < rmax)) { dmax = d; rmax = rank; }
      }
    }
    const bool incons = ballot64(inc) != 0;
    if (ninfl) imin = reduce_min<64>(imin);
    reduce_dur<64, false>(dmin, rmin);
    reduce_dur<64, true>(dmax, rmax);
    const u32 km = nd ? (nd - 1) / 2 : 0, kl = nd ? nd - 1 : 0;
    // two sorts, arrival and completion; the median of the absolute deviations is selected from each sorted
    // sequence (records still in flight carry the largest value and sort behind the nd finished ones)
    i64 stat_min[2] = {0, 0}, stat_med[2] = {0, 0}, stat_max[2] = {0, 0}, stat_mad[2] = {0, 0};
#pragma unroll 1
    for (int w = 0; w < 2; ++w) {                  // 0 arrival, 1 completion
      i64 v[E];
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const bool done = x[r] != T_INFLIGHT;      // lanes past the end hold the in-flight mark too
        v[r] = !done ? T_INFLIGHT : (w ? x[r] : e[r]);
      }
      sort_multi<E>(v, lane);
      stat_min[w] = kth_multi<E>(v, 0); stat_med[w] = kth_multi<E>(v, km); stat_max[w] = kth_multi<E>(v, kl);
      if (nd) stat_mad[w] = mad_of_sorted<E>(v, nd, km);
    }
    const bool complete = nn == a.comm_size[comm] && ninfl == 0;
    const bool barrier = hop == CCLD_OP_ALLREDUCE && hb < (u64)a.barrier_bytes;
    const bool usable = complete && !incons && !barrier;
    if (lane == 0) {
      seg_put(a, CCLD_SEG_COMM, srow, (i64)comm);
      seg_put(a, CCLD_SEG_SEQ, srow, (i64)(((k0 >> mb) & smask) + a.sf.seq_base));
      seg_put(a, CCLD_SEG_N, srow, (i64)nn);
      seg_put(a, CCLD_SEG_INFLIGHT, srow, (i64)ninfl);
      seg_put(a, CCLD_SEG_STATE, srow,
              (complete ? CCLD_SEG_COMPLETE : 0) | (!incons ? CCLD_SEG_CONSISTENT : 0) |
                  (barrier ? CCLD_SEG_BARRIER : 0) | (usable ? CCLD_SEG_USABLE : 0));
      seg_put(a, CCLD_SEG_OP, srow, (i64)hop);
      seg_put(a, CCLD_SEG_BYTES, srow, (i64)hb);
      seg_put(a, CCLD_SEG_INFLIGHT_ENTER_MIN, srow, imin);
      seg_count_alert(a, srow, ninfl, barrier, imin);
      seg_put(a, CCLD_SEG_FIRST, srow, (i64)a0);
      seg_put_group(a, srow, usable, hop, hb, dmax, dmin);
      if (nd == 0) {
        seg_put_empty_stats(a, srow);
      } else {
        seg_put(a, CCLD_SEG_ENTER_MIN, srow, stat_min[0]); seg_put(a, CCLD_SEG_ENTER_MED, srow, stat_med[0]);
        seg_put(a, CCLD_SEG_ENTER_MAX, srow, stat_max[0]); seg_put(a, CCLD_SEG_ENTER_MAD, srow, stat_mad[0]);
        seg_put(a, CCLD_SEG_EXIT_MIN, srow, stat_min[1]); seg_put(a, CCLD_SEG_EXIT_MED, srow, stat_med[1]);
        seg_put(a, CCLD_SEG_EXIT_MAX, srow, stat_max[1]); seg_put(a, CCLD_SEG_EXIT_MAD, srow, stat_mad[1]);
        seg_put(a, CCLD_SEG_DUR_MIN, srow, dmin); seg_put(a, CCLD_SEG_DUR_MAX, srow, dmax);
        seg_put(a, CCLD_SEG_ARGMIN_RANK, srow, (i64)rmin); seg_put(a, CCLD_SEG_ARGMAX_RANK, srow, (i64)rmax);
      }
    }
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const u32 i = r * CCLD_WAVE + lane;
      if (i >= nn) continue;
      const u32 j = a0 + i;
      i64 le = 0, lx = 0;
      u32 f = 0;
      if (usable) {
        le = e[r] - stat_med[0]; lx = x[r] - stat_med[1];
        if (is_late(le, a.lag_floor, a.kmad_num, a.kmad_den, stat_mad[0])) f |= CCLD_FLAG_LATE_ENTER;
        if (is_late(lx, a.lag_floor, a.kmad_num, a.kmad_den, stat_mad[1])) f |= CCLD_FLAG_LATE_EXIT;
      }
      a.rec_flag[j] = (uint8_t)f;
      if (a.lag_e) a.lag_e[j] = le;
      if (a.lag_x) a.lag_x[j] = lx;
      if (f) { a.flag_lag[j] = le; a.flag_lag[a.cap_n + j] = lx; }
    }
  }
}

// ---- collectives of 65 to SEG_TEAM_MAX records -------------------------------------------------
// length of every listed collective, capped at SEG_LARGE_MAX + 1: one wavefront per entry walks the
// sorted keys from the collective's first record until the (communicator, counter) prefix changes
__global__ __launch_bounds__(SEG_THREADS) void k_seg_lengths(SegArgs a) {
  const u32 nbig = (u32)a.counters[CNT_NBIG];
  const u32 lane = lane_id(), nw = SEG_THREADS / CCLD_WAVE;
  const int mb = a.sf.mb;
  for (u32 ent = blockIdx.x * nw + threadIdx.x / CCLD_WAVE; ent < nbig; ent += gridDim.x * nw) {
    const u32 a0 = a.big_list[3 * ent + 1];
    const u64 pref = a.key[a0] >> mb;
    u32 len = SEG_LARGE_MAX + 1;
    for (u32 o = 1; o <= (u32)SEG_LARGE_MAX + 1; o += CCLD_WAVE) {
      const u64 j = (u64)a0 + o + lane;
      const u64 m = ballot64(j >= a.n || (a.key[j] >> mb) != pref);
      if (m) { len = o + (u32)__builtin_ctzll(m); break; }
    }
    if (lane == 0) a.big_list[3 * ent + 2] = len < (u32)SEG_LARGE_MAX + 1 ? len : (u32)SEG_LARGE_MAX + 1;
  }
}

struct TeamAcc {
  unsigned long long imin;
  long long dmin, dmax;
  u32 ninfl, incons, rmin, rmax;
};

// one compare-exchange step of the network over v[0, P): partner of i is i ^ M, the element whose
// bit HB (the top bit of M) is clear keeps the smaller value
template <u32 TT = SEG_THREADS>
__device__ __forceinline__ void team_cmpx(i64* v, u32 P, u32 M, u32 HB, u32 t) {
  for (u32 p = t; p < P / 2; p += TT) {
    const u32 lo = p & (HB - 1), ia = ((p - lo) << 1) | lo, ib = ia ^ M;
    const i64 va = v[ia], vb = v[ib];
    if (vb < va) { v[ia] = vb; v[ib] = va; }
  }
  __syncthreads();
}
// ascending bitonic sort of v[0, P), P a power of two (same merges as sort_groups, in LDS)
template <u32 TT = SEG_THREADS>
__device__ __forceinline__ void team_sort(i64* v, u32 P, u32 t) {
  for (u32 k = 2; k <= P; k <<= 1) {
    team_cmpx<TT>(v, P, k - 1, k >> 1, t);
    for (u32 j = k >> 2; j; j >>= 1) team_cmpx<TT>(v, P, j, j, t);
  }
}

// One workgroup per collective of 513 to SEG_TEAM_MAX records; arrival and completion times are
// staged in LDS and a third LDS array is sorted four times (arrival, completion, and their absolute
// deviations).
__global__ __launch_bounds__(SEG_THREADS) void k_seg_team(SegArgs a) {
  constexpr u32 TEAMS = 1, TT = SEG_THREADS;
  constexpr u32 CAPN = SEG_TEAM_MAX;
  constexpr u32 LO = (u32)SEG_MULTI_MAX + 1;
  __shared__ i64 s_e[TEAMS][CAPN], s_x[TEAMS][CAPN], s_v[TEAMS][CAPN];
  __shared__ TeamAcc s_acc[TEAMS];
  const u32 team = threadIdx.x / TT, t = threadIdx.x % TT;
  i64 *E = s_e[team], *X = s_x[team], *V = s_v[team];
  TeamAcc& acc = s_acc[team];
  const int mb = a.sf.mb;
  const u64 mmask = ((u64)1 << mb) - 1, smask = ((u64)1 << a.sf.ws) - 1;
  const u32 nbig = (u32)a.counters[CNT_NBIG];
  for (u32 ent = blockIdx.x * TEAMS + team; ent < nbig; ent += gridDim.x * TEAMS) {
    const u32 nn = a.big_list[3 * ent + 2];
    if (nn < LO || nn > CAPN) continue;
    const u32 srow = a.big_list[3 * ent], a0 = a.big_list[3 * ent + 1];
    const u64 k0 = a.key[a0];
    const Rec h = load_row(a, a0);
    if (t == 0) {
      acc.imin = (unsigned long long)T_INFLIGHT; acc.dmin = INT64_MAX; acc.dmax = INT64_MIN;
      acc.ninfl = 0; acc.incons = 0; acc.rmin = 0xFFFFFFFFu; acc.rmax = 0xFFFFFFFFu;
    }
    __syncthreads();
    {
      u32 ni = 0, rmin = 0xFFFFFFFFu, rmax = 0xFFFFFFFFu;
      bool inc = false;
      i64 imin = T_INFLIGHT, dmin = INT64_MAX, dmax = INT64_MIN;
      for (u32 i = t; i < nn; i += TT) {
        const u32 j = a0 + i;
        const Rec rw = load_row(a, j);
        E[i] = rw.t_enter; X[i] = rw.t_exit;
        inc |= (rw.op != h.op || rw.bytes != h.bytes);
        if (rw.t_exit == T_INFLIGHT) {
          ++ni; imin = rw.t_enter < imin ? rw.t_enter : imin;
        } else {
          const i64 d = rw.t_exit - rw.t_enter;
          const u32 rk = (u32)(a.key[j] & mmask);
          if (d < dmin || (d == dmin && rk < rmin)) { dmin = d; rmin = rk; }
          if (d > dmax || (d == dmax && rk < rmax)) { dmax = d; rmax = rk; }
        }
      }
      if (ni) { atomicAdd(&acc.ninfl, ni); atomicMin(&acc.imin, (unsigned long long)imin); }
      if (inc) atomicOr(&acc.incons, 1u);
      if (rmin != 0xFFFFFFFFu) { atomicMin(&acc.dmin, (long long)dmin); atomicMax(&acc.dmax, (long long)dmax); }
      __syncthreads();
      if (rmin != 0xFFFFFFFFu && dmin == (i64)acc.dmin) atomicMin(&acc.rmin, rmin);
      if (rmax != 0xFFFFFFFFu && dmax == (i64)acc.dmax) atomicMin(&acc.rmax, rmax);
    }
    const u32 ninfl = acc.ninfl, nd = nn - ninfl;
    const u32 km = nd ? (nd - 1) / 2 : 0, kl = nd ? nd - 1 : 0;
    u32 P = 2;
    while (P < nn) P <<= 1;
    for (u32 i = t; i < P; i += TT) V[i] = (i < nn && X[i] != T_INFLIGHT) ? E[i] : T_INFLIGHT;
    __syncthreads();
    team_sort(V, P, t);
    const i64 min_e = V[0], med_e = V[km], max_e = V[kl];
    __syncthreads();
    for (u32 i = t; i < P; i += TT) V[i] = i < nn ? X[i] : T_INFLIGHT;
    __syncthreads();
    team_sort(V, P, t);
    const i64 min_x = V[0], med_x = V[km], max_x = V[kl];
    __syncthreads();
    for (u32 i = t; i < P; i += TT) V[i] = (i < nn && X[i] != T_INFLIGHT) ? absdiff(E[i], med_e) : T_INFLIGHT;
    __syncthreads();
    team_sort(V, P, t);
    const i64 mad_e = V[km];
    __syncthreads();
    for (u32 i = t; i < P; i += TT) V[i] = (i < nn && X[i] != T_INFLIGHT) ? absdiff(X[i], med_x) : T_INFLIGHT;
    __syncthreads();
    team_sort(V, P, t);
    const i64 mad_x = V[km];
    const u32 comm = (u32)(k0 >> (mb + a.sf.ws));
    const bool complete = nn == a.comm_size[comm] && ninfl == 0;
    const bool consistent = acc.incons == 0;
    const bool barrier = h.op == CCLD_OP_ALLREDUCE && h.bytes < (u64)a.barrier_bytes;
    const bool usable = complete && consistent && !barrier;
    if (t == 0) {
      seg_put(a, CCLD_SEG_COMM, srow, (i64)comm);
      seg_put(a, CCLD_SEG_SEQ, srow, (i64)(((k0 >> mb) & smask) + a.sf.seq_base));
      seg_put(a, CCLD_SEG_N, srow, (i64)nn);
      seg_put(a, CCLD_SEG_INFLIGHT, srow, (i64)ninfl);
      seg_put(a, CCLD_SEG_STATE, srow,
              (complete ? CCLD_SEG_COMPLETE : 0) | (consistent ? CCLD_SEG_CONSISTENT : 0) |
                  (barrier ? CCLD_SEG_BARRIER : 0) | (usable ? CCLD_SEG_USABLE : 0));
      seg_put(a, CCLD_SEG_OP, srow, (i64)h.op);
      seg_put(a, CCLD_SEG_BYTES, srow, (i64)h.bytes);
      seg_put(a, CCLD_SEG_INFLIGHT_ENTER_MIN, srow, (i64)acc.imin);
      seg_count_alert(a, srow, ninfl, barrier, (i64)acc.imin);
      seg_put(a, CCLD_SEG_FIRST, srow, (i64)a0);
      if (nd == 0) {
        seg_put_empty_stats(a, srow);
      } else {
        seg_put(a, CCLD_SEG_ENTER_MIN, srow, min_e); seg_put(a, CCLD_SEG_ENTER_MED, srow, med_e);
        seg_put(a, CCLD_SEG_ENTER_MAX, srow, max_e); seg_put(a, CCLD_SEG_ENTER_MAD, srow, mad_e);
        seg_put(a, CCLD_SEG_EXIT_MIN, srow, min_x); seg_put(a, CCLD_SEG_EXIT_MED, srow, med_x);
        seg_put(a, CCLD_SEG_EXIT_MAX, srow, max_x); seg_put(a, CCLD_SEG_EXIT_MAD, srow, mad_x);
        seg_put(a, CCLD_SEG_DUR_MIN, srow, (i64)acc.dmin); seg_put(a, CCLD_SEG_DUR_MAX, srow, (i64)acc.dmax);
        const u32* ms = a.members_sorted + a.member_off[comm];
        seg_put(a, CCLD_SEG_ARGMIN_RANK, srow, (i64)ms[acc.rmin]); seg_put(a, CCLD_SEG_ARGMAX_RANK, srow, (i64)ms[acc.rmax]);
      }
    }
    for (u32 i = t; i < nn; i += TT) {
      const u32 j = a0 + i;
      i64 le = 0, lx = 0;
      u32 f = 0;
      if (usable) {
        le = E[i] - med_e; lx = X[i] - med_x;
        if (is_late(le, a.lag_floor, a.kmad_num, a.kmad_den, mad_e)) f |= CCLD_FLAG_LATE_ENTER;
        if (is_late(lx, a.lag_floor, a.kmad_num, a.kmad_den, mad_x)) f |= CCLD_FLAG_LATE_EXIT;
      }
      a.rec_flag[j] = (uint8_t)f;
      if (a.lag_e) a.lag_e[j] = le;
      if (a.lag_x) a.lag_x[j] = lx;
      if (f) { a.flag_lag[j] = le; a.flag_lag[a.cap_n + j] = lx; }
    }
    __syncthreads();     // the staged times and the accumulator are reused by the next collective
  }
}

// One workgroup of 1,024 threads per collective of SEG_TEAM_MAX + 1 to SEG_LARGE_MAX records (a world communicator
// of thousands of ranks): the times are staged in global scratch, and one LDS array of 128 KB is filled and sorted
// four times (arrival, completion, and their absolute deviations from the medians).
constexpr u32 LARGE_THREADS = 1024;
__global__ __launch_bounds__(LARGE_THREADS) void k_seg_large(SegArgs a) {
  extern __shared__ i64 s_large[];          // [SEG_LARGE_MAX]
  __shared__ TeamAcc acc;
  i64* V = s_large;
  const u32 t = threadIdx.x;
  const int mb = a.sf.mb;
  const u64 mmask = ((u64)1 << mb) - 1, smask = ((u64)1 << a.sf.ws) - 1;
  i64* big_e = a.big_e;
  i64* big_x = a.big_x;
  const u32 nbig = (u32)a.counters[CNT_NBIG];
  for (u32 ent = blockIdx.x; ent < nbig; ent += gridDim.x) {
    const u32 nn = a.big_list[3 * ent + 2];
    if (nn <= (u32)SEG_TEAM_MAX || nn > (u32)SEG_LARGE_MAX) continue;
    const u32 srow = a.big_list[3 * ent], a0 = a.big_list[3 * ent + 1];
    const u64 k0 = a.key[a0];
    const Rec h = load_row(a, a0);
    if (t == 0) {
      acc.imin = (unsigned long long)T_INFLIGHT; acc.dmin = INT64_MAX; acc.dmax = INT64_MIN;
      acc.ninfl = 0; acc.incons = 0; acc.rmin = 0xFFFFFFFFu; acc.rmax = 0xFFFFFFFFu;
    }
    __syncthreads();
    {
      u32 ni = 0, rmin = 0xFFFFFFFFu, rmax = 0xFFFFFFFFu;
      bool inc = false;
      i64 imin = T_INFLIGHT, dmin = INT64_MAX, dmax = INT64_MIN;
      for (u32 i = t; i < nn; i += LARGE_THREADS) {
        const u32 j = a0 + i;
        const Rec rw = load_row(a, j);
        big_e[j] = rw.t_enter; big_x[j] = rw.t_exit;
        inc |= (rw.op != h.op || rw.bytes != h.bytes);
        if (rw.t_exit == T_INFLIGHT) {
          ++ni; imin = rw.t_enter < imin ? rw.t_enter : imin;
        } else {
          const i64 d = rw.t_exit - rw.t_enter;
          const u32 rk = (u32)(a.key[j] & mmask);
          if (d < dmin || (d == dmin && rk < rmin)) { dmin = d; rmin = rk; }
          if (d > dmax || (d == dmax && rk < rmax)) { dmax = d; rmax = rk; }
        }
      }
      if (ni) { atomicAdd(&acc.ninfl, ni); atomicMin(&acc.imin, (unsigned long long)imin); }
      if (inc) atomicOr(&acc.incons, 1u);
      if (rmin != 0xFFFFFFFFu) { atomicMin(&acc.dmin, (long long)dmin); atomicMax(&acc.dmax, (long long)dmax); }
      __threadfence_block();
      __syncthreads();
      if (rmin != 0xFFFFFFFFu && dmin == (i64)acc.dmin) atomicMin(&acc.rmin, rmin);
      if (rmax != 0xFFFFFFFFu && dmax == (i64)acc.dmax) atomicMin(&acc.rmax, rmax);
    }
    const u32 ninfl = acc.ninfl, nd = nn - ninfl;
    const u32 km = nd ? (nd - 1) / 2 : 0, kl = nd ? nd - 1 : 0;
    u32 P = 2;
    while (P < nn) P <<= 1;
    const i64* E = big_e + a0;
    const i64* X = big_x + a0;
    for (u32 i = t; i < P; i += LARGE_THREADS) V[i] = (i < nn && X[i] != T_INFLIGHT) ? E[i] : T_INFLIGHT;
    __syncthreads();
    team_sort<LARGE_THREADS>(V, P, t);
    const i64 min_e = V[0], med_e = V[km], max_e = V[kl];
    __syncthreads();
    for (u32 i = t; i < P; i += LARGE_THREADS) V[i] = i < nn ? X[i] : T_INFLIGHT;
    __syncthreads();
    team_sort<LARGE_THREADS>(V, P, t);
    const i64 min_x = V[0], med_x = V[km], max_x = V[kl];
    __syncthreads();
    for (u32 i = t; i < P; i += LARGE_THREADS) V[i] = (i < nn && X[i] != T_INFLIGHT) ? absdiff(E[i], med_e) : T_INFLIGHT;
    __syncthreads();
    team_sort<LARGE_THREADS>(V, P, t);
    const i64 mad_e = V[km];
    __syncthreads();
    for (u32 i = t; i < P; i += LARGE_THREADS) V[i] = (i < nn && X[i] != T_INFLIGHT) ? absdiff(X[i], med_x) : T_INFLIGHT;
    __syncthreads();
    team_sort<LARGE_THREADS>(V, P, t);
    const i64 mad_x = V[km];
    const u32 comm = (u32)(k0 >> (mb + a.sf.ws));
    const bool complete = nn == a.comm_size[comm] && ninfl == 0;
    const bool consistent = acc.incons == 0;
    const bool barrier = h.op == CCLD_OP_ALLREDUCE && h.bytes < (u64)a.barrier_bytes;
    const bool usable = complete && consistent && !barrier;
    if (t == 0) {
      seg_put(a, CCLD_SEG_COMM, srow, (i64)comm);
      seg_put(a, CCLD_SEG_SEQ, srow, (i64)(((k0 >> mb) & smask) + a.sf.seq_base));
      seg_put(a, CCLD_SEG_N, srow, (i64)nn);
      seg_put(a, CCLD_SEG_INFLIGHT, srow, (i64)ninfl);
      seg_put(a, CCLD_SEG_STATE, srow,
              (complete ? CCLD_SEG_COMPLETE : 0) | (consistent ? CCLD_SEG_CONSISTENT : 0) |
                  (barrier ? CCLD_SEG_BARRIER : 0) | (usable ? CCLD_SEG_USABLE : 0));
      seg_put(a, CCLD_SEG_OP, srow, (i64)h.op);
      seg_put(a, CCLD_SEG_BYTES, srow, (i64)h.bytes);
      seg_put(a, CCLD_SEG_INFLIGHT_ENTER_MIN, srow, (i64)acc.imin);
      seg_count_alert(a, srow, ninfl, barrier, (i64)acc.imin);
      seg_put(a, CCLD_SEG_FIRST, srow, (i64)a0);
      if (nd == 0) {
        seg_put_empty_stats(a, srow);
      } else {
        seg_put(a, CCLD_SEG_ENTER_MIN, srow, min_e); seg_put(a, CCLD_SEG_ENTER_MED, srow, med_e);
        seg_put(a, CCLD_SEG_ENTER_MAX, srow, max_e); seg_put(a, CCLD_SEG_ENTER_MAD, srow, mad_e);
        seg_put(a, CCLD_SEG_EXIT_MIN, srow, min_x); seg_put(a, CCLD_SEG_EXIT_MED, srow, med_x);
        seg_put(a, CCLD_SEG_EXIT_MAX, srow, max_x); seg_put(a, CCLD_SEG_EXIT_MAD, srow, mad_x);
        seg_put(a, CCLD_SEG_DUR_MIN, srow, (i64)acc.dmin); seg_put(a, CCLD_SEG_DUR_MAX, srow, (i64)acc.dmax);
        const u32* ms = a.members_sorted + a.member_off[comm];
        seg_put(a, CCLD_SEG_ARGMIN_RANK, srow, (i64)ms[acc.rmin]); seg_put(a, CCLD_SEG_ARGMAX_RANK, srow, (i64)ms[acc.rmax]);
      }
    }
    for (u32 i = t; i < nn; i += LARGE_THREADS) {
      const u32 j = a0 + i;
      i64 le = 0, lx = 0;
      u32 f = 0;
      if (usable) {
        le = E[i] - med_e; lx = X[i] - med_x;
        if (is_late(le, a.lag_floor, a.kmad_num, a.kmad_den, mad_e)) f |= CCLD_FLAG_LATE_ENTER;
        if (is_late(lx, a.lag_floor, a.kmad_num, a.kmad_den, mad_x)) f |= CCLD_FLAG_LATE_EXIT;
      }
      a.rec_flag[j] = (uint8_t)f;
      if (a.lag_e) a.lag_e[j] = le;
      if (a.lag_x) a.lag_x[j] = lx;
      if (f) { a.flag_lag[j] = le; a.flag_lag[a.cap_n + j] = lx; }
    }
    __syncthreads();     // the LDS array and the accumulator are reused by the next collective
  }
}

// Collectives longer than SEG_LARGE_MAX records: one workgroup per collective, values staged in
// global scratch, order statistics by counting with all reads broadcast across the workgroup.
__global__ __launch_bounds__(SEG_THREADS) void k_seg_big(SegArgs a) {
  __shared__ u32 s_end, s_ninfl, s_incons;
  __shared__ unsigned long long s_imin;
  __shared__ i64 s_stat[4];      // med_e, med_x, mad_e, mad_x
  const u32 tid = threadIdx.x;
  const int mb = a.sf.mb;
  const u64 mmask = ((u64)1 << mb) - 1, smask = ((u64)1 << a.sf.ws) - 1;
  i64* big_e = a.big_e;
  i64* big_x = a.big_x;
  const u32 nbig = (u32)a.counters[CNT_NBIG];
  for (u32 ent = blockIdx.x; ent < nbig; ent += gridDim.x) {
    if (a.big_list[3 * ent + 2] <= (u32)SEG_LARGE_MAX) continue;    // a workgroup kernel has taken it
    const u32 srow = a.big_list[3 * ent], a0 = a.big_list[3 * ent + 1];
    const u64 k0 = a.key[a0];
    const u64 pref = k0 >> mb;
    if (tid == 0) { s_end = a.n; s_ninfl = 0; s_incons = 0; s_imin = (unsigned long long)T_INFLIGHT; }
    __syncthreads();
    for (u64 j0 = (u64)a0 + 1;; j0 += SEG_THREADS) {
      const u64 j = j0 + tid;
      if (j < a.n && (a.key[j] >> mb) != pref) atomicMin(&s_end, (u32)j);
      __syncthreads();
      const bool stop = s_end != a.n || j0 + SEG_THREADS >= a.n;
      __syncthreads();
      if (stop) break;
    }
    const u32 b0 = s_end, nn = b0 - a0;
    const Rec h = load_row(a, a0);
    {
      u32 ni = 0; bool inc = false; i64 imin = T_INFLIGHT;
      for (u32 j = a0 + tid; j < b0; j += SEG_THREADS) {
        const Rec rw = load_row(a, j);
        big_e[j] = rw.t_enter; big_x[j] = rw.t_exit;
        if (rw.t_exit == T_INFLIGHT) { ++ni; imin = rw.t_enter < imin ? rw.t_enter : imin; }
        inc |= (rw.op != h.op || rw.bytes != h.bytes);
      }
      if (ni) { atomicAdd(&s_ninfl, ni); atomicMin(&s_imin, (unsigned long long)imin); }
      if (inc) atomicOr(&s_incons, 1u);
    }
    __threadfence_block();
    __syncthreads();
    const u32 ninfl = s_ninfl, nd = nn - ninfl, km = nd ? (nd - 1) / 2 : 0;
    if (tid == 0) {
      seg_put(a, CCLD_SEG_COMM, srow, (i64)(k0 >> (mb + a.sf.ws)));
      seg_put(a, CCLD_SEG_SEQ, srow, (i64)(((k0 >> mb) & smask) + a.sf.seq_base));
      seg_put(a, CCLD_SEG_N, srow, (i64)nn);
      seg_put(a, CCLD_SEG_INFLIGHT, srow, (i64)ninfl);
      seg_put(a, CCLD_SEG_OP, srow, (i64)h.op);
      seg_put(a, CCLD_SEG_BYTES, srow, (i64)h.bytes);
      seg_put(a, CCLD_SEG_INFLIGHT_ENTER_MIN, srow, (i64)s_imin);
      seg_put(a, CCLD_SEG_FIRST, srow, (i64)a0);
      if (nd == 0) seg_put_empty_stats(a, srow);
    }
    for (u32 i = a0 + tid; i < b0; i += SEG_THREADS) {
      const i64 ei = big_e[i], xi = big_x[i];
      if (xi == T_INFLIGHT) continue;
      const i64 di = xi - ei;
      u32 re = 0, rx = 0, cmin = 0, cmax = 0;
      for (u32 j = a0; j < b0; ++j) {
        const i64 ej = big_e[j], xj = big_x[j];
        if (xj == T_INFLIGHT) continue;
        const i64 dj = xj - ej;
        const bool before = j < i;
        re += (ej < ei) || (ej == ei && before);
        rx += (xj < xi) || (xj == xi && before);
        cmin += (dj < di) || (dj == di && before);
        cmax += (dj > di) || (dj == di && before);
      }
      if (re == km) { s_stat[0] = ei; seg_put(a, CCLD_SEG_ENTER_MED, srow, ei); }
      if (re == 0) seg_put(a, CCLD_SEG_ENTER_MIN, srow, ei);
      if (re == nd - 1) seg_put(a, CCLD_SEG_ENTER_MAX, srow, ei);
      if (rx == km) { s_stat[1] = xi; seg_put(a, CCLD_SEG_EXIT_MED, srow, xi); }
      if (rx == 0) seg_put(a, CCLD_SEG_EXIT_MIN, srow, xi);
      if (rx == nd - 1) seg_put(a, CCLD_SEG_EXIT_MAX, srow, xi);
      const i64 rk = (i64)a.members_sorted[a.member_off[(u32)(k0 >> (mb + a.sf.ws))] + (u32)(a.key[i] & mmask)];
      if (cmin == 0) { seg_put(a, CCLD_SEG_DUR_MIN, srow, di); seg_put(a, CCLD_SEG_ARGMIN_RANK, srow, rk); }
      if (cmax == 0) { seg_put(a, CCLD_SEG_DUR_MAX, srow, di); seg_put(a, CCLD_SEG_ARGMAX_RANK, srow, rk); }
    }
    __syncthreads();
    const i64 me = s_stat[0], mx = s_stat[1];
    for (u32 i = a0 + tid; i < b0; i += SEG_THREADS) {
      const i64 xi = big_x[i];
      if (xi == T_INFLIGHT) continue;
      const i64 dei = absdiff(big_e[i], me), dxi = absdiff(xi, mx);
      u32 rde = 0, rdx = 0;
      for (u32 j = a0; j < b0; ++j) {
        const i64 xj = big_x[j];
        if (xj == T_INFLIGHT) continue;
        const i64 dej = absdiff(big_e[j], me), dxj = absdiff(xj, mx);
        const bool before = j < i;
        rde += (dej < dei) || (dej == dei && before);
        rdx += (dxj < dxi) || (dxj == dxi && before);
      }
      if (rde == km) { s_stat[2] = dei; seg_put(a, CCLD_SEG_ENTER_MAD, srow, dei); }
      if (rdx == km) { s_stat[3] = dxi; seg_put(a, CCLD_SEG_EXIT_MAD, srow, dxi); }
    }
    __syncthreads();
    const u32 comm = (u32)(k0 >> (mb + a.sf.ws));
    const bool complete = nn == a.comm_size[comm] && ninfl == 0;
    const bool consistent = s_incons == 0;
    const bool barrier = h.op == CCLD_OP_ALLREDUCE && h.bytes < (u64)a.barrier_bytes;
    const bool usable = complete && consistent && !barrier;
    if (tid == 0) {
      seg_put(a, CCLD_SEG_STATE, srow,
              (complete ? CCLD_SEG_COMPLETE : 0) | (consistent ? CCLD_SEG_CONSISTENT : 0) |
                  (barrier ? CCLD_SEG_BARRIER : 0) | (usable ? CCLD_SEG_USABLE : 0));
      seg_count_alert(a, srow, ninfl, barrier, (i64)s_imin);
    }
    for (u32 i = a0 + tid; i < b0; i += SEG_THREADS) {
      i64 le = 0, lx = 0;
      u32 f = 0;
      if (usable) {
        le = big_e[i] - me; lx = big_x[i] - mx;
        if (is_late(le, a.lag_floor, a.kmad_num, a.kmad_den, s_stat[2])) f |= CCLD_FLAG_LATE_ENTER;
        if (is_late(lx, a.lag_floor, a.kmad_num, a.kmad_den, s_stat[3])) f |= CCLD_FLAG_LATE_EXIT;
      }
      a.rec_flag[i] = (uint8_t)f;
      if (a.lag_e) a.lag_e[i] = le;
      if (a.lag_x) a.lag_x[i] = lx;
      if (f) { a.flag_lag[i] = le; a.flag_lag[a.cap_n + i] = lx; }
    }
    __syncthreads();
  }
}

// group code and range of the collectives that a workgroup analysed (more than SEG_MULTI_MAX records), from
// their rows of the table; a row past the table's capacity is not stored and takes no part in the group stage
__global__ __launch_bounds__(256) void k_seg_group_listed(SegArgs a) {
  const u32 nbig = (u32)a.counters[CNT_NBIG];
  for (u32 ent = blockIdx.x * 256 + threadIdx.x; ent < nbig; ent += gridDim.x * 256) {
    if (a.big_list[3 * ent + 2] <= (u32)SEG_MULTI_MAX) continue;
    const u32 srow = a.big_list[3 * ent];
    if (srow >= a.seg_cap) { a.gcode[srow] = (uint16_t)NO_GROUP; a.range_c[srow] = 0; continue; }
    const u64 C = a.seg_cap;
    const bool usable = (a.seg[(u64)CCLD_SEG_STATE * C + srow] & CCLD_SEG_USABLE) != 0;
    seg_put_group(a, srow, usable, (u32)a.seg[(u64)CCLD_SEG_OP * C + srow],
                  (u64)a.seg[(u64)CCLD_SEG_BYTES * C + srow], a.seg[(u64)CCLD_SEG_DUR_MAX * C + srow],
                  a.seg[(u64)CCLD_SEG_DUR_MIN * C + srow]);
  }
}

// ---- grid placement: statistics straight from the partitioned rows --------------------------------------
// One workgroup per fine bucket: the bucket's rows (in arrival order) are placed in LDS by cell (round inside the bucket
// x member slot), which puts every collective's records side by side in rank order with empty cells where a member has
// no record; the wavefronts then take the collectives 64 / G at a time.  The kernel leaves, beside the table, the row
// of every cell (2 bytes), which the chains and the alerts look records up by, and the bucket's flagged records.
template <u32 ROUNDS>                      // most rounds of a bucket
struct GridShared {
  uint4 row[GRID_B];                     // rows by cell; y bits 16-26: number of the row in its bucket
  u32 pres[GRID_B / 32];
  unsigned short pre[ROUNDS];            // records of the bucket before each of its rounds
  u32 wave[1024 / CCLD_WAVE], rec0;      // rec0: records of the window before the bucket
  u32 odd;                               // operations in flight, rows of full width or two rows of a cell among them
  GridFlags flags;
};
// Records before fine bucket f.  The scan of the counts at the end of the partition is a chain of its own, and its workgroups
// arrive at one word; where GRID_SELF_SUM buckets are likely their sum is a load or two per thread, on their way together with
// the bucket's rows (384 buckets: a stream's step 118.7 -> 113.0 us).  At 900 and 3,900 buckets the sums cost 2 and 5 us more
// than the scan.
template <bool SELF_SUM>
struct RecordsBefore {
  u32 part;
  template <int THREADS>
  static __device__ __forceinline__ RecordsBefore load(const GridArgs& d, u32 f, bool scanned) {
    u32 v = 0;
    if (!scanned) {
#pragma unroll 2
      for (u32 i = threadIdx.x; i < f; i += THREADS) v += fill_rows(d.fill[i]);
    } else if (threadIdx.x == 0) {
      v = d.rec0[f];
    }
    return {v};
  }
  // s_sum: a word of LDS, zero before the last barrier and complete behind the next one
  __device__ __forceinline__ void add(u32* s_sum) const {
    const u32 v = wave_sum(part);
    if (lane_id() == 0 && v) atomicAdd(s_sum, v);
  }
};
template <>
struct RecordsBefore<false> { __device__ __forceinline__ void add(u32*) const {} };
// Places bucket f's rows in LDS.  Returns status bits: a cell taken twice or more rows than cells (duplicate keys), a
// round without any record (a hole in the grid).  Ends with a barrier.
template <int THREADS, u32 ROUNDS, bool SELF_SUM>
__device__ __forceinline__ u64 grid_place(const GridArgs& d, const FineDesc& D, u32 fill, const RecordsBefore<SELF_SUM>& before, GridShared<ROUNDS>& S) {
  constexpr u32 U = GRID_B / THREADS;
  const u32 tid = threadIdx.x, cells = D.K * D.size;
  typedef u32 u32x4 __attribute__((ext_vector_type(4)));
  u32x4 v[U];
  const u32 cnt = fill_rows(fill), front = fill_front(fill), back = cells - fill_back(fill);
  const bool over = cnt > cells;              // every cell has been written then (rooms.h)
  bool dup = over;
  auto holds = [&](u32 i) { return i < cells && (i < front || i >= back || over); };
#pragma unroll
  for (u32 u = 0; u < U; ++u) {
    const u32 i = tid + u * THREADS;
    if (holds(i)) v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(d.rows + D.cell0 + i));
  }
  for (u32 i = tid; i < GRID_B / 32; i += THREADS) { S.pres[i] = 0; S.flags.bits[i] = 0; }
  if (tid == 0) { S.flags.n = 0; S.rec0 = 0; S.odd = 0; }
  __syncthreads();
  before.add(&S.rec0);
  u32 most = 0;
#pragma unroll
  for (u32 u = 0; u < U; ++u) {
    const u32 i = tid + u * THREADS;
    if (!holds(i)) continue;
    most = v[u].z > most ? v[u].z : most;
    const u32 cell = (v[u].y >> ROW_CELL_SHIFT) & ROW_CELL_MASK;
    if (cell >= cells) { dup = true; continue; }
    const u32 bit = 1u << (cell & 31);
    if (atomicOr(&S.pres[cell >> 5], bit) & bit) { dup = true; continue; }
    S.row[cell] = make_uint4(v[u].x, (v[u].y & ~(ROW_CELL_MASK << ROW_CELL_SHIFT)) | (i << ROW_CELL_SHIFT), v[u].z, v[u].w);
  }
  static_assert(ROW_INFLIGHT > ROW_WIDE, "the two largest words");
  if (most >= ROW_WIDE || dup) S.odd = 1;
  __syncthreads();
#pragma unroll
  for (u32 u = 0; u < U; ++u) {
    const u32 c = tid + u * THREADS;
    if (c >= cells) continue;
    const bool on = (S.pres[c >> 5] >> (c & 31)) & 1u;
    d.cell_row[D.cell0 + c] = (uint16_t)(on ? (S.row[c].y >> ROW_CELL_SHIFT) & ROW_CELL_MASK : GRID_EMPTY);
  }
  // records per round and their exclusive scan; a bucket with as many rows as cells has a record in every cell, unless one
  // was taken twice, which fails the analysis
  bool gap = false;
  if (cnt >= cells) {
    for (u32 k = tid; k < D.K; k += THREADS) S.pre[k] = (unsigned short)(k * D.size);
    __syncthreads();
    return dup ? (u64)DS_DUPLICATE : 0;
  }
  u32 n[U], sum = 0;
  const u32 per = (D.K + THREADS - 1) / THREADS;          // <= U
#pragma unroll
  for (u32 q = 0; q < U; ++q) {
    const u32 k = per * tid + q;
    n[q] = 0;
    if (q < per && k < D.K) {
      const u32 b0 = k * D.size, b1 = b0 + D.size;      // bits [b0, b1)
      for (u32 w = b0 >> 5; w <= (b1 - 1) >> 5; ++w) {
        u32 m = S.pres[w];
        if (w == (b0 >> 5)) m &= ~0u << (b0 & 31);
        if (w == ((b1 - 1) >> 5) && (b1 & 31)) m &= (1u << (b1 & 31)) - 1;
        n[q] += (u32)__popc(m);
      }
      gap |= n[q] == 0;
    }
    sum += n[q];
  }
  u32 tot;
  u32 ex = block_exclusive_sum<THREADS>(sum, S.wave, &tot);
#pragma unroll
  for (u32 q = 0; q < U; ++q) {
    const u32 k = per * tid + q;
    if (q < per && k < D.K) S.pre[k] = (unsigned short)ex;
    ex += n[q];
  }
  __syncthreads();
  return (dup ? (u64)DS_DUPLICATE : 0) | (gap ? (u64)DS_DENSE_FALLBACK : 0);
}
// Puts the flagged records of a fine bucket in (counter, rank) order and adds them to the late columns of the blame table.
// Called by the whole workgroup behind a barrier; few buckets have any.
template <int THREADS>
__device__ __forceinline__ void grid_order_flags(const SegArgs& a, const FineDesc& D, u32 rec0, GridFlags& F, u32* s_wave,
                                                 i64* __restrict__ blame, u32 n_ranks) {
  const u32 n = F.n, tid = threadIdx.x;
  if (n == 0) return;
  static_assert(GRID_B / 32 <= CCLD_WAVE, "one word per lane");
  if (tid < CCLD_WAVE) {
    const u32 c = tid < GRID_B / 32 ? (u32)__popc(F.bits[tid]) : 0u;
    const u32 inc = wave_inclusive_sum(c);
    if (tid < GRID_B / 32) F.pre[tid] = inc - c;
  }
  __syncthreads();
  constexpr u32 U = GRID_B / THREADS;
  u32 w[U], at[U];
  i64 le[U], lx[U];
#pragma unroll
  for (u32 u = 0; u < U; ++u) {
    const u32 i = tid + u * THREADS;
    w[u] = 0;
    if (i < n) {
      w[u] = a.flag_pos[rec0 + i]; le[u] = a.flag_lag[rec0 + i]; lx[u] = a.flag_lag[a.cap_n + rec0 + i];
      const u32 cell = w[u] & 0xFFFFu;
      at[u] = F.pre[cell >> 5] + (u32)__popc(F.bits[cell >> 5] & ((1u << (cell & 31)) - 1u));
    }
  }
  __syncthreads();
#pragma unroll
  for (u32 u = 0; u < U; ++u) {
    if (__ballot(w[u] != 0) == 0) continue;
    if (w[u]) { a.flag_pos[rec0 + at[u]] = w[u]; a.flag_lag[rec0 + at[u]] = le[u]; a.flag_lag[a.cap_n + rec0 + at[u]] = lx[u]; }
    // the blame of one wavefront's records: one set of atomics per member slot that occurs
    const u32 kind = w[u] >> 16, slot = w[u] ? (w[u] & 0xFFFFu) % D.size : 0u;
    u64 todo = ballot64(w[u] != 0);
    while (todo) {
      const u32 v = (u32)__shfl((int)slot, (int)__builtin_ctzll(todo), CCLD_WAVE);
      const u64 same = ballot64(w[u] != 0 && slot == v);
      const bool me = (same >> lane_id()) & 1;
      const bool en = me && (kind & CCLD_FLAG_LATE_ENTER), ex = me && (kind & CCLD_FLAG_LATE_EXIT);
      const u64 ne = (u64)__popcll(ballot64(en)), nx = (u64)__popcll(ballot64(ex));
      u64 se = en ? (u64)le[u] : 0, sx = ex ? (u64)lx[u] : 0;
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) { se += shfl_xor_u64(se, m); sx += shfl_xor_u64(sx, m); }
      if (lane_id() < 4) {
        const u64 val = lane_id() == 0 ? ne : lane_id() == 1 ? nx : lane_id() == 2 ? se : sx;
        const u32 r = a.members_sorted[a.member_off[D.comm] + v];
        if (val) atomicAdd(reinterpret_cast<unsigned long long*>(&blame[(u64)lane_id() * n_ranks + r]), (unsigned long long)val);
      }
      todo &= ~same;
    }
  }
}
static_assert(CCLD_BLM_N_LATE_ENTER == 0 && CCLD_BLM_N_LATE_EXIT == 1 && CCLD_BLM_SUM_LAG_ENTER == 2 &&
              CCLD_BLM_SUM_LAG_EXIT == 3, "blame column order");
// position in the window's arrival order of a partitioned row
__device__ __forceinline__ u32 grid_arrival(const SegArgs& a, const GridArgs& d, u32 at) {
  return arrival_of_slot(a.win, d.slots[at]);
}

// A collective's table row waits in its own cells (16 words; from four members on they are large enough) until the
// workgroup writes the table, 64 rows per store instruction.  The words are permuted by the round's number, so that
// neither the lanes that write one row nor those that read one word of 64 rows meet in few banks.
//   0-1 x and y of the first record's row | 2-5 arrival min, median, max, MAD | 6-9 the same of the completion, all relative
//   to the first record's arrival | 10-11 T_min, T_max | 12-13 their ranks | 14 bytes, low | 15 records | inconsistent << 8
// word 15 = ROW_NOT_STAGED: the row was written directly (times that do not fit 30 bits, operations in flight).  What
// follows from these words alone is computed where the table is written: once per collective there, but once per
// lane in the passes below.
constexpr u32 ROW_WORDS = 16, ROW_NOT_STAGED = 0xFFFFFFFFu;
struct StageRow {            // where round k's words are
  u32 base, turn;            // byte offsets
  __device__ __forceinline__ StageRow(u32 k, u32 size) : base(k * size * 16 + (size >= 8 ? (k & 16u) * 4 : 0u)), turn((k & 15u) * 4) {}
  __device__ __forceinline__ u32* word(uint4* rows, u32 w) const {
    return reinterpret_cast<u32*>(reinterpret_cast<char*>(rows) + ((turn ^ (w * 4)) + base));
  }
};
// The bits of a ballot that belong to the calling lane's group of G lanes: one word below 64 lanes, and where the
// group is the wavefront the same 64 bits in every lane.
template <int G>
__device__ __forceinline__ auto group_bits(u64 m, u32 gbase) {
  if constexpr (G == 64) return m;
  else if constexpr (G == 32) return (u32)(m >> gbase);
  else return (u32)(m >> gbase) & ((1u << G) - 1u);
}
__device__ __forceinline__ u32 count_bits(u32 m) { return (u32)__builtin_popcount(m); }
__device__ __forceinline__ u32 count_bits(u64 m) { return (u32)__builtin_popcountll(m); }
__device__ __forceinline__ u32 first_bit(u32 m) { return (u32)__builtin_ctz(m); }      // m != 0
__device__ __forceinline__ u32 first_bit(u64 m) { return (u32)__builtin_ctzll(m); }

// Bound by the vector instructions of this loop, so every lane does only what its own record needs: 252 instead of 388 per 64
// records over the whole kernel, 82M records in 8.4M collectives 1,053 -> 822 us (3.0 GB: 3.7 TB/s).
// The kernel's first argument, read again where it is used: what few passes need would be kept in scalar registers over all of them,
// which are too few, and every spill and reload of one is a vector instruction.  (Not where there are FEW buckets, whose passes would
// wait for it.)  With FULL: 82M records 809 -> 778 us, 5.1M 73.1 -> 68.5, ten batches of 2M 167 -> 160.
// These two take the arguments by their places: only for the kernels whose signatures are checked below (reads_args_again), whose
// copies of the arguments are const.
__device__ __forceinline__ const SegArgs& args_again() {
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm("" : "+s"(p));
  return *(const SegArgs*)p;
}
// The second one.
__device__ __forceinline__ const GridArgs& grid_again() {
  constexpr size_t at = (sizeof(SegArgs) + alignof(GridArgs) - 1) / alignof(GridArgs) * alignof(GridArgs);
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm("" : "+s"(p));
  return *(const GridArgs*)((const char*)p + at);
}
// FULL: every cell of the bucket has a record, of a finished operation (a pass of eight lanes to a collective is 160 instructions then
// instead of 190).
template <int G, bool FULL, bool FEW>
__device__ __forceinline__ u32 grid_batches(const SegArgs& a, const GridArgs& d, const FineDesc& D, u32 rec0, i64 wref,
                                            GridShared<GRID_B>& S, u32 lane, u32 wave, u32 n_waves) {
  constexpr int SPW = CCLD_WAVE / G;
  constexpr u32 LIM = 1u << 30;
  const u32 K = D.K, size = D.size;
  const bool stage = size >= 4, per_record = a.rec_flag || a.lag_e || a.lag_x || a.perm;
  const i32 floor32 = a.lag_floor > 0x7FFFFFFF ? 0x7FFFFFFF : a.lag_floor < -0x7FFFFFFF ? -0x7FFFFFFF : (i32)a.lag_floor;
  const u32 q = lane / G, l = lane % G, gbase = q * G;
  const u32 rank = l < size ? a.members_sorted[a.member_off[D.comm] + l] : 0u;
  u32 mine = 0;                                    // records seen in this lane's member slot
  for (u32 b = wave; b * SPW < K; b += n_waves) {
    const u32 k = b * SPW + q;
    const bool in = k < K && l < size;
    const u32 cell = in ? k * size + l : 0u;
    const bool valid = FULL ? in : in && ((S.pres[cell >> 5] >> (cell & 31)) & 1u);
    const auto pm = group_bits<G>(FULL ? 0ull : ballot64(valid), gbase);
    const u32 n = FULL ? size : count_bits(pm), fl = !FULL && pm ? first_bit(pm) : 0u;
    const uint4 v = S.row[cell];
    const uint4 lead = S.row[(FULL ? k < K : pm != 0) ? k * size + fl : 0u];                // one address per group: a broadcast
    __builtin_amdgcn_wave_barrier();                                  // read before the row is staged over it
    mine += valid ? 1u : 0u;
    // arrival relative to the first record's: the 44 bits of the times sit at the bottom of x and y
    const u64 diff = (((u64)v.y << 32) | v.x) - (((u64)lead.y << 32) | lead.x);
    const i32 er = (i32)(u32)diff, xr = (i32)((u32)er + v.z);
    const bool infl = !FULL && valid && v.z == ROW_INFLIGHT, done = FULL ? valid : valid && v.z != ROW_INFLIGHT;
    // (a first record of full width shows in its own lane)
    const bool wide = (valid && ((((u32)(diff >> 32) ^ (u32)(er >> 31)) & 0xFFFu) != 0 || (u32)er + LIM >= 2 * LIM)) ||
                      (done && (v.z >= LIM || xr >= (i32)LIM));
    const u32 first = rec0 + (k < K ? S.pre[k] : 0u);
    const auto j_of = [&] { return first + (FULL ? l : G == 64 ? mbcnt64((u64)pm) : count_bits((u32)pm & ((1u << l) - 1u))); };
    if (per_record && a.perm && valid) a.perm[j_of()] = grid_arrival(a, d, D.cell0 + ((v.y >> ROW_CELL_SHIFT) & ROW_CELL_MASK));
    const StageRow at(k, size);
    if (ballot64(wide) != 0) {
      DenseLane L;
      const Rec r = valid ? unpack_row(v, wref, a.win.wide) : Rec{0, T_INFLIGHT, 0, 0};
      L.e = r.t_enter; L.x = r.t_exit; L.nb = r.bytes; L.op = r.op; L.rank = rank; L.valid = valid; L.fl = gbase + fl;
      L.n = n; L.first = first; L.j = j_of(); L.srow = D.srow0 + k; L.comm = D.comm; L.seq = D.seq0 + k;
      L.stage = nullptr; L.staged = false; L.cell = cell; L.rec0 = rec0; L.flags = &S.flags;
      const u64 gmask = (G == 64 ? ~0ull : (((u64)1 << (G & 63)) - 1)) << gbase;
      dense_pass64<G, PUT_GRID>(FEW ? a : args_again(), L, size, lane, gbase, gmask);
      if (stage && valid && l == fl) *at.word(S.row, 15) = ROW_NOT_STAGED;
      continue;
    }
    const u32 nd = FULL ? size : count_bits(group_bits<G>(ballot64(done), gbase)), ninfl = n - nd;
    const u32 kl = nd ? nd - 1 : 0, km = kl / 2;
    const i32 se = sort_groups32<G>(done ? er : REL_NONE, lane);
    const i32 sx = sort_groups32<G>(done ? xr : REL_NONE, lane);
    const i32 med_e = lane_read(se, gbase + km), med_x = lane_read(sx, gbase + km);
    // deviations of the sorted offsets (the first nd lanes of a group hold its finished records): they fall to zero
    // at the median and rise again, so one merge sorts them
    const bool held = l < nd;
    auto deviation = [](i32 x, i32 med) { const i32 t = (i32)((u32)x - (u32)med), u = (i32)(0u - (u32)t); return t > u ? t : u; };
    const i32 sde = merge_groups32<G>(held ? deviation(se, med_e) : REL_NONE, lane);
    const i32 sdx = merge_groups32<G>(held ? deviation(sx, med_x) : REL_NONE, lane);
    // T_min / T_max of the Duration Time; the first lane that attains one has the smallest rank
    const u32 dmin = reduce_u32<G, false>(done ? v.z : ~0u), dmax = reduce_u32<G, true>(done ? v.z : 0u);
    const auto mmin = group_bits<G>(ballot64(done && v.z == dmin), gbase), mmax = group_bits<G>(ballot64(done && v.z == dmax), gbase);
    const bool incons = group_bits<G>(ballot64(valid && (v.w != lead.w || ((v.y ^ lead.y) & ROW_SAME_MASK))), gbase) != 0;
    if (stage && ninfl == 0 && (FULL ? k < K : n != 0)) {
      // every lane writes the words it holds
      if (l == 0) {
        *at.word(S.row, 0) = lead.x; *at.word(S.row, 1) = lead.y; *at.word(S.row, 2) = (u32)se; *at.word(S.row, 6) = (u32)sx;
        *at.word(S.row, 10) = dmin; *at.word(S.row, 11) = dmax; *at.word(S.row, 14) = lead.w;
        *at.word(S.row, 15) = n | (incons ? 256u : 0u);
      }
      if (l == km) {
        *at.word(S.row, 3) = (u32)se; *at.word(S.row, 7) = (u32)sx;
        *at.word(S.row, 5) = (u32)sde; *at.word(S.row, 9) = (u32)sdx;
      }
      if (l == kl) { *at.word(S.row, 4) = (u32)se; *at.word(S.row, 8) = (u32)sx; }
      if (l == first_bit(mmin)) *at.word(S.row, 12) = rank;
      if (l == first_bit(mmax)) *at.word(S.row, 13) = rank;
    }
    // a lag within the floor is never late (most wavefronts end here), and only finished complete collectives have lags
    i32 le = (i32)((u32)er - (u32)med_e), lx = (i32)((u32)xr - (u32)med_x);
    const bool direct = ballot64(!stage || ninfl != 0) != 0;
    if (!direct && !per_record && ballot64(valid && (le > floor32 || lx > floor32)) == 0) continue;
    const u64 hb = row_bytes(lead);
    const u32 hop = row_op(lead);
    const bool complete = n == size && ninfl == 0;
    const bool barrier = hop == CCLD_OP_ALLREDUCE && hb < (u64)a.barrier_bytes;
    const bool usable = complete && !incons && !barrier;
    if (direct) {
      // short communicators and operations in flight: the row goes straight to the table
      const i64 ref = wref + t44_diff(row_t44(lead), (u64)wref);
      const i32 min_e = lane_read(se, gbase), max_e = lane_read(se, gbase + kl);
      const i32 min_x = lane_read(sx, gbase), max_x = lane_read(sx, gbase + kl);
      const i32 mad_e = lane_read(sde, gbase + km), mad_x = lane_read(sdx, gbase + km);
      const u32 rmin = lane_read(rank, mmin ? gbase + first_bit(mmin) : lane), rmax = lane_read(rank, mmax ? gbase + first_bit(mmax) : lane);
      const i32 imin = (i32)(reduce_u32<G, false>(infl ? (u32)er ^ 0x80000000u : ~0u) ^ 0x80000000u);
      if (valid && l == fl && (!stage || ninfl)) {
        DenseLane L;
        L.n = n; L.first = first; L.srow = D.srow0 + k; L.comm = D.comm; L.seq = D.seq0 + k; L.staged = false;
        dense_put_row<PUT_GRID>(FEW ? a : args_again(), L, ninfl, complete, incons, barrier, usable, hop, hb, ninfl ? ref + imin : T_INFLIGHT, nd,
                                ref + min_e, ref + med_e, ref + max_e, (i64)mad_e, ref + min_x, ref + med_x, ref + max_x,
                                (i64)mad_x, (i64)dmin, (i64)dmax, rmin, rmax);
        if (stage) *at.word(S.row, 15) = ROW_NOT_STAGED;
      }
    }
    u32 f = 0;
    const i32 mad_e = lane_read(sde, gbase + km), mad_x = lane_read(sdx, gbase + km);
    const SegArgs& A = FEW ? a : args_again();
    if (usable) {
      if (is_late32(le, A.lag_floor, A.kmad_num, A.kmad_den, mad_e)) f |= CCLD_FLAG_LATE_ENTER;
      if (is_late32(lx, A.lag_floor, A.kmad_num, A.kmad_den, mad_x)) f |= CCLD_FLAG_LATE_EXIT;
    } else {
      le = 0; lx = 0;
    }
    if (valid) grid_put_record(A, per_record ? j_of() : 0u, cell, rec0, &S.flags, f, (i64)le, (i64)lx);
  }
  return mine;
}

template <int GRID_THREADS, bool SELF_SUM>       // SELF_SUM: as d.self_sum
__global__ __launch_bounds__(GRID_THREADS) void k_grid_stats(const SegArgs a, const GridArgs d, i64* __restrict__ blame, u32 n_ranks) {
  __shared__ GridShared<GRID_B> S;
  __shared__ u32 s_slot[CCLD_WAVE];
  constexpr u32 NW = GRID_THREADS / CCLD_WAVE;
  const u32 f = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wave = tid / CCLD_WAVE;
  // the header and what it may turn out that there is not (every table has an entry for every workgroup) in one trip to memory
  const GridHeader H = *d.hdr;
  const FineDesc D = d.desc[f];
  const u32 fill = d.fill[f], size = D.size, scanned = SELF_SUM ? 0u : d.rec0[f];
  if (H.feasible == 0 || f >= H.n_fine) return;
  if (size > (u32)SEG_WAVE_MAX) return;                 // k_grid_long takes it
  const i64 wref = H.ref;
  if (tid < CCLD_WAVE) s_slot[tid] = 0;
  u64 bad;
  u32 rec0;
  if constexpr (SELF_SUM) {
    bad = grid_place<GRID_THREADS>(d, D, fill, RecordsBefore<true>::load<GRID_THREADS>(d, f, false), S);
    rec0 = (u32)__builtin_amdgcn_readfirstlane((int)S.rec0);
    if (tid == 0) d.rec0[f] = rec0;
  } else {
    rec0 = scanned;
    bad = grid_place<GRID_THREADS>(d, D, fill, RecordsBefore<false>{}, S);
  }
  u32 mine;
  constexpr bool FEW = GRID_THREADS == 1024;
  auto batches = [&](auto FULL) {
    if (size <= 2) mine = grid_batches<2, FULL, FEW>(a, d, D, rec0, wref, S, lane, wave, NW);
    else if (size <= 4) mine = grid_batches<4, FULL, FEW>(a, d, D, rec0, wref, S, lane, wave, NW);
    else if (size <= 8) mine = grid_batches<8, FULL, FEW>(a, d, D, rec0, wref, S, lane, wave, NW);
    else if (size <= 16) mine = grid_batches<16, FULL, FEW>(a, d, D, rec0, wref, S, lane, wave, NW);
    else if (size <= 32) mine = grid_batches<32, FULL, FEW>(a, d, D, rec0, wref, S, lane, wave, NW);
    else mine = grid_batches<64, FULL, FEW>(a, d, D, rec0, wref, S, lane, wave, NW);
  };
  // (not where a workgroup has sixteen wavefronts and there are few of them: what counts there are the instructions that are fetched
  // for the first time, 8 buckets 11.7 -> 13.2 us)
  bool full = false;
  if constexpr (!FEW) {
    full = fill_rows(fill) == D.K * size && (u32)__builtin_amdgcn_readfirstlane((int)S.odd) == 0;
    if (full) batches(std::true_type{});
  }
  if (!full) batches(std::false_type{});
  // the lane's member slot is the same in every pass
  u32 G = 2; while (G < size) G <<= 1;
  if (mine) atomicAdd(&s_slot[lane % G], mine);
  if (bad) atomicOr((unsigned long long*)&a.counters[CNT_STATUS], (unsigned long long)bad);
  __syncthreads();
  if (tid == 0) d.nflag[f] = S.flags.n;
  // the staged rows: every wavefront takes 64 of them
  if (size >= 4) {
    // a wavefront-uniform pointer that steps from column to column and a 32-bit offset per lane
    const u64 stride = a.seg_cap * 8u;
    for (u32 k = wave * CCLD_WAVE + lane; k < D.K; k += GRID_THREADS) {
      const StageRow at(k, size);
      u32 w[ROW_WORDS];
#pragma unroll
      for (u32 i = 0; i < ROW_WORDS; ++i) w[i] = *at.word(S.row, i);
      if (w[15] == ROW_NOT_STAGED) continue;
      const u32 srow = D.srow0 + k;
      const u32 n = w[15] & 255u, op = (w[1] >> 12) & 15u;
      const u64 nb = (u64)w[14] | ((u64)(w[1] >> 27) << 32);
      const bool complete = n == size, incons = w[15] >> 8 != 0, barrier = op == CCLD_OP_ALLREDUCE && nb < (u64)a.barrier_bytes;
      const bool usable = complete && !incons && !barrier;
      const u32 state = (complete ? CCLD_SEG_COMPLETE : 0) | (!incons ? CCLD_SEG_CONSISTENT : 0) | (barrier ? CCLD_SEG_BARRIER : 0) |
                        (usable ? CCLD_SEG_USABLE : 0);
      a.gcode[srow] = (uint16_t)seg_group_code(usable, op, nb);
      a.range_c[srow] = usable ? (i64)(w[11] - w[10]) : 0;
      if (srow >= a.seg_cap) continue;
      const i64 ref = wref + t44_diff((u64)w[0] | ((u64)(w[1] & 0xFFFu) << 32), (u64)wref);
      char* p = reinterpret_cast<char*>(a.seg + D.srow0);
      const u32 off = k * 8u;
      auto put = [&](i64 v) { *reinterpret_cast<i64*>(p + off) = v; p += stride; };
      put((i64)D.comm); put((i64)(D.seq0 + k)); put((i64)n); put(0); put((i64)state); put((i64)op); put((i64)nb);
      put(ref + (i32)w[2]); put(ref + (i32)w[3]); put(ref + (i32)w[4]); put((i64)w[5]);
      put(ref + (i32)w[6]); put(ref + (i32)w[7]); put(ref + (i32)w[8]); put((i64)w[9]);
      put((i64)w[10]); put((i64)w[11]); put((i64)w[12]); put((i64)w[13]);
      put(T_INFLIGHT); put((i64)(rec0 + S.pre[k]));
    }
  }
  // records per rank
  unsigned long long* nrec = (unsigned long long*)(blame + (u64)CCLD_BLM_N_RECORDS * n_ranks);
  if (tid < size && s_slot[tid]) atomicAdd(&nrec[a.members_sorted[a.member_off[D.comm] + tid]], (unsigned long long)s_slot[tid]);
  grid_order_flags<GRID_THREADS>(a, D, rec0, S.flags, S.wave, blame, n_ranks);
}

// ---- fine buckets of communicators of 65 to GRID_B members ------------------------------------------------
// Registers of 64 E members, as in k_seg_multi, on 32-bit offsets from the first record where they fit.
__device__ __forceinline__ i32 lane_xor63(i32 v) { return (i32)xor_lane_u32<63>((u32)v); }
template <int E>
__device__ __forceinline__ void sort_multi32(i32 (&v)[E], u32 lane) {
#pragma unroll
  for (int r = 0; r < E; ++r) v[r] = sort_groups32<64>(v[r], lane);
#pragma unroll
  for (int kb = 2; kb <= E; kb <<= 1) {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      if ((r & (kb >> 1)) == 0) {
        const int q = r ^ (kb - 1);
        const i32 b = lane_xor63(v[q]), lo = b < v[r] ? b : v[r], hi = b < v[r] ? v[r] : b;
        v[r] = lo; v[q] = lane_xor63(hi);
      }
    }
#pragma unroll
    for (int jb = kb >> 2; jb >= 1; jb >>= 1)
#pragma unroll
      for (int r = 0; r < E; ++r)
        if ((r & jb) == 0) {
          const i32 x = v[r], y = v[r | jb];
          v[r] = y < x ? y : x; v[r | jb] = y < x ? x : y;
        }
#pragma unroll
    for (int r = 0; r < E; ++r) v[r] = merge_groups32<64>(v[r], lane);
  }
}
// sorts a bitonic sequence
template <int E>
__device__ __forceinline__ void merge_multi32(i32 (&v)[E], u32 lane) {
#pragma unroll
  for (int jb = E >> 1; jb >= 1; jb >>= 1)
#pragma unroll
    for (int r = 0; r < E; ++r)
      if ((r & jb) == 0) {
        const i32 x = v[r], y = v[r | jb];
        v[r] = y < x ? y : x; v[r | jb] = y < x ? x : y;
      }
#pragma unroll
  for (int r = 0; r < E; ++r) v[r] = merge_groups32<64>(v[r], lane);
}
// What a collective of a long communicator leaves for its table row; the times are absolute.
struct LongRow {
  i64 stat[2][4];            // arrival, completion: min, lower median, max, MAD
  i64 imin, dmin, dmax;
  u64 bytes;
  u32 n, ninfl, state, op, rmin, rmax;
};
// Lower median of |value - median| over the nd smallest values of a sorted sequence at(0), at(1), ... (nd >= 1): see
// mad_of_sorted
template <class At>
__device__ __forceinline__ i64 mad_of(At at, u32 nd) {
  const u32 km = (nd - 1) / 2;
  const i64 med = at(km);
  const u32 nl = km + 1, nr = nd - nl, d = km + 1;
  auto under = [&](u32 j) { return med - at(km - j); };
  auto above = [&](u32 j) { return at(km + 1 + j) - med; };
  u32 lo = d > nr ? d - nr : 0u, hi = d < nl ? d : nl;
  while (lo < hi) {
    const u32 mid = (lo + hi) >> 1;
    if (under(mid) <= above(d - 1 - mid)) lo = mid + 1; else hi = mid;
  }
  i64 r = lo > 0 ? under(lo - 1) : INT64_MIN;
  if (d - lo > 0) { const i64 u = above(d - lo - 1); r = u > r ? u : r; }
  return r;
}
// most rounds of a fine bucket of such a communicator
constexpr u32 LONG_ROUNDS = GRID_B / (SEG_WAVE_MAX + 1);
using LongShared = GridShared<LONG_ROUNDS>;

// One wavefront, one collective of up to 64 E members, on 32-bit offsets from its first record's arrival.  False, and nothing
// done, if some time does not fit them.
template <int E>
__device__ __forceinline__ bool long_wave32(const SegArgs& a, const GridArgs& d, const FineDesc& D, u32 rec0, i64 wref,
                                            LongShared& S, u32 (&mine)[E], LongRow* out, u32 k, u32 lane) {
  constexpr u32 LIM = 1u << 30;
  const u32 size = D.size;
  u64 pm[E], dm[E];                 // the records present, and those of finished operations
  u32 n = 0, first_slot = 0;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const u32 slot = r * CCLD_WAVE + lane, cell = k * size + (slot < size ? slot : 0u);
    pm[r] = ballot64(slot < size && ((S.pres[cell >> 5] >> (cell & 31)) & 1u));
    if (n == 0 && pm[r]) first_slot = r * CCLD_WAVE + (u32)__builtin_ctzll(pm[r]);
    n += (u32)__popcll(pm[r]);
  }
  const uint4 lead = S.row[k * size + first_slot];
  i32 er[E];
  u32 z[E], nd = 0;
  bool wide = false, inc = false;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const u32 slot = r * CCLD_WAVE + lane, cell = k * size + (slot < size ? slot : 0u);
    const uint4 v = S.row[cell];
    const bool valid = (pm[r] >> lane) & 1u;
    const u64 diff = (((u64)v.y << 32) | v.x) - (((u64)lead.y << 32) | lead.x);
    er[r] = (i32)(u32)diff; z[r] = v.z;
    const bool done = valid && v.z != ROW_INFLIGHT;
    wide |= (valid && ((((u32)(diff >> 32) ^ (u32)(er[r] >> 31)) & 0xFFFu) != 0 || (u32)er[r] + LIM >= 2 * LIM)) ||
            (done && (v.z >= LIM || (i32)((u32)er[r] + v.z) >= (i32)LIM));
    inc |= valid && (v.w != lead.w || ((v.y ^ lead.y) & ROW_SAME_MASK));
    dm[r] = ballot64(done);
    nd += (u32)__popcll(dm[r]);
  }
  if (ballot64(wide)) return false;
  const bool incons = ballot64(inc) != 0;
  const u32 ninfl = n - nd, kl = nd ? nd - 1 : 0, km = kl / 2;
  const i64 ref = wref + t44_diff(row_t44(lead), (u64)wref);
  // T_min / T_max with the first slot, i.e. the smallest rank, that attains them
  u32 dmin = ~0u, dmax = 0, rmin = CCLD_WAVE * E, rmax = CCLD_WAVE * E;
  i32 imin = 0x7FFFFFFF;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const bool done = (dm[r] >> lane) & 1u, valid = (pm[r] >> lane) & 1u;
    mine[r] += valid ? 1u : 0u;
    if (done) { dmin = z[r] < dmin ? z[r] : dmin; dmax = z[r] > dmax ? z[r] : dmax; }
    else if (valid) imin = er[r] < imin ? er[r] : imin;
  }
  dmin = reduce_u32<64, false>(dmin); dmax = reduce_u32<64, true>(dmax);
#pragma unroll
  for (int r = E - 1; r >= 0; --r) {
    const u64 lo = ballot64(z[r] == dmin) & dm[r], hi = ballot64(z[r] == dmax) & dm[r];
    if (lo) rmin = r * CCLD_WAVE + (u32)__builtin_ctzll(lo);
    if (hi) rmax = r * CCLD_WAVE + (u32)__builtin_ctzll(hi);
  }
  i32 st[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
  for (int w = 0; w < 2; ++w) {                  // 0 arrival, 1 completion
    if (nd == 0) break;
    i32 v[E];
#pragma unroll
    for (int r = 0; r < E; ++r) v[r] = (dm[r] >> lane) & 1u ? (w ? (i32)((u32)er[r] + z[r]) : er[r]) : REL_NONE;
    sort_multi32<E>(v, lane);
    auto kth = [&](u32 q) -> i32 {               // q is the same in every lane
      i32 sel = v[0];
#pragma unroll
      for (int r = 1; r < E; ++r) if ((q >> 6) == (u32)r) sel = v[r];
      return __builtin_amdgcn_readlane(sel, (int)(q & 63));
    };
    const i32 med = kth(km);
    st[w][0] = kth(0); st[w][1] = med; st[w][2] = kth(kl);
    // deviations of the sorted offsets: one merge sorts them (see grid_batches)
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const i32 t = (i32)((u32)v[r] - (u32)med), u = (i32)(0u - (u32)t);
      v[r] = r * CCLD_WAVE + lane < nd ? (t > u ? t : u) : REL_NONE;
    }
    merge_multi32<E>(v, lane);
    st[w][3] = kth(km);
  }
  const u64 hb = row_bytes(lead);
  const u32 hop = row_op(lead);
  const bool complete = n == size && ninfl == 0;
  const bool barrier = hop == CCLD_OP_ALLREDUCE && hb < (u64)a.barrier_bytes;
  const bool usable = complete && !incons && !barrier;
  if (ninfl) imin = (i32)(reduce_u32<64, false>((u32)imin ^ 0x80000000u) ^ 0x80000000u);
  if (lane == 0) {
    const u32* ms = a.members_sorted + a.member_off[D.comm];
    LongRow& R = out[k];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      R.stat[w][0] = ref + st[w][0]; R.stat[w][1] = ref + st[w][1]; R.stat[w][2] = ref + st[w][2]; R.stat[w][3] = st[w][3];
    }
    R.imin = ninfl ? ref + imin : T_INFLIGHT;
    R.dmin = nd ? (i64)dmin : INT64_MAX; R.dmax = nd ? (i64)dmax : INT64_MIN;
    R.rmin = nd ? ms[rmin] : 0xFFFFFFFFu; R.rmax = nd ? ms[rmax] : 0xFFFFFFFFu;
    R.bytes = hb; R.n = n; R.ninfl = ninfl; R.op = hop;
    R.state = (complete ? CCLD_SEG_COMPLETE : 0) | (!incons ? CCLD_SEG_CONSISTENT : 0) | (barrier ? CCLD_SEG_BARRIER : 0) |
              (usable ? CCLD_SEG_USABLE : 0);
  }
  const bool per_record = a.rec_flag || a.lag_e || a.lag_x || a.perm;
  // a lag within the floor is never late: most collectives end here (with rare arguments read where they are used, ten batches of 2M
  // records with collectives of 128 members 99 -> 91 us, 1.1M records with collectives of 390 members 30.4 -> 28.8)
  const i32 floor32 = a.lag_floor > 0x7FFFFFFF ? 0x7FFFFFFF : a.lag_floor < -0x7FFFFFFF ? -0x7FFFFFFF : (i32)a.lag_floor;
  bool above = false;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const i32 le = (i32)((u32)er[r] - (u32)st[0][1]), lx = (i32)((u32)er[r] + z[r] - (u32)st[1][1]);
    above |= ((pm[r] >> lane) & 1u) && (le > floor32 || lx > floor32);
  }
  if (!per_record && !(usable && ballot64(above))) return true;
  const SegArgs& A = args_again();
  u32 before = rec0 + S.pre[k];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const bool valid = (pm[r] >> lane) & 1u;
    i32 le = 0, lx = 0;
    u32 f = 0;
    if (usable) {
      le = er[r] - st[0][1]; lx = (i32)((u32)er[r] + z[r]) - st[1][1];
      if (is_late32(le, A.lag_floor, A.kmad_num, A.kmad_den, st[0][3])) f |= CCLD_FLAG_LATE_ENTER;
      if (is_late32(lx, A.lag_floor, A.kmad_num, A.kmad_den, st[1][3])) f |= CCLD_FLAG_LATE_EXIT;
    }
    if (valid && (f || per_record)) {
      const u32 cell = k * size + r * CCLD_WAVE + lane, j = before + mbcnt64(pm[r]);
      if (A.perm) A.perm[j] = grid_arrival(A, grid_again(), D.cell0 + ((S.row[cell].y >> ROW_CELL_SHIFT) & ROW_CELL_MASK));
      grid_put_record(A, j, cell, rec0, &S.flags, f, (i64)le, (i64)lx);
    }
    before += (u32)__popcll(pm[r]);
  }
  return true;
}
// The same with times of any spread.
template <int E>
__device__ __forceinline__ void long_wave(const SegArgs& a, const GridArgs& d, const FineDesc& D, u32 rec0, i64 wref,
                                          LongShared& S, u32 (&mine)[E], LongRow* out, u32 k, u32 lane) {
  const u32 size = D.size, *ms = a.members_sorted + a.member_off[D.comm];
  i64 e[E], x[E];
  u32 n = 0, ninfl = 0, before[E];
  bool valid[E], inc = false;
  i64 imin = T_INFLIGHT, dmin = INT64_MAX, dmax = INT64_MIN;
  u32 rmin = 0xFFFFFFFFu, rmax = 0xFFFFFFFFu, hop = 0;
  u64 hb = 0;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const u32 slot = r * CCLD_WAVE + lane, cell = k * size + (slot < size ? slot : 0u);
    valid[r] = slot < size && ((S.pres[cell >> 5] >> (cell & 31)) & 1u);
    const u64 pm = ballot64(valid[r]);
    before[r] = n + mbcnt64(pm);
    const uint4 v = S.row[cell];
    const Rec rec = valid[r] ? unpack_row(v, wref, a.win.wide) : Rec{0, T_INFLIGHT, 0, 0};
    e[r] = rec.t_enter; x[r] = rec.t_exit;
    if (n == 0 && pm) {        // the first record of the collective
      const int fl = (int)__builtin_ctzll(pm);
      hb = shfl_u64(rec.bytes, fl); hop = __shfl(rec.op, fl, CCLD_WAVE);
    }
    n += (u32)__popcll(pm);
    inc |= valid[r] && (rec.bytes != hb || rec.op != hop);
    const bool done = valid[r] && x[r] != T_INFLIGHT;
    ninfl += (u32)__popcll(ballot64(valid[r] && !done));
    if (valid[r]) {
      ++mine[r];
      if (a.perm) a.perm[rec0 + S.pre[k] + before[r]] = grid_arrival(a, d, D.cell0 + ((v.y >> ROW_CELL_SHIFT) & ROW_CELL_MASK));
      if (!done) {
        imin = e[r] < imin ? e[r] : imin;
      } else {
        const i64 du = x[r] - e[r];
        const u32 rank = ms[slot];
        if (du < dmin || (du == dmin && rank < rmin)) { dmin = du; rmin = rank; }
        if (du > dmax || (du == dmax && rank < rmax)) { dmax = du; rmax = rank; }
      }
    }
  }
  const bool incons = ballot64(inc) != 0;
  if (ninfl) imin = reduce_min<64>(imin);
  reduce_dur<64, false>(dmin, rmin);
  reduce_dur<64, true>(dmax, rmax);
  const u32 nd = n - ninfl, km = nd ? (nd - 1) / 2 : 0, kl = nd ? nd - 1 : 0;
  i64 st_min[2] = {0, 0}, st_med[2] = {0, 0}, st_max[2] = {0, 0}, st_mad[2] = {0, 0};
#pragma unroll 1
  for (int w = 0; w < 2; ++w) {                  // 0 arrival, 1 completion
    if (nd == 0) break;
    i64 v[E];
#pragma unroll
    for (int r = 0; r < E; ++r) v[r] = x[r] != T_INFLIGHT ? (w ? x[r] : e[r]) : T_INFLIGHT;
    sort_multi<E>(v, lane);
    st_min[w] = kth_multi<E>(v, 0); st_med[w] = kth_multi<E>(v, km); st_max[w] = kth_multi<E>(v, kl);
    st_mad[w] = mad_of_sorted<E>(v, nd, km);
  }
  const bool complete = n == size && ninfl == 0;
  const bool barrier = hop == CCLD_OP_ALLREDUCE && hb < (u64)a.barrier_bytes;
  const bool usable = complete && !incons && !barrier;
  if (lane == 0) {
    LongRow& R = out[k];
#pragma unroll
    for (int w = 0; w < 2; ++w) { R.stat[w][0] = st_min[w]; R.stat[w][1] = st_med[w]; R.stat[w][2] = st_max[w]; R.stat[w][3] = st_mad[w]; }
    R.imin = imin; R.dmin = dmin; R.dmax = dmax; R.bytes = hb; R.n = n; R.ninfl = ninfl; R.op = hop; R.rmin = rmin; R.rmax = rmax;
    R.state = (complete ? CCLD_SEG_COMPLETE : 0) | (!incons ? CCLD_SEG_CONSISTENT : 0) | (barrier ? CCLD_SEG_BARRIER : 0) |
              (usable ? CCLD_SEG_USABLE : 0);
  }
#pragma unroll
  for (int r = 0; r < E; ++r) {
    if (!valid[r]) continue;
    i64 le = 0, lx = 0;
    u32 f = 0;
    if (usable) {
      le = e[r] - st_med[0]; lx = x[r] - st_med[1];
      if (is_late(le, a.lag_floor, a.kmad_num, a.kmad_den, st_mad[0])) f |= CCLD_FLAG_LATE_ENTER;
      if (is_late(lx, a.lag_floor, a.kmad_num, a.kmad_den, st_mad[1])) f |= CCLD_FLAG_LATE_EXIT;
    }
    grid_put_record(a, rec0 + S.pre[k] + before[r], k * size + r * CCLD_WAVE + lane, rec0, &S.flags, f, le, lx);
  }
}

template <int E>
__device__ __forceinline__ void long_rounds(const SegArgs& a, const GridArgs& d, const FineDesc& D, u32 rec0, i64 wref, LongShared& S,
                                            u32* s_slot, LongRow* out, u32 lane, u32 wave, u32 n_waves) {
  u32 mine[E];
#pragma unroll
  for (int r = 0; r < E; ++r) mine[r] = 0;
  for (u32 k = wave; k < D.K; k += n_waves)
    if (!long_wave32<E>(a, d, D, rec0, wref, S, mine, out, k, lane)) long_wave<E>(args_again(), grid_again(), D, rec0, wref, S, mine, out, k, lane);
#pragma unroll
  for (int r = 0; r < E; ++r) if (mine[r]) atomicAdd(&s_slot[r * CCLD_WAVE + lane], mine[r]);
}

// A workgroup takes the fine buckets on the list in turn.  E: those whose collectives go to a wavefront each, E members per
// lane (up to 64 E and more than half as many); E = 0: the larger ones (at most three in a bucket), taken by the whole
// workgroup one after the other: their times are sorted in LDS, the median of the deviations is selected from the sorted
// sequence.  A kernel each, because the sort's LDS would leave the wavefronts half of their occupancy (four workgroups per
// compute unit without it), and the registers of eight members per lane those with two.  Bound by the chain of one collective
// (two sorts, two merges of the deviations; with a binary search for their median in place of the merge a 16,384-rank stream took
// 714 instead of 702 us), so buckets of eight members per lane, of at most seven collectives, have eight wavefronts: 1.1M records
// with collectives of 390 members 211 -> 189 us.
template <int E, int THREADS>
__global__ __launch_bounds__(THREADS, E == 2 || E == 4 ? 4 : 2) void k_grid_long(const SegArgs a, const GridArgs d, i64* __restrict__ blame, u32 n_ranks) {
  constexpr bool WAVES = E > 0;
  constexpr u32 MEMBERS = WAVES ? E * CCLD_WAVE : GRID_B, ABOVE = E == 0 ? SEG_MULTI_MAX : E * CCLD_WAVE / 2;
  __shared__ LongShared S;
  __shared__ i64 s_v[WAVES ? 1 : GRID_B];      // the larger collectives' sort
  __shared__ u32 s_slot[MEMBERS];
  __shared__ LongRow s_out[LONG_ROUNDS];
  __shared__ TeamAcc s_acc;
  __shared__ u32 s_first;
  constexpr u32 NW = THREADS / CCLD_WAVE, U = GRID_B / THREADS;
  const u32 tid = threadIdx.x, wave = tid / CCLD_WAVE;
  if (d.hdr->feasible == 0) return;
  const u32 n_long = d.hdr->n_long;
  const bool scanned = !d.self_sum;
  const i64 wref = d.hdr->ref;
  for (u32 ent = blockIdx.x; ent < n_long; ent += gridDim.x) {
    const u32 f = d.long_list[ent];
    const FineDesc D = d.desc[f];
    const u32 fill = d.fill[f], size = D.size, K = D.K;
    if (size <= ABOVE || size > MEMBERS) continue;
    const RecordsBefore<true> before = RecordsBefore<true>::load<THREADS>(d, f, scanned);
    for (u32 i = tid; i < size; i += THREADS) s_slot[i] = 0;
    const u64 bad = grid_place<THREADS>(d, D, fill, before, S);
    const u32 rec0 = (u32)__builtin_amdgcn_readfirstlane((int)S.rec0);
    if (tid == 0) d.rec0[f] = rec0;
    if (bad) atomicOr((unsigned long long*)&a.counters[CNT_STATUS], (unsigned long long)bad);
    // the lane's number, not known to be the same for every bucket: what the sorts make of it is not kept over the placing of the next
    // rows, where it took 28 registers too many (with the arguments read again, ten batches of 2M records with collectives of 128
    // members 84 -> 70 us, 1.1M records with collectives of 390 members 28.3 -> 27.5; eleven registers still spill with two members per lane)
    u32 lane = lane_id();
    asm("" : "+v"(lane));
    if constexpr (WAVES) {
      long_rounds<E>(a, d, D, rec0, wref, S, s_slot, s_out, lane, wave, NW);
      __syncthreads();
    } else {
      for (u32 k = 0; k < K; ++k) {
        if (tid == 0) {
          s_acc.imin = (unsigned long long)T_INFLIGHT; s_acc.dmin = INT64_MAX; s_acc.dmax = INT64_MIN;
          s_acc.ninfl = 0; s_acc.incons = 0; s_acc.rmin = 0xFFFFFFFFu; s_acc.rmax = 0xFFFFFFFFu;
          s_first = 0xFFFFFFFFu;
        }
        __syncthreads();
        // consecutive slots per thread, so that a record's place among the present ones is one scan away
        Rec rec[U];
        bool valid[U];
        u32 here = 0, first_slot = 0xFFFFFFFFu;
#pragma unroll
        for (u32 u = 0; u < U; ++u) {
          const u32 slot = tid * U + u, cell = k * size + slot;
          valid[u] = slot < size && ((S.pres[cell >> 5] >> (cell & 31)) & 1u);
          rec[u] = valid[u] ? unpack_row(S.row[cell], wref, a.win.wide) : Rec{0, T_INFLIGHT, 0, 0};
          if (valid[u]) { ++here; if (first_slot == 0xFFFFFFFFu) first_slot = slot; }
        }
        if (here) atomicMin(&s_first, first_slot);
        u32 n;
        const u32 before = block_exclusive_sum<THREADS>(here, S.wave, &n);
        const Rec h = n ? unpack_row(S.row[k * size + s_first], wref, a.win.wide) : Rec{0, T_INFLIGHT, 0, 0};
        {
          u32 ni = 0, rmin = 0xFFFFFFFFu, rmax = 0xFFFFFFFFu;
          bool inc = false;
          i64 imin = T_INFLIGHT, dmin = INT64_MAX, dmax = INT64_MIN;
#pragma unroll
          for (u32 u = 0; u < U; ++u) {
            if (!valid[u]) continue;
            inc |= rec[u].op != h.op || rec[u].bytes != h.bytes;
            s_slot[tid * U + u] += 1;
            if (rec[u].t_exit == T_INFLIGHT) {
              ++ni; imin = rec[u].t_enter < imin ? rec[u].t_enter : imin;
            } else {
              const i64 du = rec[u].t_exit - rec[u].t_enter;      // slots ascend with the ranks: ties keep the first
              if (du < dmin) { dmin = du; rmin = tid * U + u; }
              if (du > dmax) { dmax = du; rmax = tid * U + u; }
            }
          }
          if (ni) { atomicAdd(&s_acc.ninfl, ni); atomicMin(&s_acc.imin, (unsigned long long)imin); }
          if (inc) atomicOr(&s_acc.incons, 1u);
          if (rmin != 0xFFFFFFFFu) { atomicMin(&s_acc.dmin, (long long)dmin); atomicMax(&s_acc.dmax, (long long)dmax); }
          __syncthreads();
          if (rmin != 0xFFFFFFFFu && dmin == (i64)s_acc.dmin) atomicMin(&s_acc.rmin, rmin);
          if (rmax != 0xFFFFFFFFu && dmax == (i64)s_acc.dmax) atomicMin(&s_acc.rmax, rmax);
        }
        const u32 ninfl = s_acc.ninfl, nd = n - ninfl, km = nd ? (nd - 1) / 2 : 0, kl = nd ? nd - 1 : 0;
        u32 P = 2;
        while (P < size) P <<= 1;
        i64 stat[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
        for (int w = 0; w < 2; ++w) {
          if (nd == 0) break;                          // uniform
#pragma unroll
          for (u32 u = 0; u < U; ++u) {
            const u32 i = tid * U + u;
            if (i < P) s_v[i] = valid[u] && rec[u].t_exit != T_INFLIGHT ? (w ? rec[u].t_exit : rec[u].t_enter) : T_INFLIGHT;
          }
          __syncthreads();
          team_sort<THREADS>(s_v, P, tid);
          stat[w][0] = s_v[0]; stat[w][1] = s_v[km]; stat[w][2] = s_v[kl];
          stat[w][3] = mad_of([&](u32 i) -> i64 { return s_v[i]; }, nd);
          __syncthreads();
        }
        const bool complete = n == size && ninfl == 0;
        const bool consistent = s_acc.incons == 0;
        const bool barrier = h.op == CCLD_OP_ALLREDUCE && h.bytes < (u64)a.barrier_bytes;
        const bool usable = complete && consistent && !barrier;
        if (tid == 0) {
          const u32* ms = a.members_sorted + a.member_off[D.comm];
          LongRow& R = s_out[k];
          for (int w = 0; w < 2; ++w) for (int q = 0; q < 4; ++q) R.stat[w][q] = stat[w][q];
          R.imin = (i64)s_acc.imin; R.dmin = s_acc.dmin; R.dmax = s_acc.dmax; R.bytes = h.bytes; R.n = n; R.ninfl = ninfl; R.op = h.op;
          R.rmin = nd ? ms[s_acc.rmin] : CCLD_NO_RANK; R.rmax = nd ? ms[s_acc.rmax] : CCLD_NO_RANK;
          R.state = (complete ? CCLD_SEG_COMPLETE : 0) | (consistent ? CCLD_SEG_CONSISTENT : 0) | (barrier ? CCLD_SEG_BARRIER : 0) |
                    (usable ? CCLD_SEG_USABLE : 0);
        }
        u32 j = rec0 + S.pre[k] + before;
#pragma unroll
        for (u32 u = 0; u < U; ++u) {
          if (!valid[u]) continue;
          i64 le = 0, lx = 0;
          u32 fl = 0;
          if (usable) {
            le = rec[u].t_enter - stat[0][1]; lx = rec[u].t_exit - stat[1][1];
            if (is_late(le, a.lag_floor, a.kmad_num, a.kmad_den, stat[0][3])) fl |= CCLD_FLAG_LATE_ENTER;
            if (is_late(lx, a.lag_floor, a.kmad_num, a.kmad_den, stat[1][3])) fl |= CCLD_FLAG_LATE_EXIT;
          }
          const u32 cell = k * size + tid * U + u;
          if (a.perm) a.perm[j] = grid_arrival(a, d, D.cell0 + ((S.row[cell].y >> ROW_CELL_SHIFT) & ROW_CELL_MASK));
          grid_put_record(a, j, cell, rec0, &S.flags, fl, le, lx);
          ++j;
        }
        __syncthreads();     // the accumulator and the sort array are reused by the next round
      }
    }
    __syncthreads();
    const SegArgs& A = args_again();
    if (tid == 0) grid_again().nflag[f] = S.flags.n;
    grid_order_flags<THREADS>(A, D, rec0, S.flags, S.wave, blame, n_ranks);
    // the table rows: a lane per round, a column at a time
    for (u32 col = wave; col < STAGE_COLS; col += NW) {
      const u32 k = lane;
      if (k >= K) continue;
      const LongRow& R = s_out[k];
      const u32 srow = D.srow0 + k;
      const bool none = R.n == R.ninfl, usable = (R.state & CCLD_SEG_USABLE) != 0;
      const bool barrier = (R.state & CCLD_SEG_BARRIER) != 0;
      if (col == (u32)CCLD_SEG_NCOL) { A.gcode[srow] = (uint16_t)seg_group_code(usable, R.op, R.bytes); continue; }
      if (col == (u32)CCLD_SEG_NCOL + 1) { A.range_c[srow] = usable ? R.dmax - R.dmin : 0; seg_count_alert(A, srow, R.ninfl, barrier, R.imin); continue; }
      i64 v = 0;
      switch (col) {
        case CCLD_SEG_COMM: v = (i64)D.comm; break;
        case CCLD_SEG_SEQ: v = (i64)(D.seq0 + k); break;
        case CCLD_SEG_N: v = (i64)R.n; break;
        case CCLD_SEG_INFLIGHT: v = (i64)R.ninfl; break;
        case CCLD_SEG_STATE: v = (i64)R.state; break;
        case CCLD_SEG_OP: v = (i64)R.op; break;
        case CCLD_SEG_BYTES: v = (i64)R.bytes; break;
        case CCLD_SEG_DUR_MIN: v = none ? 0 : R.dmin; break;
        case CCLD_SEG_DUR_MAX: v = none ? 0 : R.dmax; break;
        case CCLD_SEG_ARGMIN_RANK: v = none ? (i64)CCLD_NO_RANK : (i64)R.rmin; break;
        case CCLD_SEG_ARGMAX_RANK: v = none ? (i64)CCLD_NO_RANK : (i64)R.rmax; break;
        case CCLD_SEG_INFLIGHT_ENTER_MIN: v = R.imin; break;
        case CCLD_SEG_FIRST: v = (i64)(rec0 + S.pre[k]); break;
        default: v = none ? 0 : R.stat[(col - CCLD_SEG_ENTER_MIN) >> 2][(col - CCLD_SEG_ENTER_MIN) & 3]; break;
      }
      seg_put(A, (int)col, srow, v);
    }
    unsigned long long* nrec = (unsigned long long*)(blame + (u64)CCLD_BLM_N_RECORDS * n_ranks);
    for (u32 i = tid; i < size; i += THREADS)
      if (s_slot[i]) atomicAdd(&nrec[A.members_sorted[A.member_off[D.comm] + i]], (unsigned long long)s_slot[i]);
    __syncthreads();     // LDS is reused by the next bucket
  }
}
template <class Kernel>
constexpr bool reads_args_again = std::is_same_v<Kernel, void (*)(SegArgs, GridArgs, i64*, u32)>;
static_assert(reads_args_again<decltype(&k_grid_stats<256, false>)> && reads_args_again<decltype(&k_grid_long<8, 512>)>,
              "args_again and grid_again take the arguments by their places");
static_assert(LONG_ROUNDS <= CCLD_WAVE, "a lane per round");
static_assert(CCLD_SEG_ENTER_MIN == 7 && CCLD_SEG_EXIT_MIN == 11 && CCLD_SEG_DUR_MIN == 15, "four columns of arrival, four of completion");

constexpr size_t LARGE_LDS = sizeof(int64_t) * SEG_LARGE_MAX;
hipError_t allow_lds_segments() { return allow_lds(reinterpret_cast<const void*>(&k_seg_large), LARGE_LDS); }

// the collectives on the list (more than 64 records)
static void launch_seg_listed(hipStream_t st, const SegArgs& a) {
  // a collective has at most as many records as its communicator has members (a longer one holds a
  // duplicate, which ends the analysis with an error): size classes that cannot occur are not launched
  const uint32_t m = a.max_size;
  if (m <= (uint32_t)SEG_WAVE_MAX) return;
  hipLaunchKernelGGL(k_seg_lengths, dim3(1024), dim3(SEG_THREADS), 0, st, a);
  hipLaunchKernelGGL(k_seg_multi<2>, dim3(2048), dim3(SEG_THREADS), 0, st, a);
  if (m > 128) hipLaunchKernelGGL(k_seg_multi<4>, dim3(2048), dim3(SEG_THREADS), 0, st, a);
  if (m > 256) hipLaunchKernelGGL(k_seg_multi<8>, dim3(2048), dim3(SEG_THREADS), 0, st, a);
  if (m > (uint32_t)SEG_MULTI_MAX) hipLaunchKernelGGL(k_seg_team, dim3(1024), dim3(SEG_THREADS), 0, st, a);
  if (m > (uint32_t)SEG_TEAM_MAX) hipLaunchKernelGGL(k_seg_large, dim3(512), dim3(LARGE_THREADS), LARGE_LDS, st, a);
  if (m > (uint32_t)SEG_LARGE_MAX) hipLaunchKernelGGL(k_seg_big, dim3(2048), dim3(SEG_THREADS), 0, st, a);
  if (m > (uint32_t)SEG_MULTI_MAX) hipLaunchKernelGGL(k_seg_group_listed, dim3(256), dim3(256), 0, st, a);
}

void launch_grid_stats(hipStream_t st, const SegArgs& a, const GridArgs& d, uint32_t fine_bound, int64_t* blame, uint32_t n_ranks) {
  // Where there are no more fine buckets than compute units, or than two to each, a workgroup has sixteen or eight wavefronts
  // instead of four: what takes the time then is one bucket's passes one after the other (16 ranks, 8 buckets: a window
  // 70.9 -> 62.8 us).  More buckets overlap each other with four workgroups to a compute unit.
  const dim3 g(fine_bound);
  if (d.self_sum && d.likely <= 256) hipLaunchKernelGGL((k_grid_stats<1024, true>), g, dim3(1024), 0, st, a, d, blame, n_ranks);
  else if (d.self_sum) hipLaunchKernelGGL((k_grid_stats<512, true>), g, dim3(512), 0, st, a, d, blame, n_ranks);
  else hipLaunchKernelGGL((k_grid_stats<256, false>), g, dim3(256), 0, st, a, d, blame, n_ranks);
  // as many workgroups as are resident at once, which take the listed buckets in turn
  const bool few = d.likely <= 256;
  if (a.long_classes & 1) {
    if (few) hipLaunchKernelGGL((k_grid_long<2, 1024>), dim3(256), dim3(1024), 0, st, a, d, blame, n_ranks);
    else hipLaunchKernelGGL((k_grid_long<2, 256>), dim3(1024), dim3(256), 0, st, a, d, blame, n_ranks);
  }
  if (a.long_classes & 2) {
    if (few) hipLaunchKernelGGL((k_grid_long<4, 1024>), dim3(256), dim3(1024), 0, st, a, d, blame, n_ranks);
    else hipLaunchKernelGGL((k_grid_long<4, 256>), dim3(1024), dim3(256), 0, st, a, d, blame, n_ranks);
  }
  if (a.long_classes & 4) hipLaunchKernelGGL((k_grid_long<8, 512>), dim3(256), dim3(512), 0, st, a, d, blame, n_ranks);
  if (a.long_classes & 8) hipLaunchKernelGGL((k_grid_long<0, 256>), dim3(512), dim3(256), 0, st, a, d, blame, n_ranks);
}

void launch_seg_analyze(hipStream_t st, const SegArgs& a) {
  if (a.n == 0) return;
  hipLaunchKernelGGL(k_seg_wave, dim3((a.n + SEG_TILE - 1) / SEG_TILE), dim3(SEG_THREADS), 0, st, a);
  launch_seg_listed(st, a);
}

}  // namespace ccld
