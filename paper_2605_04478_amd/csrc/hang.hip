// Hang location and progress rates from progress-counter snapshots for gfx950, and Probing Frames.  Rows arrive in any
// order; they are regrouped by region (a range of member slots) and a workgroup per region works its rows off in LDS.  One
// workgroup per communicator then applies the hang decision tree, builds the ring / tree wait-for edges and follows
// them to the roots; victims are filtered across communicators at the end.
#include <algorithm>
#include <cstring>
#include <mutex>

#include "ccld_internal.h"
#include "device_utils.h"
#include "report.h"
#include "window_kernels.h"

using namespace ccld;

namespace ccld {

struct HangArgs {
  // rows
  const u32 *snap, *rank, *comm, *channel;
  const u64* seq_posted;
  const u32 *sent, *recv;
  u64 n_rows;
  u32 n_snap, n_ch;
  int mb;             // bits of the position field in the packed membership words
  DeviceTopology T;
  u64 n_members;
  // grid
  u64* cell;          // [n_members * n_ch * n_snap][2]
  u32* cnt;           // presence bitmap, one bit per cell
  int exact;          // 1: the bitmap is kept (duplicates and gaps told apart); 0: cells start from an all-ones fill and a
                      //    cell that still holds it is suspect
  ulonglong2* final;  // [n_members * n_ch] state of every (member, channel) in the last snapshot
  u32* mark;          // [n_members][2] 1 + the last snapshot that differs from the last one; 1: not stalled
  // tables
  i64* pair;          // [CCLD_HPAIR_NCOL][n_members]
  i64* hcomm;         // [CCLD_HCOMM_NCOL][n_comms]
  int* wait_slot;
  uint8_t* cand;
  u64* layer_max;
  u64* counters;
  u32 stall_snapshots, fifo_depth;
  u64 n_cell;
  int checked;        // the host has found the rows in order
  int hops_known;     // no communicator is too large for its hops to be found in LDS
  i64* root_key;      // [n_members] rank << cb | communicator of every root
  int cb;             // bits of a communicator
  i64 *out_pair, *out_comm, *out_root;
  u64 pair_cap, comm_cap, root_cap;
  u64 *host, ticket;  // pinned words of the report
  // two-step placement of large grids: rows regrouped by region of 2^rb cells
  ulonglong2* part_pay;   // [n_regions << rb] cell contents
  u32* part_idx;          // [n_regions << rb] cell number inside the region
  u32* part_fill;         // [n_regions] rows received; with `ends`, [2][SPLIT_REGIONS] rows from the front and from the end
  int rb;
  u32 n_regions;
  // hang location of large grids: rows regrouped by region of 2^sb members
  ulonglong2* part_row;   // [n_cell]
  u32* arrivals;
  int leave_clear;        // the pass clears counters and part_fill behind itself
  int sb;
  int ends;               // regions are filled from both ends (contexts; the static array has no room for the second counters)
  int pb;                 // rates: the members of a region are taken 2^pb at a time
  u32 snap_inv;           // ceil(2^32 / n_snap)
};

#define PAIR(a, col, p) (a.pair[(u64)(col) * a.n_members + (p)])
#define HCOMM(a, col, c) (a.hcomm[(u64)(col) * a.T.n_comms + (c)])

// slot of rank r inside communicator c, or -1
__device__ __forceinline__ int slot_of(const DeviceTopology& T, u32 c, u32 r) {
  const u32 off = T.member_off[c], n = T.size[c];
  u32 lo = 0, hi = n;
  while (lo < hi) { const u32 m = (lo + hi) / 2; if (T.members_sorted[off + m] < r) lo = m + 1; else hi = m; }
  if (lo < n && T.members_sorted[off + lo] == r) return (int)T.sorted_slot[off + lo];
  return -1;
}

// Row of the snapshot grid (member index) of rank r in communicator c, or -1.  m: the rank's packed row of
// rank_cell4 when that table exists (words comm << pb | member index), else of rank_memb4 (comm << mb | sorted
// position), else unused.
__device__ __forceinline__ i64 grid_row_of(const HangArgs& a, u32 c, u32 r, const uint4& m) {
  if (r >= a.T.n_ranks) return -1;
  if (a.T.rank_cell4) {
    const int pb = a.T.pb;
    const u32 w = c == (m.x >> pb) ? m.x : c == (m.y >> pb) ? m.y : c == (m.z >> pb) ? m.z : m.w;
    return c == (w >> pb) ? (i64)(w & ((1u << pb) - 1u)) : -1;
  }
  int slot = -1;
  if (a.T.rank_memb4) {
    const u32 mmask = a.mb < 32 ? (1u << a.mb) - 1 : ~0u;
    const u32 w = c == (m.x >> a.mb) ? m.x : c == (m.y >> a.mb) ? m.y : c == (m.z >> a.mb) ? m.z : m.w;
    if (c == (w >> a.mb)) slot = (int)a.T.sorted_slot[a.T.member_off[c] + (w & mmask)];
  } else {
    slot = slot_of(a.T, c, r);
  }
  return slot < 0 ? -1 : (i64)a.T.member_off[c] + slot;
}
__device__ __forceinline__ uint4 grid_row_lookup(const HangArgs& a, u32 r) {
  const uint4* __restrict__ t = reinterpret_cast<const uint4*>(a.T.rank_cell4 ? a.T.rank_cell4 : a.T.rank_memb4);
  return (t && r < a.T.n_ranks) ? t[r] : make_uint4(~0u, ~0u, ~0u, ~0u);
}

// Status of one cell as the per-member passes read it.  With the bitmap: its bit.  Without: a cell that still
// holds the all-ones fill was (almost certainly) never written; the caller then repeats the placement with the
// bitmap, which tells a gap from a duplicate and from a row that really holds that pattern.
__device__ __forceinline__ u64 cell_status(const HangArgs& a, u64 cell, u64 w0, u64 w1) {
  if (a.exact) return ((a.cnt[cell >> 5] >> (cell & 31)) & 1u) ? 0 : (u64)DS_SNAPSHOT_GAP;
  return (w0 == ~0ull && w1 == ~0ull) ? (u64)DS_SUSPECT : 0;
}

// ---- place every row in its cell ------------------------------------------------------------
template <bool EXACT>
__global__ __launch_bounds__(256) void k_hang_place(HangArgs a) {
  constexpr int U = 4;               // rows per thread in flight
  u64 status = 0;
  ulonglong2* __restrict__ cell2 = reinterpret_cast<ulonglong2*>(a.cell);
  const u64 stride = (u64)gridDim.x * 256;
  for (u64 i0 = (u64)blockIdx.x * 256 + threadIdx.x; i0 < a.n_rows; i0 += stride * U) {
    u32 c[U], r[U], ch[U], sn[U], se[U], rv[U];
    u64 sq[U];
    bool on[U];
    // the seven columns are read once: streaming loads
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const u64 i = i0 + stride * u;
      on[u] = i < a.n_rows;
      if (on[u]) {
        c[u] = __builtin_nontemporal_load(a.comm + i); r[u] = __builtin_nontemporal_load(a.rank + i);
        ch[u] = __builtin_nontemporal_load(a.channel + i); sn[u] = __builtin_nontemporal_load(a.snap + i);
        sq[u] = __builtin_nontemporal_load(a.seq_posted + i);
        se[u] = __builtin_nontemporal_load(a.sent + i); rv[u] = __builtin_nontemporal_load(a.recv + i);
      }
    }
    uint4 m[U];
#pragma unroll
    for (int u = 0; u < U; ++u) m[u] = on[u] ? grid_row_lookup(a, r[u]) : make_uint4(~0u, ~0u, ~0u, ~0u);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!on[u]) continue;
      if (c[u] >= a.T.n_comms) { status |= DS_UNKNOWN_COMM; continue; }
      const i64 p = grid_row_of(a, c[u], r[u], m[u]);
      if (p < 0) { status |= DS_NOT_MEMBER; continue; }
      if (ch[u] >= a.n_ch || sn[u] >= a.n_snap) { status |= DS_RANGE; continue; }
      const u64 k = ((u64)p * a.n_ch + ch[u]) * a.n_snap + sn[u];
      cell2[k] = make_ulonglong2(sq[u], (u64)se[u] | ((u64)rv[u] << 32));
      if (EXACT) {
        // presence bitmap (one bit per cell: small enough to stay in cache); a bit already set is a duplicate
        const u32 bit = 1u << (k & 31);
        if (atomicOr(&a.cnt[k >> 5], bit) & bit) status |= DS_DUPLICATE;
      }
    }
  }
  u64 st = status;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) st |= shfl_xor_u64(st, m);
  if (lane_id() == 0 && st) atomicOr((unsigned long long*)&a.counters[CNT_STATUS], (unsigned long long)st);
}

// ---- placement of large grids in two steps ---------------------------------------------------------
// Rows arrive in any order, so placing them directly sends one 16-byte store per row to a random line of a
// grid that is far larger than the L2.  Here the rows are first regrouped by region of 2^rb cells (at most
// PART_REGIONS regions; a round's rows of one region leave as one run), then every region's rows are placed
// by workgroups that run side by side on one XCD, so that the eight cells of a line meet in that XCD's L2
// and reach memory as whole lines.  A region takes at most 2^rb rows; more can only arrive with duplicate
// cells, which the caller's exact pass reports.
constexpr u32 PART_REGIONS = 256;
constexpr int PART_THREADS = 512, PART_U = 4;
constexpr u32 PART_CHUNK = PART_THREADS * PART_U;
constexpr u32 PLACE_ROWS = 256;           // rows per workgroup of the second step (one per thread)

__global__ __launch_bounds__(PART_THREADS) void k_hang_part(HangArgs a, u64 chunk) {
  extern __shared__ ulonglong2 s_pay[];                    // [PART_CHUNK] contents | [PART_CHUNK] cell numbers | [PART_CHUNK] destinations
  u32* s_idx = reinterpret_cast<u32*>(s_pay + PART_CHUNK);
  u32* s_dst = s_idx + PART_CHUNK;
  __shared__ u32 s_cnt[PART_REGIONS], s_pre[PART_REGIONS], s_base[PART_REGIONS], s_scan[PART_THREADS / CCLD_WAVE], s_total;
  const u32 tid = threadIdx.x;
  u64 status = 0;
  const u32 cap = 1u << a.rb, kmask = cap - 1;
  const u64 i_begin = chunk * blockIdx.x;
  const u64 i_end = chunk * (blockIdx.x + 1) < a.n_rows ? chunk * (blockIdx.x + 1) : a.n_rows;
  if (tid < PART_REGIONS) s_cnt[tid] = 0;
  __syncthreads();
  u32 c[PART_U], r[PART_U], ch[PART_U], sn[PART_U], se[PART_U], rv[PART_U];
  u64 sq[PART_U];
  u32 nc[PART_U], nr[PART_U], nch[PART_U], nsn[PART_U], nse[PART_U], nrv[PART_U];
  u64 nsq[PART_U];
  auto load_round = [&](u64 base, u32 (&C)[PART_U], u32 (&R)[PART_U], u32 (&CH)[PART_U], u32 (&SN)[PART_U], u64 (&SQ)[PART_U],
                        u32 (&SE)[PART_U], u32 (&RV)[PART_U]) {
#pragma unroll
    for (int u = 0; u < PART_U; ++u) {
      const u64 i = base + (u64)u * PART_THREADS + tid;
      if (i < i_end) {
        C[u] = __builtin_nontemporal_load(a.comm + i); R[u] = __builtin_nontemporal_load(a.rank + i);
        CH[u] = __builtin_nontemporal_load(a.channel + i); SN[u] = __builtin_nontemporal_load(a.snap + i);
        SQ[u] = __builtin_nontemporal_load(a.seq_posted + i);
        SE[u] = __builtin_nontemporal_load(a.sent + i); RV[u] = __builtin_nontemporal_load(a.recv + i);
      }
    }
  };
  load_round(i_begin, c, r, ch, sn, sq, se, rv);
  for (u64 base = i_begin; base < i_end; base += PART_CHUNK) {       // uniform over the workgroup
    u32 at[PART_U], reg[PART_U], kin[PART_U];
    bool on[PART_U];
#pragma unroll
    for (int u = 0; u < PART_U; ++u) on[u] = base + (u64)u * PART_THREADS + tid < i_end;
    load_round(base + PART_CHUNK, nc, nr, nch, nsn, nsq, nse, nrv);     // the next round's columns are on their way meanwhile
    uint4 m[PART_U];
#pragma unroll
    for (int u = 0; u < PART_U; ++u) m[u] = on[u] ? grid_row_lookup(a, r[u]) : make_uint4(~0u, ~0u, ~0u, ~0u);
#pragma unroll
    for (int u = 0; u < PART_U; ++u) {
      if (!on[u]) continue;
      on[u] = false;
      if (c[u] >= a.T.n_comms) { status |= DS_UNKNOWN_COMM; continue; }
      const i64 p = grid_row_of(a, c[u], r[u], m[u]);
      if (p < 0) { status |= DS_NOT_MEMBER; continue; }
      if (ch[u] >= a.n_ch || sn[u] >= a.n_snap) { status |= DS_RANGE; continue; }
      const u64 k = ((u64)p * a.n_ch + ch[u]) * a.n_snap + sn[u];
      reg[u] = (u32)(k >> a.rb); kin[u] = (u32)k & kmask;
      at[u] = atomicAdd(&s_cnt[reg[u]], 1u);
      on[u] = true;
    }
    __syncthreads();
    {
      const u32 cnt = tid < a.n_regions ? s_cnt[tid] : 0u;
      u32 tot;
      const u32 ex = block_exclusive_sum<PART_THREADS>(cnt, s_scan, &tot);
      if (tid < a.n_regions) {
        s_pre[tid] = ex;
        s_base[tid] = cnt ? atomicAdd(&a.part_fill[tid], cnt) : 0u;
      }
      if (tid == 0) s_total = tot;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PART_U; ++u) {
      if (!on[u]) continue;
      const u32 q = s_pre[reg[u]] + at[u];
      const u32 pos = s_base[reg[u]] + at[u];
      if (pos >= cap) status |= DS_SUSPECT;              // more rows than cells: some cell is written twice
      s_dst[q] = pos < cap ? ((reg[u] << a.rb) + pos) : ~0u;
      s_idx[q] = kin[u];
      s_pay[q] = make_ulonglong2(sq[u], (u64)se[u] | ((u64)rv[u] << 32));
    }
    __syncthreads();
    const u32 total = s_total;
    for (u32 i = tid; i < total; i += PART_THREADS) {
      const u32 D = s_dst[i];
      if (D == ~0u) continue;
      // pieces of a line that this round writes completely leave with the streaming hint
      const u32 o = D & 7;
      const bool full = i >= o && i + 7 - o < total && s_dst[i - o] == D - o && s_dst[i + 7 - o] == D + 7 - o;
      const ulonglong2 v = s_pay[i];
      if (full) {
        typedef u64 u64x2 __attribute__((ext_vector_type(2)));
        u64x2 vv = {v.x, v.y};
        __builtin_nontemporal_store(vv, reinterpret_cast<u64x2*>(a.part_pay + D));
      } else {
        a.part_pay[D] = v;
      }
      a.part_idx[D] = s_idx[i];
    }
    if (tid < PART_REGIONS) s_cnt[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PART_U; ++u) { c[u] = nc[u]; r[u] = nr[u]; ch[u] = nch[u]; sn[u] = nsn[u]; sq[u] = nsq[u]; se[u] = nse[u]; rv[u] = nrv[u]; }
  }
  u64 st = status;
#pragma unroll
  for (int m2 = 32; m2 >= 1; m2 >>= 1) st |= shfl_xor_u64(st, m2);
  if (lane_id() == 0 && st) atomicOr((unsigned long long*)&a.counters[CNT_STATUS], (unsigned long long)st);
}

// Second step: workgroup i runs on XCD i % 8 (workgroups are dealt to the XCDs in turn); XCD x takes the regions
// x, x + 8, ... one after the other, wpr consecutive workgroups of the XCD per region.
__global__ __launch_bounds__(256) void k_hang_place_regions(HangArgs a, u32 wpr) {
  const u32 xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
  const u32 reg = xcd + 8 * (j / wpr), part = j % wpr;
  if (reg >= a.n_regions) return;
  const u32 cap = 1u << a.rb;
  const u32 have = a.part_fill[reg];
  const u32 cnt = have < cap ? have : cap;
  ulonglong2* __restrict__ cell2 = reinterpret_cast<ulonglong2*>(a.cell) + ((u64)reg << a.rb);
  const ulonglong2* __restrict__ pay = a.part_pay + ((u64)reg << a.rb);
  const u32* __restrict__ idx = a.part_idx + ((u64)reg << a.rb);
  const u32 i = part * PLACE_ROWS + threadIdx.x;
  if (i >= cnt) return;
  typedef u64 u64x2 __attribute__((ext_vector_type(2)));
  const u32 k = __builtin_nontemporal_load(idx + i);                 // read once: streaming loads
  const u64x2 t = __builtin_nontemporal_load(reinterpret_cast<const u64x2*>(pay + i));
  cell2[k] = make_ulonglong2(t.x, t.y);
}

// ---- hang location: two passes over the rows instead of a grid ------------------------------------------
// Of a (member, channel)'s time series the pass needs the final state and the last snapshot that differs from it, and
// that every cell of the grid has exactly one row.  So the rows are not placed: a first pass picks the rows
// of the last snapshot, a second one compares every row with its final state and sets the row's bit in a bitmap of the cells.

// First pass: reads the snapshot numbers, and the other columns of the last snapshot's rows only.  A wavefront lists the
// rows it found in LDS and then loads them side by side: one in n_snap rows is found, and taking each
// where it is found would be a chain of misses.
constexpr int LAST_U = 8;
__global__ __launch_bounds__(256) void k_hang_last(HangArgs a) {
  __shared__ u32 s_found[4][LAST_U * CCLD_WAVE];
  const u32 tid = threadIdx.x, lane = lane_id(), wave = tid / CCLD_WAVE;
  const u64 stride = (u64)gridDim.x * 256, t0 = (u64)blockIdx.x * 256 + tid;
  // what the second pass adds to is cleared on the way
  if (blockIdx.x == 0 && tid < CNT_COUNT) a.counters[tid] = 0;
  for (u64 i = t0; i < (a.n_cell + 31) / 32; i += stride) a.cnt[i] = 0;
  for (u64 i = t0; i < 2 * a.n_members; i += stride) a.mark[i] = 0;
  const u32 L = a.n_snap - 1;
  const u64 waves = (u64)gridDim.x * 4;
  for (u64 base = ((u64)blockIdx.x * 4 + wave) * (LAST_U * CCLD_WAVE); base < a.n_rows; base += waves * (LAST_U * CCLD_WAVE)) {
    u32 sn[LAST_U];
#pragma unroll
    for (int u = 0; u < LAST_U; ++u) {
      const u64 i = base + (u64)u * CCLD_WAVE + lane;
      sn[u] = i < a.n_rows ? __builtin_nontemporal_load(a.snap + i) : ~0u;
    }
    u32 found = 0;
#pragma unroll
    for (int u = 0; u < LAST_U; ++u) {
      const u64 m = ballot64(sn[u] == L && base + (u64)u * CCLD_WAVE + lane < a.n_rows);
      if ((m >> lane) & 1) s_found[wave][found + mbcnt64(m)] = (u32)(u * CCLD_WAVE) + lane;
      found += (u32)__popcll(m);
    }
    __builtin_amdgcn_wave_barrier();
    for (u32 k = lane; k < found; k += CCLD_WAVE) {
      const u64 i = base + s_found[wave][k];
      const u32 c = a.comm[i], r = a.rank[i], ch = a.channel[i];
      const u64 sq = a.seq_posted[i];
      const u32 se = a.sent[i], rv = a.recv[i];
      const i64 p = c < a.T.n_comms ? grid_row_of(a, c, r, grid_row_lookup(a, r)) : -1;
      if (p >= 0 && ch < a.n_ch) a.final[(u64)p * a.n_ch + ch] = make_ulonglong2(sq, (u64)se | ((u64)rv << 32));
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Second pass.
template <int U>
__global__ __launch_bounds__(256) void k_hang_scan(HangArgs a) {
  u64 status = 0;
  const u32 L = a.n_snap - 1, W = a.stall_snapshots;
  const u32 s_stall = L >= W ? L - W : ~0u;
  const u64 stride = (u64)gridDim.x * 256;
  for (u64 i0 = (u64)blockIdx.x * 256 + threadIdx.x; i0 < a.n_rows; i0 += stride * U) {
    u32 c[U], r[U], ch[U], sn[U], se[U], rv[U];
    u64 sq[U];
    bool on[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const u64 i = i0 + stride * u;
      on[u] = i < a.n_rows;
      if (on[u]) {
        c[u] = __builtin_nontemporal_load(a.comm + i); r[u] = __builtin_nontemporal_load(a.rank + i);
        ch[u] = __builtin_nontemporal_load(a.channel + i); sn[u] = __builtin_nontemporal_load(a.snap + i);
        sq[u] = __builtin_nontemporal_load(a.seq_posted + i);
        se[u] = __builtin_nontemporal_load(a.sent + i); rv[u] = __builtin_nontemporal_load(a.recv + i);
      }
    }
    uint4 m[U];
#pragma unroll
    for (int u = 0; u < U; ++u) m[u] = on[u] ? grid_row_lookup(a, r[u]) : make_uint4(~0u, ~0u, ~0u, ~0u);
    i64 p[U];
    ulonglong2 f[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!on[u]) continue;
      on[u] = false;
      if (c[u] >= a.T.n_comms) { status |= DS_UNKNOWN_COMM; continue; }
      p[u] = grid_row_of(a, c[u], r[u], m[u]);
      if (p[u] < 0) { status |= DS_NOT_MEMBER; continue; }
      if (ch[u] >= a.n_ch || sn[u] >= a.n_snap) { status |= DS_RANGE; continue; }
      on[u] = true;
      f[u] = a.final[(u64)p[u] * a.n_ch + ch[u]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!on[u]) continue;
      const u64 k = ((u64)p[u] * a.n_ch + ch[u]) * a.n_snap + sn[u];
      atomicOr(&a.cnt[k >> 5], 1u << (k & 31));
      if (f[u].x == sq[u] && f[u].y == ((u64)se[u] | ((u64)rv[u] << 32))) continue;
      u32* mk = a.mark + 2 * (u64)p[u];
      if (sn[u] == s_stall) mk[1] = 1;
      // the mark only grows: one read beforehand leaves out most of the atomics
      if (mk[0] < sn[u] + 1) atomicMax(&mk[0], sn[u] + 1);
    }
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) status |= shfl_xor_u64(status, m);
  if (lane_id() == 0 && status) atomicOr((unsigned long long*)&a.counters[CNT_STATUS], (unsigned long long)status);
}

// Both of these passes touch random lines for every row (16.8M rows: the final states 150 us, the bitmap's atomics
// 400 us).  So they serve only the rows that cannot be regrouped; normally the rows are first regrouped by region, a range of
// members whose part of the bitmap and of the final states fits LDS, and a workgroup per region then streams its rows.
// A row leaves as 16 bytes:
//   x   operation counter << SPLIT_CELL_BITS | cell inside the region
//   y   sent | received << 32
// Rows with an operation counter of 2^46 or more do not fit; the host then takes the two passes above.  Bytes bound it:
// 32 in and 16 out, then 16 in.  At 16.8M rows in 256 regions the split takes 181 us (4.4 TB/s), the regions 47 us
// (5.7 TB/s), where placing the rows in a grid in memory and scanning that took 540 us.  Rounds of 3,072 rows: each
// reserves room in every region with an atomic, and those of all workgroups for one line of counters follow one another at
// about 34 ns (rounds of 2,048 rows with 512 regions: 340 us).  So there are two sets of counters: every second workgroup fills
// the regions from their ends (2.4M rows of rates 80 -> 75 us per call, hang location of 16.8M rows 268 -> 261).  Larger
// rounds leave one workgroup per CU and nothing to hide the phases behind: with 4,096 or 6,144 rows and whole lines
// stored (the rest of a line waiting in LDS for the next round) the call took 262 and 309 us, with rounds of 2,048 269.
constexpr int SPLIT_CELL_BITS = 18;
constexpr u32 SPLIT_REGIONS = HANG_REGIONS;
constexpr size_t SPLIT_LDS = 64000, RATE_LDS = 156000;      // LDS of a region: hang location, rates
constexpr int RATE_PARTS = 3;                               // a region of rates is taken in up to 2^3 parts
inline size_t rate_region_lds(u32 n_ch, u32 n_snap, int sb) {
  const u64 cells = (u64)n_ch * n_snap << sb;
  return cells * 16 + (32ull << sb) + (cells + 31) / 32 * 4;
}
inline size_t region_lds(u32 n_ch, u32 n_snap, int sb) {
  return ((20ull * n_ch + 4) << sb) + ((((u64)n_ch * n_snap << sb) + 31) / 32) * 4;
}
// A region's rows: those from the front, the room between these and the ones from the end, all.
struct RegionRows { u32 front, gap, n; };
__device__ __forceinline__ u32 region_room(const HangArgs& a, u32 reg, u32 cap) {
  const u64 left = a.n_cell - (u64)reg * cap;
  return left < cap ? (u32)left : cap;
}
__device__ __forceinline__ RegionRows region_rows(const HangArgs& a, u32 reg, u32 cap) {
  const u32 room = region_room(a, reg, cap), front = a.part_fill[reg], back = a.ends ? a.part_fill[SPLIT_REGIONS + reg] : 0u;
  if (front > room || back > room - front) {         // more rows than cells
    if (threadIdx.x == 0) atomicOr((unsigned long long*)&a.counters[CNT_STATUS], (unsigned long long)DS_DUPLICATE);
    return {room, 0, room};
  }
  return {front, room - front - back, front + back};
}
// where row i of a region lies
__device__ __forceinline__ u32 region_row(const RegionRows& r, u32 i) { return i < r.front ? i : i + r.gap; }
template <int THREADS, int U>
__global__ __launch_bounds__(THREADS) void k_hang_split(HangArgs a, u64 chunk) {
  constexpr u32 CHUNK = THREADS * U;
  extern __shared__ ulonglong2 s_row[];                                // [CHUNK] rows | [CHUNK] their regions
  unsigned short* s_reg = reinterpret_cast<unsigned short*>(s_row + CHUNK);
  __shared__ u32 s_cnt[SPLIT_REGIONS], s_pre[SPLIT_REGIONS], s_off[SPLIT_REGIONS], s_scan[THREADS / CCLD_WAVE], s_total;
  constexpr u32 PER = (SPLIT_REGIONS + THREADS - 1) / THREADS;         // regions per thread
  const u32 tid = threadIdx.x;
  const u32 L = a.n_snap - 1, per_member = a.n_ch * a.n_snap, cap = per_member << a.sb, smask = (1u << a.sb) - 1;
  u64 status = 0;
  const bool from_end = a.ends && (blockIdx.x & 1);
  u32* const fill = a.part_fill + (from_end ? SPLIT_REGIONS : 0u);
  const u64 i_begin = chunk * blockIdx.x;
  const u64 i_end = chunk * (blockIdx.x + 1) < a.n_rows ? chunk * (blockIdx.x + 1) : a.n_rows;
  u32 c[U], r[U], ch[U], sn[U], se[U], rv[U];
  u64 sq[U];
  auto load_round = [&](u64 base) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const u64 i = base + (u64)u * THREADS + tid;
      if (i < i_end) {
        c[u] = __builtin_nontemporal_load(a.comm + i); r[u] = __builtin_nontemporal_load(a.rank + i);
        ch[u] = __builtin_nontemporal_load(a.channel + i); sn[u] = __builtin_nontemporal_load(a.snap + i);
        sq[u] = __builtin_nontemporal_load(a.seq_posted + i);
        se[u] = __builtin_nontemporal_load(a.sent + i); rv[u] = __builtin_nontemporal_load(a.recv + i);
      }
    }
  };
  load_round(i_begin);
  for (u32 i = tid; i < SPLIT_REGIONS; i += THREADS) s_cnt[i] = 0;
  __syncthreads();
  for (u64 base = i_begin; base < i_end; base += CHUNK) {              // uniform over the workgroup
    uint4 m[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      m[u] = base + (u64)u * THREADS + tid < i_end ? grid_row_lookup(a, r[u]) : make_uint4(~0u, ~0u, ~0u, ~0u);
    u32 at[U];                                                         // region << 16 | rank among its rows, ~0: no row
#pragma unroll
    for (int u = 0; u < U; ++u) {
      at[u] = ~0u;
      if (base + (u64)u * THREADS + tid >= i_end) continue;
      if (c[u] >= a.T.n_comms) { status |= DS_UNKNOWN_COMM; continue; }
      const i64 p = grid_row_of(a, c[u], r[u], m[u]);
      if (p < 0) { status |= DS_NOT_MEMBER; continue; }
      if (ch[u] >= a.n_ch || sn[u] >= a.n_snap) { status |= DS_RANGE; continue; }
      if (sq[u] >> (64 - SPLIT_CELL_BITS)) { status |= DS_SUSPECT; continue; }
      if (sn[u] == L) a.final[(u64)p * a.n_ch + ch[u]] = make_ulonglong2(sq[u], (u64)se[u] | ((u64)rv[u] << 32));
      const u32 reg = (u32)p >> a.sb;
      sq[u] = sq[u] << SPLIT_CELL_BITS | (((u32)p & smask) * per_member + ch[u] * a.n_snap + sn[u]);
      at[u] = reg << 16 | atomicAdd(&s_cnt[reg], 1u);
    }
    __syncthreads();
    {
      u32 v[PER], sum = 0;
#pragma unroll
      for (u32 k = 0; k < PER; ++k) { v[k] = PER * tid + k < a.n_regions ? s_cnt[PER * tid + k] : 0u; sum += v[k]; }
      u32 f[PER];
#pragma unroll
      for (u32 k = 0; k < PER; ++k) if (v[k]) f[k] = atomicAdd(&fill[PER * tid + k], v[k]);
      u32 tot;
      u32 ex = block_exclusive_sum<THREADS>(sum, s_scan, &tot);
#pragma unroll
      for (u32 k = 0; k < PER; ++k)
        if (PER * tid + k < a.n_regions) {
          s_pre[PER * tid + k] = ex;
          if (v[k]) s_off[PER * tid + k] = (from_end ? region_room(a, PER * tid + k, cap) - f[k] - v[k] : f[k]) - ex;
          ex += v[k];
          s_cnt[PER * tid + k] = 0;
        }
      if (tid == 0) s_total = tot;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (at[u] == ~0u) continue;
      const u32 q = s_pre[at[u] >> 16] + (at[u] & 0xFFFFu);
      s_reg[q] = (unsigned short)(at[u] >> 16);
      s_row[q] = make_ulonglong2(sq[u], (u64)se[u] | ((u64)rv[u] << 32));
    }
    __syncthreads();
    load_round(base + CHUNK);                                          // on their way while this round is written
    const u32 total = s_total;
    for (u32 i = tid; i < total; i += THREADS) {
      const u32 reg = s_reg[i], pos = s_off[reg] + i;
      if (pos < region_room(a, reg, cap)) {
        a.part_row[(u64)reg * cap + pos] = s_row[i];
      } else {
        status |= DS_DUPLICATE;            // more rows than cells
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int m2 = 32; m2 >= 1; m2 >>= 1) status |= shfl_xor_u64(status, m2);
  if (lane_id() == 0 && status) atomicOr((unsigned long long*)&a.counters[CNT_STATUS], (unsigned long long)status);
}
// What a pass over regrouped rows counts in starts at zero: the context was made so, the last workgroup of the pass before left
// it so, or this launch does (61,440 rows: 38.6 -> 36.4 us without it; a context's first pass 68 -> 65.5, of 2.4M rows of
// rates 118.5 -> 112.5).
__global__ __launch_bounds__(SPLIT_REGIONS) void k_hang_clear(HangArgs a) {
  if (threadIdx.x < CNT_COUNT) a.counters[threadIdx.x] = 0;
  for (u32 i = threadIdx.x; i < (a.ends ? 2 * SPLIT_REGIONS : a.n_regions); i += SPLIT_REGIONS) a.part_fill[i] = 0;      // all: a later pass may have more
}
__device__ __forceinline__ void report_and_clear(const HangArgs& a) {
  report_words(a.counters, a.host, a.ticket);
  if (!a.leave_clear) return;
  __syncthreads();                     // the words have been read
  if (threadIdx.x < CNT_COUNT) store_agent(reinterpret_cast<i64*>(&a.counters[threadIdx.x]), 0);
  for (u32 i = threadIdx.x; i < a.n_regions; i += blockDim.x) { a.part_fill[i] = 0; a.part_fill[SPLIT_REGIONS + i] = 0; }
}
__device__ __forceinline__ void store_member(const HangArgs& a, u64 p, u64 seq, u64 S, u64 R, u32 onset, bool moved) {
  PAIR(a, CCLD_HPAIR_STALLED, p) = a.n_snap - 1 >= a.stall_snapshots && !moved ? 1 : 0;
  PAIR(a, CCLD_HPAIR_SEQ, p) = (i64)seq;
  PAIR(a, CCLD_HPAIR_SENT, p) = (i64)S;
  PAIR(a, CCLD_HPAIR_RECV, p) = (i64)R;
  PAIR(a, CCLD_HPAIR_WAITS_ON, p) = CCLD_NO_RANK;
  PAIR(a, CCLD_HPAIR_ONSET, p) = onset;
  a.wait_slot[p] = -1;
  a.cand[p] = 0;
  a.layer_max[p] = 0;          // takes the place of the marks
}
// One workgroup per region: its rows in order of arrival against the final states, then its members.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_hang_region(HangArgs a) {
  extern __shared__ ulonglong2 s_final[];                              // final states | onsets | bitmap | moved
  const u32 tid = threadIdx.x, reg = blockIdx.x;
  const u32 per_member = a.n_ch * a.n_snap, cap = per_member << a.sb, n_ser = a.n_ch << a.sb, words = (cap + 31) / 32;
  u32* s_onset = reinterpret_cast<u32*>(s_final + n_ser);
  u32* s_bits = s_onset + n_ser;
  u32* s_moved = s_bits + words;                                       // [2^sb]
  __shared__ u32 s_cells;
  const u64 p0 = (u64)reg << a.sb, q0 = p0 * a.n_ch, q_end = a.n_members * a.n_ch;
  const RegionRows R = region_rows(a, reg, cap);
  const u32 n = R.n;
  const ulonglong2* __restrict__ rows = a.part_row + (u64)reg * cap;
  for (u32 i = tid; i < n_ser; i += THREADS) {
    s_final[i] = q0 + i < q_end ? a.final[q0 + i] : make_ulonglong2(0, 0);
    s_onset[i] = 0;
  }
  for (u32 i = tid; i < words + (1u << a.sb); i += THREADS) s_bits[i] = 0;
  if (tid == 0) s_cells = 0;
  __syncthreads();
  const u32 s_stall = a.n_snap - 1 >= a.stall_snapshots ? a.n_snap - 1 - a.stall_snapshots : ~0u;
  constexpr int U = 4;
  typedef u64 u64x2 __attribute__((ext_vector_type(2)));
  for (u32 i0 = tid; i0 < n; i0 += THREADS * U) {
    u64x2 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * THREADS < n) v[u] = __builtin_nontemporal_load(reinterpret_cast<const u64x2*>(rows + region_row(R, i0 + u * THREADS)));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u * THREADS >= n) continue;
      const u32 k = (u32)v[u].x & ((1u << SPLIT_CELL_BITS) - 1);
      const u32 ser = (u32)(((u64)k * a.snap_inv) >> 32), s = k - ser * a.n_snap;
      atomicOr(&s_bits[k >> 5], 1u << (k & 31));
      const ulonglong2 f = s_final[ser];
      if (f.x == v[u].x >> SPLIT_CELL_BITS && f.y == v[u].y) continue;
      if (s_onset[ser] < s + 1) atomicMax(&s_onset[ser], s + 1);
      if (s == s_stall) s_moved[ser / a.n_ch] = 1;
    }
  }
  __syncthreads();
  u32 cells = 0;
  for (u32 i = tid; i < words; i += THREADS) cells += (u32)__popc(s_bits[i]);
  cells = wave_sum(cells);
  if (lane_id() == 0) atomicAdd(&s_cells, cells);
  for (u32 i = tid; i < (1u << a.sb) && p0 + i < a.n_members; i += THREADS) {
    u64 seq = 0, S = 0, R = 0;
    u32 onset = 0;
    for (u32 ch = 0; ch < a.n_ch; ++ch) {
      const ulonglong2 f = s_final[i * a.n_ch + ch];
      const u32 o = s_onset[i * a.n_ch + ch];
      seq = f.x > seq ? f.x : seq;
      S += f.y & 0xFFFFFFFFull;
      R += f.y >> 32;
      onset = o > onset ? o : onset;
    }
    store_member(a, p0 + i, seq, S, R, onset, s_moved[i] != 0);
  }
  __syncthreads();
  if (tid == 0) atomicAdd((unsigned long long*)&a.counters[CNT_NCELL], (unsigned long long)s_cells);
}

// Members and cells after the second pass: stalled, operation counter, chunk totals, onset of every (rank, communicator),
// eight lanes to a member, and the cells that have a row.
constexpr u32 PAIR_LANES = 8;
__global__ __launch_bounds__(256) void k_hang_pairs(HangArgs a) {
  __shared__ u32 s_cells;
  const u32 tid = threadIdx.x;
  const u64 t = (u64)blockIdx.x * 256 + tid, p = t / PAIR_LANES;
  const u32 l = tid % PAIR_LANES;
  if (tid == 0) s_cells = 0;
  __syncthreads();
  u32 cells = 0;
  for (u64 i = t; i < (a.n_cell + 31) / 32; i += (u64)gridDim.x * 256) cells += (u32)__popc(a.cnt[i]);
  cells = wave_sum(cells);
  if (lane_id() == 0) atomicAdd(&s_cells, cells);
  u64 seq = 0, S = 0, R = 0;
  if (p < a.n_members)
    for (u32 ch = l; ch < a.n_ch; ch += PAIR_LANES) {
      const ulonglong2 f = a.final[p * a.n_ch + ch];
      seq = f.x > seq ? f.x : seq;
      S += f.y & 0xFFFFFFFFull;
      R += f.y >> 32;
    }
#pragma unroll
  for (u32 m = PAIR_LANES / 2; m >= 1; m >>= 1) {
    const u64 o = shfl_xor_u64(seq, m);
    seq = o > seq ? o : seq;
    S += shfl_xor_u64(S, m); R += shfl_xor_u64(R, m);
  }
  if (p < a.n_members && l == 0) {
    store_member(a, p, seq, S, R, a.mark[2 * p], a.mark[2 * p + 1] != 0);
  }
  __syncthreads();
  if (tid == 0) atomicAdd((unsigned long long*)&a.counters[CNT_NCELL], (unsigned long long)s_cells);
}

// every row valid and exactly one for each cell
__device__ __forceinline__ bool hang_rows_ok(const HangArgs& a) {
  return a.checked || (a.counters[CNT_STATUS] == 0 && a.n_rows == a.n_cell && a.counters[CNT_NCELL] == a.n_cell);
}

// ---- per communicator: entered, idle test, decision tree, wait-for edges ------------------------
__device__ __forceinline__ u64 wave_min_u64(u64 v) { return ~wave_max_u64(~v); }
__device__ __forceinline__ u32 wave_min_u32(u32 v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) { const u32 o = __shfl_xor(v, m, CCLD_WAVE); v = o < v ? o : v; }
  return v;
}
// One workgroup per communicator; K members per thread in registers (0: communicators of any size, re-read by every
// step).  Each step is a chain of a load and a reduction, so what counts is how few there are: members are read once,
// and a wavefront reduces in registers before its one LDS atomic (atomics of all lanes on one word run one after the
// other; 4,096 members: 44 us with an atomic per thread and every step reading).
struct HangMember { u64 seq; i64 sent, recv; bool stalled; };
template <u32 THREADS, u32 K>
__global__ __launch_bounds__(THREADS) void k_hang_comm(HangArgs a) {
  __shared__ unsigned long long s_seqmax, s_minsum, s_minrecv, s_worst;
  __shared__ u32 s_flags, s_best, s_ncand;      // flags: 1 not all entered, 2 any stalled, 4 not all stalled, 8 not idle
  __shared__ u32 s_link[K ? K * THREADS : 1];   // hops << 16 | slot they lead to, LINK_ROOT set: a root
  constexpr u32 LINK_ROOT = 0x8000u;
  static_assert(K * THREADS <= LINK_ROOT / 2, "hops and slots fit 15 bits");
  const u32 c = blockIdx.x, tid = threadIdx.x, lane = lane_id();
  const u32 n = a.T.size[c], off = a.T.member_off[c];
  const bool tree = a.T.algo[c] == CCLD_ALGO_TREE, ok = hang_rows_ok(a);
  auto load_member = [&](u32 q) -> HangMember {
    const u64 p = (u64)off + q;
    return {(u64)PAIR(a, CCLD_HPAIR_SEQ, p), PAIR(a, CCLD_HPAIR_SENT, p), PAIR(a, CCLD_HPAIR_RECV, p), PAIR(a, CCLD_HPAIR_STALLED, p) != 0};
  };
  HangMember mem[K ? K : 1];
#pragma unroll
  for (u32 k = 0; k < K; ++k) if (tid + k * THREADS < n) mem[k] = load_member(tid + k * THREADS);
  auto each = [&](auto&& f) {
    if constexpr (K != 0) {
#pragma unroll
      for (u32 k = 0; k < K; ++k) if (tid + k * THREADS < n) f(tid + k * THREADS, mem[k]);
    } else {
      for (u32 q = tid; q < n; q += THREADS) f(q, load_member(q));
    }
  };
  if (tid == 0) { s_seqmax = 0; s_minsum = ~0ull; s_minrecv = ~0ull; s_worst = 0; s_flags = 0; s_best = 0xFFFFFFFFu; s_ncand = 0; }
  __syncthreads();
  if (!ok) return;                              // the same for every thread
  const bool some = (tid & ~(u32)(CCLD_WAVE - 1)) < n;      // the wavefront has members
  // depth of a slot in the tree (layers are contiguous in BFS order)
  auto depth_of = [&](u32 q) -> u32 {
    u32 d = 0;
    if (tree) { int cur = (int)q; while (a.T.tree_parent[off + cur] >= 0) { cur = a.T.tree_parent[off + cur]; ++d; } }
    return d;
  };
  {
    u32 fl = 0;
    u64 seqmax = 0, minsum = ~0ull;
    each([&](u32 q, const HangMember& m) {
      const u64 p = (u64)off + q, sum = (u64)(m.sent + m.recv);
      seqmax = m.seq > seqmax ? m.seq : seqmax;
      minsum = sum < minsum ? sum : minsum;
      fl |= m.stalled ? 2 : 4;
      // identical totals across comparable ranks: every adjacent pair of the same layer
      if (q > 0 && (!tree || depth_of(q) == depth_of(q - 1)) &&
          (m.sent != PAIR(a, CCLD_HPAIR_SENT, p - 1) || m.recv != PAIR(a, CCLD_HPAIR_RECV, p - 1)))
        fl |= 8;
      if (tree) atomicMax((unsigned long long*)&a.layer_max[off + depth_of(q)], (unsigned long long)sum);
    });
    if (some) {
      seqmax = wave_max_u64(seqmax); minsum = wave_min_u64(minsum);
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) fl |= __shfl_xor(fl, m, CCLD_WAVE);
      if (lane == 0) { atomicMax(&s_seqmax, (unsigned long long)seqmax); atomicMin(&s_minsum, (unsigned long long)minsum); atomicOr(&s_flags, fl); }
    }
  }
  __syncthreads();
  const u64 seq_max = s_seqmax, min_sum = s_minsum;
  // fewest SendCount + RecvCount, then fewest received, then smallest rank
  {
    u32 fl = 0;
    u64 mr = ~0ull;
    each([&](u32 q, const HangMember& m) {
      PAIR(a, CCLD_HPAIR_ENTERED, (u64)off + q) = m.seq == seq_max ? 1 : 0;
      if (m.seq != seq_max) fl |= 1 | 8;
      if ((u64)(m.sent + m.recv) == min_sum) mr = (u64)m.recv < mr ? (u64)m.recv : mr;
    });
    if (some) {
      mr = wave_min_u64(mr);
      const u64 late = ballot64(fl != 0);
      if (lane == 0 && mr != ~0ull) atomicMin(&s_minrecv, (unsigned long long)mr);
      if (lane == 0 && late) atomicOr(&s_flags, 1u | 8u);
    }
  }
  __syncthreads();
  {
    const u64 mr = s_minrecv;
    u32 best = 0xFFFFFFFFu;
    each([&](u32 q, const HangMember& m) {
      if ((u64)(m.sent + m.recv) != min_sum || (u64)m.recv != mr) return;
      const u32 rk = a.T.members[off + q];
      best = rk < best ? rk : best;
    });
    if (some) {
      best = wave_min_u32(best);
      if (lane == 0 && best != 0xFFFFFFFFu) atomicMin(&s_best, best);
    }
  }
  __syncthreads();
  const u32 flags = s_flags;
  const bool all_entered = !(flags & 1), any_stalled = flags & 2, all_stalled = !(flags & 4), idle_ok = !(flags & 8);
  const bool hung = !idle_ok && any_stalled;
  int cls = 0;
  if (hung) cls = !all_entered ? CCLD_HANG_H1_NOT_ENTERED : (!all_stalled ? CCLD_HANG_H2_INCONSISTENT : CCLD_HANG_H3_HARDWARE);
  if (tid == 0) {
    const i64 row[CCLD_HCOMM_NCOL] = {(i64)c, hung ? 1 : 0, cls, (i64)seq_max, hung ? (i64)s_best : CCLD_NO_RANK, 0};
    for (int col = 0; col < CCLD_HCOMM_NCOL; ++col) {
      HCOMM(a, col, c) = row[col];
      if (a.out_comm && c < a.comm_cap) a.out_comm[(u64)col * a.comm_cap + c] = row[col];
    }
    if (hung) atomicAdd((unsigned long long*)&a.counters[CNT_NALERT], 1ull);
  }
  if (!hung) return;
  if (cls == CCLD_HANG_H1_NOT_ENTERED) {
    each([&](u32 q, const HangMember& m) { if (m.seq != seq_max) a.cand[off + q] = 1; });
    return;
  }
  if (cls == CCLD_HANG_H2_INCONSISTENT) {
    each([&](u32 q, const HangMember& m) { if (!m.stalled) a.cand[off + q] = 1; });
    return;
  }
  // all entered, all hung
  if (!tree) {
    each([&](u32 q, const HangMember& m) {
      const u32 pred = q ? q - 1 : n - 1, succ = q + 1 < n ? q + 1 : 0;
      u32 on = q;                               // itself: a root
      if (n > 1 && m.recv >= PAIR(a, CCLD_HPAIR_SENT, off + pred)) on = pred;
      else if (n > 1 && m.sent - PAIR(a, CCLD_HPAIR_RECV, off + succ) >= (i64)a.fifo_depth) on = succ;
      if (on == q) {
        a.cand[off + q] = 1;
        s_ncand = 1;
      } else {
        PAIR(a, CCLD_HPAIR_WAITS_ON, off + q) = a.T.members[off + on];
        a.wait_slot[off + q] = (int)on;
      }
      if (K) s_link[q] = on == q ? q | LINK_ROOT : on | 1u << 16;
    });
  } else {
    each([&](u32 q, const HangMember& m) {
      const u64 def = a.layer_max[off + depth_of(q)] - (u64)(m.sent + m.recv);
      atomicMax(&s_worst, (unsigned long long)def);
    });
    __syncthreads();
    const u64 worst = s_worst;
    if (worst > 0)
      each([&](u32 q, const HangMember& m) {
        const u64 def = a.layer_max[off + depth_of(q)] - (u64)(m.sent + m.recv);
        if (def == worst) { a.cand[off + q] = 1; s_ncand = 1; }
      });
  }
  __syncthreads();
  const bool cycle = s_ncand == 0;      // a pure cycle: the rank with the fewest counts
  if (cycle)
    each([&](u32 q, const HangMember&) {
      if (a.T.members[off + q] != s_best) return;
      a.cand[off + q] = 1;
      if (K) s_link[q] = q | LINK_ROOT;
    });
  // Hops to a root by pointer jumping: after round r a link leads 2^r edges on, or to the root before that.
  if (K && !tree) {
    u32 link[K ? K : 1];
    for (u32 span = 1; span < n; span <<= 1) {
      __syncthreads();
#pragma unroll
      for (u32 k = 0; k < K; ++k) {
        const u32 q = tid + k * THREADS;
        if (q >= n) continue;
        link[k] = s_link[q];
        if (!(link[k] & LINK_ROOT)) {
          const u32 m = s_link[link[k] & 0xFFFFu];
          link[k] = (m & 0xFFFFu) | (((link[k] >> 16) + (m >> 16)) << 16);
        }
      }
      __syncthreads();
#pragma unroll
      for (u32 k = 0; k < K; ++k) if (tid + k * THREADS < n) s_link[tid + k * THREADS] = link[k];
    }
    __syncthreads();
    each([&](u32 q, const HangMember&) { PAIR(a, CCLD_HPAIR_HOPS, off + q) = s_link[q] & LINK_ROOT ? (i64)(s_link[q] >> 16) : -1; });
  }
}

// ---- victims, hops along the wait-for edges to a root, candidates per communicator, the tables and the roots -------
// A rank that has not entered communicator c and has entered another hung one is a victim: no candidate.  m: its packed memberships.
__device__ __forceinline__ bool is_victim(const HangArgs& a, u32 c, u32 r, const uint4& m) {
  auto entered_hung = [&](u32 c2, u64 p2) { return (HCOMM(a, CCLD_HCOMM_HUNG, c2) != 0) & (PAIR(a, CCLD_HPAIR_ENTERED, p2) != 0); };
  if (a.T.rank_cell4) {                    // the rank's (at most four) memberships in one load, then all looked at side by side
    const u32 w[4] = {m.x, m.y, m.z, m.w};
    bool hit = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const u32 c2 = w[k] == ~0u ? c : w[k] >> a.T.pb;
      hit |= entered_hung(c2, c2 == c ? 0 : w[k] & ((1u << a.T.pb) - 1)) && c2 != c;
    }
    return hit;
  }
  for (u32 k = a.T.rank_comm_off[r]; k < a.T.rank_comm_off[r + 1]; ++k) {
    const u32 c2 = a.T.rank_comms[k], off2 = a.T.member_off[c2];
    if (c2 != c && entered_hung(c2, (u64)off2 + a.T.sorted_slot[off2 + a.T.rank_slots[k]])) return true;
  }
  return false;
}

// Roots in (rank, communicator) order: the last workgroup sorts up to ROOTS_ONE of them in LDS.  More are sorted by
// the host's radix sort afterwards: that many ranks freeze at once only when whole parts of a job never enter.
constexpr u32 ROOTS_ONE = 1024;
__device__ __forceinline__ void emit_root(const HangArgs& a, u32 k, u64 key) {
  const u32 c = (u32)(key & (((u64)1 << a.cb) - 1));
  store_agent(&a.out_root[CCLD_HROOT_RANK * a.root_cap + k], (i64)(key >> a.cb));
  store_agent(&a.out_root[CCLD_HROOT_COMM * a.root_cap + k], (i64)c);
  store_agent(&a.out_root[CCLD_HROOT_CLASS * a.root_cap + k], HCOMM(a, CCLD_HCOMM_CLASS, c));
}
__global__ __launch_bounds__(256) void k_hang_final(HangArgs a) {
  __shared__ u64 s_key[ROOTS_ONE];
  __shared__ u32 s_last;
  const u64 p = (u64)blockIdx.x * 256 + threadIdx.x;
  const u32 tid = threadIdx.x, lane = lane_id();
  // Few dependent trips to memory are what this takes, so everything that is known by the member's number alone is asked for at
  // once, before it is known whether the rows are good, then what follows from its communicator and rank.
  const u64 pm = p < a.n_members ? p : 0;
  u32 c = a.T.member_comm[pm];
  const u32 rank = a.T.members[pm];
  const bool cand = a.cand[pm] != 0;
  i64 row[CCLD_HPAIR_NCOL];
#pragma unroll
  for (int col = 0; col < CCLD_HPAIR_NCOL; ++col) row[col] = col == CCLD_HPAIR_RANK || col == CCLD_HPAIR_COMM ? 0 : PAIR(a, col, pm);
  const bool ok = hang_rows_ok(a);
  const i64 cls = HCOMM(a, CCLD_HCOMM_CLASS, c);
  const bool tree = a.T.algo[c] == CCLD_ALGO_TREE;
  const uint4 memb = a.T.rank_cell4 ? grid_row_lookup(a, rank) : make_uint4(~0u, ~0u, ~0u, ~0u);
  if (ok) {
    bool root = false;
    if (p < a.n_members) {
      // only a communicator that not everyone has entered has victims, and it has no wait-for edges: no walk meets one
      root = cand && !(cls == CCLD_HANG_H1_NOT_ENTERED && is_victim(a, c, rank, memb));
      i64 hops = -1;
      if (root) {
        hops = 0;
      } else if (cls == CCLD_HANG_H3_HARDWARE && !tree) {
        if (a.hops_known) hops = row[CCLD_HPAIR_HOPS];
        const u32 off = a.T.member_off[c], n = a.T.size[c];
        u32 cur = (u32)(p - off);
        i64 walked = 0;
        while (!a.hops_known) {
          const int w = a.wait_slot[off + cur];
          if (w < 0 || walked >= (i64)n) break;
          cur = (u32)w;
          ++walked;
          if (a.cand[off + cur]) { hops = walked; break; }
        }
      }
      if (a.out_pair && p < a.pair_cap) {
        row[CCLD_HPAIR_RANK] = (i64)rank; row[CCLD_HPAIR_COMM] = (i64)c; row[CCLD_HPAIR_HOPS] = hops;
#pragma unroll
        for (int col = 0; col < CCLD_HPAIR_NCOL; ++col) store_agent(&a.out_pair[(u64)col * a.pair_cap + p], row[col]);
      }
    }
    // roots of a wavefront take their places together, and count together per communicator
    u64 m = ballot64(root);
    if (m) {
      u32 base = 0;
      if (lane == 0) base = atomicAdd(reinterpret_cast<u32*>(&a.counters[CNT_NCAND]), (u32)__popcll(m));
      base = __shfl(base, 0, CCLD_WAVE);
      if (root) store_agent(&a.root_key[base + mbcnt64(m)], (i64)(((u64)rank << a.cb) | c));
      while (m) {
        const u32 first = (u32)__builtin_ctzll(m);
        const u32 c1 = __shfl(c, (int)first, CCLD_WAVE);
        const u64 same = ballot64(root && c == c1) & m;
        if (lane == first && a.out_comm && c1 < a.comm_cap)
          atomicAdd((unsigned long long*)&a.out_comm[(u64)CCLD_HCOMM_NCAND * a.comm_cap + c1], (unsigned long long)__popcll(same));
        m &= ~same;
      }
    }
  }
  if (!last_block(reinterpret_cast<u32*>(&a.counters[CNT_DONE]), gridDim.x, &s_last)) return;
  const u32 n_root = load_agent(reinterpret_cast<const u32*>(&a.counters[CNT_NCAND]));
  if (n_root && n_root <= ROOTS_ONE && a.root_cap) {
    u32 n2 = 1;
    while (n2 < n_root) n2 <<= 1;
    for (u32 k = tid; k < n2; k += 256) {
      s_key[k] = k < n_root ? (u64)load_agent(&a.root_key[k]) : ~0ull;
    }
    __syncthreads();
    for (u32 len = 2; len <= n2; len <<= 1)
      for (u32 d = len / 2; d >= 1; d >>= 1) {
        for (u32 k = tid; k < n2 / 2; k += 256) {
          const u32 i = 2 * k - (k & (d - 1)), j = i + d;
          const bool up = (i & len) == 0;
          if ((s_key[i] > s_key[j]) == up) {
            const u64 tk = s_key[i]; s_key[i] = s_key[j]; s_key[j] = tk;
          }
        }
        __syncthreads();
      }
    for (u32 k = tid; k < n_root && k < a.root_cap; k += 256) emit_root(a, k, s_key[k]);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  }
  report_and_clear(a);
}
__global__ __launch_bounds__(256) void k_hang_root_emit(HangArgs a, const u32* sidx, u32 n_root) {
  const u32 k = blockIdx.x * 256 + threadIdx.x;
  if (k < n_root && k < a.root_cap) emit_root(a, k, (u64)a.root_key[sidx[k]]);
}

// ---- SendRate / RecvRate: count changes per operation (Section 4.1.2) ------------------------------
#define RPAIR(a, col, p) (a.pair[(u64)(col) * a.n_members + (p)])

// One wavefront per time series, lanes on consecutive snapshots.  A run of equal operation counters is committed when the
// next run starts, so the open last run never counts.
struct RateSums { u64 ops_s, chg_s, ops_r, chg_r; };
template <class Sample>
__device__ __forceinline__ void rate_series(u32 n_snap, u32 lane, RateSums& t, Sample&& sample) {
  const u64 below = ((u64)1 << lane) - 1;                // lanes before this one
  u64 c_seq = 0, c_cnt = 0;                              // last sample of the previous chunk
  u32 pend_s = 0, pend_r = 0;                            // changes seen so far in the run that is still open
  for (u32 s0 = 0; s0 < n_snap; s0 += CCLD_WAVE) {
    const u32 s = s0 + lane;
    const bool in = s < n_snap;
    u64 seq = 0, cnt = 0;
    if (in) sample(s, &seq, &cnt);
    u64 pseq = shfl_u64(seq, (int)lane - 1), pcnt = shfl_u64(cnt, (int)lane - 1);
    if (lane == 0) { pseq = c_seq; pcnt = c_cnt; }
    const bool start = in && (s == 0 || seq != pseq);
    if (start) pcnt = 0;                                 // a run's first sample is compared with zero
    const u64 B = ballot64(start);
    const u64 Cs = ballot64(in && (u32)cnt != (u32)pcnt);
    const u64 Cr = ballot64(in && (u32)(cnt >> 32) != (u32)(pcnt >> 32));
    if (B == 0) {
      pend_s += (u32)__popcll(Cs); pend_r += (u32)__popcll(Cr);
    } else {
      const u32 last = 63 - (u32)__clzll((long long)B);               // start of the run still open
      const u64 closed = ((u64)1 << last) - 1;                        // samples of runs that close here
      // this lane's run begins at the highest start at or below it (or came in from the last chunk)
      const u64 Bat = B & (below | ((u64)1 << lane));
      const bool carried = Bat == 0;
      const u32 rs = carried ? 0u : 63 - (u32)__clzll((long long)Bat);
      const u64 run_before = below & ~(((u64)1 << rs) - 1);           // lanes of my run before me
      const bool mine = ((closed >> lane) & 1) != 0;
      const bool first_s = mine && ((Cs >> lane) & 1) && (Cs & run_before) == 0 && !(carried && pend_s);
      const bool first_r = mine && ((Cr >> lane) & 1) && (Cr & run_before) == 0 && !(carried && pend_r);
      const u32 first_start = (u32)__builtin_ctzll(B);
      // the carried run closes at the chunk's first start: it is one operation if it had a change
      // earlier, else if one of its lanes here is a first change (counted below)
      t.ops_s += (u64)__popcll(ballot64(first_s)) + ((pend_s && first_start <= last) ? 1 : 0);
      t.ops_r += (u64)__popcll(ballot64(first_r)) + ((pend_r && first_start <= last) ? 1 : 0);
      t.chg_s += pend_s + (u64)__popcll(Cs & closed);
      t.chg_r += pend_r + (u64)__popcll(Cr & closed);
      pend_s = (u32)__popcll(Cs & ~closed); pend_r = (u32)__popcll(Cr & ~closed);
    }
    c_seq = shfl_u64(seq, 63); c_cnt = shfl_u64(cnt, 63);
  }
}
__device__ __forceinline__ void store_rates(const HangArgs& a, u64 p, const RateSums& t) {
  RPAIR(a, CCLD_RATE_OPS_SEND, p) = (i64)t.ops_s;
  RPAIR(a, CCLD_RATE_CHANGES_SEND, p) = (i64)t.chg_s;
  RPAIR(a, CCLD_RATE_OPS_RECV, p) = (i64)t.ops_r;
  RPAIR(a, CCLD_RATE_CHANGES_RECV, p) = (i64)t.chg_r;
}
// From the grid in memory: one wavefront per member slot.
__global__ __launch_bounds__(256) void k_rate_pairs(HangArgs a) {
  const u32 lane = lane_id();
  const u64 p = (u64)blockIdx.x * 4 + threadIdx.x / CCLD_WAVE;
  if (p >= a.n_members) return;
  RateSums t{0, 0, 0, 0};
  u64 status = 0;
  for (u32 ch = 0; ch < a.n_ch; ++ch) {
    const u64 base = (p * a.n_ch + ch) * a.n_snap;
    rate_series(a.n_snap, lane, t, [&](u32 s, u64* seq, u64* cnt) {
      *seq = a.cell[2 * (base + s)]; *cnt = a.cell[2 * (base + s) + 1];
      status |= cell_status(a, base + s, *seq, *cnt);
    });
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) status |= shfl_xor_u64(status, m);
  if (lane == 0) {
    if (status) atomicOr((unsigned long long*)&a.counters[CNT_STATUS], (unsigned long long)status);
    store_rates(a, p, t);
  }
}
// From the regrouped rows: a workgroup places the rows of its region in LDS by cell, then its wavefronts take the
// series one by one.  The grid never exists in memory.  Where the cells of a whole region do not fit LDS, a workgroup takes
// one part of its members and passes over the other rows: the parts of a region run side by side on one XCD (workgroups go
// to the eight XCDs in turn), whose L2 has the rows then.  Up to eight parts: the grid in memory, which the others take, costs
// about as much as reading the rows that often (4,096 ranks x 16 channels x 64 snapshots in four parts 545 -> 369 us per call).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_rate_region(HangArgs a) {
  extern __shared__ ulonglong2 s_cell[];                               // [cap] cells | sums of every member | bitmap
  const int db = a.sb - a.pb;
  const u32 part = (blockIdx.x >> 3) & ((1u << db) - 1);
  const u32 tid = threadIdx.x, lane = lane_id(), wave = tid / CCLD_WAVE, reg = db ? ((blockIdx.x >> 3) >> db) * 8 + (blockIdx.x & 7) : blockIdx.x;
  const u32 per_member = a.n_ch * a.n_snap, room = per_member << a.sb, cap = per_member << a.pb, words = (cap + 31) / 32, members = 1u << a.pb;
  const u32 cell0 = db ? part * cap : 0u;
  if (reg >= a.n_regions || ((u64)reg << a.sb) + (db ? (u64)part << a.pb : 0) >= a.n_members) return;
  u64* s_sum = reinterpret_cast<u64*>(s_cell + cap);
  u32* s_bits = reinterpret_cast<u32*>(s_sum + 4 * members);
  __shared__ u32 s_cells;
  const u64 p0 = ((u64)reg << a.sb) + (db ? (u64)part << a.pb : 0);
  const RegionRows R = region_rows(a, reg, room);
  const u32 n = R.n;
  const ulonglong2* __restrict__ rows = a.part_row + (u64)reg * room;
  for (u32 i = tid; i < words; i += THREADS) s_bits[i] = 0;
  for (u32 i = tid; i < 4 * members; i += THREADS) s_sum[i] = 0;
  if (tid == 0) s_cells = 0;
  __syncthreads();
  constexpr int U = 4;
  typedef u64 u64x2 __attribute__((ext_vector_type(2)));
  for (u32 i0 = tid; i0 < n; i0 += THREADS * U) {
    u64x2 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * THREADS < n) {
        const u64x2* row = reinterpret_cast<const u64x2*>(rows + region_row(R, i0 + u * THREADS));
        v[u] = db ? *row : __builtin_nontemporal_load(row);
      }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u * THREADS >= n) continue;
      const u32 k = ((u32)v[u].x & ((1u << SPLIT_CELL_BITS) - 1)) - cell0;
      if (k >= cap) continue;                                          // another part's
      s_cell[k] = make_ulonglong2(v[u].x >> SPLIT_CELL_BITS, v[u].y);
      atomicOr(&s_bits[k >> 5], 1u << (k & 31));
    }
  }
  __syncthreads();
  u32 cells = 0;
  for (u32 i = tid; i < words; i += THREADS) cells += (u32)__popc(s_bits[i]);
  cells = wave_sum(cells);
  if (lane == 0) atomicAdd(&s_cells, cells);
  const u64 left = a.n_members - p0;
  const u32 n_ser = (u32)(left < members ? left : members) * a.n_ch;
  for (u32 q = wave; q < n_ser; q += THREADS / CCLD_WAVE) {
    RateSums t{0, 0, 0, 0};
    const ulonglong2* cells_q = s_cell + q * a.n_snap;
    rate_series(a.n_snap, lane, t, [&](u32 s, u64* seq, u64* cnt) { *seq = cells_q[s].x; *cnt = cells_q[s].y; });
    unsigned long long* sum = reinterpret_cast<unsigned long long*>(s_sum + 4 * (q / a.n_ch));
    if (lane == 0) {
      if (t.ops_s) atomicAdd(&sum[0], (unsigned long long)t.ops_s);
      if (t.chg_s) atomicAdd(&sum[1], (unsigned long long)t.chg_s);
      if (t.ops_r) atomicAdd(&sum[2], (unsigned long long)t.ops_r);
      if (t.chg_r) atomicAdd(&sum[3], (unsigned long long)t.chg_r);
    }
  }
  __syncthreads();
  for (u32 i = tid; i < members && i < left; i += THREADS)
    store_rates(a, p0 + i, RateSums{s_sum[4 * i], s_sum[4 * i + 1], s_sum[4 * i + 2], s_sum[4 * i + 3]});
  if (tid == 0) atomicAdd((unsigned long long*)&a.counters[CNT_NCELL], (unsigned long long)s_cells);
}

// a rate (ops / changes, rank); changes == 0 means "no rate" and loses against everything
struct RateCand { u64 ops, chg; u32 rank; };
__device__ __forceinline__ bool rate_less(const RateCand& x, const RateCand& y) {
  if (x.chg == 0) return false;
  if (y.chg == 0) return true;
  const u128 l = (u128)x.ops * (u128)y.chg, r = (u128)y.ops * (u128)x.chg;
  if (l != r) return l < r;
  return x.rank < y.rank;
}

constexpr u32 RATE_MANY = 4;
__device__ __forceinline__ void rate_load(const HangArgs& a, u64 p, RateCand& snd, RateCand& rcv) {
  const u32 rk = a.T.members[p];
  snd = {(u64)RPAIR(a, CCLD_RATE_OPS_SEND, p), (u64)RPAIR(a, CCLD_RATE_CHANGES_SEND, p), rk};
  rcv = {(u64)RPAIR(a, CCLD_RATE_OPS_RECV, p), (u64)RPAIR(a, CCLD_RATE_CHANGES_RECV, p), rk};
}
// member p of communicator c: the caller's row, and the best of both kinds
__device__ __forceinline__ void rate_use(const HangArgs& a, u32 c, u64 p, const RateCand& snd, const RateCand& rcv, RateCand (&best)[2]) {
  if (a.out_pair && p < a.pair_cap) {
    auto put = [&](int col, u64 v) { store_agent(&a.out_pair[(u64)col * a.pair_cap + p], (i64)v); };
    put(CCLD_RATE_RANK, snd.rank); put(CCLD_RATE_COMM, c);
    put(CCLD_RATE_OPS_SEND, snd.ops); put(CCLD_RATE_CHANGES_SEND, snd.chg);
    put(CCLD_RATE_OPS_RECV, rcv.ops); put(CCLD_RATE_CHANGES_RECV, rcv.chg);
  }
  if (rate_less(snd, best[0])) best[0] = snd;
  if (rate_less(rcv, best[1])) best[1] = rcv;
}
__device__ __forceinline__ void rate_root_of(const HangArgs& a, i64* __restrict__ rate_root, u32 c, const RateCand& snd, const RateCand& rcv) {
  const RateCand both = rate_less(snd, rcv) ? snd : rcv;
  const i64 row[CCLD_RCOMM_NCOL] = {(i64)c, snd.chg ? (i64)snd.rank : (i64)CCLD_NO_RANK, rcv.chg ? (i64)rcv.rank : (i64)CCLD_NO_RANK,
                                    both.chg ? (i64)both.rank : (i64)CCLD_NO_RANK};
  if (a.out_comm && c < a.comm_cap)
    for (int col = 0; col < CCLD_RCOMM_NCOL; ++col) store_agent(&a.out_comm[(u64)col * a.comm_cap + c], row[col]);
  rate_root[c] = row[CCLD_RCOMM_ROOT];
}
// A communicator of more than SHORT_COMM members, by a workgroup.
template <u32 AHEAD>
__device__ __forceinline__ void rate_long(const HangArgs& a, i64* __restrict__ rate_root, RateCand (&s_best)[2][256], const LongComm& L) {
  const u32 tid = threadIdx.x, c = L.comm, off = L.off, n = L.size;
  RateCand best[2] = {{0, 0, 0xFFFFFFFFu}, {0, 0, 0xFFFFFFFFu}};
  // AHEAD members of a thread at a time: a load behind the stores of the member before would wait for those too, and they go
  // past the caches (16,384 members: the call 129.5 us with one at a time, 110 so, 119.6 with plain stores and a report of its own;
  // 60,000: 308, 235 and 273; 1,008 members in four communicators each: 81.0, 80.7 and 83.1)
  u32 q = tid;
  for (; AHEAD > 1 && q - tid + 256 * AHEAD <= n; q += 256 * AHEAD) {
    RateCand snd[AHEAD], rcv[AHEAD];
#pragma unroll
    for (u32 u = 0; u < AHEAD; ++u) rate_load(a, (u64)off + q + u * 256, snd[u], rcv[u]);
#pragma unroll
    for (u32 u = 0; u < AHEAD; ++u) rate_use(a, c, (u64)off + q + u * 256, snd[u], rcv[u], best);
  }
  for (; q < n; q += 256) {
    RateCand snd, rcv;
    rate_load(a, (u64)off + q, snd, rcv);
    rate_use(a, c, (u64)off + q, snd, rcv, best);
  }
  s_best[0][tid] = best[0]; s_best[1][tid] = best[1];
  __syncthreads();
  u32 w = 128;
  while (w >= 1 && w >= n) w >>= 1;             // threads beyond the members have nothing to add
  for (; w >= 1; w >>= 1) {
    if (tid < 2 * w) {                          // both kinds side by side
      const u32 k = tid >= w, i = k ? tid - w : tid;
      if (rate_less(s_best[k][i + w], s_best[k][i])) s_best[k][i] = s_best[k][i + w];
    }
    __syncthreads();
  }
  if (tid == 0) rate_root_of(a, rate_root, c, s_best[0][0], s_best[1][0]);
}
// The member of minimal SendRate, RecvRate, and of both kinds of every communicator, and the caller's tables, stored past the
// caches, since the last workgroup reports.  A long communicator (they are listed, and begin first) has a workgroup; of the others
// each has S.lanes lanes of a wavefront, a member to a lane.  With a workgroup each, most of a wavefront idled, and all of them
// arrived for the report at words that take 35 to 50 ns per arrival (the call, us: 262,144 communicators of two members 579 -> 205,
// 32,768 131 -> 82, 8,192 60.2 -> 49.5; 16,384 ranks in 3,200 83 -> 79, 4,096 of 16 83.4 -> 77.5; of 64 members, which take a wavefront,
// 79 -> 78; of 65 and more, which have a workgroup, as before).
constexpr u32 RATE_BLOCKS = 2048;               // most workgroups of the short ones
struct RateShape { const LongComm* longs; u32 n_long, lanes; };
template <u32 AHEAD>
__global__ __launch_bounds__(256) void k_rate_comm(HangArgs a, i64* __restrict__ rate_root, RateShape S) {
  __shared__ RateCand s_best[2][256];
  __shared__ u32 s_last;
  if (!hang_rows_ok(a)) {                        // the same for every thread
  } else if (blockIdx.x < S.n_long) {
    rate_long<AHEAD>(a, rate_root, s_best, S.longs[blockIdx.x]);
  } else {
    const u32 per = 256 / S.lanes, l = threadIdx.x % S.lanes, end = a.T.n_comms;
    for (u32 c0 = (blockIdx.x - S.n_long) * per; c0 < end; c0 += (gridDim.x - S.n_long) * per) {
      const u32 c = c0 + threadIdx.x / S.lanes, at = c < end ? c : end - 1, n = a.T.size[at], off = a.T.member_off[at];
      const bool mine = c < end && n <= SHORT_COMM;
      RateCand best[2] = {{0, 0, 0xFFFFFFFFu}, {0, 0, 0xFFFFFFFFu}};
      if (mine && l < n) {
        RateCand snd, rcv;
        rate_load(a, (u64)off + l, snd, rcv);
        rate_use(a, c, (u64)off + l, snd, rcv, best);
      }
      for (u32 m = 1; m < S.lanes; m <<= 1)
#pragma unroll
        for (u32 k = 0; k < 2; ++k) {
          const RateCand o{shfl_xor_u64(best[k].ops, m), shfl_xor_u64(best[k].chg, m), (u32)__shfl_xor((int)best[k].rank, (int)m, CCLD_WAVE)};
          if (rate_less(o, best[k])) best[k] = o;
        }
      if (mine && l == 0) rate_root_of(a, rate_root, c, best[0], best[1]);
    }
  }
  if (last_arrival(a.arrivals, gridDim.x, &s_last)) report_and_clear(a);
}
static void launch_rate_comm(hipStream_t st, const ccld_ctx* c, const HangArgs& a) {
  const RateShape S{c->long_comms, c->n_long_comms, c->short_lanes};
  // (the short ones' workgroups pass over the long ones' numbers)
  const u32 n = c->topo.n_comms, per = 256 / S.lanes, blocks = n > S.n_long ? std::min((n + per - 1) / per, RATE_BLOCKS) : 0u;
  // where nobody has the members for it, several at a time would only cost registers (5 wavefronts per SIMD instead of 8)
  if (c->max_comm_size >= 256 * RATE_MANY) hipLaunchKernelGGL(k_rate_comm<RATE_MANY>, dim3(S.n_long + blocks), dim3(256), 0, st, a, c->rate_root, S);
  else hipLaunchKernelGGL(k_rate_comm<1>, dim3(S.n_long + blocks), dim3(256), 0, st, a, c->rate_root, S);
}
// ---- Probing Frames (Section 5.1) -------------------------------------------------------------------
struct FrameArgs {
  const uint8_t* frames;
  const u32* frame_rank;
  u64 n_frames;
  u32 n_ch, snap;
  int mb;
  DeviceTopology T;
  u64 n_members;
  u64* last;          // [n_members][CCLD_FRAME_CHANNELS][2]
  u64* frame_of;      // [n_ranks] call << 32 | frame of the rank in that call
  u64* status;        // call << 8 | worst error of that call
  u32 call;           // number of this call: marks of earlier calls need no clearing
  u32* arrivals;
  u64 *host, ticket;
};
// errors in the order in which they are reported
enum { FRAME_DUPLICATE = 1, FRAME_RANGE, FRAME_NOT_MEMBER, FRAME_UNKNOWN_COMM };

// is rank r (r < n_ranks) a member of communicator c?
__device__ __forceinline__ bool is_member(const DeviceTopology& T, int mb, u32 c, u32 r) {
  if (T.rank_memb4) {
    const uint4 m = reinterpret_cast<const uint4*>(T.rank_memb4)[r];
    return c == (m.x >> mb) || c == (m.y >> mb) || c == (m.z >> mb) || c == (m.w >> mb);
  }
  return slot_of(T, c, r) >= 0;
}
struct BlockHead { u32 comm; bool written; u64 opc; };
__device__ __forceinline__ BlockHead block_head(const uint8_t* F, u32 b) {
  const uint4 t = *reinterpret_cast<const uint4*>(F + CCLD_FRAME_HEADER_BYTES + b * CCLD_FRAME_BLOCK_BYTES);
  return {t.x, (t.y & 1u) != 0, (u64)t.z | ((u64)t.w << 32)};
}
__device__ __forceinline__ uint4 block_counts(const uint8_t* F, u32 b, u32 ch) {
  return *reinterpret_cast<const uint4*>(F + CCLD_FRAME_HEADER_BYTES + b * CCLD_FRAME_BLOCK_BYTES + 16 + ch * 16);
}

// The validity checks, before anything is remembered: one wavefront per frame, lane = 8 * block + channel.  All of a frame's
// loads are in flight together; what the kernel takes (4 us at 4,096 frames) is that one trip to memory, the lookup
// of the rank and the exchange that finds a second frame of it.
__global__ __launch_bounds__(256) void k_frames_check(FrameArgs a) {
  const u32 lane = lane_id();
  const u64 f = (u64)blockIdx.x * 4 + threadIdx.x / CCLD_WAVE;
  if (f >= a.n_frames) return;
  const uint8_t* F = a.frames + f * CCLD_FRAME_BYTES;
  const u32 b = lane / CCLD_FRAME_CHANNELS, ch = lane % CCLD_FRAME_CHANNELS;
  const u32 r = a.frame_rank[f];
  const u32 nch = reinterpret_cast<const u32*>(F)[4];
  const BlockHead hd = block_head(F, b);
  const uint4 cnt = block_counts(F, b, ch);
  u32 worst = nch > CCLD_FRAME_CHANNELS ? FRAME_RANGE : 0;
  if (lane == 0 && r < a.T.n_ranks) {
    const u64 mark = (u64)a.call << 32;
    const u64 old = atomicExch((unsigned long long*)&a.frame_of[r], (unsigned long long)(mark | f));
    if ((old >> 32) == a.call && worst < FRAME_DUPLICATE) worst = FRAME_DUPLICATE;
  }
  if (hd.written) {
    u32 e = 0;
    if (hd.comm >= a.T.n_comms) e = FRAME_UNKNOWN_COMM;
    else if (r >= a.T.n_ranks || !is_member(a.T, a.mb, hd.comm, r)) e = FRAME_NOT_MEMBER;
    else if (ch < nch && (cnt.y | cnt.w) != 0) e = FRAME_RANGE;            // counts of 2^32 and more
    worst = e > worst ? e : worst;
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) { const u32 o = __shfl_xor(worst, m, CCLD_WAVE); worst = o > worst ? o : worst; }
  if (lane == 0 && worst) atomicMax((unsigned long long*)a.status, (unsigned long long)((u64)a.call << 8 | worst));
}

// A thread per member slot and channel: the latest kernel of the member's communicator in its rank's frame replaces
// what is remembered, unless that is newer, and the snapshot row is written from it.
__device__ __forceinline__ void frame_row(const FrameArgs& a, const ccld_snapshot_rows& o, u64 i) {
  const u64 p = i / CCLD_FRAME_CHANNELS;
  const u32 ch = (u32)(i % CCLD_FRAME_CHANNELS);
  if (p >= a.n_members) return;
  const u32 r = a.T.members[p], c = a.T.member_comm[p];
  const u64 of = a.frame_of[r];
  u64* L = a.last + i * 2;
  u64 l0 = L[0], l1 = L[1];
  if ((of >> 32) == a.call) {
    const uint8_t* F = a.frames + (of & 0xFFFFFFFFu) * CCLD_FRAME_BYTES;
    const u32 nch = reinterpret_cast<const u32*>(F)[4];
    bool any = false;
    u32 at = 0;
    u64 opc = 0;
#pragma unroll
    for (u32 b = 0; b < CCLD_FRAME_BLOCKS; ++b) {
      const BlockHead hd = block_head(F, b);
      if (hd.written && hd.comm == c && (!any || hd.opc >= opc)) { any = true; at = b; opc = hd.opc; }
    }
    if (any && opc >= l0) {
      const uint4 cnt = block_counts(F, at, ch);
      l0 = opc;
      l1 = ch < nch ? (u64)cnt.x | ((u64)cnt.z << 32) : 0ull;
      L[0] = l0; L[1] = l1;
    }
  }
  if (ch >= a.n_ch) return;
  const u64 k = p * a.n_ch + ch;
  store_agent(&o.snap[k], a.snap); store_agent(&o.rank[k], r); store_agent(&o.comm[k], c); store_agent(&o.channel[k], ch);
  store_agent(reinterpret_cast<i64*>(&o.seq_posted[k]), (i64)l0);
  store_agent(&o.chunks_sent[k], (u32)l1); store_agent(&o.chunks_recv[k], (u32)(l1 >> 32));
}
// The last workgroup reports, so the rows are stored past the caches.  (With a report in a launch of its own a call took 1 us more:
// 4,096 frames 43.5 and 42.5 us with the GPU waited for; of 65,536 ranks 116.3 and 114.4 one after another.)
__global__ __launch_bounds__(256) void k_frame_rows(FrameArgs a, ccld_snapshot_rows o) {
  __shared__ u32 s_last;
  const u64 s = *a.status;
  if ((s >> 8) != a.call) frame_row(a, o, (u64)blockIdx.x * 256 + threadIdx.x);
  if (!last_arrival(a.arrivals, gridDim.x, &s_last) || threadIdx.x != 0) return;
  __hip_atomic_store(a.host, report_word((s >> 8) == a.call ? s & 0xFF : 0, a.ticket), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace ccld

#define HIP_TRY(x) do { if ((x) != hipSuccess) { (void)hipGetLastError(); return CCLD_E_HIP; } } while (0)

static ccld_status hang_status(uint64_t bits) {
  if (bits & DS_UNKNOWN_COMM) return CCLD_E_UNKNOWN_COMM;
  if (bits & DS_NOT_MEMBER) return CCLD_E_RANK_NOT_MEMBER;
  if (bits & DS_RANGE) return CCLD_E_RANGE;
  if (bits & DS_DUPLICATE) return CCLD_E_DUPLICATE_KEY;
  if (bits & DS_SNAPSHOT_GAP) return CCLD_E_SNAPSHOT_GAP;
  return CCLD_OK;
}

// Device memory the hang and rate passes work in, beyond their inputs and outputs: either carved from the
// context's workspace or from the library's static device array.
struct HangScratch {
  uint64_t* counters;        // [CNT_COUNT]
  uint32_t* fill;            // [SPLIT_REGIONS]
  bool* clear;               // counters and fill are clear (kept from pass to pass), or null: not known
  uint64_t* cell;            // [n_cell][2]
  uint32_t* cnt;             // presence bitmap, one bit per cell
  int64_t* pair;             // [CCLD_HPAIR_NCOL][n_members]
  int64_t* hcomm;            // [CCLD_HCOMM_NCOL][n_comms]
  int32_t* wait_slot;        // [n_members]
  uint8_t* cand;             // [n_members]
  uint64_t* layer_max;       // [n_members]
  SortBuffers sb;            // root list sort: n_members items
  uint64_t* keyC;            // [n_members]
  uint64_t sort_cap;
  ulonglong2* split_row;     // [n_cell] regrouped rows, or null: no room for them
  ulonglong2* split_final;   // [n_members * n_channels]
  uint8_t* stage;            // [stage_bytes] staging for host-resident rows, or null
  uint64_t stage_bytes;
};

static HangScratch scratch_of_context(ccld_ctx* c, bool on_device) {
  HangScratch S;
  S.counters = c->h_counters; S.fill = reinterpret_cast<uint32_t*>(c->h_counters + CNT_COUNT); S.clear = &c->h_clear; S.cell = c->h_cell; S.cnt = c->h_cnt; S.pair = c->h_pair; S.hcomm = c->h_comm;
  S.wait_slot = c->h_wait_slot; S.cand = c->h_cand; S.layer_max = c->h_layer_max;
  S.sb.key[0] = c->sb.key[0]; S.sb.idx[0] = c->sb.idx[0]; S.sb.key[1] = c->sb.key[1]; S.sb.idx[1] = c->sb.idx[1];
  S.sb.table = c->table2; S.sb.totals = c->totals2;
  S.keyC = c->keyC; S.sort_cap = c->sort_cap; S.stage = c->h_stage; S.stage_bytes = c->snap_cap * 32;
  // rows that are on the device already leave the staging area free
  S.split_row = on_device ? reinterpret_cast<ulonglong2*>(c->h_stage) : nullptr;
  S.split_final = reinterpret_cast<ulonglong2*>(c->h_cell);
  return S;
}

// Stages host-resident rows; the arguments that the passes share.
static hipError_t snapshot_args(ccld_ctx* c, const HangScratch& S, const ccld_snapshots* sn, uint64_t n_rows,
                                uint64_t n_cell, HangArgs& a) {
  hipStream_t st = c->stream;
  std::memset(&a, 0, sizeof(a));
  hipError_t e = hipSuccess;
  if (sn->on_device) {
    a.snap = sn->snap; a.rank = sn->rank; a.comm = sn->comm; a.channel = sn->channel;
    a.seq_posted = sn->seq_posted; a.sent = sn->chunks_sent; a.recv = sn->chunks_recv;
  } else if (n_rows) {
    uint64_t* d_seq = (uint64_t*)S.stage;
    uint32_t* d32 = (uint32_t*)(d_seq + n_rows);
    const uint32_t* src[6] = {sn->snap, sn->rank, sn->comm, sn->channel, sn->chunks_sent, sn->chunks_recv};
    if ((e = hipMemcpyAsync(d_seq, sn->seq_posted, 8 * n_rows, hipMemcpyHostToDevice, st)) != hipSuccess) return e;
    for (int i = 0; i < 6; ++i)
      if ((e = hipMemcpyAsync(d32 + i * n_rows, src[i], 4 * n_rows, hipMemcpyHostToDevice, st)) != hipSuccess) return e;
    a.seq_posted = d_seq; a.snap = d32; a.rank = d32 + n_rows; a.comm = d32 + 2 * n_rows; a.channel = d32 + 3 * n_rows;
    a.sent = d32 + 4 * n_rows; a.recv = d32 + 5 * n_rows;
  }
  a.n_rows = n_rows; a.n_snap = sn->n_snapshots; a.n_ch = sn->n_channels; a.T = c->topo; a.mb = c->kf.mb; a.n_members = c->n_members;
  a.cell = S.cell; a.cnt = S.cnt; a.pair = S.pair; a.hcomm = S.hcomm; a.wait_slot = S.wait_slot;
  a.cand = S.cand; a.layer_max = S.layer_max; a.counters = S.counters;
  a.stall_snapshots = c->p.stall_snapshots; a.fifo_depth = c->p.fifo_depth;
  a.n_cell = n_cell; a.mark = reinterpret_cast<uint32_t*>(S.layer_max);
  a.root_key = reinterpret_cast<int64_t*>(S.keyC); a.cb = c->kf.cb; a.host = c->h_pinned; a.arrivals = c->arrivals;
  return hipSuccess;
}

constexpr size_t PART_LDS = (size_t)PART_CHUNK * (16 + 4 + 4);
hipError_t ccld::allow_lds_hang() {
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(&k_hang_part), PART_LDS);
  return e != hipSuccess ? e : allow_lds(reinterpret_cast<const void*>(&k_rate_region<1024>), RATE_LDS);
}

// Clears the grid's presence counts and places every row in its cell.
static hipError_t place_snapshots(ccld_ctx* c, const HangScratch& S, const ccld_snapshots* sn, uint64_t n_rows,
                                  uint64_t n_cell, HangArgs& a, bool exact) {
  hipStream_t st = c->stream;
  hipError_t e = hipSuccess;
  c->prof.begin(CCLD_PROF_HANG_PLACE);
  if ((e = hipMemsetAsync(S.counters, 0, sizeof(uint64_t) * CNT_COUNT, st)) != hipSuccess) return e;
  a.exact = exact ? 1 : 0;
  if (exact) e = hipMemsetAsync(S.cnt, 0, sizeof(uint32_t) * ((n_cell + 31) / 32), st);
  else e = hipMemsetAsync(S.cell, 0xFF, 16 * n_cell, st);
  if (e != hipSuccess) return e;
  // large grids whose rows are already on the device (the staging area is free then) are placed in two steps
  int rb = 16;
  while ((n_cell >> rb) >= PART_REGIONS && rb < 31) ++rb;
  const uint64_t n_regions = (n_cell + ((uint64_t)1 << rb) - 1) >> rb;
  const bool two_step = !exact && sn->on_device && S.stage && n_rows >= ((uint64_t)1 << 20) && n_cell < ((uint64_t)1 << 31) &&
                        (n_regions << rb) * 20 <= S.stage_bytes && n_regions <= PART_REGIONS;
  if (n_rows && two_step) {
    a.rb = rb; a.n_regions = (uint32_t)n_regions;
    a.part_pay = reinterpret_cast<ulonglong2*>(S.stage);
    a.part_idx = reinterpret_cast<uint32_t*>(S.stage + (n_regions << rb) * 16);
    a.part_fill = S.cnt;                       // the presence bitmap is not in use in this mode
    if ((e = hipMemsetAsync(S.cnt, 0, sizeof(uint32_t) * PART_REGIONS, st)) != hipSuccess) return e;
    uint64_t g = (n_rows + PART_CHUNK - 1) / PART_CHUNK; if (g > 1024) g = 1024;
    uint64_t chunk = (n_rows + g - 1) / g;
    chunk = (chunk + PART_CHUNK - 1) / PART_CHUNK * PART_CHUNK;
    hipLaunchKernelGGL(k_hang_part, dim3((uint32_t)g), dim3(PART_THREADS), PART_LDS, st, a, chunk);
    const uint32_t wpr = (uint32_t)((((uint64_t)1 << rb) + PLACE_ROWS - 1) / PLACE_ROWS);
    const uint64_t g2 = 8 * ((n_regions + 7) / 8) * wpr;
    hipLaunchKernelGGL(k_hang_place_regions, dim3((uint32_t)g2), dim3(256), 0, st, a, wpr);
  } else if (n_rows) {
    uint64_t g = (n_rows + 255) / 256; if (g > 4096) g = 4096;
    if (exact) hipLaunchKernelGGL(k_hang_place<true>, dim3((uint32_t)g), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(k_hang_place<false>, dim3((uint32_t)g), dim3(256), 0, st, a);
  }
  c->prof.split(CCLD_PROF_HANG_PLACE, CCLD_PROF_HANG);
  return hipSuccess;
}

// argument checks shared by the hang entry points; *n_cell receives the grid size
static ccld_status check_hang_args(ccld_ctx* c, const ccld_snapshots* sn, uint64_t n_rows, ccld_hang_result* o,
                                   uint64_t* n_cell) {
  if (!c || !sn || !o) return CCLD_E_NULL;
  o->n_root = o->n_pair = o->n_hung_comm = 0;
  o->status = CCLD_OK;
  if (!o->root && o->root_cap) return o->status = CCLD_E_NULL;
  if (n_rows && (!sn->snap || !sn->rank || !sn->comm || !sn->channel || !sn->seq_posted || !sn->chunks_sent || !sn->chunks_recv))
    return o->status = CCLD_E_NULL;
  if (sn->n_snapshots == 0 || sn->n_channels == 0) return o->status = CCLD_E_BAD_ARG;
  *n_cell = c->n_members * sn->n_channels * sn->n_snapshots;
  return CCLD_OK;
}

// The regions of a grid: false where its rows are not regrouped.  As many regions as one workgroup each keeps the chip
// busy with (129 to 256; more cost the split pass an atomic each per round), as far as a region fits LDS.
// parts: the cells of a region may be taken in up to 2^parts passes over its rows.
static bool split_regions(HangArgs& a, const HangScratch& S, size_t (*lds)(u32, u32, int), size_t lds_max, int parts) {
  const uint64_t per_member = (uint64_t)a.n_ch * a.n_snap;
  if (!S.split_row || !a.n_rows || a.n_cell >= (1ull << 31) || a.n_snap < 2 || a.n_snap > 16384 || a.n_ch > 1024) return false;
  int sb = 0;
  while (((a.n_members - 1) >> sb) >= SPLIT_REGIONS / 2) ++sb;
  while (sb > 0 && (per_member << sb) > (1ull << SPLIT_CELL_BITS)) --sb;
  int pb = sb;
  while (pb > 0 && lds(a.n_ch, a.n_snap, pb) > lds_max) --pb;
  // smaller regions rather than several parts, as far as the regions go
  while (sb > pb && ((a.n_members - 1) >> (sb - 1)) < SPLIT_REGIONS) --sb;
  const uint64_t regions = ((a.n_members - 1) >> sb) + 1;
  if (regions > SPLIT_REGIONS || per_member > (1ull << SPLIT_CELL_BITS) || lds(a.n_ch, a.n_snap, pb) > lds_max || sb - pb > parts ||
      (!S.clear && regions > a.n_cell / 32 + 1)) return false;
  a.sb = sb; a.pb = pb; a.n_regions = (uint32_t)regions; a.snap_inv = (uint32_t)((1ull << 32) / a.n_snap + 1);
  a.part_row = S.split_row; a.final = S.split_final; a.part_fill = S.fill; a.leave_clear = S.clear != nullptr; a.ends = S.clear != nullptr;
  return true;
}
template <int THREADS, int U>
static void launch_split_of(hipStream_t st, const HangArgs& a) {
  constexpr uint32_t CHUNK = THREADS * U;
  uint64_t g = std::min<uint64_t>((a.n_rows + CHUNK - 1) / CHUNK, 512);
  const uint64_t chunk = ((a.n_rows + g - 1) / g + CHUNK - 1) / CHUNK * CHUNK;
  g = (a.n_rows + chunk - 1) / chunk;
  hipLaunchKernelGGL(HIP_KERNEL_NAME(k_hang_split<THREADS, U>), dim3((uint32_t)g), dim3(THREADS), CHUNK * 18, st, a, chunk);
}
static void launch_split(hipStream_t st, const HangArgs& a, const HangScratch& S) {
  if (!S.clear || !*S.clear) hipLaunchKernelGGL(k_hang_clear, dim3(1), dim3(SPLIT_REGIONS), 0, st, a);
  if (S.clear) *S.clear = false;       // until the pass has reported
  // few rows: smaller rounds, for the sake of more workgroups
  if (a.n_rows < (1u << 18)) launch_split_of<512, 2>(st, a);
  else launch_split_of<512, 6>(st, a);
}
static void launch_scan(hipStream_t st, const HangArgs& a) {
  const uint64_t want = std::max<uint64_t>((a.n_rows + 255) / 256, 1);
  hipLaunchKernelGGL(k_hang_last, dim3((uint32_t)std::min<uint64_t>(want, 2048)), dim3(256), 0, st, a);
  if (a.n_rows) hipLaunchKernelGGL(k_hang_scan<4>, dim3((uint32_t)std::min<uint64_t>(want, 4096)), dim3(256), 0, st, a);
  hipLaunchKernelGGL(k_hang_pairs, dim3((uint32_t)((a.n_members * PAIR_LANES + 255) / 256)), dim3(256), 0, st, a);
}

// Data errors of a pass that counted the cells with a row: fewer of them than valid rows means that some cell has two.
static uint64_t snapshot_status(const ccld_ctx* c, uint64_t n_rows, uint64_t n_cell) {
  const uint64_t bits = c->h_pinned[CNT_STATUS], cells = c->h_pinned[CNT_NCELL];
  return bits ? bits : cells < n_rows ? (uint64_t)DS_DUPLICATE : cells < n_cell ? (uint64_t)DS_SNAPSHOT_GAP : 0;
}

// the hang pass proper, on scratch memory S (n_cell cells and n_rows rows fit it)
static ccld_status locate_hang_on(ccld_ctx* c, const HangScratch& S, const ccld_snapshots* sn, uint64_t n_rows,
                                  uint64_t n_cell, ccld_hang_result* o) {
  hipStream_t st = c->stream;
  HangArgs a;
  const uint32_t nm = (uint32_t)c->n_members;
  HIP_TRY(snapshot_args(c, S, sn, n_rows, n_cell, a));
  a.out_pair = o->pair; a.pair_cap = o->pair_cap; a.out_comm = o->comm; a.comm_cap = o->comm_cap;
  a.out_root = o->root; a.root_cap = o->root_cap;
  for (bool split = split_regions(a, S, region_lds, SPLIT_LDS, 0);; split = false) {
    a.ticket = take_ticket(c);
    if (!split) { a.final = reinterpret_cast<ulonglong2*>(S.cell); a.leave_clear = 0; if (S.clear) *S.clear = false; }
    c->prof.begin(CCLD_PROF_HANG_PLACE);
    if (split) {
      launch_split(st, a, S);
      const size_t lds = region_lds(a.n_ch, a.n_snap, a.sb);
      if (((uint64_t)a.n_ch * a.n_snap << a.sb) >= 8192) hipLaunchKernelGGL(k_hang_region<1024>, dim3(a.n_regions), dim3(1024), lds, st, a);
      else hipLaunchKernelGGL(k_hang_region<256>, dim3(a.n_regions), dim3(256), lds, st, a);
    } else {
      launch_scan(st, a);
    }
    c->prof.split(CCLD_PROF_HANG_PLACE, CCLD_PROF_HANG);
    const dim3 comms(c->topo.n_comms);
    a.hops_known = c->max_comm_size <= 4096;
    if (c->max_comm_size <= 256) hipLaunchKernelGGL(HIP_KERNEL_NAME(k_hang_comm<256, 1>), comms, dim3(256), 0, st, a);
    else if (c->max_comm_size <= 4096) hipLaunchKernelGGL(HIP_KERNEL_NAME(k_hang_comm<1024, 4>), comms, dim3(1024), 0, st, a);
    else hipLaunchKernelGGL(HIP_KERNEL_NAME(k_hang_comm<1024, 0>), comms, dim3(1024), 0, st, a);
    hipLaunchKernelGGL(k_hang_final, dim3((nm + 255) / 256), dim3(256), 0, st, a);
    c->prof.end(CCLD_PROF_HANG);
    HIP_TRY(hipGetLastError());
    HIP_TRY(wait_report(c));
    if (split && S.clear) *S.clear = true;
    if (!split || !(c->h_pinned[CNT_STATUS] & DS_SUSPECT)) break;      // an operation counter too large to be regrouped
  }
  const uint64_t bits = snapshot_status(c, n_rows, n_cell);
  if (bits) { c->prof.collect(); return o->status = hang_status(bits); }
  const uint32_t n_root = (uint32_t)c->h_pinned[CNT_NCAND];
  o->n_root = n_root;
  o->n_hung_comm = c->h_pinned[CNT_NALERT];
  o->n_pair = c->n_members;
  if (n_root > ROOTS_ONE && o->root_cap) {
    const SortBuffers& sb2 = S.sb;
    if (n_root > S.sort_cap) return o->status = CCLD_E_CAPACITY;
    KeySource ks; ks.key = S.keyC; ks.head = 0; ks.cap = n_root; ks.squeeze = 0; ks.hi_shift = 0; ks.lo_bits = 0; ks.lo_mask = 0; ks.lo_sub = 0;
    const int r = radix_sort_pairs(st, ks, n_root, sb2, c->kf.cb + c->rank_bits);
    if (r < 0) return o->status = CCLD_E_HIP;
    hipLaunchKernelGGL(k_hang_root_emit, dim3((n_root + 255) / 256), dim3(256), 0, st, a, (const u32*)sb2.idx[r], n_root);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(st));
  }
  c->prof.collect();
  if (o->n_root > o->root_cap || (o->pair && o->pair_cap < c->n_members) || (o->comm && o->comm_cap < c->topo.n_comms))
    o->status = CCLD_W_TRUNCATED;
  return o->status;
}

extern "C" ccld_status ccld_locate_hang(ccld_ctx* c, const ccld_snapshots* sn, uint64_t n_rows, ccld_hang_result* o) {
  uint64_t n_cell = 0;
  const ccld_status s = check_hang_args(c, sn, n_rows, o, &n_cell);
  if (s != CCLD_OK) return s;
  if (n_cell > c->snap_cap || n_rows > c->snap_cap) return o->status = CCLD_E_CAPACITY;
  c->chain_ready = false;       // the root list is sorted in the window's sort buffers
  c->inc_ok = false;
  return locate_hang_on(c, scratch_of_context(c, sn->on_device), sn, n_rows, n_cell, o);
}

// ---- hang location on the library's static device array ------------------------------------------------
// For callers that cannot allocate device memory and whose context was created without room for snapshots:
// the grid, the per-member and per-communicator tables and the sort buffers of the hang pass live in one
// file-scope device array.  Every GPU the library runs on holds its own copy of the array at its own
// address until the process ends; the address is looked up once per device.
static __device__ __align__(256) unsigned char scratch[CCLD_STATIC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
unsigned char* g_scratch_ptr[MAX_DEVICES] = {nullptr};     // device address of `scratch` on each GPU
std::mutex g_scratch_mutex;

// device address of the static array on the current device; the first call per device looks it up and allows the kernels
// their LDS
ccld_status device_scratch(unsigned char** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) { (void)hipGetLastError(); return CCLD_E_HIP; }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    for (hipError_t e : {allow_lds_window(), allow_lds_grid(), allow_lds_segments(), allow_lds_hang()})
      if (e != hipSuccess) { (void)hipGetLastError(); return CCLD_E_HIP; }
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { (void)hipGetLastError(); return CCLD_E_HIP; }
    g_scratch_ptr[dev] = static_cast<unsigned char*>(p);
  }
  *out = g_scratch_ptr[dev];
  return CCLD_OK;
}

// Bump allocator over the static array; regions start on 256-byte boundaries and are padded to them.
struct StaticCarver {
  unsigned char* base; uint64_t off;
  template <class T> T* take(uint64_t count) {
    T* p = reinterpret_cast<T*>(base + off);
    off += (count * sizeof(T) + 255) & ~(uint64_t)255;
    return p;
  }
};
}  // namespace

// called by ccld_create with the context's device current: no other call comes first on a device
ccld_status ccld_device_init() {
  unsigned char* p = nullptr;
  return device_scratch(&p);
}

extern "C" ccld_status ccld_locate_hang_static(ccld_ctx* c, const ccld_snapshots* sn, uint64_t n_rows,
                                               ccld_hang_result* o) {
  uint64_t n_cell = 0;
  const ccld_status s = check_hang_args(c, sn, n_rows, o, &n_cell);
  if (s != CCLD_OK) return s;
  unsigned char* base = nullptr;
  const ccld_status sa = device_scratch(&base);
  if (sa != CCLD_OK) return o->status = sa;
  const uint64_t nm = c->n_members, nc = c->topo.n_comms;
  // every size below is bounded before it is multiplied: a grid beyond the array is refused here
  if (n_cell > CCLD_STATIC_SCRATCH_BYTES / 16 || n_rows > CCLD_STATIC_SCRATCH_BYTES / 32 ||
      nm > CCLD_STATIC_SCRATCH_BYTES / 64 || nc > CCLD_STATIC_SCRATCH_BYTES / 64)
    return o->status = CCLD_E_CAPACITY;
  HangScratch S;
  StaticCarver w{base, 0};
  S.counters = w.take<uint64_t>(CNT_COUNT);
  S.cell = w.take<uint64_t>(2 * n_cell);
  S.cnt = w.take<uint32_t>(n_cell / 32 + 1);
  S.fill = S.cnt; S.clear = nullptr;
  S.pair = w.take<int64_t>((uint64_t)CCLD_HPAIR_NCOL * nm);
  S.hcomm = w.take<int64_t>((uint64_t)CCLD_HCOMM_NCOL * nc);
  S.wait_slot = w.take<int32_t>(nm);
  S.cand = w.take<uint8_t>(nm);
  S.layer_max = w.take<uint64_t>(nm);
  for (int i = 0; i < 2; ++i) { S.sb.key[i] = w.take<uint64_t>(nm + 1); S.sb.idx[i] = w.take<uint32_t>(nm + 1); }
  S.sb.table = w.take<uint32_t>(sort_table_words(nm + 1));
  S.sb.totals = w.take<uint32_t>(SORT_RADIX);
  S.keyC = w.take<uint64_t>(nm + 1);
  S.sort_cap = nm;
  S.stage = sn->on_device ? nullptr : w.take<uint8_t>(n_rows * 32);
  S.stage_bytes = sn->on_device ? 0 : n_rows * 32;
  if (w.off > CCLD_STATIC_SCRATCH_BYTES) return o->status = CCLD_E_CAPACITY;
  // the grid's cells take the regrouped rows, what is left of the array the final states
  const uint64_t final_bytes = nm * sn->n_channels * 16;
  S.split_row = w.off + final_bytes <= CCLD_STATIC_SCRATCH_BYTES ? reinterpret_cast<ulonglong2*>(S.cell) : nullptr;
  S.split_final = reinterpret_cast<ulonglong2*>(base + w.off);
  return locate_hang_on(c, S, sn, n_rows, n_cell, o);
}

extern "C" ccld_status ccld_progress_rates(ccld_ctx* c, const ccld_snapshots* sn, uint64_t n_rows, ccld_rate_result* o) {
  if (!c || !sn || !o) return CCLD_E_NULL;
  o->n_pair = o->n_comm = 0;
  o->status = CCLD_OK;
  if (n_rows && (!sn->snap || !sn->rank || !sn->comm || !sn->channel || !sn->seq_posted || !sn->chunks_sent || !sn->chunks_recv))
    return o->status = CCLD_E_NULL;
  if (sn->n_snapshots == 0 || sn->n_channels == 0) return o->status = CCLD_E_BAD_ARG;
  const uint64_t n_cell = c->n_members * sn->n_channels * sn->n_snapshots;
  if (n_cell > c->snap_cap || n_rows > c->snap_cap) return o->status = CCLD_E_CAPACITY;
  hipStream_t st = c->stream;
  HangArgs a;
  const HangScratch S = scratch_of_context(c, sn->on_device);
  const uint32_t nm = (uint32_t)c->n_members;
  auto tables = [&](bool checked) {
    a.checked = checked ? 1 : 0;
    a.out_pair = o->pair; a.pair_cap = o->pair_cap; a.out_comm = o->comm; a.comm_cap = o->comm_cap;
    a.ticket = take_ticket(c);
    launch_rate_comm(st, c, a);
    c->prof.end(CCLD_PROF_HANG);
  };
  HIP_TRY(snapshot_args(c, S, sn, n_rows, n_cell, a));
  bool split = split_regions(a, S, rate_region_lds, RATE_LDS, RATE_PARTS);
  if (split) {
    c->prof.begin(CCLD_PROF_HANG_PLACE);
    launch_split(st, a, S);
    c->prof.split(CCLD_PROF_HANG_PLACE, CCLD_PROF_HANG);
    const size_t lds = rate_region_lds(a.n_ch, a.n_snap, a.pb);
    const uint32_t groups = a.sb == a.pb ? a.n_regions : ((a.n_regions + 7) / 8 * 8) << (a.sb - a.pb);
    if (((uint64_t)a.n_ch * a.n_snap << a.pb) >= 2048) {
      hipLaunchKernelGGL(k_rate_region<1024>, dim3(groups), dim3(1024), lds, st, a);
    } else {
      hipLaunchKernelGGL(k_rate_region<256>, dim3(groups), dim3(256), lds, st, a);
    }
    tables(false);
    HIP_TRY(hipGetLastError());
    HIP_TRY(wait_report(c));
    *S.clear = true;
    const uint64_t bits = snapshot_status(c, n_rows, n_cell);
    split = !(bits & DS_SUSPECT);
    if (split && bits) { c->prof.collect(); return o->status = hang_status(bits); }
  }
  if (!split) {
    a.leave_clear = 0;
    *S.clear = false;
    // One row per cell is the normal case: the rows are placed without the presence bitmap (its atomics are a
    // third of the placement's time) and the per-member pass looks for cells that nobody wrote.  If it finds one
    // and no row was refused for a worse reason, or if the row count already rules the normal case out, the
    // placement is repeated with the bitmap, which tells duplicates from gaps.
    for (bool exact = n_rows != n_cell;; exact = true) {
      HIP_TRY(place_snapshots(c, S, sn, n_rows, n_cell, a, exact));
      if (nm) hipLaunchKernelGGL(k_rate_pairs, dim3((nm + 3) / 4), dim3(256), 0, st, a);
      HIP_TRY(hipGetLastError());
      HIP_TRY(hipMemcpyAsync(c->h_pinned, S.counters, sizeof(uint64_t) * CNT_COUNT, hipMemcpyDeviceToHost, st));
      HIP_TRY(hipStreamSynchronize(st));
      if (exact || c->h_pinned[CNT_STATUS] != (uint64_t)DS_SUSPECT) break;
      c->prof.end(CCLD_PROF_HANG);
    }
    if (c->h_pinned[CNT_STATUS]) { c->prof.end(CCLD_PROF_HANG); c->prof.collect(); return o->status = hang_status(c->h_pinned[CNT_STATUS]); }
    tables(true);
    HIP_TRY(hipGetLastError());
    HIP_TRY(wait_report(c));
  }
  c->prof.collect();
  o->n_pair = c->n_members;
  o->n_comm = c->topo.n_comms;
  if (o->pair_cap < o->n_pair && o->pair) o->status = CCLD_W_TRUNCATED;
  if (o->comm_cap < o->n_comm && o->comm) o->status = CCLD_W_TRUNCATED;
  return o->status;
}

extern "C" ccld_status ccld_reset_frames(ccld_ctx* c) {
  if (!c) return CCLD_E_NULL;
  HIP_TRY(hipMemsetAsync(c->f_last, 0, sizeof(uint64_t) * 2 * CCLD_FRAME_CHANNELS * c->n_members, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  return CCLD_OK;
}

extern "C" ccld_status ccld_decode_frames(ccld_ctx* c, const ccld_frames* fr, const ccld_snapshot_rows* rows,
                                          uint64_t* n_rows) {
  if (!c || !fr || !rows || !n_rows) return CCLD_E_NULL;
  *n_rows = 0;
  if (fr->n_channels == 0 || fr->n_channels > CCLD_FRAME_CHANNELS) return CCLD_E_BAD_ARG;
  if (fr->n_frames && (!fr->frames || !fr->frame_rank)) return CCLD_E_NULL;
  if (!rows->snap || !rows->rank || !rows->comm || !rows->channel || !rows->seq_posted || !rows->chunks_sent ||
      !rows->chunks_recv)
    return CCLD_E_NULL;
  const uint64_t n_out = c->n_members * fr->n_channels;
  if (n_out > rows->capacity) return CCLD_E_CAPACITY;
  hipStream_t st = c->stream;
  FrameArgs a;
  std::memset(&a, 0, sizeof(a));
  if (fr->on_device) {
    if ((reinterpret_cast<uintptr_t>(fr->frames) & 15) != 0) return CCLD_E_BAD_ARG;
    a.frames = fr->frames; a.frame_rank = fr->frame_rank;
  } else if (fr->n_frames) {
    // staging buffer of the snapshot rows: 32 bytes per row of capacity
    const uint64_t need = fr->n_frames * (CCLD_FRAME_BYTES + 4);
    if (need > c->snap_cap * 32) return CCLD_E_CAPACITY;
    uint8_t* d = c->h_stage;
    HIP_TRY(hipMemcpyAsync(d, fr->frames, fr->n_frames * CCLD_FRAME_BYTES, hipMemcpyHostToDevice, st));
    uint32_t* dr = reinterpret_cast<uint32_t*>(d + fr->n_frames * CCLD_FRAME_BYTES);
    HIP_TRY(hipMemcpyAsync(dr, fr->frame_rank, fr->n_frames * 4, hipMemcpyHostToDevice, st));
    a.frames = d; a.frame_rank = dr;
  }
  a.n_frames = fr->n_frames; a.n_ch = fr->n_channels; a.snap = fr->snapshot; a.mb = c->kf.mb; a.T = c->topo;
  a.n_members = c->n_members; a.last = c->f_last; a.frame_of = c->f_frame; a.status = c->f_status; a.call = ++c->f_call;
  a.arrivals = c->arrivals; a.host = c->h_pinned; a.ticket = take_ticket(c);
  c->prof.begin(CCLD_PROF_FRAMES);
  const uint64_t slots = c->n_members * CCLD_FRAME_CHANNELS;
  if (fr->n_frames) hipLaunchKernelGGL(k_frames_check, dim3((uint32_t)((fr->n_frames + 3) / 4)), dim3(256), 0, st, a);
  hipLaunchKernelGGL(k_frame_rows, dim3((uint32_t)((slots + 255) / 256)), dim3(256), 0, st, a, *rows);
  c->prof.end(CCLD_PROF_FRAMES);
  HIP_TRY(hipGetLastError());
  HIP_TRY(wait_report(c, 1));
  c->prof.collect();
  switch (c->h_pinned[0]) {
    case 0: break;
    case FRAME_UNKNOWN_COMM: return CCLD_E_UNKNOWN_COMM;
    case FRAME_NOT_MEMBER: return CCLD_E_RANK_NOT_MEMBER;
    case FRAME_RANGE: return CCLD_E_RANGE;
    default: return CCLD_E_DUPLICATE_KEY;
  }
  *n_rows = n_out;
  return CCLD_OK;
}
