// Root cause and secondary effects among the late-entry flags of an analysed window (Section 4.2.2: an
// anomaly may propagate across ranks; the location step separates the rank that triggered it from the
// ranks that pass it on).  Per late-entry flag: the operation its rank ran just before (found by binary
// search over the rounds of each of the rank's communicators, on the rank's own timestamps), the member
// whose late arrival ended that operation late (its parent flag), then the links from parent to parent up to
// the chain's first flag.
#include <algorithm>
#include <cstring>

#include "ccld_internal.h"
#include "grid.h"
#include "report.h"
#include "rows.h"
#include "window_kernels.h"

using namespace ccld;

namespace ccld {

constexpr i64 T_INFLIGHT = INT64_MAX;

struct ChainArgs {
  const u64* key;            // squeezed keys in (communicator, counter, rank) order
  const u32* idx;            // window slot of each sorted record
  WindowRows win;
  GridView grid;             // the window's records on the grid placement
  const u64* flag_key;       // grid placement: table row << 32 | member slot of the k-th flag
  const u32* flag_stage;     // grid placement: cell | kind << 16 of the k-th flag at flag_pos[k]
  SqueezedFormat sf;
  DeviceTopology T;
  const i64* seg;            // the analysis's collective table
  u64 seg_cap;
  u32 n_seg;
  const uint8_t* rec_flag;   // by sorted position
  const i64* flag_lag;       // [2][cap_n] lags of the flagged records by sorted position
  u64 cap_n;
  const u32* flag_pos;       // sorted position of the k-th flag; on the grid placement where its lags are
  u32 n_flag;
  u32* comm_first;           // [n_comms + 1] first table row of each communicator (sorted window; the grid's layout has it)
  u32* parent;               // [n_flag] parent flag or ~0
  u64* link;                 // [n_flag] an ancestor, links up to it << 32; a root leads to itself
  i64* per_rank;             // cleared by the parent kernel, or null
  u32* arrivals;
  u64* counters;             // CNT_CHAIN_LOOP is set if some links lead round in a loop
  u32 *anc[2], *dist[2];     // [n_flag] each: ancestors and links to them, where they do
};

// first row of the collective table of every communicator (the table is ordered by communicator)
__global__ __launch_bounds__(256) void k_chain_comm_rows(ChainArgs a) {
  const u32 c = blockIdx.x * 256 + threadIdx.x;
  if (c > a.T.n_comms) return;
  const i64* COMM = a.seg + (u64)CCLD_SEG_COMM * a.seg_cap;
  u32 lo = 0, hi = a.n_seg;
  while (lo < hi) { const u32 m = (lo + hi) >> 1; if ((u32)COMM[m] < c) lo = m + 1; else hi = m; }
  a.comm_first[c] = lo;
}

// The record of member slot `slot` in table row `row`: its times, or false if there is none.  *pos: its sorted
// position, or its row among the partitioned ones.
template <bool GRID>
__device__ __forceinline__ bool chain_record_of(const ChainArgs& a, u32 comm, u32 row, u32 slot, u32 size, u32* pos, i64* te, i64* tx) {
  if (GRID) {
    const CommLayout L = a.grid.lay[comm];
    const u32 k = row - L.seg_base, fr = k / L.rpb;
    const u32 li = a.grid.cell_row[L.cell_base + k * L.size + slot];
    if (li == GRID_EMPTY) return false;
    *pos = L.cell_base + fr * L.rpb * L.size + li;
    const Rec r = unpack_row(a.grid.rows[*pos], a.grid.hdr->ref, a.grid.wide);
    *te = r.t_enter; *tx = r.t_exit;
    return true;
  }
  const u32 first = (u32)a.seg[(u64)CCLD_SEG_FIRST * a.seg_cap + row], n = (u32)a.seg[(u64)CCLD_SEG_N * a.seg_cap + row];
  u32 p = first + slot;
  if (n != size) {
    const u64 mmask = ((u64)1 << a.sf.mb) - 1;
    u32 lo = first, hi = first + n;
    while (lo < hi) { const u32 m = (lo + hi) >> 1; if ((u32)(a.key[m] & mmask) < slot) lo = m + 1; else hi = m; }
    if (lo >= first + n || (u32)(a.key[lo] & mmask) != slot) return false;
    p = lo;
  }
  *pos = p;
  const Rec r = load_rec(a.win, a.idx[p]);
  *te = r.t_enter; *tx = r.t_exit;
  return true;
}
struct ChainFlag { u32 comm, slot, row, kind; };       // row: of the collective table, grid placement only
template <bool GRID>
__device__ __forceinline__ ChainFlag chain_flag(const ChainArgs& a, u32 k) {
  ChainFlag f;
  if (GRID) {
    const u64 w = a.flag_key[k];
    f.row = (u32)(w >> 32); f.slot = (u32)w; f.kind = a.flag_stage[a.flag_pos[k]] >> 16;
    f.comm = (u32)a.seg[(u64)CCLD_SEG_COMM * a.seg_cap + f.row];
  } else {
    const u32 j = a.flag_pos[k];
    const u64 key = a.key[j];
    f.row = 0; f.slot = (u32)(key & (((u64)1 << a.sf.mb) - 1)); f.comm = (u32)(key >> (a.sf.mb + a.sf.ws)); f.kind = a.rec_flag[j];
  }
  return f;
}

// The parent of a late entry: PARENT_LANES lanes per flag.  What takes the time is chains of dependent loads (the binary
// search over a communicator's rounds makes two per step), so the lanes of a flag search its rank's communicators side by side,
// SEARCH_LANES to a communicator: one looks at the middle and two at the middles of both halves, which is two steps of
// the same search at a time.  The flag list is searched in PARENT_LANES + 1 parts at a time.
// Up to PARENT_FEW flags 16 lanes take a flag and four a communicator; more flags, whose searches hide each other's loads, have
// four lanes, each with a communicator of its own.  The two cost the same somewhere between 16,400 and 32,800 flags on the grid and
// later on sorted windows; at the line, the last power of two before, they differ by a tenth.  (us with 16 and with 4 lanes: 7,900
// flags 16.5 and 20.5, 16,400 19.7 and 21.4, 32,800 35.9 and 25.2, 145,000 110 and 41; the whole call on sorted windows, where the
// lanes also share the walk over a collective's records: 9,800 flags 53 and 56, 12,600 59 and 63, 48,800 81 and 67, 377,000 392 and
// 208; beside a world communicator of 4,096 members 1,300 flags 89 and 178, 12,500 110 and 189, 48,700 194 and 223, 717,000 2,779
// and 2,075.  With the walk in every lane those were 560 to 4,630 us.)
constexpr u32 PARENT_FEW = 1u << 14;
struct ChainBefore { i64 exit, enter; u32 comm, row; bool have; };
template <bool GRID, u32 PARENT_LANES, u32 SEARCH_LANES>
__device__ __forceinline__ void chain_parent(const ChainArgs& a, u32 k, u32 l) {
  const u32 group0 = lane_id() & ~(PARENT_LANES - 1);
  const ChainFlag F = chain_flag<GRID>(a, k);
  u32 parent = ~0u;
  if (F.kind & CCLD_FLAG_LATE_ENTER) {
    const u32 r = a.T.members_sorted[a.T.member_off[F.comm] + F.slot];
    u32 own = a.flag_pos[k];
    i64 t, own_exit;
    if (GRID) { if (!chain_record_of<GRID>(a, F.comm, F.row, F.slot, a.T.size[F.comm], &own, &t, &own_exit)) t = 0; }
    else t = load_rec(a.win, a.idx[own]).t_enter;
    // the operation this rank ran just before: per communicator of the rank the last round that the rank left
    // before t (its rounds are in time order; a round without a record of the rank is skipped), then the latest
    ChainBefore B{0, 0, 0, 0, false};
    const auto take = [&](const ChainBefore& f) {
      if (f.have && (!B.have || f.exit > B.exit || (f.exit == B.exit && (f.enter > B.enter || (f.enter == B.enter && f.comm > B.comm))))) B = f;
    };
    const u32 sub = l % SEARCH_LANES, lane0 = lane_id() - sub;
    for (u32 q = a.T.rank_comm_off[r] + l / SEARCH_LANES; q < a.T.rank_comm_off[r + 1]; q += PARENT_LANES / SEARCH_LANES) {
      const u32 c2 = a.T.rank_comms[q], slot2 = a.T.rank_slots[q], size2 = a.T.size[c2];
      u32 lo, hi;
      if (GRID) { lo = a.grid.lay[c2].seg_base; hi = lo + a.grid.lay[c2].rounds; }
      else { lo = a.comm_first[c2]; hi = a.comm_first[c2 + 1]; }
      ChainBefore f{0, 0, c2, 0, false};
      while (lo < hi) {                          // the same in all lanes of the communicator
        const u32 mid = (lo + hi) >> 1;
        const u32 from = sub == 2 ? mid + 1 : lo, to = sub == 1 ? mid : hi, at = sub == 0 ? mid : (from + to) >> 1;
        // the nearest round at or below the middle in which the rank has a record
        u32 probe = at, pos = 0;
        i64 te = 0, tx = 0;
        bool here = false;
        if (SEARCH_LANES == 1 || (sub < 3 && from < to))
          while (true) {
            here = chain_record_of<GRID>(a, c2, probe, slot2, size2, &pos, &te, &tx);
            if (here || probe == from) break;
            --probe;
          }
        const bool ok = here && pos != own && tx != T_INFLIGHT && tx <= t;
        const u32 word = (here ? 1u : 0u) | (ok ? 2u : 0u);
        // one step of the search with what lane k of the communicator found, at the middle of [lo, hi)
        auto step = [&](u32 k) {
          const u32 w = (u32)__shfl((int)word, (int)(lane0 + k), CCLD_WAVE), p = (u32)__shfl((int)probe, (int)(lane0 + k), CCLD_WAVE);
          const i64 e = (i64)shfl_u64((u64)te, (int)(lane0 + k)), x = (i64)shfl_u64((u64)tx, (int)(lane0 + k));
          const u32 m = (lo + hi) >> 1;
          if (w & 2u) { f.have = true; f.row = p; f.exit = x; f.enter = e; lo = m + 1; }
          else if (!(w & 1u)) lo = m + 1;        // no record of the rank in [lo, m]
          else hi = p;
        };
        const u32 lo0 = lo;
        step(0);
        if (SEARCH_LANES > 1 && lo < hi && (lo != lo0 || hi == mid)) step(lo != lo0 ? 2u : 1u);      // the half that a lane has looked at
      }
      take(f);
    }
#pragma unroll
    for (u32 m = SEARCH_LANES; m < PARENT_LANES; m <<= 1) {
      const ChainBefore o{(i64)shfl_xor_u64((u64)B.exit, m), (i64)shfl_xor_u64((u64)B.enter, m), __shfl_xor(B.comm, m, CCLD_WAVE),
                          __shfl_xor(B.row, m, CCLD_WAVE), __shfl_xor((int)B.have, m, CCLD_WAVE) != 0};
      take(o);
    }
    if (B.have) {
      // who ended it late: the late entry with the largest lag (ties: smallest rank = first in rank order)
      bool any = false;
      i64 m_lag = 0;
      if (GRID) {
        u32 lo = 0, hi = a.n_flag;               // the collective's first flag: every lane of the group looks at one point
        while (lo < hi) {
          const u32 step = (hi - lo) / (PARENT_LANES + 1), m = lo + (l + 1) * step;
          const bool less = step ? (u32)(a.flag_key[m] >> 32) < B.row : (lo + l < hi && (u32)(a.flag_key[lo + l] >> 32) < B.row);
          const u32 n_less = (u32)__popcll((ballot64(less) >> group0) & ((1u << PARENT_LANES) - 1));
          if (step) {
            if (n_less < PARENT_LANES) hi = lo + (n_less + 1) * step;
            if (n_less) lo = lo + n_less * step + 1;
          } else {
            lo += n_less;
            if (n_less < PARENT_LANES) hi = lo;
          }
        }
        for (; lo < a.n_flag && (u32)(a.flag_key[lo] >> 32) == B.row; ++lo) {
          const u32 at = a.flag_pos[lo];
          if (!((a.flag_stage[at] >> 16) & CCLD_FLAG_LATE_ENTER)) continue;
          const i64 lag = a.flag_lag[at];
          if (!any || lag > m_lag) { any = true; parent = lo; m_lag = lag; }
        }
      } else {
        const u32 first = (u32)a.seg[(u64)CCLD_SEG_FIRST * a.seg_cap + B.row], n = (u32)a.seg[(u64)CCLD_SEG_N * a.seg_cap + B.row];
        u32 m_pos = 0;                           // the lanes share its records, the widest collective's 4,096 and more
        for (u32 p = first + l; p < first + n; p += PARENT_LANES)
          if (a.rec_flag[p] & CCLD_FLAG_LATE_ENTER) {
            const i64 lag = a.flag_lag[p];
            if (!any || lag > m_lag) { any = true; m_pos = p; m_lag = lag; }
          }
#pragma unroll
        for (u32 m = 1; m < PARENT_LANES; m <<= 1) {
          const bool o_any = __shfl_xor((int)any, m, CCLD_WAVE) != 0;
          const i64 o_lag = (i64)shfl_xor_u64((u64)m_lag, m);
          const u32 o_pos = __shfl_xor(m_pos, m, CCLD_WAVE);
          if (o_any && (!any || o_lag > m_lag || (o_lag == m_lag && o_pos < m_pos))) { any = true; m_lag = o_lag; m_pos = o_pos; }
        }
        if (any) {
          u32 lo = 0, hi = a.n_flag;
          while (lo < hi) { const u32 m = (lo + hi) >> 1; if (a.flag_pos[m] < m_pos) lo = m + 1; else hi = m; }
          parent = lo;
        }
      }
    }
  }
  if (l == 0) {
    a.parent[k] = parent;
    a.link[k] = parent == ~0u ? (u64)k : (u64)parent | (u64)1 << 32;
  }
}
constexpr u32 PARENT_BLOCKS = 1u << 20;
template <bool GRID, u32 PARENT_LANES, u32 SEARCH_LANES>
__global__ __launch_bounds__(256) void k_chain_parent(ChainArgs a) {
  const u32 t = blockIdx.x * 256 + threadIdx.x, threads = gridDim.x * 256;
  if (a.per_rank)
    for (u64 i = t; i < (u64)CCLD_CHR_NCOL * a.T.n_ranks; i += threads) a.per_rank[i] = 0;
  for (u64 k = t / PARENT_LANES; k < a.n_flag; k += threads / PARENT_LANES) chain_parent<GRID, PARENT_LANES, SEARCH_LANES>(a, (u32)k, t % PARENT_LANES);
}
template <bool GRID>
static void launch_parents(hipStream_t st, const ChainArgs& a) {
  auto go = [&](auto kernel, uint32_t lanes) {
    hipLaunchKernelGGL(kernel, dim3((uint32_t)std::min<uint64_t>(((uint64_t)a.n_flag * lanes + 255) / 256, PARENT_BLOCKS)), dim3(256), 0, st, a);
  };
  if (a.n_flag <= PARENT_FEW) go(k_chain_parent<GRID, 16, 4>, 16);
  else go(k_chain_parent<GRID, 4, 1>, 4);
}

// Links that lead round in a loop: jumps in step, 2^i links after the i-th, from one pair of arrays into the other.
__global__ __launch_bounds__(256) void k_chain_init(ChainArgs a) {
  const u32 k = blockIdx.x * 256 + threadIdx.x;
  if (a.per_rank)
    for (u64 i = k; i < (u64)CCLD_CHR_NCOL * a.T.n_ranks; i += (u64)gridDim.x * 256) a.per_rank[i] = 0;
  if (k >= a.n_flag) return;
  const u32 p = a.parent[k];
  a.anc[0][k] = p == ~0u ? k : p;
  a.dist[0][k] = p == ~0u ? 0u : 1u;
}
__global__ __launch_bounds__(256) void k_chain_jump(ChainArgs a) {
  const u32 k = blockIdx.x * 256 + threadIdx.x;
  if (k >= a.n_flag) return;
  const u32 a1 = a.anc[0][k], a2 = a.anc[0][a1];
  a.anc[1][k] = a2;
  a.dist[1][k] = a.dist[0][k] + (a2 != a1 ? a.dist[0][a1] : 0u);
}
// column[idx] += 1 for every lane with `on`, one atomic per distinct idx in the wavefront: a faulty rank's thousands
// of entries would otherwise queue up at one address.  Called by every active lane of the wavefront.
__device__ __forceinline__ void wave_count_by_index(i64* column, u32 idx, bool on) {
  u64 todo = ballot64(on);
  while (todo) {
    const u32 leader = (u32)__builtin_ctzll(todo);
    const u32 v = (u32)__shfl((int)idx, (int)leader, CCLD_WAVE);
    const u64 same = ballot64(on && idx == v);
    if (lane_id() == leader) atomicAdd((unsigned long long*)&column[v], (unsigned long long)__popcll(same));
    todo &= ~same;
  }
}
// Every flag follows its links to the root and keeps what it finds, in place: a link always leads to some ancestor, so
// whatever the others have written by then is right, nobody waits for anybody, and the links double in length as all
// flags go on at once (one launch in place of a jump per doubling: 14 for 8,000 flags).  Each step takes the link past the
// caches that the XCDs do not share.
// Parents end earlier, so links do not lead back; records that contradict their own clocks can make them.  Then there is
// no root and what a flag finds would depend on who was faster, so the call is repeated with LOOPED on the ancestors that
// the kernels below find, the same ones every time.
template <bool GRID, bool LOOPED>
__device__ __forceinline__ void chain_emit(const ChainArgs& a, u32 k, i64* chain, u64 chain_cap) {
  auto rank_at = [&](u32 flag) -> u32 {
    const ChainFlag f = chain_flag<GRID>(a, flag);
    return a.T.members_sorted[a.T.member_off[f.comm] + f.slot];
  };
  u64 v = (u64)load_agent(reinterpret_cast<const i64*>(&a.link[k]));
  if (LOOPED) {
    v = (u64)a.anc[0][k] | (u64)a.dist[0][k] << 32;
  } else {
    while (true) {
      const u32 up = (u32)v;
      const u64 w = (u64)load_agent(reinterpret_cast<const i64*>(&a.link[up]));
      if ((w >> 32) == 0) break;                 // up is a root: every other link has a length, a loop's included
      v = (u64)(u32)w | ((v >> 32) + (w >> 32)) << 32;
      if ((v >> 32) > a.n_flag) { store_agent(reinterpret_cast<i64*>(&a.counters[CNT_CHAIN_LOOP]), 1); break; }        // more links than flags: a loop
      store_agent(reinterpret_cast<i64*>(&a.link[k]), (i64)v);
    }
  }
  const u32 root = (u32)v, p = a.parent[k];
  i64* per_rank = a.per_rank;
  const u32 root_rank = rank_at(root);
  if (k < chain_cap) {
    auto put = [&](int col, i64 x) { store_agent(&chain[(u64)col * chain_cap + k], x); };
    put(CCLD_CHN_PARENT, p == ~0u ? -1 : (i64)p);
    put(CCLD_CHN_ROOT, (i64)root);
    put(CCLD_CHN_ROOT_RANK, (i64)root_rank);
    put(CCLD_CHN_DEPTH, (i64)(v >> 32));
  }
  if (per_rank) {
    const bool on = (chain_flag<GRID>(a, k).kind & CCLD_FLAG_LATE_ENTER) != 0;
    const u32 n_ranks = a.T.n_ranks;
    const u32 mine = on ? rank_at(k) : 0u;
    wave_count_by_index(per_rank + (u64)CCLD_CHR_ROOT_ENTRIES * n_ranks, mine, on && p == ~0u);
    wave_count_by_index(per_rank + (u64)CCLD_CHR_SECONDARY_ENTRIES * n_ranks, mine, on && p != ~0u);
    wave_count_by_index(per_rank + (u64)CCLD_CHR_CAUSED * n_ranks, root_rank, on);
  }
}
// The last workgroup reports, so the table is stored past the caches.
template <bool GRID, bool LOOPED>
__global__ __launch_bounds__(256) void k_chain_emit(ChainArgs a, i64* chain, u64 chain_cap, u64* host, u64 ticket) {
  const u32 k = blockIdx.x * 256 + threadIdx.x;
  if (k < a.n_flag) chain_emit<GRID, LOOPED>(a, k, chain, chain_cap);
  report_counters(a.counters, a.arrivals, host, ticket);
}

}  // namespace ccld

#define HIP_TRY(x) do { if ((x) != hipSuccess) { (void)hipGetLastError(); return CCLD_E_HIP; } } while (0)

extern "C" ccld_status ccld_flag_chains(ccld_ctx* c, const ccld_window_result* w, ccld_chain_result* o) {
  if (!c || !w || !o) return CCLD_E_NULL;
  o->n_chain = 0;
  o->status = CCLD_OK;
  if (o->chain_cap && !o->chain) return o->status = CCLD_E_NULL;
  // the tables and the order of the most recent analysis must still be there
  if (!c->chain_ready || w->seg != c->last_seg || w->seg_cap != c->last_seg_cap || w->n_seg != c->last_n_seg ||
      w->n_flag != c->last_n_flag)
    return o->status = CCLD_E_BAD_ARG;
  if (w->n_seg > w->seg_cap) return o->status = CCLD_E_CAPACITY;      // a truncated table cannot be searched
  hipStream_t st = c->stream;
  const uint32_t n_flag = (uint32_t)c->last_n_flag, n_ranks = c->topo.n_ranks;
  o->n_chain = n_flag;
  if (o->per_rank && !n_flag) HIP_TRY(hipMemsetAsync(o->per_rank, 0, sizeof(int64_t) * CCLD_CHR_NCOL * (uint64_t)n_ranks, st));
  if (!n_flag) {
    launch_report(st, c->counters, c->h_pinned, take_ticket(c));
    HIP_TRY(hipGetLastError());
    HIP_TRY(wait_report(c));
  } else {
    ChainArgs a;
    std::memset(&a, 0, sizeof(a));
    const bool grid = c->last_grid;
    a.key = c->sb.key[c->sorted_buf]; a.idx = c->sb.idx[c->sorted_buf]; a.win = c->last_win; a.sf = c->sf; a.T = c->topo;
    a.grid.lay = (const CommLayout*)c->g_lay; a.grid.rows = c->g_rows; a.grid.cell_row = c->g_cell_row; a.grid.wide = c->win_wide;
    a.grid.hdr = (const GridHeader*)c->g_hdr;
    a.flag_key = c->flag_key; a.flag_stage = c->flag_stage;
    a.seg = w->seg; a.seg_cap = w->seg_cap; a.n_seg = (uint32_t)w->n_seg;
    a.rec_flag = c->last_rec_flag; a.flag_lag = c->flag_lag; a.cap_n = c->cap; a.flag_pos = c->flag_pos; a.n_flag = n_flag;
    a.comm_first = c->chain_first; a.parent = c->chain_parent;
    a.link = reinterpret_cast<uint64_t*>(c->range_c);                // scratch that the analysis no longer needs
    a.per_rank = o->per_rank;
    const dim3 blocks((n_flag + 255) / 256);
    a.arrivals = c->arrivals; a.counters = c->counters;                      // CNT_CHAIN_LOOP: cleared by the analysis; its flags lead round or they do not
    take_ticket(c);
    if (grid) {
      launch_parents<true>(st, a);
      hipLaunchKernelGGL(HIP_KERNEL_NAME(k_chain_emit<true, false>), blocks, dim3(256), 0, st, a, o->chain, o->chain_cap, c->h_pinned, c->ticket);
    } else {
      hipLaunchKernelGGL(k_chain_comm_rows, dim3((c->topo.n_comms + 256) / 256), dim3(256), 0, st, a);
      launch_parents<false>(st, a);
      hipLaunchKernelGGL(HIP_KERNEL_NAME(k_chain_emit<false, false>), blocks, dim3(256), 0, st, a, o->chain, o->chain_cap, c->h_pinned, c->ticket);
    }
    HIP_TRY(hipGetLastError());
    HIP_TRY(wait_report(c));
    if (c->h_pinned[CNT_CHAIN_LOOP]) {
      a.anc[0] = reinterpret_cast<uint32_t*>(a.link); a.dist[0] = a.anc[0] + n_flag;
      a.anc[1] = c->alert_list; a.dist[1] = c->alert_ncand;
      take_ticket(c);
      hipLaunchKernelGGL(k_chain_init, blocks, dim3(256), 0, st, a);
      for (uint64_t reach = 1; reach < n_flag; reach *= 2) {
        hipLaunchKernelGGL(k_chain_jump, blocks, dim3(256), 0, st, a);
        std::swap(a.anc[0], a.anc[1]);
        std::swap(a.dist[0], a.dist[1]);
      }
      if (grid) hipLaunchKernelGGL(HIP_KERNEL_NAME(k_chain_emit<true, true>), blocks, dim3(256), 0, st, a, o->chain, o->chain_cap, c->h_pinned, c->ticket);
      else hipLaunchKernelGGL(HIP_KERNEL_NAME(k_chain_emit<false, true>), blocks, dim3(256), 0, st, a, o->chain, o->chain_cap, c->h_pinned, c->ticket);
      HIP_TRY(hipGetLastError());
      HIP_TRY(wait_report(c));
    }
  }
  if (o->n_chain > o->chain_cap) o->status = CCLD_W_TRUNCATED;
  return o->status;
}
