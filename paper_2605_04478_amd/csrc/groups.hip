// The end of an analysis, in two launches: what follows from the statistics alone (k_window_lists: the slow-detection rules
// of Eq. 1-4 per detection group, the flag list of a window on the grid placement, the blame order, a few hang alerts; workgroups of their own
// for each), then the group table and the report of the counters (k_window_end).
#include <algorithm>

#include "alerts.h"
#include "blame_order.h"
#include "device_utils.h"
#include "grid.h"
#include "report.h"
#include "rows.h"
#include "window_kernels.h"

namespace ccld {

constexpr u32 GC_THREADS = 512;
constexpr u32 GC_BATCH = 64;               // groups still averaging their baseline that one walk handles
constexpr u32 GC_WALK = 8;                 // rows of one thread per step of that walk (a byte of a word each)
constexpr u32 GC_NONE = 0xFFFFFFFFu;

// ---- groups -------------------------------------------------------------------------------------------------
// first row of the table with communicator >= c, found by one wavefront (64 probes per step)
__device__ __forceinline__ u32 first_row_of(const i64* __restrict__ comm, u32 n, u32 c, u32 lane) {
  u32 lo = 0, hi = n;
  while (hi - lo > CCLD_WAVE) {
    const u32 step = (hi - lo) / CCLD_WAVE;
    const u32 at = lo + lane * step;
    const u32 k = (u32)__popcll(ballot64((u32)comm[at] < c));       // probes before the answer: a prefix
    const u32 nlo = k ? lo + (k - 1) * step + 1 : lo;
    hi = k < CCLD_WAVE ? lo + k * step : hi;
    lo = nlo;
  }
  const u32 at = lo + lane;
  return lo + (u32)__popcll(ballot64(at < hi && (u32)comm[at] < c));
}

// Eq. 1: baseline = mean of T_max over the first m rounds (m = min(tbase_rounds, rounds within the warm-up
// span)); Eq. 2: the window's round of largest T_max - T_min; Eq. 3: slow iff (T_max - T_base) / T_base > theta;
// Eq. 4: P = (T_max - T_min) / (T_max - T_base) against alpha / beta; repetition counter.  All ratios
// cross-multiplied.
// The rows of a communicator are read as a 2-byte (op, size class) code and an 8-byte range, twice (largest range
// of every group, then the first row that attains it): 10 bytes per collective from memory, the second time from
// the L2.  Groups whose baseline is not frozen yet and that have new rounds are walked once more, 4,096 rows a step from the
// first new one on, and only until the last of them has its baseline: 100 rounds by default, which a communicator watched
// for long has in its first few thousand rows (see the walk for the times).
// At 8.4M collectives of 1,088 communicators this replaces a three-pass sort of the collectives by group (0.23 ms)
// and a wavefront per group (0.13 ms).
// What is left per group for k_window_end, in the order of the (op, class) codes at the communicator's rows:
// stage[0] = code | dynamic << 10 | slow << 11 | class << 12, stage[1] = row of Eq. 2's round, stage[2] = usable rounds.
struct GroupShared {
  unsigned long long best[GROUP_SLOTS];
  u32 cnt[GROUP_SLOTS], row[GROUP_SLOTS], last[GROUP_SLOTS];
  unsigned short list[GROUP_SLOTS];
  uint8_t map[GROUP_SLOTS];
  // the batch of groups that Eq. 1 has new rounds for
  unsigned long long wm[GC_BATCH], sum[GC_BATCH], min_wm;
  i64 t0[GC_BATCH];
  u32 i0[GC_BATCH], istar[GC_BATCH], fresh[GC_BATCH], lim[GC_BATCH], seen[GC_BATCH], m[GC_BATCH], lastb[GC_BATCH], code[GC_BATCH], rank[GC_BATCH];
  u32 wave[GC_THREADS / CCLD_WAVE], lo, hi, need, left, n_rank;
};
__device__ __forceinline__ void list_groups(const EndArgs& a, GroupShared& S, const u32 c) {
  auto &s_cnt = S.cnt, &s_row = S.row, &s_last = S.last;
  auto& s_best = S.best;
  auto& s_list = S.list;
  auto& s_wave = S.wave;
  u32 &s_lo = S.lo, &s_hi = S.hi, &s_need = S.need, &s_left = S.left, &s_n_rank = S.n_rank;
  auto& s_map = S.map;
  auto &s_wm = S.wm, &s_sum = S.sum;
  auto& s_t0 = S.t0;
  auto& s_min_wm = S.min_wm;
  auto &s_i0 = S.i0, &s_istar = S.istar, &s_new = S.fresh, &s_lim = S.lim, &s_seen = S.seen, &s_m = S.m, &s_lastb = S.lastb, &s_code = S.code,
       &s_rank = S.rank;
  const u32 tid = threadIdx.x, lane = lane_id(), wave = tid / CCLD_WAVE;
  const u64 n_seg = a.counters[CNT_NSEG];
  const u32 n = (u32)(n_seg < a.seg_cap ? n_seg : a.seg_cap);          // rows that the table holds
  const i64* __restrict__ COMM = a.seg + (u64)CCLD_SEG_COMM * a.seg_cap;
  const i64* __restrict__ SEQ = a.seg + (u64)CCLD_SEG_SEQ * a.seg_cap;
  const i64* __restrict__ EMIN = a.seg + (u64)CCLD_SEG_ENTER_MIN * a.seg_cap;
  const i64* __restrict__ DMAX = a.seg + (u64)CCLD_SEG_DUR_MAX * a.seg_cap;
  const i64* __restrict__ DMIN = a.seg + (u64)CCLD_SEG_DUR_MIN * a.seg_cap;
  const unsigned short* __restrict__ code = a.gcode;
  if (wave < 2) {
    const u32 r = first_row_of(COMM, n, c + wave, lane);
    if (lane == 0) { if (wave == 0) s_lo = r; else s_hi = r; }
  }
  if (tid == 0) s_need = 0;
  for (u32 i = tid; i < (u32)GROUP_SLOTS; i += GC_THREADS) { s_cnt[i] = 0; s_best[i] = 0; s_row[i] = GC_NONE; s_last[i] = 0; }
  __syncthreads();
  const u32 lo = s_lo, hi = s_hi;
  // The rows, GC_THREADS * U a step, those of a thread on their way together.  In a step with all of its rows none of the loads is
  // conditional, and all values are wanted before the first is used: by itself the compiler puts some of the loads behind uses of
  // others, depending on what else is in the kernel (windows of 8 ranks and 40M records, 3M rows in a communicator: 5,960 us before,
  // 6,590 at worst, 5,770 so; of 16 ranks and 10M records 1,139 and 1,113).
  constexpr u32 U = 4;
  const u32 whole = lo + (hi - lo) / (GC_THREADS * U) * (GC_THREADS * U);
  auto each_row = [&](auto use) {
    u32 g[U];
    unsigned long long r[U];
    for (u32 i0 = lo + tid; i0 < whole; i0 += GC_THREADS * U) {
#pragma unroll
      for (u32 u = 0; u < U; ++u) { g[u] = code[i0 + u * GC_THREADS]; r[u] = (unsigned long long)a.range_c[i0 + u * GC_THREADS]; }
#pragma unroll
      for (u32 u = 0; u < U; ++u) asm volatile("" : "+v"(g[u]), "+v"(r[u]));
#pragma unroll
      for (u32 u = 0; u < U; ++u) use(i0 + u * GC_THREADS, g[u], r[u]);
    }
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      const u32 i = whole + tid + u * GC_THREADS;
      g[u] = i < hi ? code[i] : NO_GROUP;
      r[u] = i < hi ? (unsigned long long)a.range_c[i] : 0ull;
    }
#pragma unroll
    for (u32 u = 0; u < U; ++u) use(whole + tid + u * GC_THREADS, g[u], r[u]);
  };
  each_row([&](u32 i, u32 g, unsigned long long r) {
    if (g >= (u32)GROUP_SLOTS) return;
    atomicAdd(&s_cnt[g], 1u);
    if (r > s_best[g]) atomicMax(&s_best[g], r);
    atomicMax(&s_last[g], i);
  });
  __syncthreads();
  each_row([&](u32 i, u32 g, unsigned long long r) {
    if (g < (u32)GROUP_SLOTS && r == s_best[g]) atomicMin(&s_row[g], i);
  });
  // the groups that occur, ascending
  u32 n_group;
  {
    constexpr u32 PER = GROUP_SLOTS / GC_THREADS;
    u32 m = 0;
#pragma unroll
    for (u32 k = 0; k < PER; ++k) m += s_cnt[tid * PER + k] != 0;
    u32 at = block_exclusive_sum<GC_THREADS>(m, s_wave, &n_group);
#pragma unroll
    for (u32 k = 0; k < PER; ++k)
      if (s_cnt[tid * PER + k]) s_list[at++] = (unsigned short)(tid * PER + k);
  }
  __syncthreads();
  GroupState* __restrict__ gs = a.gstate + (u64)c * GROUP_SLOTS;
  // Eq. 1 for the groups whose baseline still grows and that have rounds not visited before (rounds beyond the
  // watermark form a suffix: compare the last one)
  u32 mine = 0;
  for (u32 p = tid; p < n_group; p += GC_THREADS) {
    const u32 g = s_list[p];
    if (!gs[g].frozen && (u64)SEQ[s_last[g]] + 1 > gs[g].baselined_wm) ++mine;
  }
  if (mine) atomicAdd(&s_need, mine);
  __syncthreads();
  const u32 n_need = s_need;
  for (u32 done = 0; done < n_need;) {
    // the next groups of the list, GC_BATCH at a time (a group leaves the list by its new watermark)
    __syncthreads();
    if (tid == 0) { s_left = 0; s_min_wm = ~0ull; s_n_rank = 0; }
    for (u32 i = tid; i < (u32)GROUP_SLOTS; i += GC_THREADS) s_map[i] = 0xFF;
    __syncthreads();
    for (u32 p = tid; p < n_group; p += GC_THREADS) {
      const u32 g = s_list[p];
      const GroupState G = gs[g];
      if (G.frozen || (u64)SEQ[s_last[g]] + 1 <= G.baselined_wm) continue;
      const u32 m = atomicAdd(&s_left, 1u);
      if (m >= GC_BATCH) continue;
      s_map[g] = (uint8_t)m; s_code[m] = g; s_wm[m] = G.baselined_wm; s_sum[m] = 0; s_i0[m] = GC_NONE; s_istar[m] = GC_NONE;
      s_new[m] = 0; s_seen[m] = 0; s_m[m] = 0; s_lastb[m] = 0;
      s_t0[m] = G.t0; s_lim[m] = a.p.tbase_rounds > G.cnt ? a.p.tbase_rounds - G.cnt : 0u;
      atomicMin(&s_min_wm, (unsigned long long)G.baselined_wm);
    }
    __syncthreads();
    const u32 nb = s_left < GC_BATCH ? s_left : GC_BATCH;
    if (nb == 0) break;
    done += nb;
    // The walk.  A baseline ends before the first new round past the warm-up span and before the new round number s_lim, and
    // a group whose baseline has ended costs nothing from the next step on.  A step: its new rounds per group; the
    // round that ends a group by its count, where the step has it (a scan over the step's rows, once in a group's
    // life); the first one past the warm-up span; the sums up to there.  On first windows this takes the place of four passes
    // over all rows, one of them by a single wavefront (analysis of 40M records of 8 ranks, 3M rounds in a communicator:
    // 18.3 -> 6.0 ms; 10M of 16 ranks: 2.55 -> 1.19).
    if (tid == 0) s_left = nb;            // (what it says already, or more)
    u32 start = lo;
    for (u32 end = hi; end - start > GC_THREADS * GC_WALK;) {         // 512 probes at a time; few rows are walked unsearched
      const u32 step = (end - start) / GC_THREADS, was = start;
      const u32 k = (u32)__syncthreads_count((u64)SEQ[start + tid * step] < s_min_wm);     // a prefix of the probes
      if (k == 0) break;
      start = was + (k - 1) * step + 1;
      end = k < GC_THREADS ? was + k * step : end;
    }
    __syncthreads();
    bool timed = tid < nb && gs[s_code[tid]].cnt != 0, ended = false;
    for (u32 base = start, open = nb; base < hi && open;) {
      // consecutive rows per thread, so that the scan numbers them; few rows are spread over all threads
      const u32 per = hi - base < GC_THREADS * GC_WALK ? (hi - base + GC_THREADS - 1) / GC_THREADS : GC_WALK;
      const u32 i0 = base + tid * per;
      base += GC_THREADS * per;
      u64 mine8 = ~0ull;                 // a byte per row: its group in the batch, 0xFF: takes no part
#pragma unroll 1
      for (u32 u = 0; u < per; ++u) {
        const u32 i = i0 + u, g = i < hi ? code[i] : NO_GROUP, m = g < (u32)GROUP_SLOTS ? s_map[g] : 0xFFu;
        if (m == 0xFF || s_istar[m] != GC_NONE || (u64)SEQ[i] + 1 <= s_wm[m]) continue;
        atomicMin(&s_i0[m], i);
        atomicAdd(&s_new[m], 1u);
        mine8 ^= (u64)(m ^ 0xFF) << (8 * u);
      }
      if (!__syncthreads_or(mine8 != ~0ull)) continue;
      if (tid < nb && s_new[tid]) {
        if (!timed) { s_t0[tid] = EMIN[s_i0[tid]]; timed = true; }
        if (s_lim[tid] - s_seen[tid] < s_new[tid]) s_rank[atomicAdd(&s_n_rank, 1u)] = tid;      // s_seen <= s_lim while it is open
      }
      __syncthreads();
      for (u32 q = 0; q < s_n_rank; ++q) {
        const u32 who = s_rank[q];
        u32 cnt = 0, tot;
        for (u32 u = 0; u < per; ++u) cnt += (u32)(uint8_t)(mine8 >> (8 * u)) == who;
        u32 at = s_seen[who] + block_exclusive_sum<GC_THREADS>(cnt, s_wave, &tot);
        for (u32 u = 0; u < per; ++u)
          if ((u32)(uint8_t)(mine8 >> (8 * u)) == who && at++ == s_lim[who]) atomicMin(&s_istar[who], i0 + u);
      }
#pragma unroll 1
      for (u32 u = 0; u < per; ++u) {
        const u32 m = (uint8_t)(mine8 >> (8 * u));
        if (m != 0xFF && EMIN[i0 + u] - s_t0[m] > a.p.tbase_warmup_ns) atomicMin(&s_istar[m], i0 + u);
      }
      __syncthreads();
#pragma unroll 1
      for (u32 u = 0; u < per; ++u) {
        const u32 m = (uint8_t)(mine8 >> (8 * u));
        if (m != 0xFF && i0 + u < s_istar[m]) {
          atomicAdd(&s_sum[m], (unsigned long long)DMAX[i0 + u]);
          atomicAdd(&s_m[m], 1u);
          atomicMax(&s_lastb[m], i0 + u);
        }
      }
      if (tid < nb) {
        s_seen[tid] += s_new[tid]; s_new[tid] = 0;
        if (!ended && s_istar[tid] != GC_NONE) { ended = true; atomicSub(&s_left, 1u); }
      }
      if (tid == 0) s_n_rank = 0;
      __syncthreads();
      open = s_left;
    }
    __syncthreads();
    if (tid < nb) {
      const u32 g = s_code[tid];
      GroupState G = gs[g];
      G.t0 = s_t0[tid];
      G.sum = (i64)((u64)G.sum + (u64)s_sum[tid]);
      G.cnt += s_m[tid];
      if (s_m[tid]) G.baseline_last_seq = (u64)SEQ[s_lastb[tid]];
      if (s_istar[tid] != GC_NONE) { G.frozen = 1; G.tbase_dyn = G.sum / (i64)G.cnt; }
      G.baselined_wm = (u64)SEQ[s_last[g]] + 1;
      gs[g] = G;
    }
    __threadfence_block();
  }
  __syncthreads();
  // Eq. 2 to 4
  for (u32 p = tid; p < n_group; p += GC_THREADS) {
    const u32 g = s_list[p];
    GroupState G = gs[g];
    const u64 wm = (u64)SEQ[s_last[g]] + 1;
    if (wm > G.baselined_wm) G.baselined_wm = wm;
    const u32 sx = s_row[g];
    const u64 rseq = (u64)SEQ[sx];
    const i64 tmax = DMAX[sx], tmin = DMIN[sx];
    const bool dynamic = G.frozen && rseq > G.baseline_last_seq;
    const i64 tbase = dynamic ? G.tbase_dyn : a.p.tbase_init_ns;
    const bool slow = (i128)(tmax - tbase) * (i128)a.p.theta_den > (i128)a.p.theta_num * (i128)tbase;
    u32 cls = CCLD_SLOW_NONE;
    if (slow) {
      const i128 num = (i128)(tmax - tmin) * (i128)a.p.ab_den, den = (i128)(tmax - tbase);
      if (num > (i128)a.p.beta_num * den) cls = CCLD_SLOW_S1_COMPUTATION;
      else if (num < (i128)a.p.alpha_num * den) cls = CCLD_SLOW_S2_COMMUNICATION;
      else cls = CCLD_SLOW_S3_MIXED;
      if (rseq + 1 > G.detected_wm) { G.repeats += 1; G.detected_wm = rseq + 1; }
    }
    gs[g] = G;
    a.stage[0][lo + p] = g | (dynamic ? 1u << 10 : 0u) | (slow ? 1u << 11 : 0u) | (cls << 12);
    a.stage[1][lo + p] = sx;
    a.stage[2][lo + p] = s_cnt[g];
  }
  if (tid == 0) { a.comm_groups[c] = n_group; a.comm_row[c] = lo; }
}
static_assert(GROUP_SLOTS == 1024 && GROUP_SLOTS % GC_THREADS == 0, "ten bits of group code");

// ---- flags of a window on the grid placement -------------------------------------------------------------
// The statistics kernels left the flagged records of every fine bucket in (counter, rank) order; here a thread per flag finds
// its bucket by the flags before it and writes it to its place in the list and in the flag table: a few buckets hold most of the
// flags (those of a slow rank's communicators), so a workgroup or a wavefront per bucket would wait for those.  The flags before
// every bucket are scanned by each workgroup in LDS, or were scanned before (many buckets).
// Where every eighth rank is late the list is long, and what takes the time is dependent loads: a wavefront looks for its 64 flags'
// buckets at once (16 loads one after the other per flag before), and the workgroups grow with the buckets, one to 16 of them
// (64 of them, 256 where scanned, before; the whole launch, us: 82M records with 7.6M flags 591 -> 266, 20M with 1.9M 129 -> 87,
// 4M with 377,000 67 -> 31; with 132,000 flags in 82M records 73 both ways; twice as many workgroups: 258, 85, 29, 78).
constexpr u32 END_SCAN_FINE = 4096;
constexpr u32 END_FLAG_SHARE = 16, END_FLAG_BLOCKS = 1024, END_FLAG_SCANNED = 256;       // fine buckets per workgroup; at most; at least where scanned
struct FlagShared { u32 pre[END_SCAN_FINE + 1], wave[GC_THREADS / CCLD_WAVE]; };
__device__ __forceinline__ void list_flags(const EndArgs& e, const GridArgs& d, const FlagArgs& a, FlagShared& S, u32 block, u32 blocks) {
  const u32 n_fine = d.hdr->n_fine, tid = threadIdx.x;
  u32 total;
  if (e.flags_scanned) {
    total = d.nflag[n_fine];
  } else {
    constexpr u32 PER = END_SCAN_FINE / GC_THREADS;
    u32 v[PER], sum = 0;
#pragma unroll
    for (u32 q = 0; q < PER; ++q) { v[q] = tid * PER + q < n_fine ? d.nflag[tid * PER + q] : 0u; sum += v[q]; }
    u32 ex = block_exclusive_sum<GC_THREADS>(sum, S.wave, &total);
#pragma unroll
    for (u32 q = 0; q < PER; ++q) { S.pre[tid * PER + q] = ex; ex += v[q]; }
    if (block == 0 && tid == 0) e.counters[CNT_NFLAG] = total;
    __syncthreads();
  }
  const u32 lane = lane_id();
  const auto before = [&](u32 f) -> u32 { return e.flags_scanned ? d.nflag[f] : S.pre[f]; };       // flags before fine bucket f
  for (u32 k0 = block * GC_THREADS + (tid - lane); k0 < total; k0 += blocks * GC_THREADS) {        // 64 flags in a row per wavefront
    // the bucket of the first of them, the last one that starts at or before it: 64 probes at a time
    u32 lo = 0;
    for (u32 hi = n_fine;;) {
      const u32 step = (hi - lo + CCLD_WAVE - 1) / CCLD_WAVE, probe = lo + lane * step;
      lo += ((u32)__popcll(ballot64(probe < hi && before(probe) <= k0)) - 1) * step;
      if (step == 1) break;
      hi = hi - lo < step ? hi : lo + step;
    }
    // the bucket of the lane's own: as a rule among the next 64
    const u32 k = k0 + lane, next = lo + 1 + lane < n_fine ? before(lo + 1 + lane) : ~0u;
    u32 past = 0, first = before(lo);
#pragma unroll
    for (u32 m = CCLD_WAVE / 2; m; m >>= 1)
      if (lane_read(next, past + m - 1) <= k) past += m;
    if (lane_read(next, past) <= k) ++past;
    const u32 start = lane_read(next, past ? past - 1 : 0u);
    if (past) first = start;
    if (k >= total) continue;
    lo += past;
    if (past == CCLD_WAVE)
      for (u32 hi = n_fine; hi - lo > 1;) {
        const u32 m = (lo + hi) >> 1, v = before(m);
        if (v <= k) { lo = m; first = v; } else hi = m;
      }
    const FineDesc D = d.desc[lo];
    const u32 at = d.rec0[lo] + (k - first);
    const u32 w = a.flag_stage[at], cell = w & 0xFFFFu, kind = w >> 16, round = cell / D.size, slot = cell - round * D.size;
    a.flag_key[k] = ((u64)(D.srow0 + round) << 32) | slot;
    a.flag_pos[k] = at;
    if (a.flag && k < a.flag_cap) {
      auto put = [&](int col, i64 v) { a.flag[(u64)col * a.flag_cap + k] = v; };
      put(CCLD_FLG_COMM, (i64)D.comm);
      put(CCLD_FLG_SEQ, (i64)(D.seq0 + round));
      put(CCLD_FLG_RANK, (i64)rank_of_slot(a.member_off, a.members_sorted, D.comm, slot));
      put(CCLD_FLG_KIND, (i64)kind);
      put(CCLD_FLG_LAG_ENTER, a.flag_lag[at]);
      put(CCLD_FLG_LAG_EXIT, a.flag_lag[a.cap_n + at]);
    }
  }
}

// ---- blame order -----------------------------------------------------------------------------------------
// Every workgroup lists the flagged ranks in LDS for itself (a scan over two columns of the blame table), ranks its share of
// them and writes its share of the others.
constexpr u32 ORDER_TILE = 4 * GC_THREADS;
struct OrderShared { unsigned short flagged[END_ORDER_RANKS]; u32 before[END_ORDER_RANKS / ORDER_TILE], wave[GC_THREADS / CCLD_WAVE]; };
__device__ __forceinline__ void list_order(const EndArgs& a, OrderShared& S, u32 block, u32 blocks) {
  const i64* __restrict__ blame = a.blame;
  const u32 tid = threadIdx.x, lane = lane_id(), n_ranks = a.n_ranks;
  const i64* NE = blame + (u64)CCLD_BLM_N_LATE_ENTER * n_ranks;
  const i64* NX = blame + (u64)CCLD_BLM_N_LATE_EXIT * n_ranks;
  auto flags_of_four = [&](u32 r0) -> u32 {
    u32 m = 0;
#pragma unroll
    for (u32 k = 0; k < 4; ++k) if (r0 + k < n_ranks && NE[r0 + k] + NX[r0 + k] != 0) m |= 1u << k;
    return m;
  };
  u32 nb = 0;
  for (u32 t = 0; t * ORDER_TILE < n_ranks; ++t) {
    const u32 r0 = t * ORDER_TILE + tid * 4;
    const u32 m = flags_of_four(r0);
    u32 tot;
    u32 at = nb + block_exclusive_sum<GC_THREADS>((u32)__popc(m), S.wave, &tot);
#pragma unroll
    for (u32 k = 0; k < 4; ++k) if (m & (1u << k)) S.flagged[at++] = (unsigned short)(r0 + k);
    if (tid == 0) S.before[t] = nb;
    nb += tot;
  }
  __syncthreads();
  constexpr u32 NW = GC_THREADS / CCLD_WAVE;
  for (u32 q = block * NW + tid / CCLD_WAVE; q < nb; q += blocks * NW) {
    const u32 r = S.flagged[q];
    const u32 before = blamed_before(blame, n_ranks, S.flagged, nb, r, lane);
    if (lane == 0) a.order[before] = r;
  }
  for (u32 t = block; t * ORDER_TILE < n_ranks; t += blocks) {
    const u32 r0 = t * ORDER_TILE + tid * 4;
    const u32 m = flags_of_four(r0);
    u32 tot;
    u32 before = S.before[t] + block_exclusive_sum<GC_THREADS>((u32)__popc(m), S.wave, &tot);       // flagged ranks below r0
#pragma unroll
    for (u32 k = 0; k < 4; ++k) {
      if (r0 + k >= n_ranks) break;
      if (m & (1u << k)) ++before; else a.order[nb + r0 + k - before] = r0 + k;
    }
  }
}

// ---- hang alerts ------------------------------------------------------------------------------------------
// A few alerts in table order with their candidates in rank order, a wavefront each.  (Seven launches and a second wait for
// the host otherwise, which longer lists take.)  What takes the time is the trips to memory of one wavefront: ALERT_AHEAD pieces of 64
// members are on their way together, and a sorted collective's records are read in their order, where they say which members have
// one, and are the members in order where all have.  (Windows of 82K records in collectives of 2,048 members, eight alerts: 212 us on the
// grid with a piece after the other, 171 or 196 by their class so, 206 with launches of their own; sorted 543 with a search per
// member, 436 or 451, 495.)
constexpr u32 ALERT_AHEAD = 4;
struct AlertShared { u32 row[END_ALERTS], cnt[END_ALERTS]; unsigned long long hit[END_ALERTS][END_ALERT_MEMBERS / CCLD_WAVE]; };
template <bool GRID>
__device__ __forceinline__ void list_alerts(const AlertArgs& a, AlertShared& S) {
  const u32 n = (u32)a.counters[CNT_NALERT], tid = threadIdx.x, lane = lane_id(), wave = tid / CCLD_WAVE;
  if (n == 0 || n > END_ALERTS) return;
  if (tid < n) {
    const u32 row = a.alert_list[tid];
    u32 at = 0;
    for (u32 i = 0; i < n; ++i) at += a.alert_list[i] < row ? 1u : 0u;
    S.row[at] = row;
  }
  __syncthreads();
  const bool on = wave < n;
  const u64 C = a.seg_cap;
  u32 s = 0, comm = 0, size = 0, moff = 0, total = 0, before = 0;      // before: the hits of the pieces before the lane's
  int cls = 0;
  auto& hit = S.hit[wave];               // a word per 64 members
  if (on) {
    s = S.row[wave];
    comm = (u32)a.seg[CCLD_SEG_COMM * C + s];
    const u32 nn = (u32)a.seg[CCLD_SEG_N * C + s], ninfl = (u32)a.seg[CCLD_SEG_INFLIGHT * C + s], first = (u32)a.seg[CCLD_SEG_FIRST * C + s];
    size = a.topo.size[comm]; moff = a.topo.member_off[comm];
    cls = alert_class(nn, ninfl, size);
    const u32 words = (size + CCLD_WAVE - 1) / CCLD_WAVE;
    if (lane < words) hit[lane] = 0;
    __builtin_amdgcn_wave_barrier();
    CommLayout L{};
    if (GRID) L = a.grid.lay[comm];
    const u32 k = s - L.seg_base, cells = L.cell_base + k * L.size;
    for (u32 q0 = 0; cls != CCLD_HANG_H3_HARDWARE && q0 < size; q0 += CCLD_WAVE * ALERT_AHEAD) {
      u32 at[ALERT_AHEAD];
      u64 m[ALERT_AHEAD];
      bool found[ALERT_AHEAD];
      auto member = [&](u32 u) { return std::min(q0 + u * CCLD_WAVE + lane, size - 1); };
      if (cls == CCLD_HANG_H1_NOT_ENTERED && !GRID) {
        const u64 mmask = ((u64)1 << a.sf.mb) - 1;      // key slot = position among the members in ascending rank order
#pragma unroll
        for (u32 u = 0; u < ALERT_AHEAD; ++u) m[u] = a.key[first + std::min(member(u), nn - 1)] & mmask;
#pragma unroll
        for (u32 u = 0; u < ALERT_AHEAD; ++u)
          if (q0 + u * CCLD_WAVE + lane < nn) atomicOr(&hit[m[u] / CCLD_WAVE], 1ull << (m[u] % CCLD_WAVE));      // has a record
        continue;
      }
#pragma unroll
      for (u32 u = 0; u < ALERT_AHEAD; ++u) at[u] = GRID ? (u32)a.grid.cell_row[cells + member(u)] : a.idx[first + member(u)];
      if (cls == CCLD_HANG_H1_NOT_ENTERED) {
#pragma unroll
        for (u32 u = 0; u < ALERT_AHEAD; ++u) found[u] = at[u] == GRID_EMPTY;
      } else {                           // every member has a record
        i64 tx[ALERT_AHEAD];
#pragma unroll
        for (u32 u = 0; u < ALERT_AHEAD; ++u)
          tx[u] = (GRID ? unpack_row(a.grid.rows[L.cell_base + k / L.rpb * L.rpb * L.size + at[u]], a.grid.hdr->ref, a.grid.wide) : load_rec(a.win, at[u])).t_exit;
#pragma unroll
        for (u32 u = 0; u < ALERT_AHEAD; ++u) found[u] = tx[u] != INT64_MAX;
      }
#pragma unroll
      for (u32 u = 0; u < ALERT_AHEAD; ++u) {
        m[u] = ballot64(found[u] && q0 + u * CCLD_WAVE + lane < size);
        if (lane == 0 && q0 + u * CCLD_WAVE < size) hit[q0 / CCLD_WAVE + u] = m[u];
      }
    }
    __builtin_amdgcn_wave_barrier();
    u64 mine = lane < words ? hit[lane] : 0ull;
    if (cls == CCLD_HANG_H1_NOT_ENTERED && !GRID && lane < words) {
      mine = ~mine & (lane + 1 < words || size % CCLD_WAVE == 0 ? ~0ull : ((u64)1 << size % CCLD_WAVE) - 1);
      hit[lane] = mine;
    }
    const u32 inc = wave_inclusive_sum((u32)__popcll(mine));
    before = inc - (u32)__popcll(mine); total = lane_read(inc, CCLD_WAVE - 1);
    if (lane == 0) S.cnt[wave] = total;
  }
  __syncthreads();
  if (!on) return;
  u32 off = 0;
  for (u32 i = 0; i < wave; ++i) off += S.cnt[i];
  if (wave + 1 == n && lane == 0) a.counters[CNT_NCAND] = (u64)off + total;
  if (lane == 0 && wave < a.alert_cap) {
    const u64 A = a.alert_cap;
    auto put = [&](int col, i64 v) { a.alert[(u64)col * A + wave] = v; };
    put(CCLD_ALR_COMM, (i64)comm);
    put(CCLD_ALR_SEQ, a.seg[CCLD_SEG_SEQ * C + s]);
    put(CCLD_ALR_AGE, a.now_ns - a.seg[CCLD_SEG_INFLIGHT_ENTER_MIN * C + s]);
    put(CCLD_ALR_CLASS, (i64)cls);
    put(CCLD_ALR_NCAND, (i64)total);
    put(CCLD_ALR_CAND_OFF, (i64)off);
  }
  for (u32 q0 = 0; q0 < size; q0 += CCLD_WAVE * ALERT_AHEAD) {
    u32 rank[ALERT_AHEAD];
#pragma unroll
    for (u32 u = 0; u < ALERT_AHEAD; ++u) rank[u] = a.topo.members_sorted[moff + std::min(q0 + u * CCLD_WAVE + lane, size - 1)];
#pragma unroll
    for (u32 u = 0; u < ALERT_AHEAD; ++u) {
      const u32 w = q0 / CCLD_WAVE + u;
      if (w * CCLD_WAVE >= size) break;
      const u64 m = hit[w], at = (u64)off + lane_read(before, w) + mbcnt64(m);
      if (((m >> lane) & 1u) && at < a.cand_cap) a.cand[at] = (i64)rank[u];
    }
  }
}
static_assert(END_ALERT_MEMBERS <= CCLD_WAVE * CCLD_WAVE, "a lane per 64 members");
static_assert(END_ALERTS <= GC_THREADS / CCLD_WAVE, "a wavefront per alert");

// ---- the launches -----------------------------------------------------------------------------------------
// (Four workgroups per compute unit: with the registers that the compiler takes by itself there are three, and the groups of a
// stream's 3,200 communicators take 49 us instead of 38.)
template <bool GRID>
__global__ __launch_bounds__(GC_THREADS, 8) void k_window_lists(EndArgs a, GridArgs d, FlagArgs f, AlertArgs al, u32 n_flags, u32 n_order, u32 n_alerts) {
  constexpr size_t LDS = std::max(std::max(sizeof(GroupShared), sizeof(AlertShared)), std::max(sizeof(FlagShared), sizeof(OrderShared)));
  __shared__ unsigned long long s_mem[(LDS + 7) / 8];
  // a data error found by an earlier kernel of this analysis: the tables are not valid and the detection state stays as it is
  if (a.counters[CNT_STATUS] != 0) return;
  // The groups, which take longest where there are many, start behind the others: they fill the chip by themselves (in front of
  // the flags, us: 82M records 54.5 both ways, a stream of 3,200 communicators 37.5 and 38.3, 512 ranks 11.7 and 10.8).
  const u32 b = blockIdx.x;
  if (b < n_alerts) list_alerts<GRID>(al, *reinterpret_cast<AlertShared*>(s_mem));
  else if (b - n_alerts < n_order) list_order(a, *reinterpret_cast<OrderShared*>(s_mem), b - n_alerts, n_order);
  else if (GRID && b - n_alerts - n_order < n_flags) list_flags(a, d, f, *reinterpret_cast<FlagShared*>(s_mem), b - n_alerts - n_order, n_flags);
  else list_groups(a, *reinterpret_cast<GroupShared*>(s_mem), b - n_alerts - n_order - n_flags);
}
// Rows of the group table, END_COMMS communicators to a workgroup, and the report by the last one, past the caches.  The
// communicators before are summed by the workgroup itself (a few thousand counts from the L2) unless they were scanned
// before (SCANNED: many communicators, where that would be quadratic).
constexpr u32 END_COMMS = 8, END_WAVES = GC_THREADS / CCLD_WAVE;
template <bool SCANNED>
__global__ __launch_bounds__(GC_THREADS) void k_window_end(EndArgs a) {
  __shared__ u32 s_cnt[END_COMMS], s_wave[END_WAVES];
  const u32 tid = threadIdx.x, lane = lane_id(), wave = tid / CCLD_WAVE, c0 = blockIdx.x * END_COMMS;
  if (a.counters[CNT_STATUS] == 0) {
    u32 before = 0, base;
    if (SCANNED) {
      if (tid < END_COMMS) s_cnt[tid] = c0 + tid < a.n_comms ? a.comm_groups[c0 + tid + 1] - a.comm_groups[c0 + tid] : 0u;
      before = tid == 0 ? a.comm_groups[c0] : 0u;
    } else {
      if (tid < END_COMMS) s_cnt[tid] = c0 + tid < a.n_comms ? a.comm_groups[c0 + tid] : 0u;
#pragma unroll 4
      for (u32 i = tid; i < c0; i += GC_THREADS) before += a.comm_groups[i];
    }
    block_exclusive_sum<GC_THREADS>(before, s_wave, &base);
    const u64 C = a.group_cap;
    for (u32 k = wave; k < END_COMMS && c0 + k < a.n_comms; k += END_WAVES) {
      const u32 c = c0 + k, cnt = s_cnt[k], lo = a.comm_row[c];
      u32 pos = base;
      for (u32 i = 0; i < k; ++i) pos += s_cnt[i];
      if (c + 1 == a.n_comms && lane == 0) store_agent(reinterpret_cast<i64*>(&a.counters[CNT_NGROUP]), (i64)((u64)pos + cnt));
      for (u32 p = lane; p < cnt; p += CCLD_WAVE) {
        const u64 at = (u64)pos + p;
        if (at >= C) break;
        const u32 w = a.stage[0][lo + p], sx = a.stage[1][lo + p];
        const u32 code = w & 1023u, cls = w >> 12;
        const bool dynamic = (w >> 10) & 1u, slow = (w >> 11) & 1u;
        const GroupState G = a.gstate[(u64)c * GROUP_SLOTS + code];
        auto col = [&](int q) -> i64 { return a.seg[(u64)q * a.seg_cap + sx]; };
        auto put = [&](int q, i64 v) { store_agent(&a.group[(u64)q * C + at], v); };
        put(CCLD_GRP_COMM, (i64)c);
        put(CCLD_GRP_OP, (i64)(code / GROUP_CLS));
        put(CCLD_GRP_CLS, (i64)(code % GROUP_CLS));
        put(CCLD_GRP_N_USABLE, (i64)a.stage[2][lo + p]);
        put(CCLD_GRP_RSTAR_SEQ, col(CCLD_SEG_SEQ));
        put(CCLD_GRP_TMAX, col(CCLD_SEG_DUR_MAX));
        put(CCLD_GRP_TMIN, col(CCLD_SEG_DUR_MIN));
        put(CCLD_GRP_TBASE, dynamic ? G.tbase_dyn : a.p.tbase_init_ns);
        put(CCLD_GRP_STATIC, dynamic ? 0 : 1);
        put(CCLD_GRP_FROZEN, G.frozen);
        put(CCLD_GRP_M, G.cnt);
        put(CCLD_GRP_SLOW, slow ? 1 : 0);
        put(CCLD_GRP_CLASS, (i64)cls);
        put(CCLD_GRP_ROOT_S1, (slow && cls != CCLD_SLOW_S2_COMMUNICATION) ? col(CCLD_SEG_ARGMIN_RANK) : (i64)CCLD_NO_RANK);
        // communication-slow root (Eq. 4): the communicator's member of minimal SendRate / RecvRate
        put(CCLD_GRP_ROOT_S2, (cls == CCLD_SLOW_S2_COMMUNICATION || cls == CCLD_SLOW_S3_MIXED) ? a.rate_root[c] : (i64)CCLD_NO_RANK);
        put(CCLD_GRP_REPEATS, G.repeats);
        put(CCLD_GRP_LOCATE, (slow && G.repeats >= a.p.repeat_threshold) ? 1 : 0);
      }
    }
  }
  if (a.host) report_counters(a.counters, a.arrivals, a.host, a.ticket);
}

// A window without records blames nobody: the ranks in ascending order, and the report.
__global__ __launch_bounds__(GC_THREADS) void k_window_empty(u32 n_ranks, u32* order, u64* counters, u32* arrivals, u64* host, u64 ticket) {
  for (u32 r = blockIdx.x * GC_THREADS + threadIdx.x; r < n_ranks; r += gridDim.x * GC_THREADS) order[r] = r;
  report_counters(counters, arrivals, host, ticket);
}
void launch_window_empty(hipStream_t st, uint32_t n_ranks, uint32_t* order, uint64_t* counters, uint32_t* arrivals, uint64_t* host, uint64_t ticket) {
  const u32 blocks = std::min<u32>((n_ranks + GC_THREADS - 1) / GC_THREADS, 64);
  hipLaunchKernelGGL(k_window_empty, dim3(blocks), dim3(GC_THREADS), 0, st, n_ranks, order, counters, arrivals, host, ticket);
}

// From so many communicators on their counts are scanned by a launch of their own
constexpr u32 END_SCAN_COMMS = 8192;
bool launch_window_end(hipStream_t st, const EndArgs& a_in, const GridArgs* d, const FlagArgs* f, const AlertArgs* al, uint32_t fine_bound) {
  EndArgs a = a_in;
  const bool report = a.n_ranks <= END_ORDER_RANKS;
  if (!report) a.host = nullptr;
  a.flags_scanned = fine_bound > END_SCAN_FINE;                                     // the bound is the exact number there
  const u32 n_flags = !d ? 0u : std::min(std::max((fine_bound + END_FLAG_SHARE - 1) / END_FLAG_SHARE, a.flags_scanned ? END_FLAG_SCANNED : 0u), END_FLAG_BLOCKS);
  if (d && a.flags_scanned) launch_scan_tiles(st, d->nflag, fine_bound, &a.counters[CNT_NFLAG]);
  const u32 n_order = report ? std::min<u32>((a.n_ranks + 63) / 64, 64) : 0u, n_alerts = al ? 1u : 0u;
  const u32 blocks = a.n_comms + n_flags + n_order + n_alerts, ends = (a.n_comms + END_COMMS - 1) / END_COMMS;
  const AlertArgs alerts = al ? *al : AlertArgs{};
  if (d) hipLaunchKernelGGL(k_window_lists<true>, dim3(blocks), dim3(GC_THREADS), 0, st, a, *d, *f, alerts, n_flags, n_order, n_alerts);
  else hipLaunchKernelGGL(k_window_lists<false>, dim3(blocks), dim3(GC_THREADS), 0, st, a, GridArgs{}, FlagArgs{}, alerts, 0u, n_order, n_alerts);
  if (a.n_comms < END_SCAN_COMMS) {
    hipLaunchKernelGGL(k_window_end<false>, dim3(ends), dim3(GC_THREADS), 0, st, a);
  } else {
    launch_scan_tiles(st, a.comm_groups, a.n_comms, &a.counters[CNT_NGROUP]);
    hipLaunchKernelGGL(k_window_end<true>, dim3(ends), dim3(GC_THREADS), 0, st, a);
  }
  return report;
}

}  // namespace ccld
