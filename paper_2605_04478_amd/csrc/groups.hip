// Slow-detection rules (Eq. 1-4) per detection group for gfx950.  The collective table is in (communicator,
// operation counter) order, so a communicator's collectives are one run of rows and a group (communicator, op,
// size class) is a subset of that run in ascending counter order: one workgroup per communicator accumulates
// all of its groups in LDS, with no sort.
#include "window_kernels.h"
#include "device_utils.h"

namespace ccld {

constexpr u32 GC_THREADS = 512;
constexpr u32 GC_BATCH = 64;               // groups still averaging their baseline that one walk handles
constexpr u32 GC_WALK = 8;                 // rows of one thread per step of that walk (a byte of a word each)
constexpr u32 GC_NONE = 0xFFFFFFFFu;

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
// What is left per group for k_group_emit, in the order of the (op, class) codes at the communicator's rows:
// stage[0] = code | dynamic << 10 | slow << 11 | class << 12, stage[1] = row of Eq. 2's round, stage[2] = usable rounds.
// (Four workgroups per compute unit: with the registers that the compiler takes by itself there are three, and a stream's 3,200
// communicators take 49 us instead of 38.)
__global__ __launch_bounds__(GC_THREADS, 8) void k_group_comm(GroupArgs a) {
  __shared__ u32 s_cnt[GROUP_SLOTS], s_row[GROUP_SLOTS], s_last[GROUP_SLOTS];
  __shared__ unsigned long long s_best[GROUP_SLOTS];
  __shared__ unsigned short s_list[GROUP_SLOTS];
  __shared__ u32 s_wave[GC_THREADS / CCLD_WAVE];
  __shared__ u32 s_lo, s_hi, s_need, s_left, s_n_rank;
  // the batch of groups that Eq. 1 has new rounds for
  __shared__ uint8_t s_map[GROUP_SLOTS];
  __shared__ unsigned long long s_wm[GC_BATCH], s_sum[GC_BATCH];
  __shared__ i64 s_t0[GC_BATCH];
  __shared__ unsigned long long s_min_wm;
  __shared__ u32 s_i0[GC_BATCH], s_istar[GC_BATCH], s_new[GC_BATCH], s_lim[GC_BATCH], s_seen[GC_BATCH], s_m[GC_BATCH],
      s_lastb[GC_BATCH], s_code[GC_BATCH], s_rank[GC_BATCH];
  // a data error found by an earlier kernel of this analysis: the tables are not valid and the detection state
  // stays as it is
  if (a.counters[CNT_STATUS] != 0) return;
  const u32 c = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wave = tid / CCLD_WAVE;
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
  if (lo >= hi) {
    if (tid == 0) { a.comm_groups[c] = 0; a.comm_row[c] = lo; }
    return;
  }
  constexpr u32 U = 4;
  for (u32 i0 = lo + tid; i0 < hi; i0 += GC_THREADS * U) {
    u32 g[U];
    unsigned long long r[U];
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      const u32 i = i0 + u * GC_THREADS;
      g[u] = i < hi ? code[i] : NO_GROUP;
      r[u] = i < hi ? (unsigned long long)a.range_c[i] : 0ull;
    }
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      if (g[u] >= (u32)GROUP_SLOTS) continue;
      atomicAdd(&s_cnt[g[u]], 1u);
      if (r[u] > s_best[g[u]]) atomicMax(&s_best[g[u]], r[u]);
      atomicMax(&s_last[g[u]], i0 + u * GC_THREADS);
    }
  }
  __syncthreads();
  for (u32 i0 = lo + tid; i0 < hi; i0 += GC_THREADS * U) {
    u32 g[U];
    unsigned long long r[U];
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      const u32 i = i0 + u * GC_THREADS;
      g[u] = i < hi ? code[i] : NO_GROUP;
      r[u] = i < hi ? (unsigned long long)a.range_c[i] : 0ull;
    }
#pragma unroll
    for (u32 u = 0; u < U; ++u)
      if (g[u] < (u32)GROUP_SLOTS && r[u] == s_best[g[u]]) atomicMin(&s_row[g[u]], i0 + u * GC_THREADS);
  }
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

// Rows of the group table: a wavefront per communicator.  The communicators before it are summed by the wavefront
// itself (a few thousand counts from the L2) unless the counts were scanned before (SCANNED: many communicators,
// where that would be quadratic).
template <bool SCANNED>
__global__ __launch_bounds__(256) void k_group_emit(GroupArgs a) {
  if (a.counters[CNT_STATUS] != 0) return;
  const u32 c = blockIdx.x * 4 + threadIdx.x / CCLD_WAVE, lane = lane_id();
  if (c >= a.n_comms) return;
  u32 pos = 0, cnt;
  if (SCANNED) {
    pos = a.comm_groups[c];
    cnt = a.comm_groups[c + 1] - pos;
  } else {
    for (u32 i = lane; i < c; i += CCLD_WAVE) pos += a.comm_groups[i];
    pos = wave_sum(pos);
    cnt = a.comm_groups[c];
    if (c + 1 == a.n_comms && lane == 0) a.counters[CNT_NGROUP] = (u64)pos + cnt;
  }
  const u32 lo = a.comm_row[c];
  const u64 C = a.group_cap;
  i64* __restrict__ O = a.group;
  for (u32 p = lane; p < cnt; p += CCLD_WAVE) {
    const u64 g = (u64)pos + p;
    if (g >= C) break;
    const u32 w = a.stage[0][lo + p], sx = a.stage[1][lo + p];
    const u32 code = w & 1023u, cls = w >> 12;
    const bool dynamic = (w >> 10) & 1u, slow = (w >> 11) & 1u;
    const GroupState G = a.gstate[(u64)c * GROUP_SLOTS + code];
    auto col = [&](int k) -> i64 { return a.seg[(u64)k * a.seg_cap + sx]; };
    O[CCLD_GRP_COMM * C + g] = (i64)c;
    O[CCLD_GRP_OP * C + g] = (i64)(code / GROUP_CLS);
    O[CCLD_GRP_CLS * C + g] = (i64)(code % GROUP_CLS);
    O[CCLD_GRP_N_USABLE * C + g] = (i64)a.stage[2][lo + p];
    O[CCLD_GRP_RSTAR_SEQ * C + g] = col(CCLD_SEG_SEQ);
    O[CCLD_GRP_TMAX * C + g] = col(CCLD_SEG_DUR_MAX);
    O[CCLD_GRP_TMIN * C + g] = col(CCLD_SEG_DUR_MIN);
    O[CCLD_GRP_TBASE * C + g] = dynamic ? G.tbase_dyn : a.p.tbase_init_ns;
    O[CCLD_GRP_STATIC * C + g] = dynamic ? 0 : 1;
    O[CCLD_GRP_FROZEN * C + g] = G.frozen;
    O[CCLD_GRP_M * C + g] = G.cnt;
    O[CCLD_GRP_SLOW * C + g] = slow ? 1 : 0;
    O[CCLD_GRP_CLASS * C + g] = (i64)cls;
    O[CCLD_GRP_ROOT_S1 * C + g] = (slow && cls != CCLD_SLOW_S2_COMMUNICATION) ? col(CCLD_SEG_ARGMIN_RANK) : (i64)CCLD_NO_RANK;
    // communication-slow root (Eq. 4): the communicator's member of minimal SendRate / RecvRate
    O[CCLD_GRP_ROOT_S2 * C + g] =
        (cls == CCLD_SLOW_S2_COMMUNICATION || cls == CCLD_SLOW_S3_MIXED) ? a.rate_root[c] : (i64)CCLD_NO_RANK;
    O[CCLD_GRP_REPEATS * C + g] = G.repeats;
    O[CCLD_GRP_LOCATE * C + g] = (slow && G.repeats >= a.p.repeat_threshold) ? 1 : 0;
  }
}

// From this many communicators on the counts are scanned by a launch of their own
constexpr u32 GROUP_SCAN_COMMS = 8192;

void launch_groups(hipStream_t st, const GroupArgs& a) {
  hipLaunchKernelGGL(k_group_comm, dim3(a.n_comms), dim3(GC_THREADS), 0, st, a);
  const u32 blocks = (a.n_comms + 3) / 4;
  if (a.n_comms < GROUP_SCAN_COMMS) {
    hipLaunchKernelGGL(k_group_emit<false>, dim3(blocks), dim3(256), 0, st, a);
  } else {
    launch_scan_tiles(st, a.comm_groups, a.n_comms, &a.counters[CNT_NGROUP]);
    hipLaunchKernelGGL(k_group_emit<true>, dim3(blocks), dim3(256), 0, st, a);
  }
}

}  // namespace ccld
