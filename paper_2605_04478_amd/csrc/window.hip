// Window analysis kernels for gfx950: ingest (validation, keys, bucketed placement), collective
// heads per tile, compaction of the late-rank flags, per-rank blame, and hang alerts.  The
// per-collective statistics are in segments.hip, the end of an analysis (slow-detection rules, flags of a window on the grid,
// blame order) in groups.hip, the sort in radix_sort.hip.
#include "window_kernels.h"
#include "alerts.h"
#include "blame_order.h"
#include "device_utils.h"
#include "grid.h"
#include "report.h"
#include "rows.h"
#include "select.h"

namespace ccld {

constexpr i64 T_INFLIGHT = INT64_MAX;

__device__ __forceinline__ void atomic_or_u64(u64* p, u64 v) { atomicOr((unsigned long long*)p, (unsigned long long)v); }
__device__ __forceinline__ u64 atomic_add_u64(u64* p, u64 v) {
  return atomicAdd((unsigned long long*)p, (unsigned long long)v);
}

// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_fill_u64(u64* p, u64 n, u64 v) {
  for (u64 i = (u64)blockIdx.x * 256 + threadIdx.x; i < n; i += (u64)gridDim.x * 256) p[i] = v;
}
void launch_fill_u64(hipStream_t st, uint64_t* p, uint64_t n, uint64_t v) {
  if (n == 0) return;
  u32 g = (u32)((n + 255) / 256); if (g > 4096) g = 4096;
  hipLaunchKernelGGL(k_fill_u64, dim3(g), dim3(256), 0, st, p, n, v);
}

// ------------------------------------------------------------------------------------------
// Ingest: validate each record, key it by Trace ID (communicator id, operation counter) plus member slot, pack its
// payload into a 16-byte row (rows.h) and store both at the window's tail.  Small windows keep the order of arrival; in
// large ones a batch's records are placed grouped by communicator bucket, so that the grid placement, which takes the
// window bucket by bucket, meets few fine buckets at a time.
//
// Every kernel also leaves, per communicator, the batch's largest operation counter and largest complement of one (i.e.
// ~smallest) in a.range: the grid is laid out from these.  The header and the ranges of a batch start from zero: the
// ingest of the batch before cleared them (clear_next), the first ones were cleared at create.
__device__ __forceinline__ void clear_next(const IngestArgs& a, u32 n_comms, u32 tid, u32 threads) {
  if (blockIdx.x == 0 && tid == 0) {
    BatchMeta z = {};
    *a.meta_next = z;
  }
  if (a.range_next)
    for (u64 i = (u64)blockIdx.x * threads + tid; i < 2ull * n_comms; i += (u64)gridDim.x * threads) a.range_next[i] = 0;
}
// what is known of the batch before its first record is read
__device__ __forceinline__ void put_header(const IngestArgs& a, i64 ref) {
  a.meta->ref = ref; a.meta->tail = a.tail; a.meta->n = a.n;
  a.meta->chunk = a.chunk; a.meta->round0 = a.round0; a.meta->n_rounds = a.per_group * gridDim.x; a.meta->per_group = a.per_group;
}

// Records per communicator bucket in each workgroup's slice of the batch (first half of the bucketed placement).  Tables
// of no more words than this are scanned by every placement workgroup for itself, larger ones by two launches.  Streams at 6 TB/s where
// records come in a random order; in time order neighbouring lanes add to the same few words of LDS one after the other (70M records 49
// and 199 us).
constexpr u32 INGEST_SCAN_WORDS = 8192;
template <u32 THREADS>
__global__ __launch_bounds__(THREADS) void k_ingest_hist(IngestArgs a, u32 n_comms) {
  extern __shared__ u32 s_cnt[];        // [n_buckets]
  for (u32 b = threadIdx.x; b < a.n_buckets; b += THREADS) s_cnt[b] = 0;
  __syncthreads();
  const u64 chunk = a.chunk / a.hist_split;
  const u64 i_end = (chunk * (blockIdx.x + 1)) < a.n ? chunk * (blockIdx.x + 1) : a.n;
  const u32* __restrict__ in_comm = a.comm;
  for (u64 i0 = chunk * blockIdx.x + threadIdx.x; i0 < i_end; i0 += THREADS * 8) {
    u32 c[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool on = i0 + (u64)u * THREADS < i_end;
      c[u] = on ? __builtin_nontemporal_load(in_comm + i0 + (u64)u * THREADS) : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i0 + (u64)u * THREADS < i_end) atomicAdd(&s_cnt[c[u] < n_comms ? (c[u] >> a.bshift) : 0u], 1u);
  }
  __syncthreads();
  for (u32 b = threadIdx.x; b < a.n_buckets; b += THREADS) a.table[(u64)b * gridDim.x + blockIdx.x] = s_cnt[b];
}
// exclusive scan of every bucket's row of per-workgroup counts (row length <= 2048)
__global__ __launch_bounds__(256) void k_ingest_scan(u32* table, u32* totals, u32 n_blocks) {
  __shared__ u32 s_wave[4];
  u32* row = table + (u64)blockIdx.x * n_blocks;
  u32 v[8], sum = 0;
  const u32 i0 = threadIdx.x * 8;
#pragma unroll
  for (int k = 0; k < 8; ++k) { v[k] = (i0 + k) < n_blocks ? row[i0 + k] : 0u; sum += v[k]; }
  u32 tot;
  u32 ex = block_exclusive_sum<256>(sum, s_wave, &tot);
#pragma unroll
  for (int k = 0; k < 8; ++k) { if ((i0 + k) < n_blocks) row[i0 + k] = ex; ex += v[k]; }
  if (threadIdx.x == 0) totals[blockIdx.x] = tot;
}

// Validation and key of one record (Trace ID = communicator id + operation counter, then the rank's
// member slot).  mem = the rank's packed membership row when the topology has them (packed).
__device__ __forceinline__ u64 ingest_key(u32 r, u32 c, u64 sq, u32 op, i64 te, i64 tx, const uint4& mem,
                                          bool packed, const DeviceTopology& T, const KeyFormat& kf,
                                          u32 slot_mask, u64& status, u64& maxseq, u64& maxinv) {
  u64 key = 0;
  if (c >= T.n_comms) {
    status |= DS_UNKNOWN_COMM;
    return key;
  }
  bool member = false;
  u32 slot = 0;
  if (packed) {
    const u32 w = c == (mem.x >> kf.mb) ? mem.x : c == (mem.y >> kf.mb) ? mem.y : c == (mem.z >> kf.mb) ? mem.z : mem.w;
    member = c == (w >> kf.mb);
    slot = w & slot_mask;
  } else if (r < T.n_ranks) {
    for (u32 q = T.rank_comm_off[r]; q < T.rank_comm_off[r + 1]; ++q)
      if (T.rank_comms[q] == c) { member = true; slot = T.rank_slots[q]; }
    wait_vector_memory();              // nothing of this branch is waited for behind it
  }
  if (!member) status |= DS_NOT_MEMBER;
  if (op >= CCLD_OP_MAX || te < 0 || te == T_INFLIGHT || tx < te) status |= DS_RANGE;
  if (kf.sb < 64 && (sq >> kf.sb) != 0) {
    status |= DS_KEY_WIDTH;
  } else {
    key = (kf.cb ? ((u64)c << (64 - kf.cb)) : 0ull) | (sq << kf.mb) | (u64)slot;
    maxseq = sq > maxseq ? sq : maxseq;
    maxinv = ~sq > maxinv ? ~sq : maxinv;
  }
  return key;
}

// status bits and the extreme operation counters of a workgroup leave through one set of atomics, its counter ranges
// per communicator (s_rng: [n_comms][2], null if nobody wants them) through one pair per communicator that it met
template <int THREADS>
__device__ __forceinline__ void ingest_publish(u64 status, u64 maxseq, u64 maxinv, u64* s_status, u64* s_max,
                                               u64* s_inv, const IngestArgs& a, const unsigned long long* s_rng, u32 n_comms) {
  u64 st = status;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) st |= shfl_xor_u64(st, m);
  u64 mx = wave_max_u64(maxseq), mi = wave_max_u64(maxinv);
  const u32 lane = lane_id(), wave = threadIdx.x / CCLD_WAVE;
  if (lane == 0) { s_status[wave] = st; s_max[wave] = mx; s_inv[wave] = mi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    u64 S = 0, M = 0, I = 0;
    for (int w = 0; w < THREADS / CCLD_WAVE; ++w) {
      S |= s_status[w]; M = s_max[w] > M ? s_max[w] : M; I = s_inv[w] > I ? s_inv[w] : I;
    }
    if (S) atomic_or_u64(&a.meta->status, S);
    if (M) atomicMax((unsigned long long*)&a.meta->max_seq, (unsigned long long)M);
    if (I) atomicMax((unsigned long long*)&a.meta->max_inv_seq, (unsigned long long)I);
  }
  if (a.range)
    for (u32 i = threadIdx.x; i < 2 * n_comms; i += THREADS)
      if (s_rng[i]) atomicMax((unsigned long long*)&a.range[i], s_rng[i]);
}
// the counter range of a record's communicator: after the first few records of a communicator neither end moves, so the
// entries are read before they are raised
__device__ __forceinline__ void note_range(unsigned long long* s_rng, u32 c, u64 seq) {
  const unsigned long long hi = seq, lo = ~seq;
  if (hi > s_rng[2 * c]) atomicMax(&s_rng[2 * c], hi);
  if (lo > s_rng[2 * c + 1]) atomicMax(&s_rng[2 * c + 1], lo);
}

// Windows that keep the order of arrival: slot = tail + number in the batch.  One launch, a few records per thread on their way
// at a time.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_ingest(IngestArgs a, DeviceTopology T, KeyFormat kf) {
  constexpr int U = 4;               // records per thread in flight
  extern __shared__ unsigned long long s_rng[];   // [n_comms][2] if a.range
  __shared__ u64 s_status[THREADS / CCLD_WAVE], s_max[THREADS / CCLD_WAVE], s_inv[THREADS / CCLD_WAVE];
  if (a.range) for (u32 i = threadIdx.x; i < 2 * T.n_comms; i += THREADS) s_rng[i] = 0;
  const i64 ref = a.t_enter[0];
  clear_next(a, T.n_comms, threadIdx.x, THREADS);
  if (blockIdx.x == 0 && threadIdx.x == 0) put_header(a, ref);
  __syncthreads();
  u64 status = 0, maxseq = 0, maxinv = 0;      // maxinv = ~(smallest operation counter)
  const uint4* __restrict__ memb4 = reinterpret_cast<const uint4*>(T.rank_memb4);
  const u32 slot_mask = kf.mb < 32 ? (1u << kf.mb) - 1 : ~0u;
  // every workgroup walks one contiguous slice of the batch
  const u64 i_end = (a.chunk * (blockIdx.x + 1)) < a.n ? a.chunk * (blockIdx.x + 1) : a.n;
  for (u64 i0 = a.chunk * blockIdx.x + threadIdx.x; i0 < i_end; i0 += THREADS * U) {
    u32 r[U], c[U], op[U];
    u64 sq[U], nb[U];
    i64 te[U], tx[U];
    uint4 mem[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const u64 i = i0 + (u64)u * THREADS;
      if (i < i_end) {
        r[u] = __builtin_nontemporal_load(a.rank + i); c[u] = __builtin_nontemporal_load(a.comm + i);
        sq[u] = __builtin_nontemporal_load(a.seq + i); op[u] = __builtin_nontemporal_load(a.op + i);
        nb[u] = __builtin_nontemporal_load(a.bytes + i);
        te[u] = __builtin_nontemporal_load(a.t_enter + i); tx[u] = __builtin_nontemporal_load(a.t_exit + i);
      }
    }
    // the communicators of each rank with its member slot in each: one 16-byte row of words
    // comm << mb | slot when no rank is in more than four communicators
#pragma unroll
    for (int u = 0; u < U; ++u) {
      mem[u] = make_uint4(~0u, ~0u, ~0u, ~0u);
      if (i0 + (u64)u * THREADS < i_end && memb4 && r[u] < T.n_ranks) mem[u] = memb4[r[u]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const u64 i = i0 + (u64)u * THREADS;
      if (i >= i_end) continue;
      const u64 key = ingest_key(r[u], c[u], sq[u], op[u], te[u], tx[u], mem[u], memb4 != nullptr, T, kf, slot_mask, status,
                                 maxseq, maxinv);
      if (a.range && c[u] < T.n_comms) note_range(s_rng, c[u], sq[u]);
      u64 p = (u64)a.tail + i;
      if (p >= a.cap) p -= a.cap;
      a.win_key[p] = key;
      uint4 row;
      if (!pack_row(te[u], tx[u], nb[u], op[u], ref, (u32)p, &row)) {
        a.win_wide[3 * p] = te[u]; a.win_wide[3 * p + 1] = tx[u]; a.win_wide[3 * p + 2] = (i64)nb[u];
      }
      a.win_row[p] = row;
    }
  }
  ingest_publish<THREADS>(status, maxseq, maxinv, s_status, s_max, s_inv, a, s_rng, T.n_comms);
}
// Windows placed by bucket.  A workgroup takes CHUNK records per round, gives each its slot in its bucket (LDS atomic),
// then stages keys and rows in LDS ordered by (bucket, slot) and writes them out with consecutive lanes
// on consecutive pieces: every bucket's share of the round leaves as one contiguous run instead of one scattered store
// per lane.  LDS_TABLE keeps a copy of the ranks' packed membership rows in LDS, since with records in random order that
// lookup is a gather with no locality.
//
// Bound by memory: a line that a round leaves unfinished would be completed by the next one 7 us later, when it has left the
// L2 in parts.  So rows leave eight slots at a time (a line of rows, half a line of keys), with the streaming
// hint; up to seven of a bucket wait in registers for the next round.  82M records of 4,096 ranks, all in one session: 136 buckets, which
// is what such windows have, ranks' rows from the L2, 1,131 us (4.7 TB/s); 68 buckets 1,114 with the ranks' rows in LDS, 1,118 without, and
// 1,245 with every round written as it is.  (Four slots at a time took 2 % longer with 68 buckets, and 8 % with 136 beside the ranks'
// rows in LDS.)  A tenth more where one record in eight lies 2^42 ns from the batch's first and is written at full width too.
template <int THREADS, bool LDS_TABLE>
__global__ __launch_bounds__(THREADS) void k_ingest_staged(IngestArgs a, DeviceTopology T, KeyFormat kf) {
  constexpr int U = 2;
  constexpr u32 CHUNK = THREADS * U, LINE = INGEST_LINE;
  constexpr u32 HELD = INGEST_STAGED_BUCKETS * LINE / THREADS;       // rows that wait in a thread
  static_assert(CHUNK == INGEST_ROUND, "a row has room for the record's number in its round");
  static_assert(INGEST_STAGED_BUCKETS <= 256 && INGEST_STAGED_BUCKETS <= THREADS, "a byte and a thread per bucket");
  // [n_ranks] membership rows (LDS_TABLE) | [ingest_stage_rows] rows | the same number of keys | [n_comms][2] ranges
  extern __shared__ uint4 s_dyn[];
  __shared__ u64 s_status[THREADS / CCLD_WAVE], s_max[THREADS / CCLD_WAVE], s_inv[THREADS / CCLD_WAVE];
  // per bucket: its next slot; and what turns a slot into a place in the staging order, the first slot not written yet, the
  // first slot that this round leaves unwritten
  __shared__ u32 s_off[INGEST_STAGED_BUCKETS], s_total;
  __shared__ uint4 s_run[INGEST_STAGED_BUCKETS];
  __shared__ uint8_t s_bucket[ingest_stage_rows(INGEST_STAGED_BUCKETS) / LINE];   // of every LINE staged rows
  __shared__ u32 s_scan[THREADS / CCLD_WAVE];
  const u32 stage_rows = ingest_stage_rows(a.n_buckets);
  uint4* s_row = s_dyn + (LDS_TABLE ? T.n_ranks : 0u);
  u64* s_key = reinterpret_cast<u64*>(s_row + stage_rows);
  unsigned long long* s_rng = reinterpret_cast<unsigned long long*>(s_key + stage_rows);
  const u32 tid = threadIdx.x;
  // slots count from the window's first one: a.tail is the first of the batch
  u32 from = 0, start = 0;              // of the thread's bucket: first slot not written yet, next slot at the start of the round
  if (a.table_words > INGEST_SCAN_WORDS) {
    if (tid < a.n_buckets) start = a.tail + a.bucket_base[tid] + a.table[((u64)tid * gridDim.x + blockIdx.x) * a.hist_split];
  } else {
    // the buckets' records, and those of the workgroups before this one: a wavefront per bucket.  (One workgroup that scanned
    // the table at the end of the counting took 20 of its 28 us at 2M records in 32 buckets.)
    const u32 row = gridDim.x * a.hist_split, upto = blockIdx.x * a.hist_split;
    for (u32 b = tid / CCLD_WAVE; b < a.n_buckets; b += THREADS / CCLD_WAVE) {
      u32 before = 0, all = 0;
#pragma unroll 4
      for (u32 i = lane_id(); i < row; i += CCLD_WAVE) {
        const u32 v = a.table[(u64)b * row + i];
        all += v; before += i < upto ? v : 0u;
      }
      before = wave_sum(before); all = wave_sum(all);
      if (lane_id() == 0) { s_run[b].x = before; s_run[b].y = all; }
    }
    __syncthreads();
    u32 total;
    const u32 base = block_exclusive_sum<THREADS>(tid < a.n_buckets ? s_run[tid].y : 0u, s_scan, &total);
    if (tid < a.n_buckets) {
      start = a.tail + base + s_run[tid].x;
      if (blockIdx.x == 0) a.bucket_base[tid] = base;
    }
    if (blockIdx.x == 0 && tid == 0) a.bucket_base[a.n_buckets] = total;
  }
  from = start;
  if (tid < a.n_buckets) s_off[tid] = start;
  if (LDS_TABLE) {
    const uint4* __restrict__ g = reinterpret_cast<const uint4*>(T.rank_memb4);
    for (u32 r = tid; r < T.n_ranks; r += THREADS) s_dyn[r] = g[r];
  }
  if (a.range) for (u32 i = tid; i < 2 * T.n_comms; i += THREADS) s_rng[i] = 0;
  const i64 ref = a.t_enter[0];
  clear_next(a, T.n_comms, tid, THREADS);
  if (blockIdx.x == 0 && tid == 0) put_header(a, ref);
  __syncthreads();
  u64 status = 0, maxseq = 0, maxinv = 0;
  const u32* __restrict__ in_rank = a.rank;
  const u32* __restrict__ in_comm = a.comm;
  const u64* __restrict__ in_seq = a.seq;
  const uint8_t* __restrict__ in_op = a.op;
  const u64* __restrict__ in_bytes = a.bytes;
  const i64* __restrict__ in_te = a.t_enter;
  const i64* __restrict__ in_tx = a.t_exit;
  u64* __restrict__ out_key = a.win_key;
  uint4* __restrict__ out_row = a.win_row;
  const uint4* __restrict__ memb4 = reinterpret_cast<const uint4*>(T.rank_memb4);
  const u32 slot_mask = kf.mb < 32 ? (1u << kf.mb) - 1 : ~0u;
  const u64 i_begin = a.chunk * blockIdx.x;
  const u64 i_end = (a.chunk * (blockIdx.x + 1)) < a.n ? a.chunk * (blockIdx.x + 1) : a.n;
  // the next round's columns are loaded while this round is staged and written out
  u32 r[U], c[U], op[U], nr[U], nc[U], nop[U];
  u64 sq[U], nb[U], nsq[U], nnb[U];
  i64 te[U], tx[U], nte[U], ntx[U];
  auto load_round = [&](u64 base, u32 (&R)[U], u32 (&C)[U], u64 (&S)[U], u32 (&O)[U], u64 (&B)[U], i64 (&E)[U], i64 (&X)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const u64 i = base + (u64)u * THREADS + tid;
      if (i < i_end) {
        R[u] = __builtin_nontemporal_load(in_rank + i); C[u] = __builtin_nontemporal_load(in_comm + i);
        S[u] = __builtin_nontemporal_load(in_seq + i); O[u] = __builtin_nontemporal_load(in_op + i);
        B[u] = __builtin_nontemporal_load(in_bytes + i);
        E[u] = __builtin_nontemporal_load(in_te + i); X[u] = __builtin_nontemporal_load(in_tx + i);
      }
    }
  };
  u32* round_row = a.rounds + ((u64)a.round0 + (u64)blockIdx.x * a.per_group) * a.n_buckets + tid;      // used below n_buckets only
  // rows that wait: of bucket i / LINE the one at place i % LINE of its line, i = tid, tid + THREADS, ...
  // (an array of uint4 would lie in scratch memory: 82M records 1,330 us in place of 1,251)
  typedef u32 u32x4 __attribute__((ext_vector_type(4)));
  u32x4 h_row[HELD];
  u64 h_key[HELD];
  u32 held = 0;                          // a bit each
  load_round(i_begin, r, c, sq, op, nb, te, tx);
  wait_vector_memory();
  for (u64 base = i_begin; base < i_end; base += CHUNK) {        // uniform over the workgroup
    u32 at[U], bk[U];
    u64 key[U];
    bool on[U];
#pragma unroll
    for (int u = 0; u < U; ++u) on[u] = base + (u64)u * THREADS + tid < i_end;
    // the packed membership rows, if not from LDS then before the next round's columns are asked for: loads complete in order
    uint4 mem[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      mem[u] = make_uint4(~0u, ~0u, ~0u, ~0u);
      if (on[u] && (LDS_TABLE || memb4) && r[u] < T.n_ranks) mem[u] = LDS_TABLE ? s_dyn[r[u]] : memb4[r[u]];
    }
    if (!LDS_TABLE) wait_vector_memory();
    load_round(base + CHUNK, nr, nc, nsq, nop, nnb, nte, ntx);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!on[u]) continue;
      key[u] = ingest_key(r[u], c[u], sq[u], op[u], te[u], tx[u], mem[u], LDS_TABLE || memb4, T, kf, slot_mask, status, maxseq, maxinv);
      if (a.range && c[u] < T.n_comms) note_range(s_rng, c[u], sq[u]);
      bk[u] = c[u] < T.n_comms ? (c[u] >> a.bshift) : 0u;
      at[u] = atomicAdd(&s_off[bk[u]], 1u);
    }
    __syncthreads();
    // the staging order: every bucket's slots from the line on that holds its first one not written yet, in whole lines
    {
      const u32 to = tid < a.n_buckets ? s_off[tid] : 0u, first = from & ~(LINE - 1);
      const u32 cnt = tid < a.n_buckets && to != from ? (to - first + LINE - 1) & ~(LINE - 1) : 0u;
      u32 pre, all;
      if (a.n_buckets <= CCLD_WAVE) {
        const u32 inc = wave_inclusive_sum(cnt);
        pre = inc - cnt; all = inc;
        if (tid == CCLD_WAVE - 1) s_total = all;
      } else {
        pre = block_exclusive_sum<THREADS>(cnt, s_scan, &all);
        if (tid == 0) s_total = all;
      }
      if (tid < a.n_buckets) {
        // rows of lines that are not full wait, unless there is no next round
        u32 upto = to;
        if (base + CHUNK < i_end) { const u32 whole = to & ~(LINE - 1); upto = whole > from ? whole : from; }
        s_run[tid] = make_uint4(pre - first, from, upto, 0u);
        from = upto;
        *round_row = start - a.tail;
        start = to;
      }
      round_row += a.n_buckets;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!on[u]) continue;
      const u32 q = s_run[bk[u]].x + at[u];
      s_bucket[q / LINE] = (uint8_t)bk[u];       // every line has a row that names its bucket
      const u32 p = at[u] >= a.cap ? at[u] - a.cap : at[u];
      s_key[q] = key[u];
      uint4 row;
      if (!pack_row(te[u], tx[u], nb[u], op[u], ref, p, &row)) {
        a.win_wide[3 * (u64)p] = te[u]; a.win_wide[3 * (u64)p + 1] = tx[u]; a.win_wide[3 * (u64)p + 2] = (i64)nb[u];
      }
      row.y |= ((u32)u * THREADS + tid) << ROW_CELL_SHIFT;
      s_row[q] = row;
    }
#pragma unroll
    for (u32 h = 0; h < HELD; ++h) {
      const u32 i = tid + h * THREADS;
      if (held >> h & 1) {
        const u32 q = s_run[i / LINE].x + (s_run[i / LINE].y & ~(LINE - 1)) + i % LINE;
        s_bucket[q / LINE] = (uint8_t)(i / LINE);
        s_row[q] = make_uint4(h_row[h].x, h_row[h].y, h_row[h].z, h_row[h].w); s_key[q] = h_key[h];
      }
    }
    __syncthreads();
    wait_vector_memory();              // the next round's columns; the stores below have the next round's time
    const u32 total = s_total;
    // Whole lines leave with the streaming hint: they do not stay in the L2
    for (u32 q = tid; q < total; q += THREADS) {
      const uint4 run = s_run[s_bucket[q / LINE]];
      const u32 v = q - run.x, lo = run.y, hi = run.z, D = v >= a.cap ? v - a.cap : v;
      const bool full = (v & ~(LINE - 1)) >= lo && (v | (LINE - 1)) < hi;
      if (v < lo || v >= hi) continue;
      const uint4 row = s_row[q];
      const u64 k = s_key[q];
      if (full) {
        u32x4 vv = {row.x, row.y, row.z, row.w};
        __builtin_nontemporal_store(vv, reinterpret_cast<u32x4*>(out_row + D));
        __builtin_nontemporal_store(k, out_key + D);
      } else {
        out_row[D] = row; out_key[D] = k;
      }
    }
    held = 0;
#pragma unroll
    for (u32 h = 0; h < HELD; ++h) {
      const u32 i = tid + h * THREADS, b = i / LINE;
      if (b >= a.n_buckets) continue;
      const u32 to = s_off[b], v = (to & ~(LINE - 1)) + i % LINE;
      if (v >= s_run[b].z && v < to) {
        const u32 q = s_run[b].x + v;
        const uint4 row = s_row[q];
        h_row[h] = u32x4{row.x, row.y, row.z, row.w}; h_key[h] = s_key[q]; held |= 1u << h;
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      r[u] = nr[u]; c[u] = nc[u]; sq[u] = nsq[u]; op[u] = nop[u]; nb[u] = nnb[u]; te[u] = nte[u]; tx[u] = ntx[u];
    }
  }
  // rounds that this workgroup did not need: they start where it ends
  for (u32 k = (u32)((i_end > i_begin ? i_end - i_begin + CHUNK - 1 : 0) / CHUNK); k < a.per_group; ++k, round_row += a.n_buckets)
    if (tid < a.n_buckets) *round_row = start - a.tail;
  ingest_publish<THREADS>(status, maxseq, maxinv, s_status, s_max, s_inv, a, s_rng, T.n_comms);
}
// a batch without records: its header names its place in the window
__global__ __launch_bounds__(256) void k_ingest_empty(IngestArgs a, u32 n_comms) {
  clear_next(a, n_comms, threadIdx.x, 256);
  if (blockIdx.x == 0 && threadIdx.x == 0) put_header(a, 0);
}

// One 1,024-thread workgroup per compute unit; four counting workgroups per placement workgroup where a batch is large
// enough, one (and the scan of the counts without a launch of its own) otherwise.
constexpr u32 INGEST_GROUPS = 256;
IngestShape ingest_shape(uint64_t n) {
  IngestShape s = {0, 0, 1, 0};
  if (n == 0) return s;
  s.groups = (uint32_t)std::min<uint64_t>((n + INGEST_ROUND - 1) / INGEST_ROUND, INGEST_GROUPS);
  s.hist_split = n >= (1u << 23) ? 4 : 1;
  const uint64_t unit = 256ull * s.hist_split;
  s.chunk = ((n + s.groups - 1) / s.groups + unit - 1) / unit * unit;
  s.per_group = (uint32_t)((s.chunk + INGEST_ROUND - 1) / INGEST_ROUND);
  return s;
}
template <class F>
static void each_ingest_staged(F f) {
  f(&k_ingest_staged<1024, true>); f(&k_ingest_staged<1024, false>);
}
hipError_t allow_lds_window() {
  hipError_t e = hipSuccess;
  each_ingest_staged([&](auto k) { if (e == hipSuccess) e = allow_lds(reinterpret_cast<const void*>(k), INGEST_LDS); });
  return e;
}
void launch_ingest(hipStream_t st, const IngestArgs& a_in, const DeviceTopology& T, const KeyFormat& kf) {
  IngestArgs a = a_in;
  const size_t range_lds = a.range ? (size_t)16 * T.n_comms : 0;
  if (a.n == 0) {
    hipLaunchKernelGGL(k_ingest_empty, dim3(8), dim3(256), 0, st, a, T.n_comms);
    return;
  }
  if (a.n_buckets == 1) {
    // A workgroup of 256 threads per 1,024 records while that makes no more of them than compute units, then one of 1,024 threads to
    // each: every workgroup raises the ranges of the communicators that it met, and the requests for one line of them follow
    // one another at 10 to 20 ns (1,024 workgroups and 174 communicators: 32 us for 1.07M records, 21 so; a window 157 -> 146).  The line
    // is where the first kind would have more workgroups than compute units: windows of 262,860, 319,800, 390,000 and 858,000 records of
    // 390 ranks take 75, 82, 85 and 109 us with the first kind, 75, 82, 82 and 94 with the second.
    if (a.n <= INGEST_GROUPS * 1024) {
      a.chunk = 1024;
      hipLaunchKernelGGL(k_ingest<256>, dim3((u32)((a.n + 1023) / 1024)), dim3(256), range_lds, st, a, T, kf);
    } else {
      a.chunk = ((a.n + INGEST_GROUPS - 1) / INGEST_GROUPS + 255) / 256 * 256;
      hipLaunchKernelGGL(k_ingest<1024>, dim3(INGEST_GROUPS), dim3(1024), range_lds, st, a, T, kf);
    }
    return;
  }
  const IngestShape shape = ingest_shape(a.n);
  const u64 g = shape.groups;
  a.hist_split = shape.hist_split; a.chunk = shape.chunk; a.per_group = shape.per_group;
  const u32 g_hist = (u32)(g * a.hist_split);
  a.table_words = a.n_buckets * g_hist;
  // (one counting workgroup to a placement workgroup: of 1,024 threads, so that the compute units have as much on their way as with
  // four of 256)
  if (a.hist_split == 1) hipLaunchKernelGGL(k_ingest_hist<1024>, dim3(g_hist), dim3(1024), sizeof(u32) * a.n_buckets, st, a, T.n_comms);
  else hipLaunchKernelGGL(k_ingest_hist<256>, dim3(g_hist), dim3(256), sizeof(u32) * a.n_buckets, st, a, T.n_comms);
  if (a.table_words > INGEST_SCAN_WORDS) {
    hipLaunchKernelGGL(k_ingest_scan, dim3(a.n_buckets), dim3(256), 0, st, a.table, a.bucket_base, g_hist);
    launch_scan_tiles(st, a.bucket_base, a.n_buckets, a.scratch_total);
  }
  // the ranks' membership rows in LDS where they fit beside the lines: since rows leave in lines that is worth 1 % at most (15.4M records of
  // 512 ranks in a random order 220 us in place of 222; 20M of 4,096 ranks 299 both ways)
  const u32 range_comms = a.range ? T.n_comms : 0;
  const size_t lines = ingest_lds(a.n_buckets, range_comms, 0), both = ingest_lds(a.n_buckets, range_comms, T.n_ranks);
  auto go = [&](auto kernel, size_t bytes) { hipLaunchKernelGGL(kernel, dim3((u32)g), dim3(1024), bytes, st, a, T, kf); };
  if (T.rank_memb4 && both <= INGEST_LDS) go(k_ingest_staged<1024, true>, both);
  else go(k_ingest_staged<1024, false>, lines);
}

// ------------------------------------------------------------------------------------------
// In-place exclusive scan of per-tile counts by one workgroup; counts[n_tiles] and *total_out
// receive the total.
constexpr int SCAN_PER = 8;          // consecutive counts per thread and round
__device__ __forceinline__ void scan_load(const u32* counts, u32 i0, u32 n_tiles, bool vec, u32 (&v)[SCAN_PER]) {
  if (vec && i0 + SCAN_PER <= n_tiles) {
    const uint4 a = *reinterpret_cast<const uint4*>(counts + i0), b = *reinterpret_cast<const uint4*>(counts + i0 + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else {
#pragma unroll
    for (int k = 0; k < SCAN_PER; ++k) v[k] = (i0 + k) < n_tiles ? counts[i0 + k] : 0u;
  }
}
__global__ __launch_bounds__(1024) void k_scan_tiles(u32* counts, u32 n_tiles, u64* total_out) {
  static_assert(SCAN_PER == 8, "two 16-byte pieces per thread");
  __shared__ u32 s_wave[1024 / CCLD_WAVE];
  const bool vec = (reinterpret_cast<uintptr_t>(counts) & 15) == 0;
  u32 carry = 0;
  u32 v[SCAN_PER], nv[SCAN_PER];
  scan_load(counts, threadIdx.x * SCAN_PER, n_tiles, vec, v);
  for (u32 b = 0; b < n_tiles; b += 1024 * SCAN_PER) {
    const u32 i0 = b + threadIdx.x * SCAN_PER;
    // the next round's counts are on their way while this round is scanned and stored
    scan_load(counts, i0 + 1024 * SCAN_PER, n_tiles, vec, nv);
    u32 sum = 0;
#pragma unroll
    for (int k = 0; k < SCAN_PER; ++k) sum += v[k];
    u32 tot;
    u32 ex = carry + block_exclusive_sum<1024>(sum, s_wave, &tot);
    if (vec && i0 + SCAN_PER <= n_tiles) {
      u32 o[SCAN_PER];
#pragma unroll
      for (int k = 0; k < SCAN_PER; ++k) { o[k] = ex; ex += v[k]; }
      *reinterpret_cast<uint4*>(counts + i0) = make_uint4(o[0], o[1], o[2], o[3]);
      *reinterpret_cast<uint4*>(counts + i0 + 4) = make_uint4(o[4], o[5], o[6], o[7]);
    } else {
#pragma unroll
      for (int k = 0; k < SCAN_PER; ++k) { if ((i0 + k) < n_tiles) counts[i0 + k] = ex; ex += v[k]; }
    }
    carry += tot;
#pragma unroll
    for (int k = 0; k < SCAN_PER; ++k) v[k] = nv[k];
  }
  if (threadIdx.x == 0) { counts[n_tiles] = carry; *total_out = carry; }
}
void launch_scan_tiles(hipStream_t st, uint32_t* counts, uint32_t n_tiles, uint64_t* total_out) {
  hipLaunchKernelGGL(k_scan_tiles, dim3(1), dim3(1024), 0, st, counts, n_tiles, total_out);
}

// ------------------------------------------------------------------------------------------
// ------------------------------------------------------------------------------------------
// Ordered compaction of the flagged records into the flag list.
// eight consecutive flag bytes of one thread, as one 8-byte load where the tile is full
__device__ __forceinline__ u64 load_flags8(const uint8_t* __restrict__ f, u32 j0, u32 n) {
  if (j0 + 8 <= n && (reinterpret_cast<uintptr_t>(f + j0) & 7) == 0) return *reinterpret_cast<const u64*>(f + j0);
  u64 v = 0;
  for (u32 k = 0; k < 8; ++k) if (j0 + k < n) v |= (u64)f[j0 + k] << (8 * k);
  return v;
}
static_assert(SEL_TILE == 256 * 8, "one 8-byte piece of the flag bytes per thread");
__global__ __launch_bounds__(256) void k_flag_count(FlagArgs a) {
  __shared__ u32 s_wave[4];
  const u64 v = load_flags8(a.rec_flag, blockIdx.x * SEL_TILE + threadIdx.x * 8, a.n);
  u32 c = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) c += ((v >> (8 * k)) & 0xFF) != 0;
  u32 tot;
  block_exclusive_sum<256>(c, s_wave, &tot);
  if (threadIdx.x == 0) a.tile_flags[blockIdx.x] = tot;
}
__global__ __launch_bounds__(256) void k_flag_emit(FlagArgs a) {
  __shared__ u32 s_wave[4];
  const u32 j0 = blockIdx.x * SEL_TILE + threadIdx.x * 8;
  const int mb = a.sf.mb;
  const u64 mmask = ((u64)1 << mb) - 1, smask = ((u64)1 << a.sf.ws) - 1;
  const u64 v = load_flags8(a.rec_flag, j0, a.n);
  u32 c = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) c += ((v >> (8 * k)) & 0xFF) != 0;
  u32 tot;
  u32 k_out = a.tile_flags[blockIdx.x] + block_exclusive_sum<256>(c, s_wave, &tot);
  if (c == 0) return;
  for (u32 b = 0; b < 8; ++b) {
    const u32 f = (u32)(v >> (8 * b)) & 0xFF;
    if (!f) continue;
    const u32 j = j0 + b, k = k_out++;
    a.flag_pos[k] = j;
    if (a.flag && k < a.flag_cap) {
      const u64 key = a.key[j];
      const u32 comm = (u32)(key >> (mb + a.sf.ws));
      a.flag[(u64)CCLD_FLG_COMM * a.flag_cap + k] = (i64)comm;
      a.flag[(u64)CCLD_FLG_SEQ * a.flag_cap + k] = (i64)(((key >> mb) & smask) + a.sf.seq_base);
      a.flag[(u64)CCLD_FLG_RANK * a.flag_cap + k] =
          (i64)rank_of_slot(a.member_off, a.members_sorted, comm, (u32)(key & mmask));
      a.flag[(u64)CCLD_FLG_KIND * a.flag_cap + k] = (i64)f;
      a.flag[(u64)CCLD_FLG_LAG_ENTER * a.flag_cap + k] = a.flag_lag[j];
      a.flag[(u64)CCLD_FLG_LAG_EXIT * a.flag_cap + k] = a.flag_lag[a.cap_n + j];
    }
  }
}
void launch_flag_compact(hipStream_t st, const FlagArgs& a) {
  const u32 nt = (a.n + SEL_TILE - 1) / SEL_TILE;
  if (a.n) hipLaunchKernelGGL(k_flag_count, dim3(nt), dim3(256), 0, st, a);
  launch_scan_tiles(st, a.tile_flags, nt, &a.counters[CNT_NFLAG]);
  if (a.n) hipLaunchKernelGGL(k_flag_emit, dim3(nt), dim3(256), 0, st, a);
}

// ------------------------------------------------------------------------------------------
// One pass over the sorted keys for two results.
// (1) Collective heads per tile of SEG_TILE keys (a head = the first key of a (communicator,
//     operation counter) pair); equal neighbours are duplicates.
// (2) Records per rank.  The keys are sorted by communicator, so a workgroup's slice of them covers a
//     short run of communicators: it counts (communicator, member slot) pairs in an LDS table that
//     spans as many communicators as fit, then adds every non-zero cell to its rank's (zeroed) blame
//     column with one integer atomic.  A slice that covers more communicators takes several rounds.
constexpr u32 RC_CELLS = 8192;
constexpr u32 RC_MAX_TILES = 1024 + 8;      // tiles of one workgroup's slice (the launch keeps slices within 1024 tiles)
__global__ __launch_bounds__(256) void k_keys_pass(const u64* __restrict__ key, u32 n, SqueezedFormat sf,
                                                   const u32* __restrict__ member_off,
                                                   const u32* __restrict__ members_sorted,
                                                   const u32* __restrict__ comm_size, u32 n_ranks,
                                                   i64* __restrict__ blame, u32* __restrict__ tile_heads,
                                                   u64* __restrict__ counters) {
  __shared__ u32 s_h[RC_CELLS];
  __shared__ u32 s_tile[RC_MAX_TILES];
  __shared__ u32 s_end;
  const int mb = sf.mb, cshift = sf.mb + sf.ws;
  const u64 mmask = ((u64)1 << mb) - 1;
  const u32 slots = mb >= 13 ? RC_CELLS : (1u << mb);         // member slots covered by one round
  const u32 width = RC_CELLS / slots;                         // communicators covered by one round
  const u32 n_sub = mb >= 13 ? (1u << (mb - 13)) : 1u;        // rounds needed to cover every slot
  // slices of whole tiles
  const u64 per = (((u64)n + gridDim.x - 1) / gridDim.x + SEG_TILE - 1) / SEG_TILE * SEG_TILE;
  const u64 lo64 = per * blockIdx.x;
  if (lo64 >= n) return;
  const u32 lo = (u32)lo64, hi = (u32)((lo64 + per) < n ? (lo64 + per) : n);
  const u32 my_tiles = (hi - lo + SEG_TILE - 1) / SEG_TILE;
  for (u32 i = threadIdx.x; i < my_tiles; i += 256) s_tile[i] = 0;
  unsigned long long* out = (unsigned long long*)(blame + (u64)CCLD_BLM_N_RECORDS * n_ranks);
  bool dup = false;
  u32 pos = lo;
  while (pos < hi) {
    const u32 c0 = (u32)(key[pos] >> cshift);
    u32 end = hi;
    for (u32 sub = 0; sub < n_sub; ++sub) {
      const u32 s0 = sub * slots;
      for (u32 i = threadIdx.x; i < RC_CELLS; i += 256) s_h[i] = 0;
      if (threadIdx.x == 0) s_end = hi;
      __syncthreads();
      // eight keys per thread in flight; the keys are sorted, so the first one past the table's
      // communicators ends this thread's walk (that key is taken up by the next round)
      bool more = true;
      for (u32 j0 = pos + threadIdx.x; more && j0 < hi; j0 += 256 * 8) {
        u64 k[8], kp[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const u32 j = j0 + u * 256;
          k[u] = j < hi ? __builtin_nontemporal_load(key + j) : ~0ull;
        }
        // the key before each one sits in the lane below (a lane walks on no longer than the lanes
        // below it, so that lane is active); a wave's first lane reads it from memory
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const u32 j = j0 + u * 256;
          kp[u] = __shfl_up((unsigned long long)k[u], 1);
          if ((threadIdx.x & 63) == 0) kp[u] = (j < hi && j > 0) ? key[j - 1] : ~0ull;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const u32 j = j0 + u * 256;
          if (!more || j >= hi) continue;
          const u32 c = (u32)(k[u] >> cshift);
          if (c - c0 >= width) { atomicMin(&s_end, j); more = false; continue; }
          if (sub == 0) {
            if (j == 0 || (k[u] >> mb) != (kp[u] >> mb)) atomicAdd(&s_tile[(j - lo) / SEG_TILE], 1u);
            else dup |= (k[u] == kp[u]);
          }
          const u32 slot = (u32)(k[u] & mmask);
          if (slot - s0 < slots) atomicAdd(&s_h[(c - c0) * slots + (slot - s0)], 1u);
        }
      }
      __syncthreads();
      for (u32 i = threadIdx.x; i < RC_CELLS; i += 256) {
        const u32 v = s_h[i];
        if (!v) continue;
        const u32 c = c0 + i / slots, slot = s0 + i % slots;
        if (slot < comm_size[c]) atomicAdd(&out[members_sorted[member_off[c] + slot]], (unsigned long long)v);
      }
      end = s_end;
      __syncthreads();
    }
    pos = end;
  }
  for (u32 i = threadIdx.x; i < my_tiles; i += 256) tile_heads[lo / SEG_TILE + i] = s_tile[i];
  if (dup) atomic_or_u64(&counters[CNT_STATUS], DS_DUPLICATE);
}
void launch_keys_pass(hipStream_t st, const uint64_t* key, uint32_t n, const SqueezedFormat& sf,
                      const DeviceTopology& T, int64_t* blame, uint32_t* tile_heads, uint64_t* counters) {
  if (n == 0) return;
  uint32_t blocks = std::min<uint32_t>((n + 4095) / 4096, RANKCOUNT_BLOCKS);
  const uint32_t max_slice = (RC_MAX_TILES - 8) * (uint32_t)SEG_TILE;        // the per-tile counters of one slice fit in LDS
  blocks = std::max<uint32_t>(blocks, (uint32_t)(((uint64_t)n + max_slice - 1) / max_slice));
  hipLaunchKernelGGL(k_keys_pass, dim3(blocks), dim3(256), 0, st, key, n, sf, T.member_off, T.members_sorted,
                     T.size, T.n_ranks, blame, tile_heads, counters);
}

// Late columns of the blame table.  The flags are in (communicator, counter, rank) order, so a workgroup's slice of
// them names few ranks, each many times: it sums them in an LDS table keyed by rank (open addressing, a bounded number
// of probes) and adds every entry with one integer atomic per column; a rank that finds no entry goes straight to
// the blame table.  The integer sums do not depend on the order.  At 145,000 flags this takes the place of a sort by
// rank and three more launches (0.09 ms together).
constexpr u32 BH_SLOTS = 1024, BH_PROBES = 16, BH_NONE = 0xFFFFFFFFu, BH_BLOCKS = 128;
struct BlameSums {
  u32 rank[BH_SLOTS];
  unsigned long long sum[4][BH_SLOTS];
  __device__ __forceinline__ void clear() {
    for (u32 i = threadIdx.x; i < BH_SLOTS; i += blockDim.x) {
      rank[i] = BH_NONE;
#pragma unroll
      for (int k = 0; k < 4; ++k) sum[k][i] = 0;
    }
  }
  __device__ __forceinline__ void add(u32 r, u32 f, u64 le, u64 lx, i64* __restrict__ blame, u32 n_ranks) {
    u32 at = (r * 0x9E3779B1u) >> 22;                 // BH_SLOTS = 2^10
    bool found = false;
    for (u32 p = 0; p < BH_PROBES && !found; ++p) {
      const u32 was = atomicCAS(&rank[at], BH_NONE, r);
      found = was == BH_NONE || was == r;
      if (!found) at = (at + 1) & (BH_SLOTS - 1);
    }
    auto one = [&](int col, u64 v) {
      if (found) atomicAdd(&sum[col][at], (unsigned long long)v);
      else atomicAdd(reinterpret_cast<unsigned long long*>(&blame[(u64)col * n_ranks + r]), (unsigned long long)v);
    };
    if (f & CCLD_FLAG_LATE_ENTER) { one(CCLD_BLM_N_LATE_ENTER, 1); one(CCLD_BLM_SUM_LAG_ENTER, le); }
    if (f & CCLD_FLAG_LATE_EXIT) { one(CCLD_BLM_N_LATE_EXIT, 1); one(CCLD_BLM_SUM_LAG_EXIT, lx); }
  }
  __device__ __forceinline__ void flush(i64* __restrict__ blame, u32 n_ranks) {
    for (u32 i = threadIdx.x; i < BH_SLOTS; i += blockDim.x) {
      const u32 r = rank[i];
      if (r == BH_NONE) continue;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (sum[k][i]) atomicAdd(reinterpret_cast<unsigned long long*>(&blame[(u64)k * n_ranks + r]), sum[k][i]);
    }
  }
};
__global__ __launch_bounds__(256) void k_blame_sums(FlagArgs a, u32 n_ranks, i64* __restrict__ blame) {
  __shared__ BlameSums B;
  const u32 n_flag = (u32)a.counters[CNT_NFLAG], tid = threadIdx.x;
  const u32 per = ((n_flag + gridDim.x - 1) / gridDim.x + 255) / 256 * 256;
  const u64 lo = (u64)per * blockIdx.x;
  if (lo >= n_flag) return;
  const u32 hi = lo + per < n_flag ? (u32)(lo + per) : n_flag;
  B.clear();
  __syncthreads();
  const u64 mmask = ((u64)1 << a.sf.mb) - 1;
  for (u32 q = (u32)lo + tid; q < hi; q += 256) {
    const u32 j = a.flag_pos[q];
    const u64 key = a.key[j];
    const u32 r = rank_of_slot(a.member_off, a.members_sorted, (u32)(key >> (a.sf.mb + a.sf.ws)), (u32)(key & mmask));
    B.add(r, a.rec_flag[j], (u64)a.flag_lag[j], (u64)a.flag_lag[a.cap_n + j], blame, n_ranks);
  }
  __syncthreads();
  B.flush(blame, n_ranks);
}
static_assert(BH_SLOTS == 1024, "ten hash bits");
static_assert(CCLD_BLM_N_LATE_ENTER == 0 && CCLD_BLM_N_LATE_EXIT == 1 && CCLD_BLM_SUM_LAG_ENTER == 2 &&
              CCLD_BLM_SUM_LAG_EXIT == 3, "blame column order");
void launch_blame_sums(hipStream_t st, const FlagArgs& f, uint32_t n_ranks, int64_t* blame) {
  if (f.n) hipLaunchKernelGGL(k_blame_sums, dim3(std::min<u32>((f.n + 4095) / 4096, BH_BLOCKS)), dim3(256), 0, st, f, n_ranks, blame);
}

// The blame order of very many ranks (END_ORDER_RANKS and fewer: k_window_lists).
struct PredBlamed {
  const i64 *ne, *nx;
  bool want;
  __device__ bool operator()(u32 r) const { return ((ne[r] + nx[r]) != 0) == want; }
};
__global__ __launch_bounds__(256) void k_blame_order(const i64* __restrict__ blame, u32 n_ranks,
                                                     const u32* __restrict__ lists, u64* counters, u32* arrivals,
                                                     u32* __restrict__ order, u64* host, u64 ticket) {
  const u32 nb = (u32)counters[CNT_NBLAMED];
  const u32 lane = lane_id();
  for (u32 q = blockIdx.x * 4 + threadIdx.x / CCLD_WAVE; q < nb; q += gridDim.x * 4) {
    const u32 r = lists[q];
    const u32 before = blamed_before(blame, n_ranks, lists, nb, r, lane);
    if (lane == 0) order[before] = r;
  }
  const u32 stride = gridDim.x * 256;
  for (u32 i = blockIdx.x * 256 + threadIdx.x; i < n_ranks - nb; i += stride) order[nb + i] = lists[n_ranks + i];
  report_counters(counters, arrivals, host, ticket);
}
void launch_blame_order(hipStream_t st, const int64_t* blame, uint32_t n_ranks, uint32_t* lists,
                        uint32_t* tile_counts, uint64_t* counters, uint32_t* arrivals, uint32_t* order, uint64_t* host_counters,
                        uint64_t ticket) {
  PredBlamed p{blame + (u64)CCLD_BLM_N_LATE_ENTER * n_ranks, blame + (u64)CCLD_BLM_N_LATE_EXIT * n_ranks, true};
  run_select(st, p, n_ranks, tile_counts, lists, &counters[CNT_NBLAMED]);
  p.want = false;
  run_select(st, p, n_ranks, tile_counts, lists + n_ranks, &counters[CNT_NCLEAN]);
  const u32 blocks = std::min<u32>((n_ranks + 3) / 4, 512);
  hipLaunchKernelGGL(k_blame_order, dim3(blocks), dim3(256), 0, st, blame, n_ranks, (const u32*)lists, counters, arrivals, order,
                     host_counters, ticket);
}

// The end of a pass whose last kernel does not report: every launch before it is over.
__global__ __launch_bounds__(CCLD_WAVE) void k_report(const u64* counters, u64* host, u64 ticket) { report_words(counters, host, ticket); }
void launch_report(hipStream_t st, const uint64_t* counters, uint64_t* host, uint64_t ticket) {
  hipLaunchKernelGGL(k_report, dim3(1), dim3(CCLD_WAVE), 0, st, counters, host, ticket);
}

// The blame table and its order handed to the caller: the last workgroup to finish reports, so what it hands over is stored
// past the caches.  (With a report in a launch of its own a call took 11.5 in place of 9.8 us at 512 ranks, 11.7 in place of
// 10.8 at 16,384.)
__global__ __launch_bounds__(1024) void k_blame_out(const i64* __restrict__ blame, const u32* __restrict__ order_in, u32 n_ranks,
                                                    i64* __restrict__ table_out, u32* __restrict__ order_out, u64* counters,
                                                    u32* arrivals, u64* host, u64 ticket) {
  const u64 nt = (u64)CCLD_BLM_NCOL * n_ranks, stride = (u64)gridDim.x * 1024;
  for (u64 i = (u64)blockIdx.x * 1024 + threadIdx.x; i < nt; i += stride) {
    if (table_out) store_agent(&table_out[i], blame[i]);
    if (order_out && i < n_ranks) store_agent(&order_out[i], order_in[i]);
  }
  report_counters(counters, arrivals, host, ticket);
}
void launch_blame_out(hipStream_t st, const int64_t* blame, const uint32_t* order_in, uint32_t n_ranks, int64_t* table_out,
                      uint32_t* order_out, uint64_t* counters, uint32_t* arrivals, uint64_t* host, uint64_t ticket) {
  const u64 nt = (u64)CCLD_BLM_NCOL * n_ranks;
  const u32 blocks = (u32)std::min<u64>((nt + 1023) / 1024, 256);
  hipLaunchKernelGGL(k_blame_out, dim3(blocks), dim3(1024), 0, st, blame, order_in, n_ranks, table_out, order_out, counters, arrivals, host, ticket);
}

// ------------------------------------------------------------------------------------------
// Hang alerts: a collective with an operation in flight longer than the threshold, barriers
// excepted; class by the first two questions of the hang decision tree.
struct PredAlert {
  const i64 *inflight, *state, *imin;
  i64 now, thr;
  __device__ bool operator()(u32 s) const {
    return inflight[s] > 0 && !(state[s] & CCLD_SEG_BARRIER) && now - imin[s] > thr;
  }
};
void launch_alert_select(hipStream_t st, const AlertArgs& a) {
  PredAlert p{a.seg + (u64)CCLD_SEG_INFLIGHT * a.seg_cap, a.seg + (u64)CCLD_SEG_STATE * a.seg_cap,
              a.seg + (u64)CCLD_SEG_INFLIGHT_ENTER_MIN * a.seg_cap, a.now_ns, a.hang_threshold_ns};
  run_select(st, p, a.n_seg, a.tile_counts, a.alert_list, &a.counters[CNT_NALERT]);
}

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
// candidates of one alert, in ascending rank order; EMIT = false only counts them
template <bool EMIT, bool GRID>
__global__ __launch_bounds__(256) void k_alert_cand(AlertArgs a, u32 n_alert) {
  __shared__ u32 s_wave[4];
  const u32 al = blockIdx.x, tid = threadIdx.x;
  const u32 s = a.alert_list[al];
  const u64 C = a.seg_cap;
  const u32 comm = (u32)a.seg[CCLD_SEG_COMM * C + s];
  const u32 nn = (u32)a.seg[CCLD_SEG_N * C + s], ninfl = (u32)a.seg[CCLD_SEG_INFLIGHT * C + s];
  const u32 first = (u32)a.seg[CCLD_SEG_FIRST * C + s];
  const u32 size = a.topo.size[comm], moff = a.topo.member_off[comm];
  const u32 off = EMIT ? a.alert_ncand[al] : 0u;
  const int cls = alert_class(nn, ninfl, size);
  u32 total = 0;
  if (cls != CCLD_HANG_H3_HARDWARE) {
    for (u32 q0 = 0; q0 < size; q0 += 256) {
      const u32 q = q0 + tid;
      bool hit = false;
      u32 r = 0;
      if (q < size) {
        r = a.topo.members_sorted[moff + q];
        i64 tx = T_INFLIGHT;
        const bool here = alert_record<GRID>(a, s, comm, first, nn, q, &tx);
        hit = cls == CCLD_HANG_H1_NOT_ENTERED ? !here : (here && tx != T_INFLIGHT);
      }
      u32 tot;
      const u32 ex = block_exclusive_sum<256>(hit ? 1u : 0u, s_wave, &tot);
      if (EMIT && hit && (u64)off + total + ex < a.cand_cap) a.cand[off + total + ex] = (i64)r;
      total += tot;
    }
  }
  if (tid != 0) return;
  if (!EMIT) { a.alert_ncand[al] = total; return; }
  if (al < a.alert_cap) {
    const u64 A = a.alert_cap;
    a.alert[CCLD_ALR_COMM * A + al] = comm;
    a.alert[CCLD_ALR_SEQ * A + al] = a.seg[CCLD_SEG_SEQ * C + s];
    a.alert[CCLD_ALR_AGE * A + al] = a.now_ns - a.seg[CCLD_SEG_INFLIGHT_ENTER_MIN * C + s];
    a.alert[CCLD_ALR_CLASS * A + al] = cls;
    a.alert[CCLD_ALR_NCAND * A + al] = total;
    a.alert[CCLD_ALR_CAND_OFF * A + al] = off;
  }
}
void launch_alert_candidates(hipStream_t st, const AlertArgs& a, uint32_t n_alert) {
  if (n_alert == 0) return;
  const bool grid = a.grid.lay != nullptr;
  if (grid) hipLaunchKernelGGL((k_alert_cand<false, true>), dim3(n_alert), dim3(256), 0, st, a, n_alert);
  else hipLaunchKernelGGL((k_alert_cand<false, false>), dim3(n_alert), dim3(256), 0, st, a, n_alert);
  launch_scan_tiles(st, a.alert_ncand, n_alert, &a.counters[CNT_NCAND]);
  if (grid) hipLaunchKernelGGL((k_alert_cand<true, true>), dim3(n_alert), dim3(256), 0, st, a, n_alert);
  else hipLaunchKernelGGL((k_alert_cand<true, false>), dim3(n_alert), dim3(256), 0, st, a, n_alert);
}

// ------------------------------------------------------------------------------------------
// position of every sorted record in the window's arrival order
__global__ __launch_bounds__(256) void k_perm(const u32* __restrict__ idx, WindowRows win, u32 n, u32* perm) {
  const u32 j = blockIdx.x * 256 + threadIdx.x;
  if (j < n) perm[j] = arrival_of_slot(win, idx[j]);
}
void launch_perm(hipStream_t st, const uint32_t* idx, const WindowRows& win, uint32_t n, uint32_t* perm) {
  if (n) hipLaunchKernelGGL(k_perm, dim3((n + 255) / 256), dim3(256), 0, st, idx, win, n, perm);
}

}  // namespace ccld
