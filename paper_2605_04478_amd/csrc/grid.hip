// Grid placement for gfx950: the layout of the (communicator, operation counter, member slot) grid from the
// window's counter ranges, and the partition pass that moves every payload row into the fine bucket of its cell.
#include <algorithm>
#include <type_traits>

#include "grid.h"
#include "rows.h"

namespace ccld {

// A division by n as a multiplication: x * 2^s / d = x / n for x < 2^31, with the smallest 2^s >= n and 2^(31 + s) / n rounded up
// (below 2^32; its error of less than one adds less than 1 / n to the quotient).  The doubles round up as they should: the
// quotient is whole or at least 1 / n away from a whole number.
__device__ __forceinline__ void divide_by(u32 n, u32* div, u32* shift) {
  *shift = n > 1 ? 32 - (u32)__clz((int)(n - 1)) : 0u;
  *div = (u32)ceil(ldexp(1.0, 31 + (int)*shift) / (double)n);
}
// ---- layout ------------------------------------------------------------------------------------------
// One workgroup: data errors of the batches; per communicator the rounds in the window, its fine buckets, cells and rows
// of the collective table (exclusive scans over the communicators); the pieces of the window that hold each coarse
// bucket.  The layout is infeasible (the host then sorts) when the grid has more cells or rounds than the buffers and
// the records allow (counters that are far apart), when a coarse bucket spans more fine buckets than a partition
// workgroup addresses, or when the batches lie so far apart that no single time serves all rows.
// Bound by its few dependent loads and, with many batches, by one workgroup reading all their ranges: 4 to 5 us at up to
// 1,024 communicators and one batch, 12 at 3,200, and 18.5 with ten batches (31 with fewer loads on their way).
// PER: most communicators of a thread; AHEAD: batches whose ranges are on their way at a time.
template <u32 PER, u32 AHEAD>
__global__ __launch_bounds__(1024) void k_grid_layout(GridArgs d) {
  __shared__ u32 s_wave[1024 / CCLD_WAVE];
  __shared__ uint4 s_sums[CCLD_WAVE];
  __shared__ u32 s_bad, s_any, s_empty;
  __shared__ unsigned long long s_status;
  __shared__ i64 s_ref;
  const u32 tid = threadIdx.x;
  if (tid == 0) { s_bad = 0; s_status = 0; s_any = 0xFFFFFFFFu; s_empty = 0; }
  if (tid < CNT_COUNT) d.counters[tid] = 0;
  // the headers of the batches (those of the first 1,024 stay in registers), the pieces and the counter ranges are on their way together
  auto meta_of = [&](u32 i) -> const BatchMeta& { return d.meta[(d.slot0 + i) % d.n_meta]; };
  u64 m_status = 0, m_n = 0;
  i64 m_ref = 0;
  if (tid < d.nb) { const BatchMeta& m = meta_of(tid); m_status = m.status; m_n = m.n; m_ref = m.ref; }
  // piece k: its records and its first window slot
  const u32 n_stretches = d.n_buckets == 1 ? 0u : d.n_buckets * d.nb;
  auto piece = [&](u32 k, u32* slot) -> u32 {
    if (k >= n_stretches) return 0;
    const u32 b = k / d.nb, i = k % d.nb, m = (d.slot0 + i) % d.n_meta;
    const u32* bb = d.bucket_base + (u64)m * (d.n_buckets + 1);
    const u32 from = bb[b], to = bb[b + 1];
    const u64 p = d.meta[m].tail + from;
    *slot = (u32)(p >= d.cap ? p - d.cap : p);
    return d.meta[m].n ? to - from : 0u;
  };
  u32 slot0 = 0;
  const u32 cnt0 = piece(tid, &slot0);
  bool bad = false;
  // thread t has the communicators t, 1,024 + t, ..., so that neighbouring lanes read neighbouring ranges (with consecutive ones per
  // thread every line went to the compute unit four times at 3,200 communicators)
  constexpr u32 WAVES = 1024 / CCLD_WAVE;
  static_assert(PER * WAVES <= CCLD_WAVE, "a lane per wavefront's sums");
  u64 mx[PER], inv[PER];
  u32 size[PER];
#pragma unroll
  for (u32 k = 0; k < PER; ++k) {
    mx[k] = 0; inv[k] = 0; size[k] = 0;
    if (k * 1024 + tid < d.n_comms) size[k] = d.comm_size[k * 1024 + tid];
  }
  for (u32 i0 = 0, m = d.slot0; i0 < d.nb; i0 += AHEAD) {
    ulonglong2 r[AHEAD][PER];           // none of the loads is conditional: the compiler would wait for each
#pragma unroll
    for (u32 u = 0; u < AHEAD; ++u) {
      const ulonglong2* __restrict__ row = reinterpret_cast<const ulonglong2*>(d.range) + (u64)m * d.n_comms;
#pragma unroll
      for (u32 k = 0; k < PER; ++k) r[u][k] = row[std::min(k * 1024 + tid, d.n_comms - 1)];
      m = i0 + u + 1 < d.nb ? (m + 1 == d.n_meta ? 0 : m + 1) : m;
    }
#pragma unroll
    for (u32 u = 0; u < AHEAD; ++u)
#pragma unroll
      for (u32 k = 0; k < PER; ++k) { mx[k] = r[u][k].x > mx[k] ? r[u][k].x : mx[k]; inv[k] = r[u][k].y > inv[k] ? r[u][k].y : inv[k]; }
  }
#pragma unroll
  for (u32 k = 0; k < PER; ++k)
    if (k * 1024 + tid >= d.n_comms) { mx[k] = 0; inv[k] = 0; }
  __syncthreads();
  if (m_status) atomicOr(&s_status, (unsigned long long)m_status);
  if (m_n) atomicMin(&s_any, tid);
  for (u32 i = tid + 1024; i < d.nb; i += 1024) {
    const BatchMeta& b = meta_of(i);
    if (b.status) atomicOr(&s_status, (unsigned long long)b.status);
    if (b.n) atomicMin(&s_any, i);
  }
  // the sum of the cells can pass 32 bits, so it is taken in halves (where it does, the layout is refused, and where it
  // does not, the sums of buckets and rounds do not either)
  const bool lines = d.lines != 0;
  u32 rounds[PER], empty = 0;
  uint4 before[PER];                    // fine buckets, rounds, cells (low and high half) before the communicator
  const u32 lane = lane_id(), wave = tid / CCLD_WAVE;
  auto sums = [](const uint4& v) { return make_uint4(wave_inclusive_sum(v.x), wave_inclusive_sum(v.y), wave_inclusive_sum(v.z), wave_inclusive_sum(v.w)); };
  auto less = [](const uint4& a, const uint4& b) { return make_uint4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w); };
  auto from = [](const uint4& v, u32 l) { return make_uint4(__shfl(v.x, l, CCLD_WAVE), __shfl(v.y, l, CCLD_WAVE), __shfl(v.z, l, CCLD_WAVE), __shfl(v.w, l, CCLD_WAVE)); };
#pragma unroll
  for (u32 k = 0; k < PER; ++k) {
    rounds[k] = 0;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (mx[k] | inv[k]) {
      const u64 r = mx[k] - ~inv[k] + 1;                 // largest >= smallest; r == 0 only for the full 64-bit range
      if (r == 0 || r > 0x7FFFFFFFull || r * size[k] > (u64)d.cell_cap) {
        bad = true;
      } else {
        rounds[k] = (u32)r;
        const u32 rpb = bucket_rounds(size[k], lines);   // size <= GRID_B: the host checked
        const u64 cells = grid_cells(size[k], rounds[k], lines);
        empty += (u32)(cells - r * size[k]);
        v = make_uint4((rounds[k] + rpb - 1) / rpb, rounds[k], (u32)cells & 0xFFFFu, (u32)(cells >> 16));
      }
    }
    const uint4 inc = sums(v);
    if (lane == CCLD_WAVE - 1) s_sums[k * WAVES + wave] = inc;
    before[k] = less(inc, v);
  }
  if (lines) { empty = wave_sum(empty); if (lane == 0 && empty) atomicAdd(&s_empty, empty); }
  __syncthreads();
  const uint4 part = lane < PER * WAVES ? s_sums[lane] : make_uint4(0, 0, 0, 0), upto = sums(part), total = from(upto, CCLD_WAVE - 1);
  const uint4 ahead = less(upto, part);
  // one time serves the whole window, that of its first batch with records, unless its batches lie too far apart
  const u32 any = s_any;
  if (tid == (any < 1024 ? any : 0u)) s_ref = any < 1024 ? m_ref : meta_of(any < d.nb ? any : 0).ref;
  const u64 cell_total = (u64)total.z + ((u64)total.w << 16), cell_used = cell_total - s_empty;
  const u32 fb_total = total.x, seg_total = total.y;
#pragma unroll
  for (u32 k = 0; k < PER; ++k) {
    const uint4 w = from(ahead, k * WAVES + wave);
    const u32 c = k * 1024 + tid;
    if (c >= d.n_comms) continue;
    CommLayout L;
    L.seq_min = (mx[k] | inv[k]) ? ~inv[k] : 0; L.rpb = bucket_rounds(size[k], lines); L.rounds = rounds[k]; L.size = size[k];
    L.fb_base = w.x + before[k].x; L.seg_base = w.y + before[k].y;
    L.cell_base = (u32)((u64)w.z + before[k].z + ((u64)(w.w + before[k].w) << 16));
    divide_by(L.rpb, &L.div, &L.shift);
    d.lay[c] = L;
  }
  // more rounds than records means a round without any record: the sort handles such windows
  if (cell_used > d.cell_cap || fb_total > d.fine_cap || seg_total > d.n) bad = true;        // uniform
  const u64 fb_carry = fb_total, seg_carry = seg_total, cell_carry = cell_total;
  if (tid == 0) {
    CommLayout L;
    L.seq_min = 0; L.fb_base = (u32)(fb_carry > d.fine_cap ? d.fine_cap : fb_carry); L.rpb = 1; L.rounds = 0;
    L.seg_base = (u32)seg_carry; L.cell_base = (u32)cell_carry; L.size = 1; L.div = 0; L.shift = 0;
    d.lay[d.n_comms] = L;
  }
  if (d.n_buckets == 1 && fb_total > GRID_SPAN) bad = true;
  if (bad) atomicOr(&s_bad, 1u);
  __threadfence_block();
  __syncthreads();
  const i64 ref = s_ref;
  auto far = [&](i64 t) { return (((u64)t - (u64)ref + ((u64)1 << 42)) >> 43) != 0; };
  bool apart = m_n && far(m_ref);
  for (u32 i = tid + 1024; i < d.nb; i += 1024) { const BatchMeta& b = meta_of(i); apart |= b.n && far(b.ref); }
  if (apart) atomicOr(&s_bad, 1u);
  if (d.n_buckets > 1) {
    bool wide = false;
    for (u32 b = tid; b < d.n_buckets; b += 1024) {
      u64 c0 = (u64)b << d.bshift, c1 = (u64)(b + 1) << d.bshift;
      if (c0 > d.n_comms) c0 = d.n_comms;
      if (c1 > d.n_comms) c1 = d.n_comms;
      if (d.lay[c1].fb_base - d.lay[c0].fb_base > GRID_SPAN) wide = true;
    }
    if (wide) atomicOr(&s_bad, 1u);
  }
  __syncthreads();
  const bool ok = s_bad == 0 && s_status == 0;
  const u32 n_fine = ok ? (u32)fb_carry : 0u;
  // pieces: a window placed without buckets is one contiguous stretch of slots; otherwise every batch holds its own
  // stretch of every bucket
  u32 n_pieces = 1;
  if (d.n_buckets == 1) {
    if (tid == 0) { d.piece_at[0] = 0; d.piece_at[1] = d.n; d.piece_slot[0] = d.head; }
  } else {
    n_pieces = n_stretches;
    u32 carry = 0;
    for (u32 base = 0; base < n_pieces; base += 1024) {
      const u32 k = base + tid;
      u32 slot = slot0;
      const u32 cnt = base ? piece(k, &slot) : cnt0;
      u32 tot;
      const u32 ex = block_exclusive_sum<1024>(cnt, s_wave, &tot);
      if (k < n_pieces) { d.piece_at[k] = carry + ex; d.piece_slot[k] = slot; }
      carry += tot;
    }
    if (tid == 0) d.piece_at[n_pieces] = carry;
  }
  for (u32 f = tid; f <= n_fine; f += 1024) d.fill[f] = 0;
  if (tid == 0) {
    GridHeader h;
    h.feasible = ok ? 1u : 0u; h.n_fine = n_fine; h.n_seg = ok ? (u32)seg_carry : 0u; h.n_pieces = n_pieces; h.ref = ref;
    h.n_long = 0; h.done = 0;
    *d.hdr = h;
    if (s_status) d.counters[CNT_STATUS] = s_status;
    else if (!ok) d.counters[CNT_STATUS] = DS_DENSE_FALLBACK;
    d.counters[CNT_NSEG] = ok ? seg_carry : 0;
    __hip_atomic_store(d.host_fine, ok ? (n_fine + 1) | (cell_used == d.n ? GRID_FULL : 0u) : GRID_INFEASIBLE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

void launch_grid_layout(hipStream_t st, const GridArgs& d) {
  // One communicator per thread where there are no more than threads, and no loads ahead of a single batch: with the general form
  // a window of one batch takes 7.3 us in place of 4.7 at 512 ranks, ten batches of that job 9.3 in place of 4.9.  Two, five or ten
  // batches ahead: 3,200 communicators with four batches 11.2, 11.3 and 13.6, with ten 19.3, 18.4 and 18.6, with 16 24.7, 25.6 and 26.1.
  constexpr u32 MANY = (GRID_MAX_COMMS + 1023) / 1024;
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(1), dim3(1024), 0, st, d); };
  if (d.n_comms <= 1024) { if (d.nb > 1) go(k_grid_layout<1, 5>); else go(k_grid_layout<1, 1>); }
  else { if (d.nb > 1) go(k_grid_layout<MANY, 5>); else go(k_grid_layout<MANY, 1>); }
}

// ---- partition --------------------------------------------------------------------------------------
// A workgroup takes one slice of the window, bucket by bucket: a few thousand records per round, each counted into its fine
// bucket in LDS; rooms in the fine buckets are reserved, the rows are staged in LDS in (bucket, rank) order and leave with
// consecutive lanes on consecutive 16-byte pieces.  A fine bucket takes as many rows as it has cells; more can only be duplicate keys.
//
// Runs: a round's share of every fine bucket is reserved with one atomic and leaves as it is.  Pieces of a line that the round
// writes completely leave with the streaming hint, which keeps them from displacing the partially written lines at the
// buckets' frontiers from the L2.  Bound by memory and by the instructions and LDS traffic of a round, between which there are
// barriers: the fields of a key are 32-bit words, the division is a multiplication, the next round's keys are asked for behind the
// reservations (operations of vector memory are waited for in the order of their issue) and its rows when this round's are staged:
// 20.5M records 205 -> 164 us (4.9 TB/s, buckets of half the communicators included), 5.1M 55.7 -> 52.1, 2M-record batches of
// 16,384 ranks, ten in the window, 215 -> 185.
//
// Lines (part_lines): the largest windows have more lines on their way than the caches hold, and what a round left of one unwritten
// leaves in parts before the next completes it.  There rooms are reserved eight rows at a time from the fine bucket's start, up to
// seven rows of a fine bucket wait in registers for the next round, and what is left when the workgroup's share of the coarse
// bucket ends goes to the fine bucket's end: 82M records 959 us before, 842 as runs, 703 so (4.7 TB/s).  The layout starts fine
// buckets on lines there (bucket_rounds), since eight rows that lie across two lines are two parts of lines: communicators of 6, 8 and 64
// members, 60M / 100M records 530 / 1,042 us as runs, 613 / 1,277 as rows in eights anywhere, 532 / 962 so; of 3, 9 and 13 members 497 /
// 976, 622 / 1,320, 507 / 905.  (Coarse buckets with a communicator that has too few rounds in a fine bucket for that leave as runs.)
//
// One workgroup per compute unit.  Workgroups go to the eight XCDs in turn and every XCD has an L2 of its own: those of one XCD
// take neighbouring slices, so that the lines that several workgroups write are completed in one L2.
constexpr u32 PART_THREADS = 1024, PART_U = 4, PART_CHUNK = PART_THREADS * PART_U;
constexpr u32 PART_BLOCKS = 256, PART_XCDS = 8;
constexpr u32 PART_LAY = 256;          // communicators of a bucket whose layout waits in LDS
constexpr u32 LINES_U = 3, LINES_CHUNK = PART_THREADS * LINES_U;
constexpr u32 LINES_SPAN = 384;        // most fine buckets of a coarse bucket whose rows leave in whole lines
constexpr u32 LINES_STAGE = LINES_CHUNK + 2 * (LINE_ROWS - 1) * LINES_SPAN;     // and rows that waited, and lines that are not filled
constexpr u32 LINES_MIN = 16 * LINES_CHUNK;      // fewest records of a workgroup in such a bucket: its rows that wait at the end are few beside them
constexpr u32 LINES_SLICE = 64 * LINES_CHUNK;    // fewest records of a workgroup in such a window
static_assert(LINES_SPAN <= PART_THREADS, "a thread per fine bucket");
static_assert(GRID_B == 2048 && (u64)LINES_SPAN * GRID_B < 1u << 21, "a bucket's first cell and cells in a word");

// The pieces of a coarse bucket, walked from front to back: the piece that held the first record of the last round asked for.
struct PartCursor {
  const u32 *at, *slot0;               // records of the window before each piece, its first slot
  u32 piece, first, last, slot;
  __device__ __forceinline__ PartCursor(const u32* at_, const u32* slot0_) : at(at_), slot0(slot0_), piece(0) { load(); }
  __device__ __forceinline__ void load() { first = scalar(at[piece]); last = scalar(at[piece + 1]); slot = scalar(slot0[piece]); }
  static __device__ __forceinline__ u32 scalar(u32 v) { return (u32)__builtin_amdgcn_readfirstlane((int)v); }
};
// slots and keys of a round, its rows: asked for without conditions, since the compiler waits for what is issued before
// conditional loads with them
template <u32 U>
__device__ __forceinline__ void part_keys(const GridArgs& d, PartCursor& C, u32 base, u32 end, u32 (&src)[U], u64 (&key)[U]) {
  base = std::min(base, end - 1);
  while (base >= C.last) { ++C.piece; C.load(); }    // base < end <= the last entry of the table
  if (std::min(base + U * PART_THREADS, end) <= C.last) {            // one piece holds the round
#pragma unroll
    for (u32 u = 0; u < U; ++u) src[u] = C.slot + (std::min(base + u * PART_THREADS + threadIdx.x, end - 1) - C.first);
  } else {
    u32 k = C.piece;
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      const u32 j = std::min(base + u * PART_THREADS + threadIdx.x, end - 1);
      while (j >= C.at[k + 1]) ++k;
      src[u] = C.slot0[k] + (j - C.at[k]);
    }
  }
#pragma unroll
  for (u32 u = 0; u < U; ++u) { src[u] = src[u] >= d.cap ? src[u] - d.cap : src[u]; key[u] = __builtin_nontemporal_load(d.win_key + src[u]); }
}
typedef u32 u32x4 __attribute__((ext_vector_type(4)));
template <u32 U>
__device__ __forceinline__ void part_rows(const GridArgs& d, const u32 (&src)[U], uint4 (&row)[U]) {
#pragma unroll
  for (u32 u = 0; u < U; ++u) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(d.win_row + src[u]));
    row[u] = make_uint4(v.x, v.y, v.z, v.w);
  }
}
// The fields of a key in 32-bit words: a round's number inside the window has fewer bits.
struct PartKey {
  u32 comm_shift, comm_mask, mb, seq_mask, slot_mask;
  __device__ __forceinline__ PartKey(const KeyFormat& kf) {
    comm_shift = kf.cb ? 32 - kf.cb : 0; comm_mask = kf.cb ? ~0u : 0u; mb = kf.mb;
    seq_mask = kf.sb >= 32 ? ~0u : (1u << kf.sb) - 1;
    slot_mask = (1u << kf.mb) - 1;
  }
  __device__ __forceinline__ u32 comm(u64 k) const { return (u32)(k >> 32) >> comm_shift & comm_mask; }
  __device__ __forceinline__ u32 seq(u64 k) const { return (u32)(k >> mb) & seq_mask; }
  __device__ __forceinline__ u32 slot(u64 k) const { return (u32)k & slot_mask; }
};
static_assert(GRID_MAX_COMMS <= 1u << 16 && GRID_B <= 1u << 16, "communicator and slot fields of fewer than 32 bits");
// A communicator of a coarse bucket: the smallest counter's low word, its first fine bucket relative to the coarse bucket's, rounds
// per fine bucket | members << 12 | shift << 24, and the multiplier that divides by the rounds per fine bucket.
struct PartComm {
  u32 seq, fb, rss, div;
  __device__ __forceinline__ PartComm() = default;
  __device__ __forceinline__ PartComm(const CommLayout& L, u32 f_lo)
      : seq((u32)L.seq_min), fb(L.fb_base - f_lo), rss(L.rpb | (L.size << 12) | (L.shift << 24)), div(L.div) {}
  __device__ __forceinline__ u32 rpb() const { return rss & 0xFFFu; }
  __device__ __forceinline__ u32 size() const { return (rss >> 12) & 0xFFFu; }
  __device__ __forceinline__ u32 bucket(u32 rel) const { return __umulhi(rel << 1, div) >> (rss >> 24); }
};
__device__ __forceinline__ uint4 part_row(const uint4& row, u32 cell) {
  return make_uint4(row.x, (row.y & ~(ROW_CELL_MASK << ROW_CELL_SHIFT)) | (cell << ROW_CELL_SHIFT), row.z, row.w);
}

// The thread's number, not known to be the same every time: what follows from it is worked out again in every round.  Kept over the
// rounds, a thread's places and addresses take thirty registers, and a kernel that spills needs scratch memory (1 us more to start;
// part_lines still spills eleven, around its loop).
__device__ __forceinline__ u32 thread_here() { u32 t = threadIdx.x; asm("" : "+v"(t)); return t; }

struct PartLines {
  u32x4 row[LINES_STAGE];              // a round's rows by fine bucket, each bucket's from a whole line on
  uint2 place[2][LINES_SPAN];          // of each fine bucket: place of its first new row; first place that stays | rows that stay << 16
  uint2 leave[2][LINES_SPAN];          // what turns a place into a destination; first place that does not leave
  u32 cnt[LINES_SPAN];                 // rows of the next round
  u32 fine[LINES_SPAN];                // first cell relative to the coarse bucket's << 11 | cells - 1
  uint16_t line[LINES_STAGE / LINE_ROWS];      // fine bucket of every line
};
// The records [pos, end) of a coarse bucket of `span` fine buckets from f_lo on, whose n_lay communicators (from c0 on) are in s_lay
// and s_base (first cell, rounds).  Ends with a barrier.
//
// Vector memory operations are waited for in the order of their issue, so a round asks for its rooms first, then for rows two
// rounds ahead, and stores last; the stores are as many in every round (those of places without a row lie outside the
// buffer and are dropped), so that the wait for rows does not become one for everything.
__device__ __forceinline__ void part_lines(const GridArgs& d, PartLines& S, const PartComm* s_lay, const uint2* s_base, u32 c0, u32 n_lay, const PartKey& pk,
                                           const u32* s_at, const u32* s_slot0, u32* s_wave, u32 pos, u32 end, u32 f_lo, u32 span, u64& status) {
  constexpr u32 HELD = LINES_SPAN * LINE_ROWS / PART_THREADS, OUT = (LINES_STAGE + PART_THREADS - 1) / PART_THREADS, OUT_MOST = 6;
  static_assert(LINES_SPAN * LINE_ROWS % PART_THREADS == 0, "rows that wait: as many places in every thread");
  const u32 tid = threadIdx.x;
  const u32 cell_lo = s_base[0].x;
  uint4 row0[LINES_U], row1[LINES_U];
  u64 key0[LINES_U], key1[LINES_U];
  u32 src0[LINES_U], src1[LINES_U];
  // round r: rows in set r % 2; the keys of the round behind it in the other set; slots of a round where its keys were
  PartCursor C(s_at, s_slot0);
  part_keys(d, C, pos, end, src0, key0);
  part_rows(d, src0, row0);
  part_keys(d, C, pos + LINES_CHUNK, end, src1, key1);
  part_rows(d, src1, row1);
  u32 left = 0;                        // rows of the thread's fine bucket that wait
  if (tid < span) {
    u32 lo = 0, hi = n_lay;
    while (lo < hi) { const u32 m = (lo + hi) >> 1; if (s_lay[m].fb <= tid) lo = m + 1; else hi = m; }
    const PartComm L = s_lay[lo - 1];
    const uint2 B = s_base[lo - 1];
    const u32 r0 = (tid - L.fb) * L.rpb(), k = B.y - r0;
    S.fine[tid] = (B.x + r0 * L.size() - cell_lo) << 11 | ((k < L.rpb() ? k : L.rpb()) * L.size() - 1);
    S.cnt[tid] = 0;
  }
  __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(d.rows + cell_lo, 0, (int)(span * GRID_B * 16), 0x00027000);
  u32 total = 0, held = 0;
  u32x4 h_row[HELD];
  u32 h_at[HELD];                      // place relative to the bucket's first new row
  u32 fi_cell[LINES_U], at[LINES_U];
  auto count = [&](u32 base, const u64 (&key)[LINES_U]) {
#pragma unroll
    for (u32 u = 0; u < LINES_U; ++u) {
      fi_cell[u] = ~0u;
      if (base + u * PART_THREADS + tid >= end) continue;
      const PartComm L = s_lay[pk.comm(key[u]) - c0];
      const u32 rel = pk.seq(key[u]) - L.seq, fr = L.bucket(rel), fi = L.fb + fr;
      if (fi >= span) continue;
      fi_cell[u] = fi | (__umul24(rel - __umul24(fr, L.rpb()), L.size()) + pk.slot(key[u])) << 16;
      at[u] = atomicAdd(&S.cnt[fi], 1u);
    }
  };
  // rooms for the lines that the counted rows make up, and their places
  u32 t = 0, got = 0;                  // rows of the thread's bucket, and those of others that have a room
  auto ask = [&] {
    const u32 tid = thread_here();
    t = left + (tid < span ? S.cnt[tid] : 0u);
    const u32 out = t & ~(LINE_ROWS - 1);
    if (out) got = atomicAdd(&d.fill[f_lo + tid], out);
  };
  auto places = [&](u32* all) { return block_exclusive_sum<PART_THREADS>((t + LINE_ROWS - 1) & ~(LINE_ROWS - 1), s_wave, all); };
  auto settle = [&](u32 b, u32 pre) {
    const u32 tid = thread_here();
    if (tid >= span) return;
    S.cnt[tid] = 0;
    const u32 fine = S.fine[tid], out = t & ~(LINE_ROWS - 1), first = fine >> 11, cells = (fine & 2047u) + 1;
    if (out && fill_rows(got) + out > cells) status |= DS_DUPLICATE;
    S.place[b][tid] = make_uint2(pre + left, (pre + out) | ((t - out) << 16));
    S.leave[b][tid] = make_uint2(first + fill_front(got) - pre, pre + front_room(got, out, cells));
    left = t - out;
  };
  auto round = [&](u32 base, u32 b, uint4 (&row)[LINES_U], u64 (&key)[LINES_U], u32 (&src)[LINES_U], u32 (&src_key)[LINES_U]) {
    const u32 tid = thread_here();
#pragma unroll
    for (u32 u = 0; u < LINES_U; ++u) {
      if (fi_cell[u] == ~0u) continue;
      const u32 fi = fi_cell[u] & 0xFFFFu, q = S.place[b][fi].x + at[u];
      if (q % LINE_ROWS == 0) S.line[q / LINE_ROWS] = (uint16_t)fi;      // every line has a row at its first place
      const uint4 v = part_row(row[u], (fi_cell[u] >> 16) & ROW_CELL_MASK);
      S.row[q] = u32x4{v.x, v.y, v.z, v.w};
    }
#pragma unroll
    for (u32 h = 0; h < HELD; ++h) {
      const u32 fi = (tid + h * PART_THREADS) / LINE_ROWS;
      if (held >> h & 1) { const u32 q = S.place[b][fi].x + h_at[h]; S.row[q] = h_row[h]; if (q % LINE_ROWS == 0) S.line[q / LINE_ROWS] = (uint16_t)fi; }
    }
    count(base + LINES_CHUNK, key);
    __syncthreads();
    const u32 here = total;
    __builtin_amdgcn_sched_barrier(0);
    ask();
    part_rows(d, src, row);
    part_keys(d, C, base + 3 * LINES_CHUNK, end, src_key, key);
    held = 0;
#pragma unroll
    for (u32 h = 0; h < HELD; ++h) {
      const u32 i = tid + h * PART_THREADS, fi = i / LINE_ROWS, k = i % LINE_ROWS;
      const u32 stay = fi < span ? S.place[b][fi].y : 0u;
      if (k < stay >> 16) { h_row[h] = S.row[(stay & 0xFFFFu) + k]; h_at[h] = k - (stay >> 16); held |= 1u << h; }
    }
    const u32 pre = places(&total);
    __builtin_amdgcn_sched_barrier(0);
    auto leave = [&](u32 i) {
      const u32 q = std::min(tid + i * PART_THREADS, LINES_STAGE - 1);
      const uint2 L = S.leave[b][q < here ? S.line[q / LINE_ROWS] : 0u];
      // whole lines, with the streaming hint
      __builtin_amdgcn_raw_buffer_store_b128(S.row[q], rsrc, q < here && q < L.y && tid + i * PART_THREADS < LINES_STAGE ? (int)((q + L.x) * 16) : -1, 0, 2);
      if (i % 3 == 2) __builtin_amdgcn_sched_barrier(0);        // three rows in registers at a time
    };
#pragma unroll
    for (u32 i = 0; i < OUT_MOST; ++i) leave(i);
    if (here > OUT_MOST * PART_THREADS) {
#pragma unroll
      for (u32 i = OUT_MOST; i < OUT; ++i) leave(i);
    }
    settle(b ^ 1, pre);
    __syncthreads();
  };
  __syncthreads();
  count(pos, key0);
  part_keys(d, C, pos + 2 * LINES_CHUNK, end, src0, key0);
  __syncthreads();
  ask();
  settle(0, places(&total));
  __syncthreads();
  for (u32 base = pos; base < end; base += 2 * LINES_CHUNK) {
    round(base, 0, row0, key1, src0, src1);
    if (base + LINES_CHUNK < end) round(base + LINES_CHUNK, 1, row1, key0, src1, src0);
  }
  // what did not make up a line goes to the fine buckets' ends
  const u32 t_end = thread_here();
  if (t_end < span && left) {
    const u32 old = atomicAdd(&d.fill[f_lo + t_end], left << 16);
    const u32 fine = S.fine[t_end], cells = (fine & 2047u) + 1;
    if (fill_rows(old) + left > cells) status |= DS_DUPLICATE;
    S.cnt[t_end] = (u32)back_place(old, 0, cells);
  }
  __syncthreads();
#pragma unroll
  for (u32 h = 0; h < HELD; ++h) {
    if (!(held >> h & 1)) continue;
    const u32 fi = (t_end + h * PART_THREADS) / LINE_ROWS;
    const i32 place = (i32)(S.cnt[fi] + h_at[h]);
    if (place >= 0) *reinterpret_cast<u32x4*>(d.rows + (cell_lo + (S.fine[fi] >> 11) + (u32)place)) = h_row[h];
  }
  __syncthreads();
}

// U: records of a thread in a round.  With one, a workgroup has a single round of every coarse bucket: what such a window takes is the
// fetching of instructions that run once (16K records 8.6 -> 7.5 us).
template <bool SLOTS, bool LINES, u32 U>
__global__ __launch_bounds__(PART_THREADS) void k_grid_partition(GridArgs d) {
  extern __shared__ uint4 s_row[];      // [PART_CHUNK] staged rows | [PART_CHUNK] destinations | 3 x [GRID_SPAN] tables | [PART_CHUNK] slots
  __shared__ u32 s_wave[PART_THREADS / CCLD_WAVE];
  __shared__ u32 s_at[GRID_MAX_BATCHES + 1], s_slot0[GRID_MAX_BATCHES];
  __shared__ u32 s_total, s_last;
  __shared__ u32 s_off;                // 1 + the last coarse bucket with a fine bucket that does not start on a line
  __shared__ PartComm s_lay[PART_LAY];
  __shared__ uint2 s_base[PART_LAY];    // first cell, rounds
  const u32 tid = threadIdx.x;
  if (d.hdr->feasible == 0) return;
  u32* s_dst = reinterpret_cast<u32*>(s_row + PART_CHUNK);
  u32* s_cnt = s_dst + PART_CHUNK;      // rows of the round per fine bucket, then their exclusive scan
  u32* s_next = s_cnt + GRID_SPAN;      // the same of the next round: cleared one round ahead
  u32* s_start = s_next + GRID_SPAN;    // first row reserved in each bucket
  u32* s_src = s_start + GRID_SPAN;
  // the fine buckets' descriptors and the blame table: every workgroup's share
  const u32 n_fine = d.hdr->n_fine, G = gridDim.x;
  u32* const s_first = reinterpret_cast<u32*>(s_row);      // the communicators' first buckets, searched in LDS: 4 of 16 us of a window
  if (blockIdx.x * PART_THREADS < n_fine) {                // of 600K records went by with a search in memory
    for (u32 c = tid; c < d.n_comms; c += PART_THREADS) s_first[c] = d.lay[c].fb_base;
    __syncthreads();
  }
  for (u32 f = blockIdx.x * PART_THREADS + tid; f < n_fine; f += G * PART_THREADS) {
    // the communicator whose fine buckets include f: the last one whose first bucket is <= f
    u32 lo = 0, hi = d.n_comms;
    while (lo < hi) { const u32 m = (lo + hi) >> 1; if (s_first[m] <= f) lo = m + 1; else hi = m; }
    const u32 c = lo - 1;
    const CommLayout L = d.lay[c];
    const u32 r0 = (f - L.fb_base) * L.rpb;
    FineDesc D;
    D.comm = c; D.size = L.size;
    D.K = (L.rounds - r0) < L.rpb ? (L.rounds - r0) : L.rpb;
    D.srow0 = L.seg_base + r0; D.cell0 = L.cell_base + r0 * L.size; D.pad = 0; D.seq0 = L.seq_min + r0;
    d.desc[f] = D;
    if (L.size > CCLD_WAVE) d.long_list[atomicAdd(&d.hdr->n_long, 1u)] = f;
    d.nflag[f] = 0;
  }
  for (u32 i = blockIdx.x * PART_THREADS + tid; i < d.n_blame; i += G * PART_THREADS) d.blame[i] = 0;
  const PartKey pk(d.kf);
  const u32 per = ((d.n + G - 1) / G + CCLD_WAVE - 1) / CCLD_WAVE * CCLD_WAVE;
  // a permutation of the slices for grids of whole XCD rounds, which all windows of more than 256K records take
  const u32 slice = G % PART_XCDS == 0 ? (blockIdx.x % PART_XCDS) * (G / PART_XCDS) + blockIdx.x / PART_XCDS : blockIdx.x;
  const u64 lo64 = (u64)per * slice;
  const u32 lo = lo64 < d.n ? (u32)lo64 : d.n, hi = lo64 + per < d.n ? (u32)(lo64 + per) : d.n;
  u64 status = 0;
  const u32 nb = d.n_buckets == 1 ? 1u : d.nb;          // pieces of one coarse bucket
  // the coarse bucket that holds record lo: the last one that starts at or before it
  static_assert(INGEST_STAGED_BUCKETS <= PART_THREADS, "a thread per coarse bucket");
  const u32 b_lo = d.n_buckets == 1 ? 0u : (u32)__syncthreads_count(tid < d.n_buckets && d.piece_at[(u64)tid * nb] <= lo) - 1;
  if (tid == 0) s_off = 0;
  __syncthreads();
  u32 pos = lo;
  for (u32 b = lo < hi ? b_lo : d.n_buckets; b < d.n_buckets && pos < hi; ++b) {
    // the bucket's pieces, its records of this slice, its communicators and fine buckets, all on their way together
    const u32 c0 = (u32)std::min<u64>((u64)b << d.bshift, d.n_comms), c1 = (u32)std::min<u64>((u64)(b + 1) << d.bshift, d.n_comms);
    const bool near = c1 - c0 <= PART_LAY;
    static_assert(GRID_MAX_BATCHES < PART_THREADS && PART_LAY <= PART_THREADS, "a thread per piece and per communicator");
    u32 at = 0, slot = 0;
    CommLayout L;
    if (tid <= nb) at = d.piece_at[b * nb + tid];
    if (tid < nb) slot = d.piece_slot[b * nb + tid];
    if (near && tid < c1 - c0) L = d.lay[c0 + tid];
    const u32 f_lo = d.lay[c0].fb_base, span = d.lay[c1].fb_base - f_lo;
    if (tid <= nb) s_at[tid] = at;
    if (tid < nb) s_slot0[tid] = slot;
    if (near && tid < c1 - c0) { s_lay[tid] = PartComm(L, f_lo); s_base[tid] = make_uint2(L.cell_base, L.rounds); }
    if constexpr (LINES) if (near && tid < c1 - c0 && off_lines(L.size, L.rpb, L.rounds)) s_off = b + 1;
    __syncthreads();
    const u32 end = s_at[nb] < hi ? s_at[nb] : hi;
    if (end <= pos) { __syncthreads(); continue; }         // no record of the bucket in the slice
    if constexpr (LINES) if (near && s_off != b + 1 && span <= LINES_SPAN && end - pos >= LINES_MIN) {
      part_lines(d, *reinterpret_cast<PartLines*>(s_row), s_lay, s_base, c0, c1 - c0, pk, s_at, s_slot0, s_wave, pos, end, f_lo, span, status);
      pos = end;
      continue;
    }
    for (u32 i = tid; i < span; i += PART_THREADS) s_cnt[i] = 0;
    PartCursor C(s_at, s_slot0);
    u64 key[U], nkey[U];
    uint4 row[U];
    u32 src[U], nsrc[U];
    part_keys(d, C, pos, end, src, key);
    part_rows(d, src, row);
    wait_vector_memory();        // so that no register of the loop below is waited for behind the loads inside it
    __syncthreads();
    // MORE: another round follows
    auto round = [&](auto MORE, u32 base) {
      const u32 tid = thread_here();
      // (packed: at 128 registers per thread the kernel spills with a word for each)
      u32 fi_cell[U], at_room[U], first[U];       // fi | cell << 16, at | room << 16
      bool on[U];
#pragma unroll
      for (u32 u = 0; u < U; ++u) {
        on[u] = base + u * PART_THREADS + tid < end;
        if (!on[u]) continue;
        const u64 k = key[u];
        PartComm L;
        uint2 B;                       // first cell, rounds
        if (near) {
          L = s_lay[pk.comm(k) - c0]; B = s_base[pk.comm(k) - c0];
        } else {
          const CommLayout G = d.lay[pk.comm(k)];
          wait_vector_memory();        // nothing of this branch is waited for behind it
          L = PartComm(G, f_lo); B = make_uint2(G.cell_base, G.rounds);
        }
        const u32 rel = pk.seq(k) - L.seq, fr = L.bucket(rel), r0 = fr * L.rpb(), left = B.y - r0;
        const u32 fi = L.fb + fr, room = (left < L.rpb() ? left : L.rpb()) * L.size();
        first[u] = B.x + r0 * L.size();
        on[u] = fi < span;
        fi_cell[u] = fi | (((rel - r0) * L.size() + pk.slot(k)) << 16);
        if (on[u]) at_room[u] = atomicAdd(&s_cnt[fi], 1u) | (room << 16);
      }
      __syncthreads();
      {     // one reservation per bucket, all on their way at once, behind them the next rows, and meanwhile the exclusive scan of
            // the round's counts
        constexpr u32 PER = GRID_SPAN / PART_THREADS;
        u32 v[PER], got[PER], sum = 0;
#pragma unroll
        for (u32 i = 0; i < PER; ++i) {
          const u32 q = tid + i * PART_THREADS, c = q < span ? s_cnt[q] : 0u;
          got[i] = 0;
          if (c) got[i] = atomicAdd(&d.fill[f_lo + q], c);
        }
        if constexpr (MORE) part_keys(d, C, base + U * PART_THREADS, end, nsrc, nkey);
#pragma unroll
        for (u32 i = 0; i < PER; ++i) { const u32 q = PER * tid + i; v[i] = q < span ? s_cnt[q] : 0u; sum += v[i]; }
        u32 tot;
        u32 ex = block_exclusive_sum<PART_THREADS>(sum, s_wave, &tot);
#pragma unroll
        for (u32 i = 0; i < PER; ++i) { const u32 q = PER * tid + i; if (q < span) s_cnt[q] = ex; ex += v[i]; }
#pragma unroll
        for (u32 i = 0; i < PER; ++i) { const u32 q = tid + i * PART_THREADS; if (q < span) s_start[q] = got[i]; }
        if (tid == 0) s_total = tot;
      }
      __syncthreads();
      for (u32 i = tid; i < span; i += PART_THREADS) s_next[i] = 0;
#pragma unroll
      for (u32 u = 0; u < U; ++u) {
        if (!on[u]) continue;
        const u32 fi = fi_cell[u] & 0xFFFFu, at = at_room[u] & 0xFFFFu, room = at_room[u] >> 16;
        const u32 q = s_cnt[fi] + at, w = fill_front(s_start[fi]) + at;
        if (w >= room) status |= DS_DUPLICATE;
        s_dst[q] = w < room ? first[u] + w : ~0u;
        s_row[q] = part_row(row[u], (fi_cell[u] >> 16) & ROW_CELL_MASK);
        if (SLOTS) s_src[q] = src[u];
      }
      // the next round's rows take the place of this one's; its keys are here (4: the loads behind theirs)
      if constexpr (MORE) {
#pragma unroll
        for (u32 u = 0; u < U; ++u) src[u] = nsrc[u];
        part_rows(d, src, row);
        __builtin_amdgcn_s_waitcnt(0x0F74);
#pragma unroll
        for (u32 u = 0; u < U; ++u) key[u] = nkey[u];
      }
      __syncthreads();
      // Pieces of a line that the round writes completely leave with the streaming hint, which keeps them from displacing the
      // partially written lines at the buckets' frontiers from the L2.
      const u32 total = s_total;
      for (u32 i = tid; i < total; i += PART_THREADS) {
        const u32 D = s_dst[i];
        if (D == ~0u) continue;
        const u32 o = D & 7;
        const bool full = i >= o && i + 7 - o < total && s_dst[i - o] == D - o && s_dst[i + 7 - o] == D + 7 - o;
        const uint4 v = s_row[i];
        u32x4 vv = {v.x, v.y, v.z, v.w};
        if (full) __builtin_nontemporal_store(vv, reinterpret_cast<u32x4*>(d.rows + D));
        else d.rows[D] = v;
        if (SLOTS) d.slots[D] = s_src[i];
      }
      // no barrier here: the staging area is written again behind two barriers of the next round
      u32* const t = s_cnt; s_cnt = s_next; s_next = t;
    };
    u32 base = pos;
    if constexpr (U > 1) for (; base + U * PART_THREADS < end; base += U * PART_THREADS) round(std::true_type{}, base);
    round(std::false_type{}, base);
    pos = end;
    __syncthreads();        // the piece table is rewritten for the next bucket
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) status |= shfl_xor_u64(status, m);
  if (lane_id() == 0 && status) atomicOr((unsigned long long*)&d.counters[CNT_STATUS], (unsigned long long)status);
  // the last workgroup to finish scans the records per fine bucket; few buckets are summed by the statistics kernels' workgroups
  // for themselves
  if (d.self_sum || !last_block(&d.hdr->done, G, &s_last)) return;
  u32 carry = 0;
  for (u32 base = 0; base < n_fine; base += PART_THREADS * 4) {
    u32 v[4], sum = 0;
#pragma unroll
    for (u32 i = 0; i < 4; ++i) { const u32 f = base + tid * 4 + i; v[i] = f < n_fine ? fill_rows(load_agent(&d.fill[f])) : 0u; sum += v[i]; }
    u32 tot;
    u32 ex = carry + block_exclusive_sum<PART_THREADS>(sum, s_wave, &tot);
#pragma unroll
    for (u32 i = 0; i < 4; ++i) { const u32 f = base + tid * 4 + i; if (f < n_fine) d.rec0[f] = ex; ex += v[i]; }
    carry += tot;
  }
  if (tid == 0) d.rec0[n_fine] = carry;
}
static_assert(GRID_SPAN % PART_THREADS == 0, "whole buckets per thread");
static_assert(GRID_MAX_COMMS * 4 <= PART_CHUNK * 16, "the first buckets fit the staging area");
static_assert(ROW_CELL_SHIFT == 16 && ROW_CELL_MASK == GRID_B - 1, "the cell is packed as the row has it");

constexpr size_t PART_LDS = (size_t)PART_CHUNK * 20 + (size_t)GRID_SPAN * 12, PART_LDS_SLOTS = PART_LDS + (size_t)PART_CHUNK * 4;
constexpr size_t PART_LDS_LINES = std::max(PART_LDS, sizeof(PartLines));
template <class F>
static hipError_t each_partition(F f) {
  hipError_t e = f(&k_grid_partition<false, false, PART_U>, PART_LDS);
  if (e == hipSuccess) e = f(&k_grid_partition<true, false, PART_U>, PART_LDS_SLOTS);
  if (e == hipSuccess) e = f(&k_grid_partition<false, false, 1>, PART_LDS);
  if (e == hipSuccess) e = f(&k_grid_partition<true, false, 1>, PART_LDS_SLOTS);
  return e != hipSuccess ? e : f(&k_grid_partition<false, true, PART_U>, PART_LDS_LINES);
}
hipError_t allow_lds_grid() {
  return each_partition([](auto k, size_t bytes) { return allow_lds(reinterpret_cast<const void*>(k), bytes); });
}
// 33M, 41M, 57M and 82M records (communicators of 8 and 64 members): 270, 367, 500 and 844 us as runs, 304, 378, 489 and 704 in whole
// lines; 61M of 8 and 60: 503 and 552.  (The order of the records is wanted for small windows, so rows with slots have no lines.)
bool grid_in_lines(uint64_t n, bool with_slots) { return !with_slots && n / PART_BLOCKS >= LINES_SLICE; }
void launch_grid_partition(hipStream_t st, const GridArgs& d) {
  // small windows: a thousand records per workgroup, so that there are several of them
  const u32 g = std::min<u32>(PART_BLOCKS, std::max<u32>((d.n + PART_THREADS - 1) / PART_THREADS, 1));
  const bool one = d.n <= PART_BLOCKS * PART_THREADS;        // a record per thread
  auto go = [&](auto kernel, size_t bytes) { hipLaunchKernelGGL(kernel, dim3(g), dim3(PART_THREADS), bytes, st, d); };
  if (d.slots) one ? go(k_grid_partition<true, false, 1>, PART_LDS_SLOTS) : go(k_grid_partition<true, false, PART_U>, PART_LDS_SLOTS);
  else if (one) go(k_grid_partition<false, false, 1>, PART_LDS);
  else if (!d.lines) go(k_grid_partition<false, false, PART_U>, PART_LDS);
  else go(k_grid_partition<false, true, PART_U>, PART_LDS_LINES);
}

// ---- rounds without any record ------------------------------------------------------------------------
// The statistics find them too, but behind them the whole window has still to be sorted: here they end the placement of a
// window whose statistics take long, before these run.  A round can only be missing from a fine bucket that has at least
// that many records fewer than cells; such buckets mark the rounds of their rows, a wavefront each.  Taken by windows of
// more than GRID_FINE_BOUND fine buckets that have fewer records than cells: 20M records with one round missing 1.99 -> 1.79 ms,
// the steps of a 20M-record stream that have one in the window 1.41 -> 1.27; where no round is missing it costs 5 us.
constexpr u32 GAP_THREADS = 256, GAP_BLOCKS = 2048;
__global__ __launch_bounds__(GAP_THREADS) void k_grid_gaps(GridArgs d) {
  constexpr u32 NW = GAP_THREADS / CCLD_WAVE, WORDS = GRID_B / 32, U = 8;
  static_assert(WORDS <= CCLD_WAVE, "a word of the bitmap per lane");
  __shared__ u32 s_round[NW][WORDS];
  const u32 n_fine = d.hdr->n_fine, lane = lane_id(), wave = threadIdx.x / CCLD_WAVE;
  u32* const mark = s_round[wave];
  for (u32 f = blockIdx.x * NW + wave; f < n_fine; f += gridDim.x * NW) {
    const FineDesc D = d.desc[f];
    const u32 cells = D.K * D.size, fill = d.fill[f], front = fill_front(fill), back = cells - fill_back(fill);
    if (fill_rows(fill) + D.size > cells) continue;
    if (lane < WORDS) mark[lane] = 0;
    __builtin_amdgcn_wave_barrier();
    auto on = [&](u32 i) { return i < front || (i >= back && i < cells); };
    for (u32 i0 = lane; i0 < cells; i0 += U * CCLD_WAVE) {
      u32 y[U];
#pragma unroll
      for (u32 u = 0; u < U; ++u) y[u] = on(i0 + u * CCLD_WAVE) ? d.rows[D.cell0 + i0 + u * CCLD_WAVE].y : ~0u;
#pragma unroll
      for (u32 u = 0; u < U; ++u) {
        const u32 cell = (y[u] >> ROW_CELL_SHIFT) & ROW_CELL_MASK, round = cell / D.size;
        if (on(i0 + u * CCLD_WAVE) && round < D.K) atomicOr(&mark[round >> 5], 1u << (round & 31));
      }
    }
    __builtin_amdgcn_wave_barrier();
    const u32 left = lane * 32 < D.K ? D.K - lane * 32 : 0u, want = left >= 32 ? ~0u : (1u << left) - 1;
    const u32 have = lane < WORDS ? mark[lane] : 0u;
    if (have != want && lane < WORDS) {
      atomicOr((unsigned long long*)&d.counters[CNT_STATUS], (unsigned long long)DS_DENSE_FALLBACK);
      d.hdr->feasible = 0;
    }
    __builtin_amdgcn_wave_barrier();
  }
}
void launch_grid_gaps(hipStream_t st, const GridArgs& d, uint32_t n_fine) {
  const u32 blocks = std::min<u32>((n_fine + 3) / 4, GAP_BLOCKS);
  hipLaunchKernelGGL(k_grid_gaps, dim3(blocks), dim3(GAP_THREADS), 0, st, d);
}

}  // namespace ccld
