// extern "C" entry points: context set-up, workspace carving, ingest, window analysis, blame.
#include <algorithm>
#include <chrono>
#include <cstring>
#include <new>

#include "ccld_internal.h"
#include "device_utils.h"
#include "window_kernels.h"
#include "grid.h"
#include "host_copy.h"
#include "merge.h"

using namespace ccld;

#define HIP_TRY(x) do { if ((x) != hipSuccess) { (void)hipGetLastError(); return CCLD_E_HIP; } } while (0)

// words of the pinned buffer: the counters come first
constexpr size_t PINNED_FINE = 32, PINNED_META = 64;
static_assert(CNT_COUNT <= PINNED_FINE, "the counters come first");


namespace {

CopyStreams g_copy_streams;

// Bump allocator over the caller's workspace; with base == nullptr it only measures.
struct Carver {
  uint8_t* base; uint64_t off;
  template <class T> T* take(uint64_t count) {
    off = (off + 255) & ~(uint64_t)255;
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

struct TopoCounts { uint64_t n_members; };

void carve_all(ccld_ctx* c, Carver& w, uint32_t n_ranks, uint32_t n_comms, uint64_t n_members) {
  const uint64_t N = std::max<uint64_t>(c->cap, 1), B = std::max<uint64_t>(c->batch_cap, 1);
  // topology
  c->topo.algo = w.take<uint8_t>(n_comms);
  c->topo.size = w.take<uint32_t>(n_comms);
  c->topo.member_off = w.take<uint32_t>(n_comms);
  c->topo.members = w.take<uint32_t>(n_members);
  c->topo.members_sorted = w.take<uint32_t>(n_members);
  c->topo.sorted_slot = w.take<uint32_t>(n_members);
  c->topo.tree_parent = w.take<int32_t>(n_members);
  c->topo.rank_comm_off = w.take<uint32_t>((uint64_t)n_ranks + 1);
  c->topo.rank_comms = w.take<uint32_t>(n_members);
  c->topo.rank_slots = w.take<uint32_t>(n_members);
  c->topo.rank_memb4 = w.take<uint32_t>(4ull * n_ranks);
  c->topo.rank_cell4 = w.take<uint32_t>(4ull * n_ranks);
  c->topo.member_comm = w.take<uint32_t>(n_members);
  c->comm_info = w.take<uint2>(n_comms);
  // window
  c->win_key = w.take<uint64_t>(N);
  c->win_row = w.take<uint4>(N);
  c->win_wide = w.take<int64_t>(3 * N);
  c->rounds_cap = c->n_buckets > 1 ? ingest_rounds_cap(N, c->p.window_batches) : 0;
  c->ing_rounds = w.take<uint32_t>(c->rounds_cap * c->n_buckets + 1);
  c->batch_meta = w.take<BatchMeta>((uint64_t)c->p.window_batches + 2);
  const uint64_t n_meta = (uint64_t)c->p.window_batches + 2;
  c->ing_table = w.take<uint32_t>((uint64_t)c->n_buckets * INGEST_BLOCKS);
  c->ing_base = w.take<uint32_t>(n_meta * (c->n_buckets + 1) + 4);
  c->comm_range = c->grid_capable ? w.take<uint64_t>(n_meta * n_comms * 2) : nullptr;
  // sort
  // (the hang pass sorts its root list, at most one entry per communicator member, in these buffers too)
  const uint64_t NS = std::max<uint64_t>(N, n_members);
  c->sort_cap = NS;
  const uint64_t tw = sort_table_words(NS);
  // The partitioned rows of the grid placement and the arrays that run beside them.  A window is either sorted or placed
  // on the grid, so in large contexts they lie over the sort buffers; small ones, and contexts that ask for
  // the placement, have them apart.
  auto take_grid = [&](Carver& g) {
    const uint64_t cells = c->cell_cap + (grid_in_lines(N, false) ? (LINE_ROWS - 1) * (uint64_t)n_comms : 0);
    c->g_rows = g.take<uint4>(cells);
    c->g_slots = g.take<uint32_t>(cells);
    c->g_cell_row = g.take<uint16_t>(cells);
    c->flag_stage = g.take<uint32_t>(N);
  };
  const uint64_t sort_begin = w.off;
  for (int i = 0; i < 2; ++i) { c->sb.key[i] = w.take<uint64_t>(NS); c->sb.idx[i] = w.take<uint32_t>(NS); }
  c->keyC = w.take<uint64_t>(NS);
  if (c->grid_capable && c->grid_over_sort) {
    Carver g{w.base, sort_begin};
    take_grid(g);
    w.off = std::max(w.off, g.off);
  } else if (c->grid_capable) {
    take_grid(w);
  }
  c->sb.table = w.take<uint32_t>(tw);
  c->sb.totals = w.take<uint32_t>(SORT_RADIX);
  c->table2 = w.take<uint32_t>(tw);
  c->totals2 = w.take<uint32_t>(SORT_RADIX);
  // analysis scratch
  const uint64_t NT = std::max<uint64_t>(N, std::max<uint64_t>(n_members, n_comms));   // the tile-count scratch also serves the hang pass
  const uint64_t seg_tiles = (NT + SEG_TILE - 1) / SEG_TILE, sel_tiles = (NT + SEL_TILE - 1) / SEL_TILE;
  c->tile_heads = w.take<uint32_t>(seg_tiles + 2);
  c->tile_flags = w.take<uint32_t>(sel_tiles + 2);
  c->blame_list = w.take<uint32_t>(2ull * n_ranks);
  c->blame_tiles = w.take<uint32_t>(n_ranks / SEL_TILE + 3);
  c->blame_order = w.take<uint32_t>(n_ranks);
  // per-record scratch of one analysis; nothing in it outlives the next ingest, so a batch that arrives in host
  // memory is staged in the same bytes (48 per record of batch capacity)
  c->stage = w.take<uint8_t>(0);
  const uint64_t scratch_begin = w.off;
  c->rec_flag = w.take<uint8_t>(N);
  c->flag_pos = w.take<uint32_t>(N);
  c->flag_lag = w.take<int64_t>(2 * N);
  c->big_list = w.take<uint32_t>(3 * (N / 65 + 2));
  c->flag_key = w.take<uint64_t>(N);
  c->range_c = w.take<int64_t>(N);
  c->gcode = w.take<uint16_t>(N);
  c->comm_groups = w.take<uint32_t>((uint64_t)n_comms + 1);
  c->comm_row = w.take<uint32_t>(n_comms);
  c->chain_parent = w.take<uint32_t>(N + 1);
  c->alert_rows = w.take<uint32_t>(END_ALERTS);
  c->alert_list = w.take<uint32_t>(NT);
  c->alert_ncand = w.take<uint32_t>(N + 2);
  if (w.off - scratch_begin < B * 48) (void)w.take<uint8_t>(B * 48 - (w.off - scratch_begin));
  c->gstate = w.take<GroupState>((uint64_t)n_comms * GROUP_SLOTS);
  c->chain_first = w.take<uint32_t>((uint64_t)n_comms + 2);
  c->arrivals = w.take<uint32_t>(ARRIVAL_WORDS);
  // the counters and the blame table are cleared together at the start of every analysis
  c->counters = w.take<uint64_t>(CNT_COUNT);
  c->blame = w.take<int64_t>((uint64_t)CCLD_BLM_NCOL * n_ranks);
  c->g_lay = nullptr; c->g_hdr = nullptr; c->g_desc = nullptr;
  if (c->grid_capable) {
    const uint64_t F = (uint64_t)c->fine_cap + 4;
    c->g_lay = w.take<CommLayout>((uint64_t)n_comms + 1);
    c->g_hdr = w.take<GridHeader>(1);
    c->g_desc = w.take<FineDesc>(F);
    const uint64_t pieces = c->n_buckets == 1 ? 1 : (uint64_t)c->n_buckets * c->p.window_batches;
    c->g_piece_at = w.take<uint32_t>(pieces + 1); c->g_piece_slot = w.take<uint32_t>(pieces);
    c->g_fill = w.take<uint32_t>(F); c->g_rec0 = w.take<uint32_t>(F);
    c->g_nflag = w.take<uint32_t>(F); c->g_long = w.take<uint32_t>(F);
  }
  // hang location
  const uint64_t SN = std::max<uint64_t>(c->snap_cap, 1);
  c->n_members = n_members;
  c->rate_root = w.take<int64_t>(n_comms);
  c->long_comms = w.take<LongComm>(n_comms);
  c->h_counters = w.take<uint64_t>(CNT_COUNT + HANG_REGIONS);
  c->h_cell = w.take<uint64_t>(2 * SN);
  c->h_cnt = w.take<uint32_t>(SN / 32 + 1);
  c->h_pair = w.take<int64_t>((uint64_t)CCLD_HPAIR_NCOL * n_members);
  c->h_comm = w.take<int64_t>((uint64_t)CCLD_HCOMM_NCOL * n_comms);
  c->h_wait_slot = w.take<int32_t>(n_members);
  c->h_cand = w.take<uint8_t>(n_members);
  c->h_layer_max = w.take<uint64_t>(n_members);
  c->f_last = w.take<uint64_t>(2ull * CCLD_FRAME_CHANNELS * n_members);
  c->f_frame = w.take<uint64_t>((uint64_t)n_ranks + 1);
  c->h_stage = w.take<uint8_t>(SN * 32);
}

ccld_status check_params(const ccld_params* p) {
  if (!p) return CCLD_E_NULL;
  if (p->tbase_rounds < 1 || p->theta_den < 1 || p->ab_den < 1 || p->kmad_den < 1 || p->tbase_warmup_ns < 0 ||
      p->window_batches < 1 || p->window_batches > 4096 || p->hang_threshold_ns < 0 ||
      p->placement > CCLD_PLACEMENT_DENSE)
    return CCLD_E_BAD_ARG;
  return CCLD_OK;
}

ccld_status check_topology(const ccld_topology* t, uint64_t* n_members) {
  if (!t) return CCLD_E_NULL;
  if (t->n_ranks == 0 || t->n_comms == 0) return CCLD_E_BAD_TOPOLOGY;
  if (!t->algo || !t->size || !t->member_off || !t->members) return CCLD_E_NULL;
  uint64_t total = 0;
  for (uint32_t c = 0; c < t->n_comms; ++c) {
    if (t->size[c] == 0 || t->algo[c] > CCLD_ALGO_TREE) return CCLD_E_BAD_TOPOLOGY;
    if (t->member_off[c] != total) return CCLD_E_BAD_TOPOLOGY;     // packed CSR
    total += t->size[c];
    if (total > 0xFFFFFFFFull) return CCLD_E_BAD_TOPOLOGY;
  }
  for (uint32_t c = 0; c < t->n_comms; ++c) {
    std::vector<uint32_t> m(t->members + t->member_off[c], t->members + t->member_off[c] + t->size[c]);
    std::sort(m.begin(), m.end());
    for (size_t i = 0; i < m.size(); ++i)
      if (m[i] >= t->n_ranks || (i > 0 && m[i] == m[i - 1])) return CCLD_E_BAD_TOPOLOGY;
    if (t->algo[c] == CCLD_ALGO_TREE) {
      if (!t->tree_parent) return CCLD_E_BAD_TOPOLOGY;
      int roots = 0;
      for (uint32_t q = 0; q < t->size[c]; ++q) {
        int32_t par = t->tree_parent[t->member_off[c] + q];
        if (par < 0) ++roots;
        else if ((uint32_t)par >= q) return CCLD_E_BAD_TOPOLOGY;   // BFS order: parents come first
      }
      if (roots != 1 || t->tree_parent[t->member_off[c]] >= 0) return CCLD_E_BAD_TOPOLOGY;
      std::vector<uint32_t> depth(t->size[c], 0);                  // BFS order: layers are contiguous
      for (uint32_t q = 1; q < t->size[c]; ++q) {
        depth[q] = depth[t->tree_parent[t->member_off[c] + q]] + 1;
        if (depth[q] < depth[q - 1]) return CCLD_E_BAD_TOPOLOGY;
      }
    }
  }
  *n_members = total;
  return CCLD_OK;
}

// What follows from the parameters, the topology and the capacities: the key format, whether windows can be placed on the
// grid, and the communicator buckets of the ingest.
void plan(ccld_ctx* c, const ccld_params* p, const ccld_topology* t, uint64_t n_members, uint64_t cap, uint64_t batch_cap, uint64_t snap_cap) {
  c->p = *p;
  c->cap = cap; c->batch_cap = batch_cap; c->snap_cap = snap_cap;
  uint32_t max_size = 1;
  for (uint32_t k = 0; k < t->n_comms; ++k) max_size = std::max(max_size, t->size[k]);
  const int mb = bits_for(max_size - 1), cb = bits_for(t->n_comms - 1);
  c->max_comm_size = max_size;
  c->long_classes = 0;
  for (uint32_t k = 0; k < t->n_comms; ++k) if (t->size[k] > 64) c->long_classes |= t->size[k] <= 128 ? 1u : t->size[k] <= 256 ? 2u : t->size[k] <= 512 ? 4u : 8u;
  c->kf.mb = mb; c->kf.cb = cb; c->kf.sb = 64 - mb - cb;
  const uint64_t N = std::max<uint64_t>(cap, 1), W = p->window_batches;
  c->grid_capable = cap > 0 && max_size <= GRID_B && t->n_comms <= GRID_MAX_COMMS && (W + 2) * t->n_comms * 16 <= (64ull << 20);
  c->dense_asked = p->placement == CCLD_PLACEMENT_DENSE && W == 1;
  // cells beyond the records: a fifth, so that windows with members missing here and there stay on the grid; small
  // contexts can afford twice the records and take the arrays of their own
  c->grid_over_sort = N >= (4u << 20) && p->placement != CCLD_PLACEMENT_DENSE;
  c->cell_cap = (uint32_t)std::min<uint64_t>(N >= (4u << 20) ? N + N / 5 : 2 * N + 4096, 0xFFFFFF00u);
  c->fine_cap = c->cell_cap / GRID_MIN_FILL + t->n_comms + 16;
  // Communicator buckets of the ingest.  A window that cannot be placed on the grid takes buckets whose rows (16 bytes per record) stay
  // within about 100 MB, which the memory-side cache holds while the statistics gather from one.
  int bb = 0;
  if (c->grid_capable) {
    bb = grid_bucket_bits(N / 1400 + t->n_comms, W, t->n_comms);
    if (bb > 0 && W > GRID_MAX_BATCHES) c->grid_capable = false;
  }
  if (!c->grid_capable) { bb = 0; while (bb < 6 && ((N * 16) >> bb) > 100000000ull) ++bb; }
  c->bshift = bucket_shift(bb, t->n_comms);
  c->n_buckets = bucket_count(bb, t->n_comms);
  c->n_members = n_members;
}

ccld_status data_status(uint64_t bits) {
  if (bits & DS_UNKNOWN_COMM) return CCLD_E_UNKNOWN_COMM;
  if (bits & DS_NOT_MEMBER) return CCLD_E_RANK_NOT_MEMBER;
  if (bits & DS_RANGE) return CCLD_E_RANGE;
  if (bits & DS_KEY_WIDTH) return CCLD_E_KEY_WIDTH;
  if (bits & DS_DUPLICATE) return CCLD_E_DUPLICATE_KEY;
  if (bits & DS_SNAPSHOT_GAP) return CCLD_E_SNAPSHOT_GAP;
  return CCLD_OK;
}

}  // namespace

extern "C" {

ccld_status ccld_default_params(ccld_params* p) {
  if (!p) return CCLD_E_NULL;
  std::memset(p, 0, sizeof(*p));
  p->hang_threshold_ns = 300000000000ll;
  p->tbase_init_ns = INT64_MAX / 4;
  p->tbase_rounds = 100;
  p->repeat_threshold = 2;
  p->tbase_warmup_ns = 120000000000ll;
  p->theta_num = 3; p->theta_den = 1;
  p->alpha_num = 4; p->beta_num = 6; p->ab_den = 10;
  p->barrier_bytes = 4;
  p->kmad_num = 9; p->kmad_den = 2;
  p->lag_floor_ns = 300000;
  p->stall_snapshots = 30;
  p->fifo_depth = 8;
  p->window_batches = 1;
  return CCLD_OK;
}

ccld_status ccld_query_workspace(const ccld_params* params, const ccld_topology* topo, uint64_t max_window_records,
                                 uint64_t max_batch_records, uint64_t max_snapshot_rows, uint64_t* bytes) {
  if (!bytes) return CCLD_E_NULL;
  ccld_status s = check_params(params);
  if (s != CCLD_OK) return s;
  uint64_t n_members = 0;
  s = check_topology(topo, &n_members);
  if (s != CCLD_OK) return s;
  if (max_window_records >= (1ull << 31) || max_batch_records > max_window_records ||
      max_snapshot_rows >= (1ull << 31))
    return CCLD_E_CAPACITY;
  ccld_ctx tmp;
  plan(&tmp, params, topo, n_members, max_window_records, max_batch_records, max_snapshot_rows);
  Carver w{nullptr, 0};
  carve_all(&tmp, w, topo->n_ranks, topo->n_comms, n_members);
  *bytes = w.off + 256;
  return CCLD_OK;
}

ccld_status ccld_create(const ccld_params* params, const ccld_topology* topo, uint64_t max_window_records,
                        uint64_t max_batch_records, uint64_t max_snapshot_rows, void* workspace,
                        uint64_t workspace_bytes, void* hip_stream, ccld_ctx** out) {
  if (!out || !workspace) return CCLD_E_NULL;
  *out = nullptr;
  uint64_t need = 0;
  ccld_status s = ccld_query_workspace(params, topo, max_window_records, max_batch_records, max_snapshot_rows, &need);
  if (s != CCLD_OK) return s;
  if (workspace_bytes < need || ((uintptr_t)workspace & 255) != 0) return CCLD_E_WORKSPACE;
  ccld_ctx* c = new (std::nothrow) ccld_ctx();
  if (!c) return CCLD_E_BAD_ARG;
  uint64_t n_members = 0;
  check_topology(topo, &n_members);
  plan(c, params, topo, n_members, max_window_records, max_batch_records, max_snapshot_rows);
  const int mb = c->kf.mb, cb = c->kf.cb;
  if (mb + cb > 63) { delete c; return CCLD_E_KEY_WIDTH; }
  c->stream = (hipStream_t)hip_stream;
  c->copy_earned = 0;
  if (hipGetDevice(&c->device) != hipSuccess || c->device >= COPY_DEVICES) { (void)hipGetLastError(); delete c; return CCLD_E_HIP; }
  c->chain_ready = false;
  c->rank_bits = bits_for(topo->n_ranks - 1);
  c->head = 0; c->count = 0; c->next_slot = 0; c->rounds_next = 0; c->total_ingested = 0;
  c->inc_ok = false; c->inc_head = c->inc_count = c->inc_total = 0;
  c->sorted_buf = 0; c->blame_valid = false; c->sort_passes = 0;
  c->sf.mb = mb; c->sf.ws = 0; c->sf.seq_base = 0;
  Carver w{(uint8_t*)workspace, 0};
  carve_all(c, w, topo->n_ranks, topo->n_comms, n_members);
  c->topo.n_ranks = topo->n_ranks; c->topo.n_comms = topo->n_comms;
  c->h_pinned = nullptr;
  c->ticket = 0; c->h_clear = true;

  // derived host tables: sorted member lists, rank -> communicators CSR
  std::vector<uint32_t> sorted(topo->members, topo->members + n_members), sslot(n_members);
  std::vector<uint32_t> rc_off((size_t)topo->n_ranks + 1, 0), rc(n_members), rs_slot(n_members);
  std::vector<int32_t> parent(n_members, -1);
  for (uint32_t k = 0; k < topo->n_comms; ++k) {
    {
      std::vector<uint32_t> ord(topo->size[k]);
      for (uint32_t q = 0; q < topo->size[k]; ++q) ord[q] = q;
      const uint32_t* mem = topo->members + topo->member_off[k];
      std::sort(ord.begin(), ord.end(), [mem](uint32_t a, uint32_t b) { return mem[a] < mem[b]; });
      for (uint32_t q = 0; q < topo->size[k]; ++q) {
        sorted[topo->member_off[k] + q] = mem[ord[q]];
        sslot[topo->member_off[k] + q] = ord[q];
      }
    }
    for (uint32_t q = 0; q < topo->size[k]; ++q) rc_off[topo->members[topo->member_off[k] + q] + 1] += 1;
  }
  for (uint32_t r = 0; r < topo->n_ranks; ++r) rc_off[r + 1] += rc_off[r];
  {
    std::vector<uint32_t> fill(rc_off.begin(), rc_off.end() - 1);
    for (uint32_t k = 0; k < topo->n_comms; ++k)
      for (uint32_t q = 0; q < topo->size[k]; ++q) {
        const uint32_t at = fill[sorted[topo->member_off[k] + q]]++;
        rc[at] = k; rs_slot[at] = q;
      }
  }
  if (topo->tree_parent) parent.assign(topo->tree_parent, topo->tree_parent + n_members);
  std::vector<uint32_t> rc4(4ull * topo->n_ranks, 0xFFFFFFFFu);
  bool fits4 = mb + cb <= 31;       // a padding word then never matches a communicator id
  for (uint32_t r = 0; fits4 && r < topo->n_ranks; ++r) {
    if (rc_off[r + 1] - rc_off[r] > 4) { fits4 = false; break; }
    for (uint32_t q = rc_off[r]; q < rc_off[r + 1]; ++q) rc4[4ull * r + (q - rc_off[r])] = (rc[q] << mb) | rs_slot[q];
  }

  // the same rows with the member index (the row of the snapshot grid) in place of the sorted position: the
  // snapshot placement then needs one lookup per row instead of three
  const int pb = bits_for(n_members ? n_members - 1 : 0);
  std::vector<uint32_t> rp4(4ull * topo->n_ranks, 0xFFFFFFFFu);
  const bool fits_cell4 = fits4 && pb + cb <= 31;
  for (uint32_t r = 0; fits_cell4 && r < topo->n_ranks; ++r)
    for (uint32_t q = rc_off[r]; q < rc_off[r + 1]; ++q) {
      const uint32_t k = rc[q], off = topo->member_off[k];
      rp4[4ull * r + (q - rc_off[r])] = (k << pb) | (off + sslot[off + rs_slot[q]]);
    }
  c->topo.pb = pb;
  std::vector<uint32_t> mcomm(n_members);
  for (uint32_t k = 0; k < topo->n_comms; ++k)
    std::fill_n(mcomm.begin() + topo->member_off[k], topo->size[k], k);

  ccld_status rs = CCLD_OK;
  auto up = [&](const void* dst, const void* src, size_t bytes) {
    if (bytes && hipMemcpyAsync(const_cast<void*>(dst), src, bytes, hipMemcpyHostToDevice, c->stream) != hipSuccess)
      rs = CCLD_E_HIP;
  };
  up(c->topo.algo, topo->algo, topo->n_comms);
  up(c->topo.size, topo->size, 4ull * topo->n_comms);
  up(c->topo.member_off, topo->member_off, 4ull * topo->n_comms);
  up(c->topo.members, topo->members, 4ull * n_members);
  up(c->topo.members_sorted, sorted.data(), 4ull * n_members);
  up(c->topo.sorted_slot, sslot.data(), 4ull * n_members);
  up(c->topo.tree_parent, parent.data(), 4ull * n_members);
  up(c->topo.rank_comm_off, rc_off.data(), 4ull * rc_off.size());
  up(c->topo.rank_comms, rc.data(), 4ull * n_members);
  up(c->topo.rank_slots, rs_slot.data(), 4ull * n_members);
  up(c->topo.rank_memb4, rc4.data(), 4ull * rc4.size());
  if (!fits4) c->topo.rank_memb4 = nullptr;
  std::vector<uint2> cinfo(topo->n_comms);
  for (uint32_t k = 0; k < topo->n_comms; ++k) cinfo[k] = make_uint2(topo->member_off[k], topo->size[k]);
  up(c->comm_info, cinfo.data(), sizeof(uint2) * cinfo.size());
  up(c->topo.member_comm, mcomm.data(), 4ull * n_members);
  std::vector<LongComm> longs;
  c->short_lanes = 1;
  for (uint32_t k = 0; k < topo->n_comms; ++k) {
    if (topo->size[k] > SHORT_COMM) longs.push_back({k, topo->member_off[k], topo->size[k], 0});
    else while (c->short_lanes < topo->size[k]) c->short_lanes *= 2;
  }
  c->n_long_comms = (uint32_t)longs.size();
  up(c->long_comms, longs.data(), sizeof(LongComm) * longs.size());
  up(c->topo.rank_cell4, rp4.data(), 4ull * rp4.size());
  if (!fits_cell4) c->topo.rank_cell4 = nullptr;
  if (hipMemsetAsync(c->gstate, 0, sizeof(GroupState) * (uint64_t)topo->n_comms * GROUP_SLOTS, c->stream) != hipSuccess) rs = CCLD_E_HIP;
  if (hipMemsetAsync(c->batch_meta, 0, sizeof(BatchMeta) * ((uint64_t)c->p.window_batches + 2), c->stream) != hipSuccess) rs = CCLD_E_HIP;
  if (c->comm_range && hipMemsetAsync(c->comm_range, 0, 16ull * topo->n_comms * ((uint64_t)c->p.window_batches + 2), c->stream) != hipSuccess) rs = CCLD_E_HIP;
  if (hipMemsetAsync(c->counters, 0, sizeof(uint64_t) * CNT_COUNT, c->stream) != hipSuccess) rs = CCLD_E_HIP;
  if (hipMemsetAsync(c->h_counters, 0, sizeof(uint64_t) * (CNT_COUNT + HANG_REGIONS), c->stream) != hipSuccess) rs = CCLD_E_HIP;
  if (hipMemsetAsync(c->arrivals, 0, sizeof(uint32_t) * ARRIVAL_WORDS, c->stream) != hipSuccess) rs = CCLD_E_HIP;
  launch_fill_u64(c->stream, (uint64_t*)c->rate_root, topo->n_comms, (uint64_t)CCLD_NO_RANK);
  c->f_status = c->f_frame + topo->n_ranks;
  if (hipMemsetAsync(c->f_frame, 0, 8ull * ((uint64_t)topo->n_ranks + 1), c->stream) != hipSuccess) rs = CCLD_E_HIP;
  if (hipMemsetAsync(c->f_last, 0, sizeof(uint64_t) * 2 * CCLD_FRAME_CHANNELS * n_members, c->stream) != hipSuccess) rs = CCLD_E_HIP;
  if (hipMemsetAsync(c->blame, 0, sizeof(int64_t) * CCLD_BLM_NCOL * (uint64_t)topo->n_ranks, c->stream) != hipSuccess) rs = CCLD_E_HIP;
  {     // pinned words: the counters, the ticket and the fine buckets of a layout, then the headers of every batch slot
    const size_t bytes = std::max<size_t>(4096 * sizeof(uint64_t), (PINNED_META) * sizeof(uint64_t) + sizeof(BatchMeta) * ((size_t)c->p.window_batches + 2));
    if (hipHostMalloc((void**)&c->h_pinned, bytes, hipHostMallocDefault) != hipSuccess) rs = CCLD_E_HIP;
    else std::memset(c->h_pinned, 0, bytes);
  }
  if (ccld_device_init() != CCLD_OK) rs = CCLD_E_HIP;
  if (hipStreamSynchronize(c->stream) != hipSuccess) rs = CCLD_E_HIP;   // host vectors above die at return
  if (rs != CCLD_OK) {
    (void)hipGetLastError();
    if (c->h_pinned) (void)hipHostFree(c->h_pinned);
    delete c;
    return rs;
  }
  g_copy_streams.join(c->device);
  *out = c;
  return CCLD_OK;
}

ccld_status ccld_destroy(ccld_ctx* c) {
  if (!c) return CCLD_E_NULL;
  (void)hipStreamSynchronize(c->stream);
  g_copy_streams.leave(c->device);
  if (c->h_pinned) (void)hipHostFree(c->h_pinned);
  c->prof.destroy();
  delete c;
  return CCLD_OK;
}

ccld_status ccld_reset_window(ccld_ctx* c) {
  if (!c) return CCLD_E_NULL;
  c->head = 0; c->count = 0; c->batch_n.clear(); c->batch_slot.clear();
  c->inc_ok = false;
  c->chain_ready = false;
  return CCLD_OK;
}

ccld_status ccld_ingest(ccld_ctx* c, const ccld_records* b, uint64_t n) {
  if (!c || !b) return CCLD_E_NULL;
  if (n && (!b->rank || !b->comm || !b->seq || !b->op || !b->bytes || !b->t_enter || !b->t_exit)) return CCLD_E_NULL;
  if (n > c->batch_cap) return CCLD_E_CAPACITY;
  // drop the oldest batch once the window holds window_batches of them
  uint64_t head = c->head, count = c->count;
  size_t drop = 0;
  if (c->batch_n.size() >= c->p.window_batches) {
    drop = c->batch_n.size() - c->p.window_batches + 1;
    for (size_t i = 0; i < drop; ++i) { head = (head + c->batch_n[i]) % std::max<uint64_t>(c->cap, 1); count -= c->batch_n[i]; }
  }
  if (count + n > c->cap) return CCLD_E_CAPACITY;
  c->chain_ready = false;
  IngestArgs a;
  std::memset(&a, 0, sizeof(a));
  const uint32_t slot = c->next_slot;
  const uint32_t n_meta = c->p.window_batches + 2, next = (slot + 1) % n_meta;
  a.meta = c->batch_meta + slot; a.meta_next = c->batch_meta + next;
  if (b->on_device) {
    a.rank = b->rank; a.comm = b->comm; a.seq = b->seq; a.op = b->op; a.bytes = b->bytes;
    a.t_enter = b->t_enter; a.t_exit = b->t_exit;
  } else if (n) {
    // host batch: copy the seven columns into the staging area, 8-byte columns first
    uint8_t* s = c->stage;
    uint64_t* d_seq = (uint64_t*)s; uint64_t* d_bytes = d_seq + n; int64_t* d_te = (int64_t*)(d_bytes + n);
    int64_t* d_tx = d_te + n; uint32_t* d_rank = (uint32_t*)(d_tx + n); uint32_t* d_comm = d_rank + n;
    uint8_t* d_op = (uint8_t*)(d_comm + n);
    const HostCopy copies[] = {{d_seq, b->seq, 8 * n}, {d_bytes, b->bytes, 8 * n}, {d_te, b->t_enter, 8 * n}, {d_tx, b->t_exit, 8 * n},
                               {d_rank, b->rank, 4 * n}, {d_comm, b->comm, 4 * n}, {d_op, b->op, n}};
    HIP_TRY(copy_from_host(g_copy_streams, c->device, c->copy_earned, c->stream, copies, 7));
    a.rank = d_rank; a.comm = d_comm; a.seq = d_seq; a.op = d_op; a.bytes = d_bytes; a.t_enter = d_te; a.t_exit = d_tx;
  }
  a.n = n; a.win_key = c->win_key; a.win_row = c->win_row; a.win_wide = c->win_wide;
  a.tail = (uint32_t)((head + count) % std::max<uint64_t>(c->cap, 1));
  a.cap = (uint32_t)c->cap;
  a.table = c->ing_table; a.bucket_base = c->ing_base + (uint64_t)slot * (c->n_buckets + 1); a.scratch_total = &c->counters[CNT_COUNT - 1];
  a.n_buckets = c->n_buckets; a.bshift = c->bshift;
  uint64_t rounds_end = c->rounds_next;
  if (c->n_buckets > 1) {
    const IngestShape shape = ingest_shape(n);
    const uint64_t r = (uint64_t)shape.groups * shape.per_group, at = c->rounds_next + r <= c->rounds_cap ? c->rounds_next : 0;
    a.rounds = c->ing_rounds; a.round0 = (uint32_t)at;
    rounds_end = at + r;
  }
  if (c->grid_capable) {
    a.range = c->comm_range + (uint64_t)slot * c->topo.n_comms * 2;
    a.range_next = c->comm_range + (uint64_t)next * c->topo.n_comms * 2;
  }
  c->prof.begin(CCLD_PROF_INGEST);
  launch_ingest(c->stream, a, c->topo, c->kf);
  c->prof.end(CCLD_PROF_INGEST);
  HIP_TRY(hipGetLastError());
  if (!b->on_device && n) HIP_TRY(hipStreamSynchronize(c->stream));   // the host buffers may go away on return
  c->batch_n.erase(c->batch_n.begin(), c->batch_n.begin() + drop);
  c->batch_slot.erase(c->batch_slot.begin(), c->batch_slot.begin() + drop);
  c->batch_n.push_back(n);
  c->batch_slot.push_back(slot);
  c->rounds_next = rounds_end;
  c->next_slot = next;
  c->head = head; c->count = count + n;
  c->total_ingested += n;
  return CCLD_OK;
}

// Waits until the device has reported the counters of the current ticket into pinned memory.  The report is the last
// thing on the stream: what the caller asked for is in memory by then, although the reporting kernel may still be on its
// way out.  Spinning on the words costs about 10 us less than copying the counters with a queued copy and synchronising.
// A wait that takes long (a very large window, or a device error) ends in hipStreamSynchronize, as does every wait while
// spans are timed (their events must have completed).
static bool reported(const ccld_ctx* c, int words) {
  for (int i = 0; i < words; ++i)
    if (!report_arrived(__atomic_load_n(c->h_pinned + i, __ATOMIC_RELAXED), c->ticket)) return false;
  return true;
}
extern "C++" hipError_t wait_report(ccld_ctx* c, int words) {
  bool there = false;
  if (!c->prof.on) {
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t i = 1; !(there = reported(c, words)); ++i) {
      if ((i & 255) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(50)) break;
      __builtin_ia32_pause();
    }
  }
  if (!there) {
    const hipError_t e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return e;
    if (!reported(c, words)) return hipErrorUnknown;
  }
  for (int i = 0; i < words; ++i) c->h_pinned[i] = report_value(c->h_pinned[i]);
  return hipSuccess;
}

static void zero_counts(ccld_window_result* o) {
  o->n_records = o->n_seg = o->n_flag = o->n_group = o->n_alert = o->n_cand = 0;
}

// Waits for the number of fine buckets of a layout (a window large enough that launching for the most there could be
// would cost more than the wait): 0 = the layout is not feasible.  *full: there may be a record for every cell.
static hipError_t wait_fine(ccld_ctx* c, uint32_t* n_fine, bool* full) {
  const uint32_t* word = reinterpret_cast<const uint32_t*>(c->h_pinned + PINNED_FINE);
  const auto t0 = std::chrono::steady_clock::now();
  uint32_t v;
  for (uint32_t i = 1; (v = __atomic_load_n(word, __ATOMIC_ACQUIRE)) == 0; ++i) {
    if ((i & 255) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(50)) {
      const hipError_t e = hipStreamSynchronize(c->stream);
      if (e != hipSuccess) return e;
      if ((v = __atomic_load_n(word, __ATOMIC_ACQUIRE)) == 0) return hipErrorUnknown;
      break;
    }
    __builtin_ia32_pause();
  }
  *full = (v & GRID_FULL) != 0;
  *n_fine = (v & GRID_INFEASIBLE) ? 0u : (v & ~GRID_FULL) - 1;
  return hipSuccess;
}
// The last launches of an analysis: groups, flags (d and f: a window on the grid placement), blame order, report.
static void launch_end(ccld_ctx* c, EndArgs& e, const GridArgs* d, const FlagArgs* f, const AlertArgs* al, uint32_t fine) {
  e.counters = c->counters; e.blame = c->blame; e.n_ranks = c->topo.n_ranks; e.order = c->blame_order;
  e.arrivals = c->arrivals; e.host = c->h_pinned; e.ticket = c->ticket;
  if (!launch_window_end(c->stream, e, d, f, al, fine))
    launch_blame_order(c->stream, c->blame, c->topo.n_ranks, c->blame_list, c->blame_tiles, c->counters, c->arrivals, c->blame_order, c->h_pinned, c->ticket);
}

// Everything behind the statistics: what the last launch does, its report, and the alerts.  d, f and fine are those of a window
// on the grid placement.
static ccld_status finish_analysis(ccld_ctx* c, int64_t now_ns, ccld_window_result* o, const SegArgs& sa, const GridArgs* d, const FlagArgs* f,
                                   uint32_t fine, bool* fallback) {
  hipStream_t st = c->stream;
  const bool grid = d != nullptr;
  EndArgs e;
  std::memset(&e, 0, sizeof(e));
  e.seg = o->seg; e.seg_cap = o->seg_cap; e.gcode = c->gcode; e.range_c = c->range_c; e.n_comms = c->topo.n_comms;
  e.gstate = c->gstate; e.rate_root = c->rate_root; e.group = o->group; e.group_cap = o->group_cap; e.p = c->p;
  e.comm_groups = c->comm_groups; e.comm_row = c->comm_row;
  e.stage[0] = c->alert_list; e.stage[1] = c->alert_ncand; e.stage[2] = c->chain_parent;      // nothing lives there yet
  AlertArgs aa;
  std::memset(&aa, 0, sizeof(aa));
  aa.seg = o->seg; aa.seg_cap = o->seg_cap; aa.now_ns = now_ns;
  aa.hang_threshold_ns = c->p.hang_threshold_ns; aa.key = sa.key; aa.idx = sa.idx; aa.win = sa.win; aa.n = sa.n;
  if (grid) {
    aa.grid.lay = (const CommLayout*)c->g_lay; aa.grid.rows = c->g_rows; aa.grid.cell_row = c->g_cell_row; aa.grid.wide = c->win_wide;
    aa.grid.hdr = (const GridHeader*)c->g_hdr;
  }
  aa.sf = c->sf; aa.topo = c->topo; aa.tile_counts = c->tile_heads; aa.alert_list = c->alert_rows;
  aa.alert_ncand = c->alert_ncand; aa.alert = o->alert; aa.alert_cap = o->alert_cap; aa.cand = o->cand;
  aa.cand_cap = o->cand_cap; aa.counters = c->counters;
  launch_end(c, e, d, f, c->max_comm_size <= END_ALERT_MEMBERS ? &aa : nullptr, fine);
  c->prof.end(CCLD_PROF_GROUPS);
  HIP_TRY(hipGetLastError());
  HIP_TRY(wait_report(c));
  if (c->h_pinned[CNT_STATUS]) {
    const uint64_t bad = c->h_pinned[CNT_STATUS];
    c->prof.collect();
    zero_counts(o);
    if (grid && (bad & DS_DENSE_FALLBACK)) { *fallback = true; return CCLD_OK; }
    return o->status = data_status(bad);
  }
  o->n_seg = c->h_pinned[CNT_NSEG];
  o->n_flag = c->h_pinned[CNT_NFLAG];
  o->n_alert = c->h_pinned[CNT_NALERT];
  o->n_group = c->h_pinned[CNT_NGROUP];
  if (o->n_seg > o->seg_cap || o->n_flag > o->flag_cap || o->n_group > o->group_cap) o->status = CCLD_W_TRUNCATED;

  // hang alerts: the collectives that raise one in table order, and the candidates of every alert; a few are listed already
  if (o->n_alert > END_ALERTS || (o->n_alert && c->max_comm_size > END_ALERT_MEMBERS)) {
    aa.n_seg = (uint32_t)std::min<uint64_t>(o->n_seg, o->seg_cap); aa.alert_list = c->alert_list;
    c->prof.begin(CCLD_PROF_ALERTS);
    launch_alert_select(st, aa);
    launch_alert_candidates(st, aa, (uint32_t)o->n_alert);
    c->prof.end(CCLD_PROF_ALERTS);
    launch_report(st, c->counters, c->h_pinned, take_ticket(c));
    HIP_TRY(hipGetLastError());
    HIP_TRY(wait_report(c));
  }
  o->n_cand = o->n_alert ? c->h_pinned[CNT_NCAND] : 0;
  if (o->n_alert > o->alert_cap || o->n_cand > o->cand_cap) o->status = CCLD_W_TRUNCATED;
  c->prof.collect();
  c->blame_valid = true;
  c->chain_ready = true;
  c->last_seg = o->seg; c->last_seg_cap = o->seg_cap; c->last_n_seg = o->n_seg; c->last_n_flag = o->n_flag;
  c->last_rec_flag = sa.rec_flag; c->last_grid = grid; c->last_win = sa.win;
  return o->status;
}

// what the statistics kernels of both placements share
static SegArgs seg_args(ccld_ctx* c, int64_t now_ns, const ccld_window_result* o, uint32_t n) {
  SegArgs sa;
  std::memset(&sa, 0, sizeof(sa));
  sa.n = n; sa.comm_size = c->topo.size;
  sa.member_off = c->topo.member_off; sa.members_sorted = c->topo.members_sorted; sa.comm_info = c->comm_info;
  sa.seg = o->seg; sa.seg_cap = o->seg_cap;
  sa.lag_e = o->lag_enter; sa.lag_x = o->lag_exit; sa.flag_lag = c->flag_lag; sa.cap_n = c->cap;
  sa.counters = c->counters; sa.alert_rows = c->alert_rows;
  sa.lag_floor = c->p.lag_floor_ns; sa.kmad_num = c->p.kmad_num; sa.kmad_den = c->p.kmad_den;
  sa.barrier_bytes = c->p.barrier_bytes; sa.now_ns = now_ns; sa.hang_threshold_ns = c->p.hang_threshold_ns; sa.max_size = c->max_comm_size; sa.long_classes = c->long_classes;
  sa.gcode = c->gcode; sa.range_c = c->range_c;
  const uint32_t n_meta = c->p.window_batches + 2;
  sa.win.row = c->win_row; sa.win.wide = c->win_wide; sa.win.meta = c->batch_meta; sa.win.n_meta = n_meta;
  sa.win.n_batch = (uint32_t)c->batch_slot.size(); sa.win.slot0 = c->batch_slot.empty() ? 0 : c->batch_slot[0];
  sa.win.head = (uint32_t)c->head; sa.win.cap = (uint32_t)std::max<uint64_t>(c->cap, 1);
  sa.win.bucket_base = c->ing_base; sa.win.rounds = c->n_buckets > 1 ? c->ing_rounds : nullptr; sa.win.n_buckets = c->n_buckets;
  return sa;
}

// One analysis of the resident window on the grid placement.  Nothing waits for the host before the end, unless the window
// is large enough to ask for its number of fine buckets.  *fallback is set (and nothing of the context's detection state
// has changed) when the window turns out not to fill a grid; the caller then sorts.
static ccld_status analyze_on_grid(ccld_ctx* c, int64_t now_ns, ccld_window_result* o, bool* fallback) {
  hipStream_t st = c->stream;
  const uint32_t n = (uint32_t)c->count, n_ranks = c->topo.n_ranks;
  o->path = c->dense_asked ? 1 : 0;
  o->n_records = n;
  SegArgs sa = seg_args(c, now_ns, o, n);
  sa.rec_flag = o->rec_flag; sa.perm = o->perm; sa.flag_pos = c->flag_stage;
  GridArgs d;
  std::memset(&d, 0, sizeof(d));
  d.win_key = c->win_key; d.win_row = c->win_row; d.head = sa.win.head; d.cap = sa.win.cap; d.n = n;
  d.meta = c->batch_meta; d.n_meta = sa.win.n_meta; d.slot0 = sa.win.slot0; d.nb = sa.win.n_batch;
  d.kf = c->kf; d.comm_size = c->topo.size; d.n_comms = c->topo.n_comms;
  d.bucket_base = c->ing_base; d.n_buckets = c->n_buckets; d.bshift = c->bshift; d.range = c->comm_range;
  d.lay = (CommLayout*)c->g_lay; d.hdr = (GridHeader*)c->g_hdr; d.piece_at = c->g_piece_at; d.piece_slot = c->g_piece_slot;
  d.fill = c->g_fill; d.rec0 = c->g_rec0; d.nflag = c->g_nflag; d.desc = (FineDesc*)c->g_desc; d.long_list = c->g_long;
  // cells that this window may take, and the fine buckets that they can make
  d.cell_cap = (uint32_t)std::min<uint64_t>(c->cell_cap, (c->cap >= (4u << 20) ? (uint64_t)n + n / 5 : 2ull * n) + 4096);
  d.fine_cap = std::min(c->fine_cap, d.cell_cap / GRID_MIN_FILL + c->topo.n_comms);
  d.likely = n / GRID_B + c->topo.n_comms / 2;
  d.self_sum = d.likely <= GRID_SELF_SUM && d.fine_cap <= GRID_FINE_BOUND;
  d.lines = grid_in_lines(n, o->perm != nullptr);
  d.rows = c->g_rows; d.slots = o->perm ? c->g_slots : nullptr;
  d.cell_row = c->g_cell_row; d.counters = c->counters;
  d.blame = (uint64_t*)c->blame; d.n_blame = CCLD_BLM_NCOL * n_ranks;
  d.host_fine = reinterpret_cast<uint32_t*>(c->h_pinned + PINNED_FINE);
  *d.host_fine = 0;
  c->prof.begin(CCLD_PROF_DENSE_PARTITION);
  launch_grid_layout(st, d);
  launch_grid_partition(st, d);
  c->prof.split(CCLD_PROF_DENSE_PARTITION, CCLD_PROF_SEGMENTS);
  c->sort_passes = 1;
  uint32_t fine = d.fine_cap;
  if (fine > GRID_FINE_BOUND) {
    HIP_TRY(hipGetLastError());
    bool full;
    HIP_TRY(wait_fine(c, &fine, &full));
    if (fine && !full) launch_grid_gaps(st, d, fine);
  }
  if (fine) launch_grid_stats(st, sa, d, fine, c->blame, n_ranks);
  c->prof.split(CCLD_PROF_SEGMENTS, CCLD_PROF_GROUPS);
  FlagArgs fa;
  std::memset(&fa, 0, sizeof(fa));
  fa.flag_lag = c->flag_lag; fa.cap_n = c->cap; fa.n = n; fa.member_off = c->topo.member_off; fa.members_sorted = c->topo.members_sorted;
  fa.flag_pos = c->flag_pos; fa.flag_key = c->flag_key; fa.flag_stage = c->flag_stage; fa.flag = o->flag; fa.flag_cap = o->flag_cap;
  fa.counters = c->counters;
  return finish_analysis(c, now_ns, o, sa, &d, &fa, fine, fallback);
}

// The order of a window that still holds at least half of the one that was sorted last: the new records are sorted on their
// own and merged with that order, whose keys are re-based to this window's format and whose entries of the batches that
// left are dropped on the way.  Half the time of sorting a window of ten batches again (20M records at 16,384 ranks in
// 5,184 communicators: 0.25 instead of 0.49 ms, a step 1.18 instead of 1.49).  Returns the buffer of the result, -1 for a
// failed launch, -2 where there is no such order.
static int merge_new_records(ccld_ctx* c, const KeySource& src, uint32_t n) {
  const uint64_t cap = std::max<uint64_t>(c->cap, 1), n_new = c->total_ingested - c->inc_total;
  const int bits = src.lo_bits + c->kf.cb;
  if (!c->inc_ok || n_new == 0 || n_new >= n || bits > 64 || src.lo_bits >= 64 || c->inc_sf.mb != c->sf.mb || c->inc_sf.mb + c->inc_sf.ws >= 64)
    return -2;
  const uint64_t kept = n - n_new, old_tail = (c->inc_head + c->inc_count) % cap;       // kept: records of that window still here
  if (kept < n_new || kept > c->inc_count) return -2;
  const uint64_t exp_n = c->inc_count - kept;
  if ((c->inc_head + exp_n) % cap != c->head || (old_tail + n_new) % cap != (c->head + n) % cap) return -2;
  // the new records end in a third pair of buffers (a sort of p passes ends in its buffer (p - 1) % 2), so that the merge can
  // read the kept order where it lies and write beside it; flag_pos is written by the flags, later
  const int s = c->sorted_buf, passes = bits <= 0 ? 1 : (bits + SORT_RBITS - 1) / SORT_RBITS, third = (passes - 1) % 2;
  SortBuffers fresh;
  fresh.key[third] = c->keyC; fresh.idx[third] = c->flag_pos;
  fresh.key[1 - third] = c->sb.key[1 - s]; fresh.idx[1 - third] = c->sb.idx[1 - s];
  fresh.table = c->table2; fresh.totals = c->totals2;
  KeySource from = src;
  from.head = (uint32_t)old_tail;
  const int r = radix_sort_pairs(c->stream, from, (uint32_t)n_new, fresh, bits, &c->prof, CCLD_PROF_SORT_HIST, CCLD_PROF_SORT_SCAN,
                                 CCLD_PROF_SORT_SCATTER);
  if (r < 0) return -1;
  if (r != third &&       // few records are sorted in one launch, whose result may be in the other pair
      (hipMemcpyAsync(c->keyC, fresh.key[r], sizeof(uint64_t) * n_new, hipMemcpyDeviceToDevice, c->stream) != hipSuccess ||
       hipMemcpyAsync(c->flag_pos, fresh.idx[r], sizeof(uint32_t) * n_new, hipMemcpyDeviceToDevice, c->stream) != hipSuccess))
    return -1;
  c->prof.begin(CCLD_PROF_SORT_SCATTER);
  RetainArgs ra;
  ra.key = c->sb.key[s]; ra.idx = c->sb.idx[s]; ra.n = (uint32_t)c->inc_count; ra.from = c->inc_sf; ra.to = c->sf;
  ra.exp_lo = (uint32_t)c->inc_head; ra.exp_n = (uint32_t)exp_n; ra.cap = (uint32_t)cap;
  ra.tile_counts = c->tile_flags; ra.total_out = &c->counters[CNT_COUNT - 1];
  ra.key_out = c->sb.key[1 - s]; ra.idx_out = c->sb.idx[1 - s];
  launch_merge_kept(c->stream, ra, c->keyC, c->flag_pos, (uint32_t)n_new, c->tile_heads);
  c->prof.end(CCLD_PROF_SORT_SCATTER);
  return 1 - s;
}

// One analysis of the resident window by sorting it.
static ccld_status analyze_sorted(ccld_ctx* c, int64_t now_ns, ccld_window_result* o) {
  hipStream_t st = c->stream;
  const uint32_t n = (uint32_t)c->count, n_ranks = c->topo.n_ranks;
  o->path = 0;
  // 1. data errors found at ingest, and the range of the operation counters in the window
  SegArgs sa = seg_args(c, now_ns, o, n);
  uint64_t bits = 0, max_seq = 0, min_seq = ~0ull;
  if (!c->batch_slot.empty()) {
    BatchMeta* hm = (BatchMeta*)(c->h_pinned + PINNED_META);
    HIP_TRY(hipMemcpyAsync(hm, c->batch_meta, sizeof(BatchMeta) * sa.win.n_meta, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    bool first = true;
    for (uint32_t slot : c->batch_slot) {
      const BatchMeta& m = hm[slot];
      bits |= m.status;
      if (m.n == 0) continue;
      max_seq = std::max(max_seq, m.max_seq); min_seq = std::min(min_seq, ~m.max_inv_seq);
      if (first) { sa.win.ref = m.ref; first = false; }
      else if ((((uint64_t)m.ref - (uint64_t)sa.win.ref + (1ull << 42)) >> 43) != 0) sa.win.far = 1;
    }
  }
  if (bits) return o->status = data_status(bits);
  o->n_records = n;
  HIP_TRY(hipMemsetAsync(c->counters, 0, sizeof(uint64_t) * CNT_COUNT, st));
  HIP_TRY(hipMemsetAsync(c->blame, 0, sizeof(int64_t) * CCLD_BLM_NCOL * (uint64_t)n_ranks, st));
  take_ticket(c);
  // 2. sort by (communicator, operation counter, rank) on the significant bits only, the operation counters relative to
  //    the smallest one of the window
  if (min_seq > max_seq) min_seq = max_seq;
  const int mb = c->kf.mb, cb = c->kf.cb, ws = bits_for(max_seq - min_seq);
  c->sf.mb = mb; c->sf.ws = ws; c->sf.seq_base = min_seq;
  KeySource src;
  src.key = c->win_key; src.head = sa.win.head; src.cap = sa.win.cap;
  src.squeeze = 1;
  src.hi_shift = 64 - cb;                                  // 64 when there is a single communicator
  src.lo_bits = mb + ws;
  src.lo_mask = cb > 0 ? (((uint64_t)1 << (64 - cb)) - 1) : ~0ull;      // everything below the communicator field
  src.lo_sub = min_seq << mb;
  int sorted = merge_new_records(c, src, n);
  c->inc_ok = false;
  if (sorted == -2)
    sorted = radix_sort_pairs(st, src, n, c->sb, mb + ws + cb, &c->prof, CCLD_PROF_SORT_HIST, CCLD_PROF_SORT_SCAN, CCLD_PROF_SORT_SCATTER);
  c->sort_passes = (mb + ws + cb) <= 0 ? 1 : (mb + ws + cb + SORT_RBITS - 1) / SORT_RBITS;
  if (sorted < 0) return o->status = CCLD_E_HIP;
  c->sorted_buf = sorted;

  // 3. collectives: heads per tile, their scan, statistics, flags
  sa.key = c->sb.key[sorted]; sa.idx = c->sb.idx[sorted]; sa.sf = c->sf;
  sa.tile_heads = c->tile_heads; sa.rec_flag = o->rec_flag ? o->rec_flag : c->rec_flag;
  sa.big_list = c->big_list; sa.big_cap = c->cap / 65 + 2;
  sa.big_e = reinterpret_cast<int64_t*>(c->sb.key[1 - sorted]); sa.big_x = reinterpret_cast<int64_t*>(c->keyC);
  const uint32_t seg_tiles = (n + SEG_TILE - 1) / SEG_TILE;
  c->prof.begin(CCLD_PROF_SEG_HEADS);
  launch_keys_pass(st, sa.key, n, c->sf, c->topo, c->blame, c->tile_heads, c->counters);
  launch_scan_tiles(st, c->tile_heads, seg_tiles, &c->counters[CNT_NSEG]);
  c->prof.split(CCLD_PROF_SEG_HEADS, CCLD_PROF_SEGMENTS);          // one event ends a timed span and begins the next
  launch_seg_analyze(st, sa);
  c->prof.split(CCLD_PROF_SEGMENTS, CCLD_PROF_FLAGS);
  FlagArgs fa;
  std::memset(&fa, 0, sizeof(fa));
  fa.key = sa.key; fa.rec_flag = sa.rec_flag; fa.flag_lag = c->flag_lag; fa.cap_n = c->cap; fa.n = n; fa.sf = c->sf;
  fa.member_off = c->topo.member_off; fa.members_sorted = c->topo.members_sorted;
  fa.tile_flags = c->tile_flags; fa.flag_pos = c->flag_pos; fa.flag = o->flag; fa.flag_cap = o->flag_cap;
  fa.counters = c->counters;
  launch_flag_compact(st, fa);
  if (o->perm) launch_perm(st, sa.idx, sa.win, n, o->perm);
  // 4. per-rank blame
  c->prof.split(CCLD_PROF_FLAGS, CCLD_PROF_BLAME);
  launch_blame_sums(st, fa, n_ranks, c->blame);
  c->prof.split(CCLD_PROF_BLAME, CCLD_PROF_GROUPS);
  bool fallback = false;
  const ccld_status s = finish_analysis(c, now_ns, o, sa, nullptr, nullptr, 0, &fallback);
  // the order serves the next analysis (windows of several batches only)
  c->inc_ok = s >= 0 && c->p.window_batches > 1;
  c->inc_sf = c->sf; c->inc_head = c->head; c->inc_count = n; c->inc_total = c->total_ingested;
  return s;
}

// a window without records: an all-zero blame table and the ranks in ascending order
static ccld_status analyze_empty(ccld_ctx* c, ccld_window_result* o) {
  hipStream_t st = c->stream;
  const uint32_t n_ranks = c->topo.n_ranks;
  HIP_TRY(hipMemsetAsync(c->counters, 0, sizeof(uint64_t) * CNT_COUNT, st));
  HIP_TRY(hipMemsetAsync(c->blame, 0, sizeof(int64_t) * CCLD_BLM_NCOL * (uint64_t)n_ranks, st));
  take_ticket(c);
  launch_window_empty(st, n_ranks, c->blame_order, c->counters, c->arrivals, c->h_pinned, c->ticket);
  HIP_TRY(hipGetLastError());
  HIP_TRY(wait_report(c));
  c->blame_valid = true;
  return o->status;
}

ccld_status ccld_analyze_window(ccld_ctx* c, int64_t now_ns, ccld_window_result* o) {
  if (!c || !o) return CCLD_E_NULL;
  zero_counts(o);
  o->status = CCLD_OK;
  o->path = 0;
  c->chain_ready = false;
  c->blame_valid = false;
  if (!o->seg || o->seg_cap == 0) return o->status = CCLD_E_NULL;
  if ((o->flag_cap && !o->flag) || (o->group_cap && !o->group) || (o->alert_cap && !o->alert) ||
      (o->cand_cap && !o->cand))
    return o->status = CCLD_E_NULL;
  ccld_status s = CCLD_OK;
  if (c->count == 0) {
    s = analyze_empty(c, o);
  } else {
    bool fallback = !c->grid_capable;
    if (c->grid_capable) {
      take_ticket(c);
      c->inc_ok = false;       // the grid's rows lie where the order is kept
      s = analyze_on_grid(c, now_ns, o, &fallback);
    }
    if (s >= 0 && fallback) s = analyze_sorted(c, now_ns, o);
  }
  if (s < 0) {       // an error return may have left work queued and timed spans open
    (void)hipStreamSynchronize(c->stream);
    (void)hipGetLastError();
    c->prof.abandon();
    c->inc_ok = false;
  }
  return s;
}

ccld_status ccld_rank_blame(ccld_ctx* c, int64_t* blame, uint32_t* order) {
  if (!c) return CCLD_E_NULL;
  if (!c->blame_valid) return CCLD_E_BAD_ARG;
  const uint32_t n_ranks = c->topo.n_ranks;
  launch_blame_out(c->stream, c->blame, c->blame_order, n_ranks, blame, order, c->counters, c->arrivals, c->h_pinned, take_ticket(c));
  HIP_TRY(hipGetLastError());
  HIP_TRY(wait_report(c));
  return CCLD_OK;
}

ccld_status ccld_profile_enable(ccld_ctx* c, int32_t on) {
  if (!c) return CCLD_E_NULL;
  HIP_TRY(hipStreamSynchronize(c->stream));
  if (on < 0 || on >= 2 + CCLD_PROF_NCLASS) return CCLD_E_BAD_ARG;
  return c->prof.enable(c->stream, on != 0, on >= 2 ? on - 2 : -1) ? CCLD_OK : CCLD_E_HIP;
}

ccld_status ccld_profile_read(ccld_ctx* c, double* ms, uint64_t* launches, uint64_t* sort_passes) {
  if (!c) return CCLD_E_NULL;
  HIP_TRY(hipStreamSynchronize(c->stream));
  c->prof.collect();
  for (int i = 0; i < CCLD_PROF_NCLASS; ++i) {
    if (ms) ms[i] = c->prof.ms[i];
    if (launches) launches[i] = c->prof.cnt[i];
  }
  if (sort_passes) *sort_passes = (uint64_t)c->sort_passes;
  return CCLD_OK;
}

const char* ccld_status_str(ccld_status s) {
  switch (s) {
    case CCLD_OK: return "OK";
    case CCLD_E_UNKNOWN_COMM: return "E_UNKNOWN_COMM";
    case CCLD_E_RANK_NOT_MEMBER: return "E_RANK_NOT_MEMBER";
    case CCLD_E_RANGE: return "E_RANGE";
    case CCLD_E_DUPLICATE_KEY: return "E_DUPLICATE_KEY";
    case CCLD_E_SNAPSHOT_GAP: return "E_SNAPSHOT_GAP";
    case CCLD_E_BAD_ARG: return "E_BAD_ARG";
    case CCLD_E_NULL: return "E_NULL";
    case CCLD_E_CAPACITY: return "E_CAPACITY";
    case CCLD_E_KEY_WIDTH: return "E_KEY_WIDTH";
    case CCLD_E_BAD_TOPOLOGY: return "E_BAD_TOPOLOGY";
    case CCLD_E_HIP: return "E_HIP";
    case CCLD_E_WORKSPACE: return "E_WORKSPACE";
    case CCLD_W_TRUNCATED: return "W_TRUNCATED";
    default: return "E_UNKNOWN";
  }
}

}  // extern "C"
