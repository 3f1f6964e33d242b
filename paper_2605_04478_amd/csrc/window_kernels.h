// Host-callable launchers of the window-analysis kernels (defined in window.hip).
#pragma once
#include "ccld_internal.h"

namespace ccld {

struct IngestArgs {
  const uint32_t *rank, *comm;
  const uint64_t* seq;
  const uint8_t* op;
  const uint64_t* bytes;
  const int64_t *t_enter, *t_exit;
  uint64_t n;
  uint64_t* win_key;
  uint4* win_row;
  int64_t* win_wide;         // [cap][3]
  uint32_t tail, cap;
  BatchMeta *meta, *meta_next;   // this batch's header and the one that the next batch will use
  uint32_t* table;           // [n_buckets][workgroups] records per communicator bucket and workgroup
  uint32_t* bucket_base;     // [n_buckets + 1] of this batch
  uint32_t table_words;      // words of the table
  uint64_t* scratch_total;
  uint32_t n_buckets;
  int bshift;                // bucket = comm >> bshift
  uint32_t* rounds;          // [rounds][n_buckets] of the window's batches; this batch's start at round0
  uint32_t round0;
  uint64_t *range, *range_next;  // [n_comms][2] per communicator: largest operation counter, largest complement of one; null:
                             // not wanted.  At most INGEST_RANGE_COMMS communicators.
  uint64_t chunk;            // records per placement workgroup (a multiple of 256 * hist_split)
  uint32_t hist_split;       // counting workgroups per placement workgroup
  uint32_t per_group;        // rounds per placement workgroup
};
// How a batch that is placed by bucket is dealt out: workgroups, records and rounds of each, counting workgroups per workgroup
struct IngestShape { uint32_t groups, per_group, hist_split; uint64_t chunk; };
IngestShape ingest_shape(uint64_t n);
constexpr uint32_t INGEST_BLOCKS = 1024;
void launch_ingest(hipStream_t st, const IngestArgs& a, const DeviceTopology& T, const KeyFormat& kf);
void launch_fill_u64(hipStream_t st, uint64_t* p, uint64_t n, uint64_t v);

constexpr uint32_t NO_GROUP = 0xFFFFu;
constexpr uint32_t END_ALERTS = 8;                // most hang alerts that k_window_lists lists, a wavefront each ...
constexpr uint32_t END_ALERT_MEMBERS = 2048;      // ... where no communicator has more members
struct SegArgs {
  const uint64_t* key;       // sorted squeezed keys
  const uint32_t* idx;       // window slot of each sorted record
  WindowRows win;
  uint32_t n;
  SqueezedFormat sf;
  const uint32_t* comm_size;
  const uint32_t *member_off, *members_sorted;   // key slot -> rank
  const uint2* comm_info;    // [n_comms] (member_off, comm_size) side by side
  uint32_t* tile_heads;      // [tiles + 1] head counts, then (after the scan) first segment ordinal of each tile
  int64_t* seg;
  uint64_t seg_cap;
  uint8_t* rec_flag;         // (optional on the grid placement)
  int64_t *lag_e, *lag_x;    // optional per-record outputs
  uint32_t* perm;            // optional, grid placement only (a sorted window's comes from launch_perm)
  int64_t* flag_lag;         // [2][cap_n] lags of flagged records: by sorted position; on the grid placement with flag_pos
  uint32_t* flag_pos;        // grid placement: cell | kind << 16 of the flagged records of each fine bucket
  uint64_t cap_n;
  uint32_t* big_list;
  uint64_t big_cap;          // entries the list holds
  int64_t *big_e, *big_x;    // [cap_n] each: times of the collectives that do not fit LDS
  uint64_t* counters;
  int64_t lag_floor;
  uint32_t kmad_num, kmad_den, barrier_bytes;
  int64_t now_ns, hang_threshold_ns;             // collectives in flight for longer are counted in counters[CNT_NALERT]
  uint32_t* alert_rows;      // [END_ALERTS] rows of the first ones, in any order
  uint32_t max_size;         // members of the largest communicator (host-side: which size classes can occur)
  uint32_t long_classes;     // which there are: bit 0 65 to 128 members, 1 up to 256, 2 up to 512, 3 more
  // (op, size class) code and T_max - T_min of every collective, for the group stage; a collective that takes
  // no part gets NO_GROUP
  uint16_t* gcode;
  int64_t* range_c;
};
void launch_scan_tiles(hipStream_t st, uint32_t* counts, uint32_t n_tiles, uint64_t* total_out);
void launch_seg_analyze(hipStream_t st, const SegArgs& a);        // small collectives, then the oversized ones

struct FlagArgs {
  const uint64_t* key;
  const uint8_t* rec_flag;
  const int64_t* flag_lag;
  uint64_t cap_n;
  uint32_t n;
  SqueezedFormat sf;
  const uint32_t *member_off, *members_sorted;
  uint32_t* tile_flags;      // [tiles + 1]
  uint32_t* flag_pos;        // list: sorted position of each flagged record; on the grid placement its place in flag_stage
  uint64_t* flag_key;        // grid placement, list: row of the collective table << 32 | member slot
  const uint32_t* flag_stage;// grid placement: what the statistics kernels collected, cell | kind << 16
  int64_t* flag;             // caller's table (may be NULL)
  uint64_t flag_cap;
  uint64_t* counters;
};
void launch_flag_compact(hipStream_t st, const FlagArgs& a);

// one pass over the sorted keys: collective heads per tile (tile_heads), duplicates (status counter),
// records per rank (added into the zeroed records column of blame)
void launch_keys_pass(hipStream_t st, const uint64_t* key, uint32_t n, const SqueezedFormat& sf,
                      const DeviceTopology& T, int64_t* blame, uint32_t* tile_heads, uint64_t* counters);
// adds the flag list (its length is read from the counters) to the late columns of the blame table
void launch_blame_sums(hipStream_t st, const FlagArgs& f, uint32_t n_ranks, int64_t* blame);
// order[] = ranks by (flags, summed lag, rank); then the counters are reported to host_counters (pinned host memory), each
// word with `ticket`: the last words of an analysis of more than END_ORDER_RANKS ranks
void launch_blame_order(hipStream_t st, const int64_t* blame, uint32_t n_ranks, uint32_t* lists,
                        uint32_t* tile_counts, uint64_t* counters, uint32_t* arrivals, uint32_t* order, uint64_t* host_counters,
                        uint64_t ticket);

// The end of an analysis (groups.hip)
struct EndArgs {
  const int64_t* seg;        // collective table; its row count is read from counters[CNT_NSEG]
  uint64_t seg_cap;
  uint64_t* counters;
  const uint16_t* gcode;     // [rows] op * GROUP_CLS + size class of each usable collective, NO_GROUP of the others
  const int64_t* range_c;    // [rows] T_max - T_min (written with the collectives' statistics)
  uint32_t n_comms;
  uint32_t* comm_groups;     // [n_comms + 1] groups of each communicator
  uint32_t* comm_row;        // [n_comms] its first row of the table
  uint32_t* stage[3];        // [rows] what k_window_lists leaves for k_window_end
  GroupState* gstate;
  const int64_t* rate_root;  // [n_comms] minimal-rate member per communicator (CCLD_NO_RANK before any rate pass)
  int64_t* group;
  uint64_t group_cap;
  ccld_params p;
  // blame order
  const int64_t* blame;
  uint32_t n_ranks;
  uint32_t* order;
  uint32_t flags_scanned;    // the flags per fine bucket were scanned before
  uint32_t* arrivals;
  uint64_t* host;            // pinned words of the report
  uint64_t ticket;
};
constexpr uint32_t END_ORDER_RANKS = 16384;       // most ranks whose blame order k_window_lists finds
// a window without records: its blame order and the report
void launch_window_empty(hipStream_t st, uint32_t n_ranks, uint32_t* order, uint64_t* counters, uint32_t* arrivals, uint64_t* host, uint64_t ticket);
void launch_report(hipStream_t st, const uint64_t* counters, uint64_t* host, uint64_t ticket);
void launch_blame_out(hipStream_t st, const int64_t* blame, const uint32_t* order_in, uint32_t n_ranks, int64_t* table_out,
                      uint32_t* order_out, uint64_t* counters, uint32_t* arrivals, uint64_t* host, uint64_t ticket);

struct CommLayout;
struct GridHeader;
// What the chains and the alerts need of a window on the grid placement (grid.h).
struct GridView {
  const CommLayout* lay;
  const uint4* rows;         // partitioned rows
  const uint16_t* cell_row;  // row of every cell inside its fine bucket
  const int64_t* wide;
  const GridHeader* hdr;
};

struct AlertArgs {
  const int64_t* seg;
  uint64_t seg_cap;
  uint32_t n_seg;
  int64_t now_ns, hang_threshold_ns;
  const uint64_t* key;
  const uint32_t* idx;
  WindowRows win;
  uint32_t n;
  SqueezedFormat sf;
  GridView grid;             // lay is null for a sorted window
  DeviceTopology topo;
  uint32_t* tile_counts;
  uint32_t* alert_list;      // rows of the collectives that raise one: ascending; for k_window_lists in any order
  uint32_t* alert_ncand;
  int64_t* alert;
  uint64_t alert_cap;
  int64_t* cand;
  uint64_t cand_cap;
  uint64_t* counters;
};
void launch_alert_select(hipStream_t st, const AlertArgs& a);
void launch_alert_candidates(hipStream_t st, const AlertArgs& a, uint32_t n_alert);

void launch_perm(hipStream_t st, const uint32_t* idx, const WindowRows& win, uint32_t n, uint32_t* perm);

}  // namespace ccld
