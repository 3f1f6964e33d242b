// Context layout and kernel-launcher declarations shared by the translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <vector>

#include "ccld.h"
#include "buckets.h"
#include "radix_sort.h"
#include "profiler.h"
#include "ticket.h"

namespace ccld {

// Key layout at ingest: comm << (64 - cb) | seq << mb | slot.  slot is the record's rank counted
// among its communicator's members in ascending rank order, so keys order like (comm, seq, rank)
// while the field needs only as many bits as the largest communicator has members; mb / cb are
// the bit widths of the largest slot / communicator id.  The sort squeezes the unused middle bits out.
struct KeyFormat {
  int mb, cb;          // member-slot bits, communicator bits
  int sb;              // bits available to the sequence number: 64 - mb - cb
};

// Squeezed key used from the sort onwards: comm << (mb + ws) | (seq - seq_base) << mb | slot, with
// seq_base the window's smallest operation counter: a long-running job's large counters do not
// widen the key.
struct SqueezedFormat {
  int mb, ws;          // member-slot bits, bits of (largest - smallest operation counter) in this window
  uint64_t seq_base;   // the window's smallest operation counter
};

struct DeviceTopology {
  uint32_t n_ranks, n_comms;
  const uint8_t* algo;
  const uint32_t* size;
  const uint32_t* member_off;
  const uint32_t* members;
  const uint32_t* members_sorted;   // each communicator's members in ascending rank order
  const uint32_t* sorted_slot;      // slot (position in members[]) of each entry of members_sorted
  const int32_t* tree_parent;
  const uint32_t* rank_comm_off;    // [n_ranks + 1] CSR: communicators each rank belongs to
  const uint32_t* rank_comms;
  const uint32_t* rank_slots;       // parallel to rank_comms: the rank's position in members_sorted of that communicator
  const uint32_t* rank_memb4;       // [n_ranks][4] words comm << mb | position (padded with 0xFFFFFFFF); null if a rank is in more than four communicators or cb + mb > 31
  const uint32_t* rank_cell4;       // [n_ranks][4] words comm << pb | member index (member_off[comm] + slot in members[]), padded alike; null if a rank is in more than four communicators or cb + pb > 31
  int pb;                           // bits of the largest member index
  const uint32_t* member_comm;      // [members] communicator of every member slot
};

// rank of the record whose key carries (comm, slot)
__device__ __forceinline__ uint32_t rank_of_slot(const uint32_t* __restrict__ member_off,
                                                 const uint32_t* __restrict__ members_sorted, uint32_t comm,
                                                 uint32_t slot) {
  return members_sorted[member_off[comm] + slot];
}

// Eq. 1 state and repetition counter of one detection group (communicator, op, size class).
struct GroupState {
  uint32_t cnt, frozen, repeats, pad;
  int64_t sum, t0, tbase_dyn;
  uint64_t baselined_wm, baseline_last_seq, detected_wm;
};
constexpr int GROUP_CLS = 64;
constexpr int GROUP_SLOTS = CCLD_OP_MAX * GROUP_CLS;

// status bits accumulated on the device
enum { DS_UNKNOWN_COMM = 1, DS_NOT_MEMBER = 2, DS_RANGE = 4, DS_KEY_WIDTH = 8, DS_DUPLICATE = 16,
       DS_SNAPSHOT_GAP = 32,
       DS_SUSPECT = 64,     // snapshot grid placed without the presence bitmap: a cell still holds the fill pattern
       DS_DENSE_FALLBACK = 128 };   // the window does not fill a dense grid (far-apart counters, a round without any record): sort instead

// device-side header of a batch: status bits, largest operation counter and largest complement of one (i.e.
// ~smallest counter), so that a zeroed header means "no record yet"; the time its rows are relative to, its first
// window slot and its records
struct BatchMeta {
  uint64_t status; uint64_t max_seq; uint64_t max_inv_seq; int64_t ref; uint64_t tail; uint64_t n;
  // a batch placed by bucket: records per placement workgroup, and its rounds in the rounds table (the first one's
  // number, how many, how many per workgroup)
  uint64_t chunk; uint32_t round0, n_rounds, per_group, pad;
};

// The window's rows (rows.h) and what it takes to read one by its slot.
struct WindowRows {
  const uint4* row;          // [cap] 16-byte rows
  const int64_t* wide;       // [cap][3] t_enter, t_exit, bytes of the rows that do not fit
  int64_t ref;               // time the rows are relative to ...
  uint32_t far;              // ... unless the window's batches lie hours apart: then the batch's own
  const BatchMeta* meta;     // headers of the window's batches: n_batch of them from slot0 on, modulo n_meta
  uint32_t n_meta, slot0, n_batch;
  uint32_t head, cap;
  // batches placed by bucket (null: slots are in order of arrival): first record of every bucket in each batch, first record
  // of every round in each bucket
  const uint32_t* bucket_base;   // [n_meta][n_buckets + 1]
  const uint32_t* rounds;        // [rounds][n_buckets]
  uint32_t n_buckets;
};
// Rounds of all resident batches and of one more: a batch of n records has at most 3 n / 2048 + 2, and as much again keeps
// a batch's rounds in one piece where the table starts over.
inline uint64_t ingest_rounds_cap(uint64_t records, uint64_t batches) { return 2 * (3 * records / INGEST_ROUND + 2 * batches) + 64; }

constexpr int SEG_TILE = 1024;       // sorted records owned by one workgroup of the segment kernels
constexpr int SEG_THREADS = 256;
constexpr int SEL_TILE = 2048;       // records per workgroup of the compaction kernels
constexpr int RANKCOUNT_BLOCKS = 2048;
constexpr uint32_t SHORT_COMM = 64;          // most members of a communicator whose rates part of a wavefront compares
struct LongComm { uint32_t comm, off, size, unused; };
constexpr uint32_t HANG_REGIONS = 512;       // most regions that snapshot rows are regrouped by

// device counters written by kernels and read back by the host
enum { CNT_NSEG, CNT_NFLAG, CNT_NBIG, CNT_NGROUP, CNT_NALERT, CNT_NCAND, CNT_STATUS, CNT_NBLAMED, CNT_NCLEAN,
       CNT_CHAIN_LOOP, CNT_DONE, CNT_NCELL, CNT_COUNT = 16 };

}  // namespace ccld

struct ccld_ctx {
  ccld_params p;
  hipStream_t stream;
  uint64_t cap, batch_cap, snap_cap;
  ccld::KeyFormat kf;
  int rank_bits;                      // bit width of the largest rank
  // topology
  ccld::DeviceTopology topo;
  // window (circular)
  uint64_t head, count;
  std::vector<uint64_t> batch_n;      // sizes of the resident batches, oldest first
  std::vector<uint32_t> batch_slot;   // meta slot of each resident batch
  uint32_t next_slot;
  uint64_t* win_key;
  uint4* win_row;                     // [cap] 16-byte rows (rows.h)
  int64_t* win_wide;                  // [cap][3] values of the rows that do not fit
  uint32_t* ing_rounds;               // [rounds_cap][n_buckets] (batches placed by bucket)
  uint64_t rounds_cap, rounds_next;   // the next batch's rounds start there
  ccld::BatchMeta* batch_meta;        // [window_batches + 2]
  uint32_t* ing_table;                // [n_buckets][INGEST_BLOCKS]
  uint32_t* ing_base;                 // [window_batches + 2][n_buckets + 1]
  uint32_t n_buckets; int bshift;
  // sort
  ccld::SortBuffers sb;               // main sort
  uint64_t* keyC;                     // third array of keys
  uint32_t* table2; uint32_t* totals2;
  // analysis scratch
  uint32_t* tile_heads;               // [seg tiles + 1]
  uint32_t* tile_flags;               // [sel tiles + 1]
  uint8_t* rec_flag;                  // [cap]
  uint32_t* flag_pos;                 // [cap] sorted position of the k-th flagged record
  int64_t* flag_lag;                  // [2][cap]
  uint32_t* big_list;                 // [cap / 65 + 2][3]  (segment ordinal, first position, length) of the collectives over 64 records
  uint64_t* flag_key;                 // [cap] grid placement: table row << 32 | member slot of the k-th flagged record
  int64_t* range_c;                   // [cap] T_max - T_min of every usable collective
  int64_t* blame;                     // [CCLD_BLM_NCOL][n_ranks]
  uint32_t* blame_list;               // [2][n_ranks] flagged ranks, then the others, each ascending (many ranks only)
  uint32_t* blame_tiles;              // [n_ranks / SEL_TILE + 3]
  uint32_t* blame_order;              // [n_ranks] ranks by (flags, summed lag, rank), written at the end of every analysis
  uint16_t* gcode;                    // [cap] (op, size class) of every usable collective
  uint32_t* comm_groups;              // [n_comms + 1] detection groups of each communicator
  uint32_t* comm_row;                 // [n_comms] its first row of the collective table
  uint32_t* chain_parent;             // [cap + 1] scratch of ccld_flag_chains: parent of every flag
  uint32_t* alert_rows;               // [END_ALERTS]
  uint32_t* alert_list;               // [cap]
  uint32_t* alert_ncand;              // [cap + 1]
  uint2* comm_info;                   // [n_comms] (first member index, members) of every communicator: one load for both
  ccld::GroupState* gstate;           // [n_comms][GROUP_SLOTS]
  uint64_t* counters;                 // [CNT_COUNT] device
  uint32_t* arrivals;                 // [ARRIVAL_WORDS] of the kernels whose last workgroup reports; zero between launches
  uint32_t max_comm_size;             // members of the largest communicator
  ccld::LongComm* long_comms;         // [n_comms] the first n_long_comms: communicators of more than SHORT_COMM members, ascending
  uint32_t n_long_comms;
  uint32_t short_lanes;               // the smallest power of two that no other communicator's members exceed
  uint32_t long_classes;              // which sizes beyond 64 members there are (SegArgs)
  uint64_t sort_cap;                  // items the sort buffers hold: max(window records, communicator members)
  uint64_t* h_pinned;                 // pinned host staging
  uint64_t ticket;                    // of the latest report that the device was asked for
  int device;                         // the device that the context was created on
  uint64_t copy_earned;               // bytes of large host batches that the caller has copied alone (host_copy.h)
  // staging for host-resident batches
  uint8_t* stage;                     // [batch_cap * 41] device
  // hang location and rates
  uint64_t* h_counters;               // [CNT_COUNT] counters, then two words per region: its rows
  bool h_clear;                       // both are clear
  uint64_t n_members;                 // member slots over all communicators
  uint64_t* h_cell;                   // [snap_cap][2]  (operation counter, sent | recv << 32)
  uint32_t* h_cnt;                    // [snap_cap / 32 + 1] presence bitmap of the grid cells
  int64_t* h_pair;                    // [CCLD_HPAIR_NCOL][n_members]
  int64_t* h_comm;                    // [CCLD_HCOMM_NCOL][n_comms]
  int32_t* h_wait_slot;               // [n_members] slot waited on, -1 = none
  uint8_t* h_cand;                    // [n_members]
  uint64_t* h_layer_max;              // [n_members]
  int64_t* rate_root;                 // [n_comms] member of minimal SendRate / RecvRate from the latest rate pass, or CCLD_NO_RANK
  uint64_t* f_last;                   // [n_members][CCLD_FRAME_CHANNELS][2] remembered (operation counter, sent | recv << 32) per member and channel
  uint64_t* f_frame;                  // [n_ranks] call << 32 | frame that the rank delivered in it
  uint64_t* f_status;                 // call << 8 | error of it
  uint32_t f_call;                    // calls so far
  uint8_t* h_stage;                   // [snap_cap * 32] device staging for host-resident snapshots
  // grid placement (grid.h)
  bool grid_capable;                  // communicators fit a fine bucket, few enough of them, few enough batches
  bool grid_over_sort;                // its arrays lie over the sort buffers
  bool dense_asked;                   // CCLD_PLACEMENT_DENSE and windows of one batch: results name the path taken
  uint64_t* comm_range;               // [window_batches + 2][n_comms][2] per batch and communicator: largest counter, largest complement
  void* g_lay;                        // [n_comms + 1] CommLayout
  void* g_hdr;                        // GridHeader
  void* g_desc;                       // [fine_cap] FineDesc
  uint32_t *g_piece_at, *g_piece_slot;
  uint32_t *g_fill, *g_rec0, *g_nflag, *g_long;   // [fine_cap + 1]
  uint4* g_rows;                      // [cell_cap, and what stays empty where rows leave in whole lines]
  uint32_t* g_slots;                  // [cell_cap]
  uint16_t* g_cell_row;               // [cell_cap]
  uint32_t* flag_stage;               // [cap]
  uint32_t fine_cap, cell_cap;
  // what ccld_flag_chains needs of the most recent analysis
  bool chain_ready;                   // its order (sorted or on the grid), flag positions and lags are still in the workspace
  const int64_t* last_seg; uint64_t last_seg_cap, last_n_seg, last_n_flag;
  const uint8_t* last_rec_flag;
  bool last_grid;                     // the analysis ran on the grid placement
  ccld::WindowRows last_win;          // the window's rows
  uint32_t* chain_first;              // [n_comms + 2] first table row of each communicator
  // the order of the latest analysis that sorted, for windows of several batches (merge.h)
  uint64_t total_ingested;
  bool inc_ok;                        // sb.key/idx[sorted_buf] hold it, in format inc_sf
  ccld::SqueezedFormat inc_sf;
  uint64_t inc_head, inc_count, inc_total;   // that window's first slot, records, and total_ingested at the time
  // last analysis
  int sorted_buf;                     // which ping-pong buffer holds the sorted window
  ccld::SqueezedFormat sf;
  bool blame_valid;
  ccld::Profiler prof;
  int sort_passes;                    // passes of the last main sort
};

namespace ccld {
// Kernels that take more than 64 KB of dynamic LDS have to be allowed it on every device (one function per file of kernels,
// called by ccld_device_init).
inline hipError_t allow_lds(const void* kernel, size_t bytes) {
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}
hipError_t allow_lds_window();
hipError_t allow_lds_grid();
hipError_t allow_lds_segments();
hipError_t allow_lds_hang();
}  // namespace ccld

// what every device needs once, for the current one (hang.hip): kernels with much LDS allowed it, and the device address of
// the library's static scratch array
ccld_status ccld_device_init();
// the ticket of the report that the device is asked for next
inline uint64_t take_ticket(ccld_ctx* c) { return c->ticket = ccld::next_ticket(c->ticket); }
// waits for the report of the current ticket (api.hip): its words are then in h_pinned
hipError_t wait_report(ccld_ctx* c, int words = ccld::CNT_COUNT);
