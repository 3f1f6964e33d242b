// The grid placement of a window.  Every rank bumps the same operation counter per communicator (the Trace ID of
// Section 5.1), so (communicator, counter - smallest counter, member slot) is a grid in which the cell of every record
// follows from its key.  The grid is cut into fine buckets of whole collectives that fit LDS; one partition pass
// moves every 16-byte row into its fine bucket, and the statistics kernel places a bucket's rows in LDS by cell and
// reads the collectives in (communicator, counter, rank) order.  Windows that do not fill such a grid (counters far
// apart, rounds without any record, communicators larger than a fine bucket) are sorted instead.
#pragma once
#include "ccld_internal.h"
#include "rooms.h"
#include "window_kernels.h"

namespace ccld {

constexpr uint32_t GRID_SPAN = 4096;         // fine buckets of one coarse bucket that a partition workgroup addresses
constexpr uint32_t GRID_FINE_BOUND = 4096;   // most fine buckets that a launch is sized for without asking for their number
constexpr uint32_t GRID_SELF_SUM = 512;      // where so many fine buckets are likely, each workgroup of the statistics sums the records before its own
constexpr uint32_t GRID_MAX_COMMS = INGEST_RANGE_COMMS;
constexpr uint32_t GRID_MAX_BATCHES = 256;   // batches of a window whose batches are placed by communicator bucket

// Per communicator: where its part of the grid lies.  Rounds are numbered from the window's smallest
// operation counter of the communicator; rpb rounds make one fine bucket.
struct __attribute__((aligned(16))) CommLayout {
  uint64_t seq_min;        // smallest operation counter in the window
  uint32_t fb_base;        // first fine bucket
  uint32_t rpb;            // rounds per fine bucket (bucket_rounds)
  uint32_t rounds;         // largest - smallest operation counter + 1 (0: no record)
  uint32_t seg_base;       // row of the collective table of the first round
  uint32_t cell_base;      // first cell
  uint32_t size;           // members
  uint32_t div, shift;     // a round's fine bucket is its number * 2 * div >> (32 + shift) (partition)
};

// One fine bucket (written by the partition kernel).
struct __attribute__((aligned(16))) FineDesc {
  uint32_t comm, size;     // communicator and its members
  uint32_t K;              // collectives (rounds) in the bucket
  uint32_t srow0;          // row of the collective table of the bucket's first round
  uint32_t cell0;          // first cell, and first row of the partitioned rows
  uint32_t pad;
  uint64_t seq0;           // operation counter of the first round
};

// device-side header of the layout
struct GridHeader {
  uint32_t feasible, n_fine, n_seg, n_pieces;
  int64_t ref;             // time the window's rows are relative to
  uint32_t n_long, done;   // fine buckets of communicators of more than 64 members; workgroups that have finished
};

struct GridArgs {
  // window: n records, nb batches whose headers start at slot0 (modulo n_meta)
  const uint64_t* win_key;
  const uint4* win_row;
  uint32_t head, cap, n;
  const BatchMeta* meta;
  uint32_t n_meta, slot0, nb;
  KeyFormat kf;
  const uint32_t* comm_size;
  uint32_t n_comms;
  // coarse buckets (communicator >> bshift) as ingest placed them: first record of each bucket in every batch
  const uint32_t* bucket_base;   // [n_meta][n_buckets + 1]
  uint32_t n_buckets;
  int bshift;
  // counter ranges per batch and communicator: largest counter, largest complement (zero pair: no record)
  const uint64_t* range;         // [n_meta][n_comms][2]
  // layout
  CommLayout* lay;               // [n_comms + 1]
  GridHeader* hdr;
  uint32_t* piece_at;            // [pieces + 1] records before each (coarse bucket, batch) piece, bucket by bucket
  uint32_t* piece_slot;          // [pieces] its first window slot
  // fine buckets
  uint32_t* fill;                // [fine_cap + 1] rows of each (rooms.h)
  uint32_t* rec0;                // [fine_cap + 1] records before each (from the statistics on, where these sum them)
  uint32_t* nflag;               // [fine_cap + 1] flagged records of each
  FineDesc* desc;                // [fine_cap]
  uint32_t* long_list;           // [fine_cap] fine buckets of communicators of more than 64 members
  uint32_t fine_cap, cell_cap;
  uint32_t lines;                // 1: rows leave in whole lines (grid_in_lines), and up to seven cells behind those of a communicator stay empty
  uint32_t likely, self_sum;     // fine buckets that the window most likely has; 1: they are not scanned (RecordsBefore)
  uint4* rows;                   // [cell_cap, and what stays empty] partitioned rows
  uint32_t* slots;               // [cell_cap] their window slots, or null: not wanted
  uint16_t* cell_row;            // [cell_cap] row of each cell inside its bucket, GRID_EMPTY: no record
  uint64_t* counters;
  uint64_t* blame;               // cleared here: [n_blame] words
  uint32_t n_blame;
  // pinned host word: 1 + fine buckets once the layout is known, GRID_FULL if the window has as many records as the grid has
  // cells (GRID_INFEASIBLE: it is not feasible)
  uint32_t* host_fine;
};
constexpr uint32_t GRID_INFEASIBLE = 0x80000000u, GRID_FULL = 0x40000000u;
constexpr uint32_t GRID_EMPTY = 0xFFFFu;

// whether the rows of n records leave in whole lines
bool grid_in_lines(uint64_t n, bool with_slots);
void launch_grid_layout(hipStream_t st, const GridArgs& d);
void launch_grid_partition(hipStream_t st, const GridArgs& d);
// ends the placement of a window that has a round without any record (behind the partition)
void launch_grid_gaps(hipStream_t st, const GridArgs& d, uint32_t n_fine);

// statistics of every collective (segments.hip); fine_bound: no fewer than the layout's fine buckets
void launch_grid_stats(hipStream_t st, const SegArgs& a, const GridArgs& d, uint32_t fine_bound, int64_t* blame, uint32_t n_ranks);

// groups, blame order, a few alerts and report, and the flags of a window on the grid placement (groups.hip); d and f null: a
// sorted window, whose flags are listed; al null: alerts are not listed here.  True if it reports.
bool launch_window_end(hipStream_t st, const EndArgs& a, const GridArgs* d, const FlagArgs* f, const AlertArgs* al, uint32_t fine_bound);

}  // namespace ccld
