// Communicator buckets of windows that are placed by bucket, and the LDS that a placement workgroup takes for them.  Plain C++: the
// rule is tested without a GPU.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace ccld {

constexpr uint32_t INGEST_ROUND = 2048;           // records that a placement workgroup regroups at a time
constexpr uint32_t INGEST_LINE = 8;               // rows of a 128-byte line, which leave together
constexpr uint32_t INGEST_STAGED_BUCKETS = 256;   // most buckets of the placement
constexpr uint32_t INGEST_RANGE_COMMS = 3584;     // most communicators whose counter ranges the placement keeps in LDS
constexpr size_t INGEST_LDS = 152 * 1024;         // beside the 8 KB of the static tables

// Rows staged in a round: those that waited and lines that are not filled come on top of the round's records.
constexpr uint32_t ingest_stage_rows(uint32_t n_buckets) { return INGEST_ROUND + 2 * (INGEST_LINE - 1) * n_buckets; }
// LDS bytes of a placement workgroup: rows and keys of a round, a counter range per communicator (range_comms of them), and a
// membership row per rank where the table is in LDS.
constexpr size_t ingest_lds(uint32_t n_buckets, uint32_t range_comms, uint32_t table_ranks) {
  return (size_t)ingest_stage_rows(n_buckets) * 24 + (size_t)range_comms * 16 + (size_t)table_ranks * 16;
}

constexpr uint32_t GRID_ONE_BUCKET = 3500;        // windows of no more fine buckets are partitioned in one go, without communicator buckets
constexpr uint32_t GRID_TARGET = 300;             // fine buckets per communicator bucket of the others
constexpr uint32_t GRID_MAX_PIECES = 4096;        // (coarse bucket, batch) pairs of such a window
constexpr int GRID_BUCKET_BITS = 8;

// A bucket is a communicator's number without its lower bits.
constexpr int bits_for(uint64_t v) { return v ? 1 + bits_for(v >> 1) : 0; }
constexpr int bucket_shift(int bits, uint32_t n_comms) { return bits_for(n_comms - 1) > bits ? bits_for(n_comms - 1) - bits : 0; }
constexpr uint32_t bucket_count(int bits, uint32_t n_comms) { return ((n_comms - 1) >> bucket_shift(bits, n_comms)) + 1; }

// Bits of a communicator's number that name its bucket, for a window of `batches` batches placed on a grid that may have `fine`
// fine buckets.  A partition workgroup addresses a few thousand fine buckets at a time, so a window that may have more of them is
// placed by bucket, into as many buckets as leave about GRID_TARGET fine buckets in one: fewer fine buckets in one lengthen the runs
// that the partition writes, more those that the ingest writes (82M records with 300 / 600 in one: ingest 1,131 / 1,114 us, partition
// 704 / 910, a window 2,820 / 3,010; 20M: ingest 299 / 300, partition 164 / 190).  Half as many buckets where the ingest could not
// stage whole lines of so many beside the counter ranges (the largest windows of 1,833 to 2,048 and of 2,877 or more communicators:
// 60M records of 16,384 ranks in 3,200, 200 / 100 buckets: ingest 1,142 / 805 us, partition 541 / 551, a window 2,557 / 2,214; 100M:
// ingest 1,880 / 1,425, partition 925 / 1,106, a window 4,166 / 3,738).
constexpr int grid_bucket_bits(uint64_t fine, uint64_t batches, uint32_t n_comms) {
  int bits = 0;
  if (fine > GRID_ONE_BUCKET) while (bits < GRID_BUCKET_BITS && (fine >> bits) > GRID_TARGET) ++bits;
  while (bits > 0 && (batches << bits) > GRID_MAX_PIECES) --bits;
  if (ingest_lds(bucket_count(bits, n_comms), n_comms, 0) > INGEST_LDS) --bits;
  return bits;
}
static_assert(1u << GRID_BUCKET_BITS <= INGEST_STAGED_BUCKETS, "the placement takes them");
static_assert(ingest_lds(INGEST_STAGED_BUCKETS / 2, INGEST_RANGE_COMMS, 0) <= INGEST_LDS, "half as many are few enough");

}  // namespace ccld
