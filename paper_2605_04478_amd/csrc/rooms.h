// Places of a fine bucket's rows.  One word per fine bucket counts the rows that were placed from its first cell on (lower half)
// and those that end with its last cell (upper half); whoever adds to a half has the places behind what it found there.  More rows
// than cells can only be duplicate keys, which end the analysis with an error, but the statistics have been launched by then and read
// what the word says is there: so that nothing is read that nobody wrote, every row whose place is a cell is written, also where others
// of the same request have none.  (Past 65,535 rows a half starts again or runs into the other one.  All cells have been written by then.)
// Plain C++: the rules are tested without a GPU.
#pragma once
#include <stdint.h>

namespace ccld {

constexpr uint32_t GRID_B = 2048;            // grid cells (= LDS cells of the statistics kernels) per fine bucket
constexpr uint32_t GRID_MIN_FILL = 1025;     // a full fine bucket holds at least this many cells (whole rounds of <= GRID_B members)
constexpr uint32_t LINE_ROWS = 8;            // rows of a 128-byte line

// Rounds of a communicator of `size` members that make one fine bucket.  Where rows leave in whole lines a bucket starts on a line, so
// its cells are whole lines: with the last rounds of it left out that this takes, up to seven (not for those of the communicators of
// more than 256 members that have too few).
constexpr uint32_t bucket_rounds(uint32_t size, bool lines) {
  const uint32_t most = GRID_B / size, off = lines ? 7u >> __builtin_ctz(size | 8) : 0u;      // 0 to 7: a multiple of off + 1 rounds
  return most > off ? most & ~off : most;
}
// A communicator with several fine buckets that do not all start on a line.
constexpr bool off_lines(uint32_t size, uint32_t rpb, uint32_t rounds) { return rounds > rpb && rpb * size % LINE_ROWS != 0; }
// Cells of a communicator's part of the grid.
constexpr uint64_t grid_cells(uint32_t size, uint32_t rounds, bool lines) {
  const uint64_t off = lines ? LINE_ROWS - 1 : 0u;
  return ((uint64_t)size * rounds + off) & ~off;
}

constexpr uint32_t fill_front(uint32_t fill) { return fill & 0xFFFFu; }
constexpr uint32_t fill_back(uint32_t fill) { return fill >> 16; }
constexpr uint32_t fill_rows(uint32_t fill) { return fill_front(fill) + fill_back(fill); }

// Of n rows asked for from the front with `fill` in the word, the first so many have a cell: fill_front(fill) + 0, 1, ...
constexpr uint32_t front_room(uint32_t fill, uint32_t n, uint32_t cells) {
  const uint32_t left = fill_front(fill) < cells ? cells - fill_front(fill) : 0u;
  return n < left ? n : left;
}
// The k-th last (1, 2, ...) of the rows asked for from the back has this place, if it is not negative.
constexpr int32_t back_place(uint32_t fill, uint32_t k, uint32_t cells) { return (int32_t)(cells - fill_back(fill) - k); }

}  // namespace ccld
