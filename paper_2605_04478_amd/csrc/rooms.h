// Places of a fine bucket's rows.  One word per fine bucket counts the rows that were placed from its first cell on (lower half)
// and those that end with its last cell (upper half); whoever adds to a half has the places behind what it found there.  More rows
// than cells can only be duplicate keys, which end the analysis with an error, but the statistics have been launched by then and read
// what the word says is there: so that nothing is read that nobody wrote, every row whose place is a cell is written, also where others
// of the same request have none.  (Past 65,535 rows a half starts again or runs into the other one.  All cells have been written by then.)
// Plain C++: the rule is tested without a GPU.
#pragma once
#include <stdint.h>

namespace ccld {

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
