"""Places of the rows of a fine bucket: csrc/rooms.h compiled for the host, with workgroups that ask for rooms in a random order as
the partition does (rows eight at a time from the front and the rest from the back, or runs of any length from the front).  Whatever
the word of a bucket says is there, which is what the statistics read, has been written, with duplicate keys too."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_04478_amd", "csrc")

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>
#include "rooms.h"
using namespace ccld;
typedef uint32_t u32;
struct Bucket {
  u32 cells, fill = 0;
  u32 total = 0;                                   // rows, however many
  bool dup = false;
  std::vector<u32> written;
  void write(u32 place) { if (place >= cells) { std::printf("place %u of %u\n", place, cells); std::exit(1); } ++written[place]; }
  void lines(u32 n) {                              // n % 8 == 0, from the front
    const u32 old = fill; fill += n; total += n;
    dup |= fill_rows(old) + n > cells;
    for (u32 k = 0; k < front_room(old, n, cells); ++k) write(fill_front(old) + k);
  }
  void rest(u32 n) {                               // n < 8, from the back
    const u32 old = fill; fill += n << 16; total += n;
    dup |= fill_rows(old) + n > cells;
    for (u32 k = 1; k <= n; ++k) if (back_place(old, k, cells) >= 0) write((u32)back_place(old, k, cells));
  }
  void run(u32 n) {                                // any number, from the front; each row for itself
    const u32 old = fill; fill += n; total += n;
    for (u32 k = 0; k < n; ++k) { const u32 w = fill_front(old) + k; if (w >= cells) dup = true; else write(w); }
  }
};
int main() {
  std::mt19937 rng(7);
  auto below = [&](u32 n) { return (u32)(rng() % n); };
  int over = 0, wrapped = 0;
  for (int trial = 0; trial < 40000; ++trial) {
    Bucket B;
    B.cells = trial % 3 ? 1 + below(2048) : 2048 - below(16);
    B.written.assign(B.cells, 0);
    // rows in all: fewer than cells, as many, a few more, many more than a half of the word can tell
    const int kind = trial % 5;
    u32 rows = kind == 0 ? below(B.cells + 1) : kind == 1 ? B.cells : kind == 2 ? B.cells + 1 + below(8) : kind == 3 ? B.cells + below(4000) : 60000 + below(120000);
    const u32 groups = 1 + below(kind == 4 ? 40 : 12), mixed = below(3);       // all whole lines, all runs, both
    struct Group { u32 rows, wait; bool runs; };
    std::vector<Group> g(groups, Group{0, 0, false});
    for (auto& x : g) x.runs = mixed == 1 || (mixed == 2 && below(2));
    for (u32 r = rows; r;) { const u32 k = std::min(r, 1 + below(kind == 4 ? 4096 : 512)); g[below(groups)].rows += k; r -= k; }
    while (!g.empty()) {
      const u32 i = below((u32)g.size());
      Group& x = g[i];
      if (x.rows == 0) { if (x.wait) B.rest(x.wait); g.erase(g.begin() + i); continue; }
      const u32 k = std::min(x.rows, 1 + below(kind == 4 ? 3072 : 300));
      x.rows -= k;
      if (x.runs) B.run(k);
      else { x.wait += k; const u32 out = x.wait & ~7u; if (out) B.lines(out); x.wait -= out; }
    }
    const u32 front = fill_front(B.fill), back = fill_back(B.fill), cnt = fill_rows(B.fill);
    if (B.total > B.cells) {
      ++over;
      wrapped += B.total > 65535;
      if (!B.dup && cnt <= B.cells) { std::printf("trial %d: %u rows in %u cells not noticed\n", trial, B.total, B.cells); return 1; }
    } else {
      if (B.dup || cnt != B.total) { std::printf("trial %d: duplicates where there are none\n", trial); return 1; }
      for (u32 w : B.written) if (w > 1) { std::printf("trial %d: two rows in one place\n", trial); return 1; }
    }
    // what is read: every cell where there are more rows than cells, else those of the two ends
    for (u32 i = 0; i < B.cells; ++i)
      if ((cnt > B.cells || i < front || i + back >= B.cells) && !B.written[i]) {
        std::printf("trial %d: cell %u of %u is read, nobody wrote it (%u rows, %u from the front, %u from the back)\n", trial, i, B.cells, B.total, front, back);
        return 1;
      }
  }
  return over > 10000 && wrapped > 5000 ? 0 : 2;
}
"""


def test_every_row_that_the_statistics_read_was_written(tmp_path):
    src, exe = tmp_path / "rooms.cpp", tmp_path / "rooms"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-I", CSRC, "-o", str(exe), str(src)])
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout


def test_the_partition_takes_its_rooms_by_this_rule():
    text = open(os.path.join(CSRC, "grid.hip")).read()
    lines = text[text.index("void part_lines("):text.index("void k_grid_partition(")]
    assert lines.count("atomicAdd(&d.fill[") == 2 and "front_room(got, out, cells)" in lines and "back_place(old, 0, cells)" in lines and "if (place >= 0)" in lines


LAYOUT = r"""
#include <cstdio>
#include "rooms.h"
using namespace ccld;
int main() {
  for (uint32_t size = 1; size <= GRID_B; ++size)
    for (int lines = 0; lines < 2; ++lines) {
      const uint32_t rpb = bucket_rounds(size, lines), cells = rpb * size;
      if (cells > GRID_B || (size < GRID_B && cells < GRID_MIN_FILL && GRID_B / size > 1) || (!lines && rpb != GRID_B / size)) { std::printf("%u members: %u cells\n", size, cells); return 1; }
      if (lines && size <= 256 && off_lines(size, rpb, rpb + 1)) { std::printf("%u members: a second bucket that starts at cell %u\n", size, cells); return 1; }
      if (off_lines(size, rpb, rpb) || off_lines(size, rpb, rpb + 1) != (cells % 8 != 0)) return 2;
      for (uint32_t rounds : {1u, rpb, rpb + 1, 3 * rpb, 3 * rpb + 2, 100000u}) {
        const uint64_t have = grid_cells(size, rounds, lines), want = (uint64_t)size * rounds;
        if (have < want || have - want > 7 || (lines ? have % 8 != 0 : have != want)) { std::printf("%u members, %u rounds: %llu cells\n", size, rounds, (unsigned long long)have); return 3; }
        // the fine buckets' cells, 2,048 at most, hold the communicator's
        if (have > (uint64_t)((rounds + rpb - 1) / rpb) * GRID_B) return 4;
      }
    }
  return 0;
}
"""


def test_fine_buckets_start_on_lines_where_rows_leave_in_lines(tmp_path):
    src, exe = tmp_path / "layout.cpp", tmp_path / "layout"
    src.write_text("#include <initializer_list>\n" + LAYOUT)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-I", CSRC, "-o", str(exe), str(src)])
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, (run.returncode, run.stdout)
