"""Communicator buckets of the ingest: csrc/buckets.h compiled for the host and run over every number of communicators that the grid takes and
windows of every size.  A placement workgroup can always stage whole lines, and the buckets are no fewer than half of what the fine
buckets ask for."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_04478_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "buckets.h"
using namespace ccld;
int main() {
  int halved = 0;
  for (uint32_t c = 1; c <= INGEST_RANGE_COMMS; ++c)
    for (uint64_t n = 100000; n < 1ull << 31; n += n / 16)
      for (uint64_t w : {1, 2, 10, 16, 17, 100, 256}) {
        const uint64_t fine = n / 1400 + c;
        const int bits = grid_bucket_bits(fine, w, c);
        int asked = 0;
        if (fine > GRID_ONE_BUCKET) while (asked < GRID_BUCKET_BITS && (fine >> asked) > GRID_TARGET) ++asked;
        while (asked > 0 && (w << asked) > GRID_MAX_PIECES) --asked;
        const uint32_t k = bucket_count(bits, c);
        if (k > INGEST_STAGED_BUCKETS || ingest_lds(k, c, 0) > INGEST_LDS) { std::printf("%u communicators, %llu records: %u buckets, %zu bytes\n", c, (unsigned long long)n, k, ingest_lds(k, c, 0)); return 1; }
        if (bits != asked) {
          ++halved;
          if (bits != asked - 1 || ingest_lds(bucket_count(asked, c), c, 0) <= INGEST_LDS) { std::printf("%u communicators, %llu records: %d bits, asked for %d\n", c, (unsigned long long)n, bits, asked); return 1; }
        }
        if ((c - 1) >> bucket_shift(bits, c) != k - 1) return 1;
      }
  return halved ? 0 : 2;
}
"""


def test_lines_always_fit_beside_the_counter_ranges(tmp_path):
    src, exe = tmp_path / "buckets.cpp", tmp_path / "buckets"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-I", CSRC, "-o", str(exe), str(src)])
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
