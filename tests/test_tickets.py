"""The tags that tell a report of the device from the words of the call before: csrc/ticket.h compiled for the host and run
over several turns of the tag."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_04478_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "ticket.h"
using namespace ccld;
int main() {
  uint64_t word = 0, ticket = 0;                  // as at create: cleared words, no ticket yet
  for (uint32_t i = 0; i < (3u << 16); ++i) {
    const uint64_t before = ticket, value = (i * 0x9E3779B97F4Aull + i) & REPORT_MASK;
    ticket = next_ticket(ticket);
    if (ticket <= before || ticket > before + 2) { std::printf("order at %u\n", i); return 1; }
    if (report_arrived(word, ticket)) { std::printf("ticket %llu: the call before taken for a report\n", (unsigned long long)ticket); return 1; }
    word = report_word(value, ticket);            // the device reports
    if (!report_arrived(word, ticket)) { std::printf("ticket %llu: not seen\n", (unsigned long long)ticket); return 1; }
    if (report_arrived(word, next_ticket(ticket))) { std::printf("ticket %llu: taken for the next one\n", (unsigned long long)ticket); return 1; }
    word = report_value(word);                    // the host has read it
    if (word != value) { std::printf("value at %u\n", i); return 1; }
  }
  return 0;
}
"""


def test_a_read_report_is_never_taken_for_the_next_one(tmp_path):
    src, exe = tmp_path / "tickets.cpp", tmp_path / "tickets"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(exe), str(src)])
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout


def test_every_ticket_is_taken_by_the_one_rule():
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".hip", ".h")):
            continue
        text = re.sub(r"//.*", "", open(os.path.join(CSRC, name)).read())
        assigned = re.findall(r"(?:\+\+\s*c->ticket|c->ticket\s*(?:\+\+|[-+|]?=(?!=))[^;]*)", text)
        assert [a for a in assigned if a not in ("c->ticket = 0", "c->ticket = ccld::next_ticket(c->ticket)")] == [], name
