// How the device reports a counter to the host: its value in the lower bits of a pinned word, the ticket of the call that
// waits for it in the upper ones.  Plain C++: the host logic is tested without a GPU.
#pragma once
#include <stdint.h>

namespace ccld {

constexpr int REPORT_BITS = 48;
constexpr uint64_t REPORT_MASK = (1ull << REPORT_BITS) - 1;

// A word whose report has been read holds its value alone, that is, tag zero: no ticket may have that tag, or the wait for
// it would take the words of the call before for its own.
constexpr uint64_t ticket_tag(uint64_t ticket) { return ticket & (~0ull >> REPORT_BITS); }
constexpr uint64_t next_ticket(uint64_t ticket) { return ticket_tag(ticket + 1) ? ticket + 1 : ticket + 2; }
constexpr uint64_t report_word(uint64_t value, uint64_t ticket) { return (value & REPORT_MASK) | (ticket_tag(ticket) << REPORT_BITS); }
constexpr uint64_t report_value(uint64_t word) { return word & REPORT_MASK; }
constexpr bool report_arrived(uint64_t word, uint64_t ticket) { return (word >> REPORT_BITS) == ticket_tag(ticket); }

}  // namespace ccld
