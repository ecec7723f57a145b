// csr_entries.hpp — positions of a CSR row's entries, a wave's or a group's
// worth at a time.  Plain C++, used in device code.
#pragma once

namespace wise {

// Entries beg .. end - 1.  Offsets are int32 and the last row may end at
// 2^31 - 1: a position past the end is never formed, what is left is compared
// instead.
struct Entries {
  int at, end;
  constexpr Entries(int beg, int end_) : at(beg), end(end_) {}
  constexpr bool more() const { return at < end; }
  constexpr bool holds(int i) const { return i < end - at; }   // is there an entry at + i
  constexpr void advance(int n) { at = end - at > n ? at + n : end; }
};

}  // namespace wise
