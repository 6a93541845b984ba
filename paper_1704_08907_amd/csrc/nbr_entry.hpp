// An entry of a recorded neighbour list: the neighbour's slot, with the top bit set when
// the box search reached it through a nonzero image shift.  In a list of up to 2^30 slots
// the next bit is set when it is the first neighbour of its stencil row; larger lists (whose
// sums are not formed by rows) use all 31 bits for the slot.  Plain C++, so that it can be
// checked without a GPU.
#pragma once

#include <stdint.h>

namespace aboria {

constexpr uint32_t kNbrShift = 0x80000000u;
constexpr uint32_t kNbrOverflow = 0xFFFFFFFFu;  // a count above every capacity

// The row flag of a list of n slots (0: none), and the slot of an entry of such a list.
constexpr uint32_t nbr_row_flag(uint32_t n) { return n <= 0x40000000u ? 0x40000000u : 0u; }
constexpr uint32_t nbr_slot(uint32_t entry, uint32_t row_flag) { return entry & ~(kNbrShift | row_flag); }

}  // namespace aboria
