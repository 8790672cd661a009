// Byte offsets of buffer loads that may lie outside their buffer.  The
// hardware compares the whole 32-bit offset, unsigned, with the buffer's size,
// and a load beyond it reads zero; so the sums wrap by intent, and are formed
// in unsigned arithmetic, where wrapping is defined.  (A buffer holds one
// projection or one decimated angle: at most 4096 rows of 4096 columns of 4
// bytes, 2^26 bytes.  Plain C++: a host test includes this file.)
#pragma once

#include <cstdint>

namespace fdkod {

// the offset of a column outside its row: 2^31 plus or minus the rows' offsets
// of a whole buffer stays beyond every buffer
constexpr uint32_t kOutside = 0x80000000u;

constexpr uint32_t column_offset(bool inside, int bytes) { return inside ? (uint32_t)bytes : kOutside; }

// offset `off` moved by a signed number of bytes (rows up or down)
constexpr uint32_t moved(uint32_t off, int bytes) { return off + (uint32_t)bytes; }

}  // namespace fdkod
