// Sizes of the raw buffers that kernels load x through, evaluated by the kernels and on the CPU.
#pragma once

#include <cstdint>

namespace ppc {

// Records of the buffer over what is left of x, `room` bytes from the first image of a tile on.  A tile's own offsets end below 2^31 (the
// plan sees to it), and 0x80000000 is outside.
constexpr uint32_t buffer_records(int64_t room) { return room > 0x7FFFFFFC ? 0x7FFFFFFCu : (uint32_t)room; }

// ... and of the one that begins `at` bytes further, at a channel.  A 16-byte load of a row's last pixels may run past the row: in the last row
// of the last channel past x.  Only a buffer that begins at the channel ends where x does for the offsets of that channel: the range check of a
// load with the channel in its scalar offset need not cover that offset.
constexpr uint32_t buffer_records_from(uint32_t records, uint32_t at) { return records - at; }

}  // namespace ppc
