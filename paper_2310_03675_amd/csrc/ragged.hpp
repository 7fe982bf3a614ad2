// Where the loads of a line that starts on any byte lie (load_units in gemm_small.hip): apart from the kernel, so
// that the host can go over every one of them against the operand's first and last byte.
#pragma once

#include <stdint.h>

namespace hdqt {

// A lane's aligned dwords of a line: 16 bytes from here, and from every 32 bytes on (`half`: of the wave).
constexpr uint32_t ragged_at(uint32_t line, int half) { return (line & ~3u) + 16 * (uint32_t)half; }

// The last of the line's first `bytes` bytes' dwords, where it is.  (Not from the aligned dword behind the others: that
// one may reach past the operand, whose last line can have less behind these bytes than it would read on.)
constexpr uint32_t ragged_last_at(uint32_t line, uint32_t bytes) { return line + bytes - 4; }

} // namespace hdqt
