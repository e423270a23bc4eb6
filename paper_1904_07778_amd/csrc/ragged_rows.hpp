// ragged_rows.hpp - byte counts of the time rows that the 16-row ring kernel
// takes in phases (LD_CHUNK and LD_DWORD of xcorr16.hpp).  A phase's rows lie
// `stride` bytes apart (a whole number of load units), each `sub` bytes into
// its first unit; plain integers, so that they can be checked on the host.
#pragma once
#include <stdint.h>

namespace xeng {
namespace x16 {

// What a phase's last row leaves of its stride, to the last 4 bytes that hold
// some of it.  Loads are checked against the byte count in steps of 4, so at
// most 3 bytes past the row are read, in the dword that holds its last byte;
// without this the last units of a block reached up to 15 bytes past its end.
constexpr uint32_t row_slack(uint32_t stride, uint32_t sub, uint32_t row_bytes) {
  return stride - ((sub + row_bytes + 3) & ~3u);
}
// Bytes that the loads of a stage of `rows` rows may read from its first row's
// unit on.
constexpr uint32_t stage_bytes(int rows, uint32_t stride, uint32_t slack) {
  return rows > 0 ? (uint32_t)rows * stride - slack : 0;
}

}  // namespace x16
}  // namespace xeng
