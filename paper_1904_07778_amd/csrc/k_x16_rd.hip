// Instantiations of the 16-row-tile ring kernel (xcorr16.hpp) for any N, with
// 13, 14 tiles loaded in 16-byte chunks.
// (Several translation units so that they compile in parallel.)
#include "x16_ragged.hpp"

namespace xeng {
namespace x16 {
namespace {

const KernelInfo kTable[2] = {ragged_info<13, LD_CHUNK>(), ragged_info<14, LD_CHUNK>()};

}  // namespace
}  // namespace x16

const KernelInfo* x16_ragged_d(int nt) { return nt >= 13 && nt <= 14 ? &x16::kTable[nt - 13] : nullptr; }

}  // namespace xeng
