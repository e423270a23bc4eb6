// Instantiations of the 16-row-tile ring kernel (xcorr16.hpp) for any N, with
// 11, 12 tiles loaded in 16-byte chunks.
// (Several translation units so that they compile in parallel.)
#include "x16_ragged.hpp"

namespace xeng {
namespace x16 {
namespace {

const KernelInfo kTable[2] = {ragged_info<11, LD_CHUNK>(), ragged_info<12, LD_CHUNK>()};

}  // namespace
}  // namespace x16

const KernelInfo* x16_ragged_c(int nt) { return nt >= 11 && nt <= 12 ? &x16::kTable[nt - 11] : nullptr; }

}  // namespace xeng
