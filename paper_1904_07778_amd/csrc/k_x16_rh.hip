// Instantiations of the 16-row-tile ring kernel (xcorr16.hpp) for any N, with
// 12, 13 tiles loaded in 4-byte units.
// (Several translation units so that they compile in parallel.)
#include "x16_ragged.hpp"

namespace xeng {
namespace x16 {
namespace {

const KernelInfo kTable[2] = {ragged_info<12, LD_DWORD>(), ragged_info<13, LD_DWORD>()};

}  // namespace
}  // namespace x16

const KernelInfo* x16_ragged_h(int nt) { return nt >= 12 && nt <= 13 ? &x16::kTable[nt - 12] : nullptr; }

}  // namespace xeng
