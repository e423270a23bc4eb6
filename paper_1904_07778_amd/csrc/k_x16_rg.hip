// Instantiations of the 16-row-tile ring kernel (xcorr16.hpp) for any N, with
// 8, 9, 10, 11 tiles loaded in 4-byte units.
// (Several translation units so that they compile in parallel.)
#include "x16_ragged.hpp"

namespace xeng {
namespace x16 {
namespace {

const KernelInfo kTable[4] = {ragged_info<8, LD_DWORD>(), ragged_info<9, LD_DWORD>(), ragged_info<10, LD_DWORD>(), ragged_info<11, LD_DWORD>()};

}  // namespace
}  // namespace x16

const KernelInfo* x16_ragged_g(int nt) { return nt >= 8 && nt <= 11 ? &x16::kTable[nt - 8] : nullptr; }

}  // namespace xeng
