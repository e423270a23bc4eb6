// Instantiations of the 16-row-tile ring kernel (xcorr16.hpp) for any N, with
// 16 tiles loaded in 4-byte units.
// (Several translation units so that they compile in parallel.)
#include "x16_ragged.hpp"

namespace xeng {
namespace x16 {
namespace {

const KernelInfo kTable[1] = {ragged_info<16, LD_DWORD>()};

}  // namespace
}  // namespace x16

const KernelInfo* x16_ragged_k(int nt) { return nt >= 16 && nt <= 16 ? &x16::kTable[nt - 16] : nullptr; }

}  // namespace xeng
