// Instantiations of the 16-row-tile ring kernel (xcorr16.hpp) for any N, with
// 8, 9, 10 tiles loaded in 16-byte chunks.
// (Several translation units so that they compile in parallel.)
#include "x16_ragged.hpp"

namespace xeng {
namespace x16 {
namespace {

const KernelInfo kTable[3] = {ragged_info<8, LD_CHUNK>(), ragged_info<9, LD_CHUNK>(), ragged_info<10, LD_CHUNK>()};

}  // namespace
}  // namespace x16

const KernelInfo* x16_ragged_b(int nt) { return nt >= 8 && nt <= 10 ? &x16::kTable[nt - 8] : nullptr; }

}  // namespace xeng
