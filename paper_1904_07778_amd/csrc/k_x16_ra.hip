// Instantiations of the 16-row-tile ring kernel (xcorr16.hpp) for any N, with
// 1, 2, 3, 4, 5, 6, 7 tiles loaded in 16-byte chunks.
// (Several translation units so that they compile in parallel.)
#include "x16_ragged.hpp"

namespace xeng {
namespace x16 {
namespace {

const KernelInfo kTable[7] = {ragged_info<1, LD_CHUNK>(), ragged_info<2, LD_CHUNK>(), ragged_info<3, LD_CHUNK>(), ragged_info<4, LD_CHUNK>(), ragged_info<5, LD_CHUNK>(), ragged_info<6, LD_CHUNK>(), ragged_info<7, LD_CHUNK>()};

}  // namespace
}  // namespace x16

const KernelInfo* x16_ragged_a(int nt) { return nt >= 1 && nt <= 7 ? &x16::kTable[nt - 1] : nullptr; }

}  // namespace xeng
