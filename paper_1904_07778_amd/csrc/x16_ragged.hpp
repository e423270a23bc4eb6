// x16_ragged.hpp - launches and table entries of the 16-row-tile ring kernel
// for any N (LD_CHUNK and LD_DWORD of xcorr16.hpp), by tile count.
#pragma once
#include "kernels.hpp"
#include "xcorr16.hpp"

namespace xeng {
namespace x16 {

// Ring depth: as for N = 16 NT; the dword loads count one per row against
// the 63 a wave can wait for, which allows 5 stages.
template <int NT, int LD>
constexpr int ragged_stages() {
  return LD == LD_DWORD ? 5 : stages_for(16 * NT, KPS_DEFAULT);
}

template <int NT, int LD>
hipError_t ragged_launch(dim3 grid, hipStream_t s, const Args& a) {
  constexpr int N = 16 * NT, CPW = LD == LD_DWORD ? 1 : cpw_for(N), S = ragged_stages<NT, LD>();
  hipLaunchKernelGGL((kernel<N, CPW, S, KPS_DEFAULT, LD>), grid,
                     dim3(Shape<N, CPW, S, KPS_DEFAULT, LD>::THREADS), 0, s, a);
  return hipGetLastError();
}

template <int NT, int LD>
constexpr KernelInfo ragged_info() {
  constexpr int N = 16 * NT, CPW = LD == LD_DWORD ? 1 : cpw_for(N), S = ragged_stages<NT, LD>();
  using C = Shape<N, CPW, S, KPS_DEFAULT, LD>;
  return KernelInfo{C::NT, C::W, CPW, S, C::THREADS, C::LDS_BYTES, MAX_T_PER_WG, MAX_ROW_BYTES, TILE_ROWS,
                    &ragged_launch<NT, LD>, load_unit(LD), true, 0};
}

}  // namespace x16
}  // namespace xeng
