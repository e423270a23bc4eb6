// kernels.hpp - the table of compiled X-engine kernels seen by the host code.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xcorr.hpp"

namespace xeng {

using LaunchFn = hipError_t (*)(dim3 grid, hipStream_t s, const Args& a);

struct KernelInfo {
  int nt, w, cpw, stages, threads, lds_bytes;
  int64_t max_t_per_wg;  // longest time range one workgroup may integrate
  int64_t max_row_bytes; // largest time row F*N the kernel addresses (0: any)
  int tile_rows;         // rows of its tiles: 16 or 32
  LaunchFn launch;
  int load_unit = 0;     // ragged kernels: bytes that every row offset must share
                         // (rows are taken in phases where F*N is no multiple); 0: none
  bool chunks = false;   // honours Args::chunk_stride
  int split = 1;         // default time split: workgroups per CU to aim for; 0: modelled (choose_split)
};

// Staging kernel (any N), by 16-row tile count nt = ceil(N/16), 1..16.
const KernelInfo* stage_kernel(int nt);
// 32-row-tile ring kernel, N a multiple of 16 up to 256 (one function per
// translation unit; x32_kernel asks each).
const KernelInfo* x32_kernel_a(int n);
const KernelInfo* x32_kernel_b(int n);
const KernelInfo* x32_kernel_c(int n);
const KernelInfo* x32_kernel_d(int n);
inline const KernelInfo* x32_kernel(int n) {
  const KernelInfo* k = x32_kernel_a(n);
  if (!k) k = x32_kernel_b(n);
  if (!k) k = x32_kernel_c(n);
  if (!k) k = x32_kernel_d(n);
  return k;
}
// 16-row-tile ring kernel on v_mfma_i32_16x16x64_i8, N a multiple of 16 up
// to 256 (several translation units; x16_kernel asks each).
const KernelInfo* x16_kernel_a(int n);
const KernelInfo* x16_kernel_b(int n);
const KernelInfo* x16_kernel_c(int n);
const KernelInfo* x16_kernel_d(int n);
const KernelInfo* x16_kernel_e(int n);
const KernelInfo* x16_kernel_f(int n);
inline const KernelInfo* x16_kernel(int n) {
  const KernelInfo* k = x16_kernel_a(n);
  if (!k) k = x16_kernel_b(n);
  if (!k) k = x16_kernel_c(n);
  if (!k) k = x16_kernel_d(n);
  if (!k) k = x16_kernel_e(n);
  if (!k) k = x16_kernel_f(n);
  return k;
}
// The same kernel for any other N, by tile count: _a .. _f load 16-byte
// chunks (1 .. 16 tiles), _g .. _k 4-byte units (8 .. 16 tiles).
const KernelInfo* x16_ragged_a(int nt);
const KernelInfo* x16_ragged_b(int nt);
const KernelInfo* x16_ragged_c(int nt);
const KernelInfo* x16_ragged_d(int nt);
const KernelInfo* x16_ragged_e(int nt);
const KernelInfo* x16_ragged_f(int nt);
const KernelInfo* x16_ragged_g(int nt);
const KernelInfo* x16_ragged_h(int nt);
const KernelInfo* x16_ragged_i(int nt);
const KernelInfo* x16_ragged_j(int nt);
const KernelInfo* x16_ragged_k(int nt);
constexpr int gcd(int64_t a, int b) {
  while (b) {
    const int r = (int)(a % b);
    a = b;
    b = r;
  }
  return (int)a;
}
constexpr int ragged_tiles(int n, int unit) { return (n + unit - gcd(n, unit) + 15) / 16; }
// The kernel for rows of f channels of n inputs.  The tiles start at the
// whole load unit that holds a channel's first byte, up to unit - gcd(n, unit)
// bytes before it, so they must cover that many positions more than n.  From
// 8 tiles up, chunks are taken where they need no tile more than n alone and
// every row starts on a chunk: at F = 1024, T = 4096 they are 3-13% faster
// there (N = 200: 299 against 319 us; a chunk load moves 1 KB, a dword load
// one row of at most 256 bytes).  With a tile more they are slower (N = 230:
// 461 against 388), and where rows do not start on a chunk they take up to
// 16 phases against 4, each with its own sums to store and add.  Below 8
// tiles the array is bound by memory and a tile more costs little.  N = 255
// fits neither (its 258 positions are 17 tiles).
inline const KernelInfo* x16_any_kernel(int n, int64_t f) {
  if (n % 16 == 0) return x16_kernel(n);
  const KernelInfo* k = nullptr;
  int nt = ragged_tiles(n, 16);
  if (nt >= 8 && (nt > (n + 15) / 16 || f * n % 16 != 0)) {
    nt = ragged_tiles(n, 4);
    if (nt > 16) return nullptr;
    if (nt >= 8) {
      k = x16_ragged_g(nt);
      if (!k) k = x16_ragged_h(nt);
      if (!k) k = x16_ragged_i(nt);
      if (!k) k = x16_ragged_j(nt);
      if (!k) k = x16_ragged_k(nt);
      return k;
    }
    nt = ragged_tiles(n, 16);
  }
  k = x16_ragged_a(nt);
  if (!k) k = x16_ragged_b(nt);
  if (!k) k = x16_ragged_c(nt);
  if (!k) k = x16_ragged_d(nt);
  if (!k) k = x16_ragged_e(nt);
  if (!k) k = x16_ragged_f(nt);
  return k;
}
// Phases of time rows of a ragged kernel for rows of row_bytes = F*N.
inline int row_phases(const KernelInfo* k, int64_t row_bytes) {
  return k->load_unit ? k->load_unit / gcd(row_bytes, k->load_unit) : 1;
}

// Copy n[k] int2 values (re, im) from acc[k] to dst[k] for k < count; a
// null acc[k] writes zeros.  Pointers are 8-byte aligned device memory.
constexpr int DUMP_MAX = 24;
struct DumpParams {
  const int2* acc[DUMP_MAX];
  int2* dst[DUMP_MAX];
  int64_t n[DUMP_MAX];
  int count;
};
hipError_t dump_launch(int grid, hipStream_t s, const DumpParams& d);
// dst[i] = (prev ? prev[i] : 0) + sum of part[c * n + i] over c < chunks
hipError_t sum_launch(hipStream_t s, const int2* prev, const int2* part, int2* dst, int64_t n, int chunks);

}  // namespace xeng
