// k_chan.hip - F-stage channeliser (paper Sec. 2.1, Eq. 1-2) and its C
// entry points (include/xeng.h).
//
// Per spectrum s and input pair (2q, 2q + 1):
//  1. polyphase FIR: v[n] = sum_{p<4} h[pL + n] x[sL + pL + n] for both
//     inputs (L = 2F real samples per spectrum, h the Hamming-windowed sinc
//     prototype), packed as y[n] = v_2q[n] + j v_2q+1[n] (Eq. 1);
//  2. Stockham FFT of y, L points, natural order out;
//  3. Eq. 2: X_2q[k] = (Y[k] + conj Y[-k]) / 2, X_2q+1[k] = (Y[k] -
//     conj Y[-k]) / 2j, k < F, written to out[s][k][2q .. 2q + 1] (the
//     [time, channel, input] order of the X side).
// Float32 arithmetic; the tables (h and the twiddles e^{-2 pi i t / L}) are
// computed in double and rounded once, at compile time (chan_tables.hpp).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/xeng.h"
#include "chan_tables.hpp"

namespace xeng {
namespace {

constexpr int MAX_L = 2048;

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// e^{-2 pi i t / L} for 0 <= t < L from the half table
template <int L>
__device__ __forceinline__ float2 twiddle(const float2* tw, int t) {
  const float2 w = tw[t & (L / 2 - 1)];
  return t < L / 2 ? w : make_float2(-w.x, -w.y);
}

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }

// 4-point forward DFT in place
__device__ __forceinline__ void dft4(float2& x0, float2& x1, float2& x2, float2& x3) {
  const float2 s02 = cadd(x0, x2), d02 = csub(x0, x2);
  const float2 s13 = cadd(x1, x3);
  const float2 d13 = make_float2(x1.y - x3.y, x3.x - x1.x);  // -i (x1 - x3)
  x0 = cadd(s02, s13);
  x2 = csub(s02, s13);
  x1 = cadd(d02, d13);
  x3 = csub(d02, d13);
}

// 8-point forward DFT in place, natural order: X[2r] = DFT4(a_n + a_n+4)[r],
// X[2r+1] = DFT4((a_n - a_n+4) e^{-2 pi i n / 8})[r]
__device__ __forceinline__ void dft8(float2 (&a)[8]) {
  constexpr float R = 0.70710678118654752440f;
  float2 e0 = cadd(a[0], a[4]), e1 = cadd(a[1], a[5]), e2 = cadd(a[2], a[6]), e3 = cadd(a[3], a[7]);
  float2 o0 = csub(a[0], a[4]), o1 = csub(a[1], a[5]), o2 = csub(a[2], a[6]), o3 = csub(a[3], a[7]);
  o1 = make_float2((o1.x + o1.y) * R, (o1.y - o1.x) * R);      // x (1 - i) / sqrt 2
  o2 = make_float2(o2.y, -o2.x);                               // x (-i)
  o3 = make_float2((o3.y - o3.x) * R, -(o3.x + o3.y) * R);     // x (-1 - i) / sqrt 2
  dft4(e0, e1, e2, e3);
  dft4(o0, o1, o2, o3);
  a[0] = e0; a[2] = e1; a[4] = e2; a[6] = e3;
  a[1] = o0; a[3] = o1; a[5] = o2; a[7] = o3;
}

// Input pairs (units) per workgroup, L / 8 threads each.  `wide` for work
// that fills the chip: a store then writes 64 (L = 2048, where more do not
// fit the LDS) to 512 contiguous bytes.  With two pairs at L = 2048 (32 bytes)
// the cylinder case below took 1948 us against 1204: lines reached HBM half
// filled.  Narrow for less work, so that more CUs share it (N = 6, F = 1024,
// 23 spectra: 7.6 us against 11.0; N = 10, F = 256, 19 spectra: 5.3 against
// 9.7).
constexpr int pairs_per_wg(int L, bool wide) {
  if (L <= 64) return L == 64 ? 16 : 32;
  if (wide) return L == 2048 ? 4 : L == 1024 ? 8 : 16;
  return L >= 1024 ? 2 : L == 512 ? 4 : 8;
}
// Spectra per run at most.  L = 2048: 16 gave 1227 us, 8 1204, 4 1255; L =
// 1024 1063, 1128, 1278 (192 inputs, 4096 spectra).
constexpr int run_max(int L) { return L == 2048 ? 8 : 16; }
// Points of a unit's LDS buffer: a point of padding per 32, and a pitch that
// spreads the P units over the 32 banks of 8 bytes in the last step's reads
// (P units x 32 / P channels per half wave).
constexpr int buf_points(int L, int P) {
  int n = L + L / 32;
  while (n % (64 / P) != 32 / P) ++n;
  return n;
}

// A workgroup takes P units, a unit being one input pair over a run of
// `run` consecutive spectra (pair fastest), L / 8 threads per unit:
//  - thread t of a unit owns the points n = t + m L/8 (m < 8) of every
//    stage, which are the inputs of its first radix-8 butterfly, and keeps
//    their 32 filter taps in registers for the run;
//  - each input block of L samples is loaded once per run (one byte per
//    point), a spectrum ahead, and kept as packed bytes while the four
//    spectra that use it are formed;
//  - Stockham FFT: radix-8 passes and, where log2 L is no multiple of 3, one
//    radix-2 or radix-4 pass, butterflies in registers; between passes the
//    points go through LDS (two buffers per unit, one barrier per exchange);
//    the twiddles come from tables in LDS;
//  - Eq. 2 reads Y[k] and Y[L - k] from LDS; neighbouring lanes take the P
//    pairs of one channel, so each store writes 16 P contiguous bytes.
// 128 registers, so that 16 waves fit a CU: the input window as bytes instead
// of floats, twiddles from LDS, and exchange addresses that are a lane base
// plus a constant (hoisted per-point addresses alone took 64 registers).
//
// What bounds it: memory, with the stores first.  Cylinder shape (192 streams,
// 1024 channels, 2048 spectra: 3.2 GB out, 0.8 GB in): 1197 us, 3.4 TB/s,
// against 1682 with two pairs and 256 registers (8 waves per CU).  Without
// its stores it takes 800 us, without loads and stores 680; a plain fill
// writes 3.2 GB in 470 us.  F = 512, 4096 spectra: 1034 against 1330 us; F =
// 256, 8192: 957 against 1764.  F <= 128, formerly one workgroup per spectrum
// and pair with all points in LDS: N = 162, F = 64, 3014 spectra 94 against
// 554 us; N = 150, F = 16, 9000: 51 against 1003.
template <int L, int P>
__global__ __launch_bounds__(P * L / 8) __attribute__((amdgpu_waves_per_eu(4, 4))) void channelise(
    const int8_t* __restrict__ adc, int64_t n_samples, int pairs, int n_spec, int run, float4* __restrict__ out) {
  constexpr int TH = L / 8, F = L / 2, THREADS = P * TH;
  constexpr int N8 = L >= 512 ? 3 : L >= 64 ? 2 : 1;      // radix-8 passes
  constexpr int RL = L >> (3 * N8);                       // radix of the last pass (1: none)
  constexpr int BUF = buf_points(L, P);
  __shared__ float2 lds_all[2][P][BUF];
  __shared__ float2 w2_all[N8 > 1 ? 56 : 1], w3_all[N8 > 2 ? 448 : 1], wl_all[RL > 1 ? L / 2 : 1];
  const int pp = threadIdx.x / TH;
  const int t = threadIdx.x % TH;
  // workgroups are dealt to the 8 XCDs in turn: each takes a contiguous range
  const int64_t total = gridDim.x, b = blockIdx.x;
  const int64_t xq = total / 8, xr = total % 8, xcd = b % 8;
  const int64_t w = xcd * xq + (xcd < xr ? xcd : xr) + b / 8;
  const int64_t units = (int64_t)pairs * ((n_spec + run - 1) / run);
  const int64_t unit = min(w * P + pp, units - 1);        // past the end: computed, not stored
  const int q = (int)(unit % pairs), s0 = (int)(unit / pairs) * run;
  // runs never get longer from unit to unit: the first one's length bounds all
  const int first_s0 = (int)(w * P / pairs) * run;
  const int len = min(run, n_spec - first_s0);
  const float* tab = chan_tables<L>.h;
  const float2* tw = reinterpret_cast<const float2*>(chan_tables<L>.tw);

  if constexpr (N8 > 1)
    for (int i = threadIdx.x; i < 56; i += THREADS) w2_all[i] = twiddle<L>(tw, ((i / 8 + 1) * (i % 8) * (L / 64)) & (L - 1));
  if constexpr (N8 > 2)
    for (int i = threadIdx.x; i < 448; i += THREADS) w3_all[i] = twiddle<L>(tw, ((i / 64 + 1) * (i % 64) * (L / 512)) & (L - 1));
  if constexpr (RL > 1)
    for (int i = threadIdx.x; i < L / 2; i += THREADS) wl_all[i] = tw[i];

  float hr[4][8];
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int m = 0; m < 8; ++m) hr[p][m] = tab[p * L + t + m * TH];

  const int8_t* xs[2] = {adc + (int64_t)(2 * q) * n_samples + t, adc + (int64_t)(2 * q + 1) * n_samples + t};
  int inc[2][8];       // loads of the next block
  auto load_block = [&](int blk) {   // (a unit past its own end reloads the last block)
    const int64_t at = (int64_t)min(blk, n_spec + 2) * L;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int m = 0; m < 8; ++m) inc[c][m] = xs[c][at + m * TH];
  };
  // the four blocks of a spectrum, a byte per point
  uint32_t win[4][2][2];
  auto pack = [&](uint32_t (&to)[2][2]) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t lo = __builtin_amdgcn_perm(inc[c][4 * h + 1], inc[c][4 * h], 0x0c0c0400u);
        const uint32_t hi = __builtin_amdgcn_perm(inc[c][4 * h + 3], inc[c][4 * h + 2], 0x04000c0cu);
        to[c][h] = lo | hi;
      }
  };
  auto point = [&](const uint32_t (&b)[2][2], int c, int m) {
    return (float)(int8_t)(b[c][m >> 2] >> (8 * (m & 3)));
  };
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    load_block(s0 + k);
    pack(win[k]);
  }

  // the pairs and spectra this thread stores: unit u % P of the workgroup
  const int p2 = threadIdx.x % P, k2 = threadIdx.x / P;
  const int64_t unit2 = w * P + p2;
  const int s2 = (int)(unit2 / pairs) * run;
  const int len2 = unit2 < units ? min(run, n_spec - s2) : 0;
  float4* o = out + ((int64_t)s2 * F + k2) * pairs + unit2 % pairs;

  int e = 0;  // buffer of the next exchange
  // Exchanges: write at w(m), barrier, read the thread's points t + m TH back
  // at r(m).  Both are a lane base plus a constant (or, the second exchange,
  // xor a constant), without bank conflicts:
  //   PAD  point i at i + i / 32 (writes 8 t + m, and rows of 64);
  //   XOR  point i at i ^ 8 (i / 64 % 4) (writes 64 (t / 8) + t % 8 + 8 m).
  const int pad_r = t + (t >> 5), xor_r = t ^ (((t >> 6) & 3) << 3);
  auto put = [&](const float2 (&a)[8], auto w) {
    float2* to = &lds_all[e][pp][0];
#pragma unroll
    for (int m = 0; m < 8; ++m) to[w(m)] = a[m];
    __syncthreads();
  };
  auto get = [&](float2 (&a)[8], auto r) {
    const float2* from = &lds_all[e][pp][0];
#pragma unroll
    for (int m = 0; m < 8; ++m) a[m] = from[r(m)];
    e ^= 1;
  };
  auto read_pad = [&](int m) { return pad_r + m * TH + ((m * TH) >> 5); };
  auto read_xor = [&](int m) { return (xor_r ^ ((((m * TH) >> 6) & 3) << 3)) + m * TH; };
  const int w1 = 8 * t + (t >> 2);
  const int w2 = 8 * (t & ~7) + (t & 7), w2x = w2 | (((t >> 3) & 3) << 3);
  const int w3 = 8 * (t & ~63) + (t & 63), w3p = w3 + (w3 >> 5);
  __syncthreads();  // the twiddles
#pragma unroll 1
  for (int j = 0; j < len; ++j) {
    // Eq. 1 after the polyphase filter: y = v_2q + j v_2q+1
    float2 a[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      float v[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        v[c] = hr[0][m] * point(win[0], c, m);
        v[c] = fmaf(hr[1][m], point(win[1], c, m), v[c]);
        v[c] = fmaf(hr[2][m], point(win[2], c, m), v[c]);
        v[c] = fmaf(hr[3][m], point(win[3], c, m), v[c]);
      }
      a[m] = make_float2(v[0], v[1]);
    }
    load_block(s0 + j + 4);
    // pass 1 (Ns = 1): outputs to 8 t + m
    dft8(a);
    put(a, [&](int m) { return w1 + m; });
    get(a, read_pad);
    if constexpr (N8 > 1) {  // pass 2 (Ns = 8)
#pragma unroll
      for (int m = 1; m < 8; ++m) a[m] = cmul(a[m], w2_all[(m - 1) * 8 + (t & 7)]);
      dft8(a);
      if constexpr (N8 == 2 && RL == 1) {
        put(a, [&](int m) { return w2 + 8 * m; });
      } else {
        put(a, [&](int m) { return w2x ^ (8 * m); });
        get(a, read_xor);
      }
    }
    if constexpr (N8 > 2) {  // pass 3 (Ns = 64)
#pragma unroll
      for (int m = 1; m < 8; ++m) a[m] = cmul(a[m], w3_all[(m - 1) * 64 + (t & 63)]);
      dft8(a);
      if constexpr (RL == 1) {
        put(a, [&](int m) { return w3 + 64 * m; });
      } else {
        put(a, [&](int m) { return w3p + 66 * m; });
        get(a, read_pad);
      }
    }
    // last pass (Ns = L / RL): butterfly j = t + i L/8 reads points j + m L/RL
    if constexpr (RL == 4) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int jj = t + i * TH;
        float2 b0 = a[i], b1 = cmul(a[i + 2], wl_all[jj]), b2 = cmul(a[i + 4], twiddle<L>(wl_all, 2 * jj)),
               b3 = cmul(a[i + 6], twiddle<L>(wl_all, 3 * jj));
        dft4(b0, b1, b2, b3);
        a[i] = b0; a[i + 2] = b1; a[i + 4] = b2; a[i + 6] = b3;
      }
      put(a, [&](int m) { return t + m * TH; });
    } else if constexpr (RL == 2) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 b = cmul(a[i + 4], wl_all[t + i * TH]);
        const float2 u = a[i];
        a[i] = cadd(u, b);
        a[i + 4] = csub(u, b);
      }
      put(a, [&](int m) { return t + m * TH; });
    }
    // The next block's bytes are taken here, before this spectrum's stores: a
    // wait for loads that are younger than stores waits for the stores too.
    uint32_t next[2][2];
    pack(next);
    asm volatile("" : "+v"(next[0][0]), "+v"(next[0][1]), "+v"(next[1][0]), "+v"(next[1][1]));
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        win[0][c][h] = win[1][c][h], win[1][c][h] = win[2][c][h], win[2][c][h] = win[3][c][h];
        win[3][c][h] = next[c][h];
      }
    // Eq. 2 split
    if (j < len2) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float2 yk = lds_all[e][p2][k2 + r * TH];
        const float2 ym = r == 0 ? lds_all[e][p2][(L - k2) & (L - 1)] : lds_all[e][p2][L - k2 - r * TH];
        const float dr = yk.x - ym.x, di = yk.y + ym.y;   // Y[k] - conj(Y[-k])
        o[(int64_t)r * TH * pairs] = make_float4(0.5f * (yk.x + ym.x), 0.5f * (yk.y - ym.y), 0.5f * di, -0.5f * dr);
      }
    }
    o += (int64_t)F * pairs;
    e ^= 1;
  }
}

template <int L, bool WIDE>
hipError_t launch_channelise(const int8_t* adc, int64_t n_samples, int pairs, int n_spec, float* out, hipStream_t st) {
  constexpr int P = pairs_per_wg(L, WIDE);
  // Run length: the fewest rounds of workgroups over the CUs (16 waves each)
  // times the spectra of a run and its start (taps, tables, three more
  // blocks: about half a spectrum's time).  Up to L = 64 a wave's byte loads
  // touch a line per unit and bound the kernel well before the CUs are full,
  // so the blocks loaded count, r + 3 per run (N = 70, F = 8, 4806 spectra:
  // 40, 26, 16 and 22 us in runs of 1, 2, 7 and 16; N = 178, F = 16, 700: 13,
  // 11, 16 and 23).
  constexpr int64_t SLOTS = 256 * (1024 / (P * L / 8));
  int run = 1;
  double best = 0;
  for (int r = 1; r <= run_max(L); ++r) {
    const int64_t w = ((int64_t)pairs * ((n_spec + r - 1) / r) + P - 1) / P;
    const double cost = L <= 64 ? (4.0 * w / SLOTS + 1.0) * (r + 3) : (double)((w + SLOTS - 1) / SLOTS) * (r + 0.5);
    if (best == 0 || cost <= best) best = cost, run = r;
  }
  const int64_t wgs = ((int64_t)pairs * ((n_spec + run - 1) / run) + P - 1) / P;
  if (wgs > 2147483647LL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((channelise<L, P>), dim3((unsigned)wgs), dim3(P * L / 8), 0, st, adc, n_samples, pairs, n_spec,
                     run, reinterpret_cast<float4*>(out));
  return hipGetLastError();
}

// Wide workgroups where single spectra of them would fill the CUs.
template <int L>
hipError_t launch_channelise(const int8_t* adc, int64_t n_samples, int pairs, int n_spec, float* out, hipStream_t st) {
  if ((int64_t)pairs * n_spec >= 256 * pairs_per_wg(L, true) && pairs >= pairs_per_wg(L, false))
    return launch_channelise<L, true>(adc, n_samples, pairs, n_spec, out, st);
  return launch_channelise<L, false>(adc, n_samples, pairs, n_spec, out, st);
}

int log2_exact(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return (1 << l) == v ? l : -1;
}

}  // namespace
}  // namespace xeng

extern "C" int64_t xeng_channelise_spectra(int64_t n_samples, int32_t n_chans) {
  if (n_samples < 0 || n_chans < 1) return -1;
  const int64_t L = 2LL * n_chans;
  const int64_t s = n_samples / L - xeng::TAPS + 1;
  return s > 0 ? s : 0;
}

extern "C" int64_t xeng_channelise_table_floats(int32_t n_chans) {
  if (n_chans < 1) return -1;
  return (int64_t)xeng::TAPS * 2 * n_chans + 2 * n_chans;  // h[4L] + L/2 complex twiddles
}

namespace xeng {
namespace {

int channelise_impl(const int8_t* d_adc, int64_t n_samples, int32_t n_inputs, int32_t n_chans, float* d_out,
                    void* hip_stream) {
  const int L = 2 * n_chans;
  if (!d_adc || n_inputs < 2 || n_inputs % 2 || n_chans < 8 || L > MAX_L || log2_exact(L) < 0 || n_samples < 0 ||
      n_samples % 8 || (reinterpret_cast<uintptr_t>(d_adc) & 7u) || (reinterpret_cast<uintptr_t>(d_out) & 15u))
    return XENG_EINVAL;
  const int64_t S = xeng_channelise_spectra(n_samples, n_chans);
  if (S == 0) return XENG_OK;  // (d_out is not touched and may be null)
  if (!d_out || S > 2147483647LL - 64) return XENG_EINVAL;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  const int pairs = n_inputs / 2;
  hipError_t e = hipErrorInvalidValue;
  switch (L) {
    case 16: e = launch_channelise<16>(d_adc, n_samples, pairs, (int)S, d_out, st); break;
    case 32: e = launch_channelise<32>(d_adc, n_samples, pairs, (int)S, d_out, st); break;
    case 64: e = launch_channelise<64>(d_adc, n_samples, pairs, (int)S, d_out, st); break;
    case 128: e = launch_channelise<128>(d_adc, n_samples, pairs, (int)S, d_out, st); break;
    case 256: e = launch_channelise<256>(d_adc, n_samples, pairs, (int)S, d_out, st); break;
    case 512: e = launch_channelise<512>(d_adc, n_samples, pairs, (int)S, d_out, st); break;
    case 1024: e = launch_channelise<1024>(d_adc, n_samples, pairs, (int)S, d_out, st); break;
    case 2048: e = launch_channelise<2048>(d_adc, n_samples, pairs, (int)S, d_out, st); break;
  }
  return e == hipSuccess ? XENG_OK : e == hipErrorInvalidValue ? XENG_EINVAL : XENG_EDEVICE;
}

}  // namespace
}  // namespace xeng

extern "C" int xeng_channelise(const int8_t* d_adc, int64_t n_samples, int32_t n_inputs, int32_t n_chans,
                               float* d_out, float* d_tables, void* hip_stream) {
  if (!d_tables || (reinterpret_cast<uintptr_t>(d_tables) & 15u)) return XENG_EINVAL;
  return xeng::channelise_impl(d_adc, n_samples, n_inputs, n_chans, d_out, hip_stream);
}

extern "C" int xeng_channelise_noalloc(const int8_t* d_adc, int64_t n_samples, int32_t n_inputs,
                                       int32_t n_chans, float* d_out, void* hip_stream) {
  return xeng::channelise_impl(d_adc, n_samples, n_inputs, n_chans, d_out, hip_stream);
}
