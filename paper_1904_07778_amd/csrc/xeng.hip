// xeng.hip - host side of the X-engine C ABI (declared in include/xeng.h).
//
// A plan holds, per array slot, the HBM-resident int32 accumulator
// [F][nbl][2], the number of samples integrated since the last dump, and the
// kernel configuration chosen for its N.  xeng_correlate validates, applies
// the overflow guard and launches: one launch per array in a plain plan, one
// captured graph around the batch kernel in a batched plan.
// xeng_dump copies the accumulators out and clears them on the plan's
// stream.  Slots can be attached and detached between calls (admission in a
// serving loop).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/xeng.h"
#include "batch.hpp"
#include "kernels.hpp"

namespace {

using xeng::KernelInfo;

struct ArrayState {
  xeng_array_desc d{};
  bool active = false;  // slot holds an array (attached, not detached)
  int32_t* acc = nullptr;
  size_t acc_bytes = 0;
  int64_t n_integrated = 0;
  bool clean = true;   // integration is empty (no launch since the last dump or clear)
  bool zeroed = true;  // accumulator memory holds zeros (a dump does not clear it:
                       // the next launch overwrites it with plain stores, or
                       // zeroes it first when it must add atomically)
  const int32_t* prev = nullptr;  // during xeng_correlate_dump: the earlier samples' sums,
                                  // while acc is the caller's destination
  const KernelInfo* k = nullptr;  // kernel of the plain launch
  int split = 0;                  // plain launch: aim for split * n_cu workgroups; 0: modelled (choose)
  const KernelInfo* other = nullptr;  // the kernel of the calls it is modelled faster for (choose)
  int32_t* part = nullptr;        // plain plan: room for time chunks' sums, of which a call
  int part_chunks = 0;            // uses part_chunks; allocated for part_room
  int part_room = 0;
  int32_t* old_part = nullptr;    // the room before the autotuner chose a larger one
  mutable int64_t chosen_T = -1;  // choose's last pick, of calls of this length
  mutable const KernelInfo* chosen_k = nullptr;
  mutable int64_t chosen_ts = 0;
  bool own_launch = false;        // batched plan: a plain launch of its own inside the
                                  // graph instead of items of the batch launch
};

// ---- tuning cache: the launch shapes the autotuner picked, by GPU
// architecture, plan kind, N and the power-of-two buckets of F and T, for the
// whole process (xeng_tune_cache_save / _load write and read it as text).
enum KernelKind { KIND_X16 = 0, KIND_X32 = 1, KIND_STAGE = 2 };
const char* const kKindNames[] = {"ring16", "ring32", "staging"};

const KernelInfo* kernel_of(int kind, const xeng_array_desc& d) {
  const int32_t n = d.n_inputs;
  switch (kind) {
    case KIND_X16: return xeng::x16_any_kernel(n, d.n_chans);
    case KIND_X32: return xeng::x32_kernel(n);
    case KIND_STAGE: return xeng::stage_kernel((n + 15) / 16);
    default: return nullptr;
  }
}

int kind_of(const KernelInfo* k, const xeng_array_desc& d) {
  if (k == xeng::x16_any_kernel(d.n_inputs, d.n_chans)) return KIND_X16;
  if (k == xeng::x32_kernel(d.n_inputs)) return KIND_X32;
  return KIND_STAGE;
}

int bucket(int64_t v) {  // ceil(log2 v)
  int b = 0;
  while (((int64_t)1 << b) < v && b < 62) ++b;
  return b;
}

struct TuneKey {
  std::string arch;
  int batched, n, fb, tb;
  int phases;  // of the 16-row ring kernel (row_phases): they depend on F itself
  bool operator<(const TuneKey& o) const {
    return std::tie(arch, batched, n, fb, tb, phases) < std::tie(o.arch, o.batched, o.n, o.fb, o.tb, o.phases);
  }
};
struct TuneVal {
  int kind, split, own;
};
std::mutex g_tune_mu;
std::map<TuneKey, TuneVal> g_tune;

}  // namespace

struct xeng_plan_s {
  int device = 0;
  int n_cu = 256;
  std::string arch;       // gcnArchName of the device (tuning-cache key)
  hipStream_t stream = nullptr;
  bool own_stream = false;
  bool dead = false;
  bool batched = false;   // calls go through the batch launch
  int batch_split = 0;    // batch: cut items to about batch_split per CU; 0: modelled
  std::vector<ArrayState> arrays;
  int32_t* counters = nullptr;  // batch queue heads, zero between launches
  // Ring of instantiated graphs of batched calls, each with the event of its
  // last launch (a graph is updated only once that launch has completed).
  static constexpr int GRAPH_RING = 4;
  hipGraphExec_t exec[GRAPH_RING] = {};
  hipEvent_t done[GRAPH_RING] = {};
  int next_graph = 0;
  xeng_stats_t stats{};   // counters since the plan was made
  bool trace = false;     // XENG_TRACE set: one stderr line per launch
  std::string err;
};

namespace {

int fail(xeng_plan_t* p, int status, const char* fmt, ...) {
  if (p) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    p->err = buf;
    if (status == XENG_EDEVICE) p->dead = true;
  }
  return status;
}

int hip_fail(xeng_plan_t* p, hipError_t e, const char* what) {
  return fail(p, XENG_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

bool aligned16(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15u) == 0; }

int64_t nbl_of(int32_t n) { return (int64_t)n * (n + 1) / 2; }

// Modelled time of a call of the 16-row ring kernel in ts time chunks per
// channel group and phase: rounds of workgroups over the CUs, each a start
// (launch or hand-over, ring fill, epilogue: 4 us, 3 for a single channel)
// plus its rows.  A CU's rows go at 1.2 times its matrix-core cycles (at 2 GHz) and at no more than 25 bytes
// per ns (what one CU streams through its ring, also with most of the chip
// idle: 24-28 measured for N = 32 .. 112); a workgroup alone takes 1 ns a row
// longer and no less than 4 (N = 16, where four share a CU, gains by more of
// them: F = 1024, T = 8192 36 us in one chunk, 32 in two).  Measured against
// it, kernel times in us for N x F x T: 100x64x4096 in 1, 4, 8, 16 chunks 80,
// 36, 27, 30 (105 with atomics in 16); 192x35x6736 in 1, 4, 8 chunks 82, 35,
// 45; 96x200x4096 in 1, 4, 8 67, 37, 51; 32x64x4096 in 1, 4, 8, 16 25, 16, 12,
// 13; 128x64x2048 in 1, 2, 4 18, 20, 22.
// Nanoseconds per row of a workgroup's CU (busy), and of one workgroup alone.
double busy_ns(const KernelInfo* k) {
  const double mfma = k->nt * (k->nt + 1) / (double)k->w / 2.0 / 2.0;  // 16 cycles per unit and 32 rows
  return std::max(1.2 * mfma, k->cpw * 16.0 * k->nt / 25.0);
}
double row_ns(const KernelInfo* k) {
  const double mfma = k->nt * (k->nt + 1) / (double)k->w / 2.0 / 2.0;
  return std::max({1.2 * mfma + 1.0, busy_ns(k), 4.0});
}

// Workgroups of a 16-row ring kernel that run on one CU together: by LDS, and
// by registers (36 a lane at one tile, 84 at two, 224-248 at 8 tiles over four
// waves, over 256 at any other count from 4 up).
int together(const KernelInfo* k) {
  const int regs = k->nt <= 3 ? 4 : k->nt == 8 ? 2 : 1;
  return std::max(1, std::min(regs, 160 * 1024 / k->lds_bytes));
}

// Adding up the sums of n workgroups per channel group: stored and summed by
// a second kernel (its launch, and the store, the read and the sum at 6 bytes
// per ps, out of the caches mostly), or without room for them added
// atomically (140 G adds/s: F = 1001, N = 61 in 16 phases 485 us, N = 201 in 4
// 1157, N = 250 in 2 919).
double combine_us(const ArrayState& s, int64_t n) {
  if (n == 1) return 0;
  const double acc = (double)s.acc_bytes;
  return 5.0 + (n <= s.part_chunks ? (2 * n + 1) * acc / 6e6 : n * acc / 4.0 / 140e3);
}

double split_us(const xeng_plan_t* p, const ArrayState& s, int64_t rows, int phases, int ts) {
  const int64_t groups = (s.d.n_chans + s.k->cpw - 1) / s.k->cpw;
  const int64_t wgs = groups * phases * ts;
  const int64_t per_cu = (wgs + p->n_cu - 1) / p->n_cu;
  const int64_t rounds = (per_cu + together(s.k) - 1) / together(s.k);
  const double rows_us = (double)((rows + ts - 1) / ts) * std::max(per_cu * busy_ns(s.k), rounds * row_ns(s.k)) * 1e-3;
  return rounds * (s.k->cpw == 1 ? 3.0 : 4.0) + rows_us + combine_us(s, (int64_t)ts * phases);
}

// Modelled time of a call of the staging kernel: `row` ns from row to row of
// a workgroup (loads to registers, transpose, LDS, matrix products one after
// the other), `more` for every further workgroup of its CU, by the waves of a
// channel (five tiles stand out: 15 tile pairs in one wave); byte loads, or
// dwords where N is a multiple of 4.  Measured us, F = 1001, T = 4096: N = 7
// 171, 61 342, 75 963, 113 894, 145 1536, 201 2948, 250 3093; N = 52 96, 100
// 280, 152 455, 200 879, 252 840.
double stage_us(const xeng_plan_t* p, const ArrayState& s, const KernelInfo* k, int64_t T, int64_t ts) {
  const bool dwords = s.d.n_inputs % 4 == 0;
  const double row = k->nt == 5 ? (dwords ? 54 : 154) : (dwords ? 30 : 80) + k->nt;
  const double more = k->nt == 5 ? 240 : k->w == 1 ? 30 + 12 * k->nt : k->w == 2 ? 108 : k->w <= 4 ? 95 : 190;
  const int64_t groups = (s.d.n_chans + k->cpw - 1) / k->cpw;
  const int64_t per_cu = (groups * ts + p->n_cu - 1) / p->n_cu;
  return 5.0 + (T + ts - 1) / ts * (row + (per_cu - 1) * more * (dwords ? 0.3 : 1.0)) * 1e-3 + combine_us(s, ts) +
         (double)s.acc_bytes / 6e6;
}

// Kernel and time chunks (per channel group and phase) of a call of T
// samples.  A tuned array takes the kernel and the split it was given.  An
// untuned one on the 16-row ring kernel takes the chunks with the least
// modelled time; and where its rows come in phases, each of which leaves its
// own sums to store and add, it takes the staging kernel for the calls that
// this is modelled faster for: few rows per phase, or no room for the sums
// (kernel times in us, staging against ring: N = 37, F = 1001, T = 512 48 and
// 98, T = 4096 231 and 130; N = 201, F = 1001, T = 512, whose sums do not fit
// the room, 330 and 1161, T = 4096 2948 and 1247; in a batched plan, which
// keeps no room, N = 37, F = 1001, T = 512 64 and 216.  Over 660 calls of 38
// N in both forms of plan the pick is 0.7% slower than the better one on
// average, and 21 times by more than 10%; the ring kernel is 271 times).
struct Choice {
  const KernelInfo* k;
  int64_t ts;
};

int64_t aimed_chunks(const xeng_plan_t* p, const KernelInfo* k, int32_t F, int64_t rows, int phases, int split) {
  const int64_t wgs = (int64_t)((F + k->cpw - 1) / k->cpw) * phases;
  const int64_t ts = ((int64_t)split * p->n_cu + wgs - 1) / wgs;
  return std::max<int64_t>(1, std::min<int64_t>(ts, rows / 256));
}

Choice choose(const xeng_plan_t* p, const ArrayState& s, int64_t T) {
  const int phases = xeng::row_phases(s.k, (int64_t)s.d.n_chans * s.d.n_inputs);
  const int64_t rows = (T + phases - 1) / phases;  // of the longest phase
  if (s.split > 0) return Choice{s.k, aimed_chunks(p, s.k, s.d.n_chans, rows, phases, s.split)};
  if (T == s.chosen_T) return Choice{s.chosen_k, s.chosen_ts};
  double best = 0;
  Choice c{s.k, 1};
  for (int ts = 1; ts <= 64 && (ts == 1 || rows / ts >= 64); ++ts) {
    const double us = split_us(p, s, rows, phases, ts);
    if (best == 0 || us < best) best = us, c.ts = ts;
  }
  if (s.other) {
    const int64_t ts = aimed_chunks(p, s.other, s.d.n_chans, T, 1, s.other->split);
    if (stage_us(p, s, s.other, T, ts) < best) c = Choice{s.other, ts};
  }
  s.chosen_T = T;
  s.chosen_k = c.k;
  s.chosen_ts = c.ts;
  return c;
}

// One call's launch, and how its sums reach the accumulator.
struct Grid {
  const KernelInfo* k;
  dim3 dim;         // channel groups x time chunks
  int64_t t_chunk;  // rows of a chunk
  int mode;         // EpiMode
  bool parts;       // the chunks are stored in s.part and summed by a second kernel
  int chunks;       // of them, those that hold samples
};

Grid grid_for(const xeng_plan_t* p, const ArrayState& s, int64_t T) {
  const Choice c = choose(p, s, T);
  const int ngroups = (s.d.n_chans + c.k->cpw - 1) / c.k->cpw;
  const int phases = xeng::row_phases(c.k, (int64_t)s.d.n_chans * s.d.n_inputs);
  const int64_t rows = (T + phases - 1) / phases;  // of the longest phase
  int64_t ts = std::max<int64_t>(c.ts, (rows + c.k->max_t_per_wg - 1) / c.k->max_t_per_wg);
  Grid g{};
  g.k = c.k;
  g.t_chunk = (rows + ts - 1) / ts;
  g.t_chunk = (g.t_chunk + xeng::KS - 1) / xeng::KS * xeng::KS;
  ts = (rows + g.t_chunk - 1) / g.t_chunk * phases;
  g.dim = dim3((unsigned)ngroups, (unsigned)ts, 1);
  g.parts = c.k->chunks && ts > 1 && ts <= s.part_chunks;
  // the last chunk of a phase may be empty: phase ph has rows left while
  // last * t_chunk * phases + ph < T
  const int64_t before = ts - phases;
  g.chunks = (int)(before + std::min<int64_t>(phases, T - before / phases * g.t_chunk * phases));
  g.mode = ts > 1 ? (g.parts ? xeng::EPI_STORE : xeng::EPI_ATOMIC) : (s.clean ? xeng::EPI_STORE : xeng::EPI_ADD);
  return g;
}


bool valid_desc(const xeng_array_desc& d) {
  return d.n_inputs >= 1 && d.n_inputs <= XENG_MAX_INPUTS && d.n_chans >= 1 &&
         (int64_t)d.n_chans * d.n_inputs <= INT32_MAX &&  // one time row indexes in 32 bits
         d.max_time_per_call >= 1 && d.max_time_per_call <= XENG_MAX_INTEGRATION;
}

bool kernel_fits(const KernelInfo* k, const xeng_array_desc& d) {
  if (!k) return false;
  const int64_t row_bytes = (int64_t)d.n_chans * d.n_inputs;
  return k->max_row_bytes == 0 || row_bytes * xeng::row_phases(k, row_bytes) <= k->max_row_bytes;
}

// Default kernel for an array: the 16-row-tile ring kernel where it takes N
// (all but 255) and the time rows fit its 32-bit offsets, else the
// 32-row-tile ring kernel when N is a multiple of 16, else the staging
// kernel of 16-row tiles.
const KernelInfo* default_kernel(const xeng_array_desc& d) {
  const KernelInfo* k = xeng::x16_any_kernel(d.n_inputs, d.n_chans);
  if (kernel_fits(k, d)) return k;
  if (d.n_inputs % 16 == 0 && (k = xeng::x32_kernel(d.n_inputs))) return k;
  return xeng::stage_kernel((d.n_inputs + 15) / 16);
}

void set_kernel(ArrayState& s, const KernelInfo* k, int split) {
  s.k = k;
  s.split = split;
  s.other = split == 0 && xeng::row_phases(k, (int64_t)s.d.n_chans * s.d.n_inputs) > 1
                ? xeng::stage_kernel((s.d.n_inputs + 15) / 16)
                : nullptr;
  s.chosen_T = -1;
}

TuneKey tune_key(const xeng_plan_t* p, const ArrayState& s, int64_t T) {
  const KernelInfo* k = kernel_of(KIND_X16, s.d);
  return TuneKey{p->arch, p->batched ? 1 : 0, s.d.n_inputs, bucket(s.d.n_chans), bucket(T),
                 k ? xeng::row_phases(k, (int64_t)s.d.n_chans * s.d.n_inputs) : 1};
}

void apply_cached(const xeng_plan_t* p, ArrayState& s, int64_t T) {
  TuneKey key = tune_key(p, s, T);
  std::lock_guard<std::mutex> lock(g_tune_mu);
  auto it = g_tune.find(key);
  if (it == g_tune.end() && key.phases > 1) {
    // A choice made for rows of whole load units (and all lines of older
    // files) says nothing of the ring kernel in phases.
    key.phases = 1;
    it = g_tune.find(key);
    if (it != g_tune.end() && it->second.kind == KIND_X16) return;
  }
  if (it == g_tune.end()) return;
  const KernelInfo* k = kernel_of(it->second.kind, s.d);
  if (!kernel_fits(k, s.d)) return;
  set_kernel(s, k, it->second.split);
  s.own_launch = p->batched && it->second.own;
}

// The batched plan's own choice (items per workgroup) is kept under N = 0,
// keyed by the base-2 bucket of the plan's array count.
TuneKey plan_key(const xeng_plan_t* p, int32_t n_arrays) { return TuneKey{p->arch, 1, 0, 0, bucket(n_arrays), 1}; }

void apply_cached_plan(xeng_plan_t* p, int32_t n_arrays) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  auto it = g_tune.find(plan_key(p, n_arrays));
  if (it != g_tune.end()) p->batch_split = it->second.split;
}

void record_choice(const xeng_plan_t* p, const ArrayState& s, int64_t T) {
  const TuneKey key = tune_key(p, s, T);
  std::lock_guard<std::mutex> lock(g_tune_mu);
  g_tune[key] = TuneVal{kind_of(s.k, s.d), s.split, s.own_launch ? 1 : 0};
}

constexpr size_t MAX_PART_BYTES = (size_t)256 << 20;

// Chunks of the longest call that a plain plan keeps room for (bounded; calls
// split further add atomically).
int room_chunks(const xeng_plan_t* p, ArrayState& s) {
  if (p->batched || !s.k->chunks) return 0;
  const int keep = s.part_chunks;
  s.part_chunks = (int)std::min<size_t>(INT_MAX, MAX_PART_BYTES / s.acc_bytes);
  const Grid g = grid_for(p, s, s.d.max_time_per_call);
  s.part_chunks = keep;
  s.chosen_T = -1;  // (that was with the most room)
  return g.parts ? (int)g.dim.y : 0;
}

int init_slot(xeng_plan_t* p, ArrayState& s, const xeng_array_desc& d) {
  s = ArrayState{};
  s.d = d;
  s.acc_bytes = (size_t)d.n_chans * nbl_of(d.n_inputs) * 2 * sizeof(int32_t);
  const KernelInfo* k = default_kernel(d);
  set_kernel(s, k, k->split);
  apply_cached(p, s, d.max_time_per_call);
  hipError_t e = hipMalloc(&s.acc, s.acc_bytes);
  if (e != hipSuccess) {
    s.acc = nullptr;
    return e == hipErrorOutOfMemory ? fail(p, XENG_ENOMEM, "accumulator of %zu bytes", s.acc_bytes)
                                    : hip_fail(p, e, "accumulator allocation");
  }
  // The room is not needed: where there is no memory for it, split calls add
  // atomically.
  s.part_chunks = room_chunks(p, s);
  if (s.part_chunks && hipMalloc(&s.part, s.part_chunks * s.acc_bytes) != hipSuccess) {
    (void)hipGetLastError();
    s.part = nullptr;
    s.part_chunks = 0;
  }
  s.part_room = s.part_chunks;
  e = hipMemsetAsync(s.acc, 0, s.acc_bytes, p->stream);
  if (e != hipSuccess) return hip_fail(p, e, "accumulator clear");
  s.active = true;
  return XENG_OK;
}

// Give the accumulators of the given arrays the values that atomic adds start
// from, with one launch of the dump kernel (which may be recorded into a
// graph): the earlier samples' sums, or zeros.
int init_for_atomics(xeng_plan_t* p, const std::vector<ArrayState*>& arrays) {
  xeng::DumpParams dp{};
  int64_t most = 0;
  auto flush = [&]() -> int {
    if (dp.count == 0) return XENG_OK;
    const int64_t blocks = std::min<int64_t>((most + 1023) / 1024, 8LL * p->n_cu);
    hipError_t e = xeng::dump_launch((int)std::max<int64_t>(1, blocks), p->stream, dp);
    dp.count = 0;
    most = 0;
    return e == hipSuccess ? XENG_OK : hip_fail(p, e, "accumulator clear");
  };
  for (ArrayState* s : arrays) {
    dp.acc[dp.count] = reinterpret_cast<const int2*>(s->prev);
    dp.dst[dp.count] = reinterpret_cast<int2*>(s->acc);
    dp.n[dp.count] = (int64_t)(s->acc_bytes / sizeof(int2));
    most = std::max(most, dp.n[dp.count]);
    s->zeroed = s->clean;
    if (++dp.count == xeng::DUMP_MAX) {
      const int st = flush();
      if (st != XENG_OK) return st;
    }
  }
  return flush();
}

// Whether a launch that adds atomically needs that first: an empty
// integration in memory that does not hold zeros, or earlier sums elsewhere.
bool needs_init(const ArrayState& s) { return s.clean ? !s.zeroed : s.prev != nullptr; }

xeng::Args base_args(const ArrayState& s, const KernelInfo* k, const uint8_t* v, int64_t T) {
  xeng::Args a{};
  a.v = v;
  a.acc = s.acc;
  a.T = T;
  a.F = s.d.n_chans;
  a.N = s.d.n_inputs;
  a.period = xeng::row_phases(k, (int64_t)s.d.n_chans * s.d.n_inputs);
  if (s.prev)
    a.prev_off = (int64_t)(reinterpret_cast<uintptr_t>(s.prev) - reinterpret_cast<uintptr_t>(s.acc)) /
                 (int64_t)sizeof(int32_t);
  return a;
}

int launch_plain(xeng_plan_t* p, ArrayState& s, const uint8_t* v, int64_t T) {
  const Grid g = grid_for(p, s, T);
  xeng::Args args = base_args(s, g.k, v, T);
  args.t_chunk = g.t_chunk;
  args.mode = g.mode;
  if (g.parts) {
    args.acc = s.part;
    args.chunk_stride = (int64_t)(s.acc_bytes / sizeof(int32_t));
  }
  ++p->stats.launches;
  if (p->trace)
    fprintf(stderr, "xeng: plan %p plain launch N=%d F=%d T=%lld kernel=%s grid=%ux%u threads=%d mode=%d chunks=%d\n",
            (void*)p, args.N, args.F, (long long)T, kKindNames[kind_of(g.k, s.d)], g.dim.x, g.dim.y, g.k->threads,
            args.mode, g.parts ? g.chunks : 0);
  if (args.mode == xeng::EPI_ATOMIC && needs_init(s)) {
    const int st = init_for_atomics(p, {&s});
    if (st != XENG_OK) return st;
  }
  hipError_t e = g.k->launch(g.dim, p->stream, args);
  if (e == hipSuccess && g.parts)
    e = xeng::sum_launch(p->stream, s.clean ? nullptr : reinterpret_cast<const int2*>(s.prev ? s.prev : s.acc),
                         reinterpret_cast<const int2*>(s.part), reinterpret_cast<int2*>(s.acc),
                         (int64_t)(s.acc_bytes / sizeof(int2)), g.chunks);
  return e == hipSuccess ? XENG_OK : hip_fail(p, e, "kernel launch");
}

// Batched call.  Arrays whose N the batch kernel covers become items of one
// launch (several when there are more than batch::MAX_ARRAYS); the rest get
// their plain launch.  Per array the time range is cut into chunks so that
// the items come to about `split` per CU, by the modelled time of a row
// (row_ns) and a start per item; arrays are queued longest item first.
// Untuned plans take the split with the least modelled time: the work spread
// over the CUs, half of the longest item (what the CUs wait for at the end)
// and the atomic adds of the arrays that are cut.  (96x1024, 32x1024 and
// 32x256, 1024 samples: 68 us per call uncut, 188 cut for two items per CU.)
constexpr double ITEM_START_US = 4.0;

struct BatchEntry {
  int32_t a;
  int32_t ngroups, nchunks;
  int64_t t_chunk;
  double item_us;
};

// Cut the items to about split per CU (0: not at all, but for the longest
// range a workgroup takes); returns the modelled time of the call.
double cut_items(const xeng_plan_t* p, const int64_t* n_time, int split, std::vector<BatchEntry>& items) {
  double total = 0, longest = 0, adds = 0;
  for (const BatchEntry& b : items)
    total += b.ngroups * (n_time[b.a] * row_ns(p->arrays[b.a].k) * 1e-3 + ITEM_START_US);
  const double target = split ? total / ((double)split * p->n_cu) : 1e30;
  total = 0;
  for (BatchEntry& b : items) {
    const ArrayState& s = p->arrays[b.a];
    const int64_t T = n_time[b.a];
    const double full = T * row_ns(s.k) * 1e-3;
    int64_t nc = (int64_t)std::ceil(full / std::max(target, 1.0));
    nc = std::max<int64_t>(1, std::min<int64_t>(nc, T / 256));
    nc = std::max<int64_t>(nc, (T + s.k->max_t_per_wg - 1) / s.k->max_t_per_wg);
    int64_t tc = (T + nc - 1) / nc;
    tc = (tc + xeng::KS - 1) / xeng::KS * xeng::KS;
    b.t_chunk = tc;
    b.nchunks = (int32_t)((T + tc - 1) / tc);
    b.item_us = tc * row_ns(s.k) * 1e-3 + ITEM_START_US;
    total += b.ngroups * b.nchunks * b.item_us;
    longest = std::max(longest, b.item_us);
    if (b.nchunks > 1) adds += 2.0 + b.nchunks * (double)s.acc_bytes / 4.0 / 115e3;
  }
  return std::max(total / p->n_cu, longest / 2) + longest / 2 + adds;
}

int record_batched(xeng_plan_t* p, const uint8_t* const* v, const int64_t* n_time) {
  std::vector<BatchEntry> items;
  std::vector<int32_t> others;
  for (int32_t a = 0; a < (int32_t)p->arrays.size(); ++a) {
    const ArrayState& s = p->arrays[a];
    if (!s.active || n_time[a] == 0) continue;
    if (s.own_launch || !xeng::batch::supports(s.d.n_inputs) || s.k != xeng::x16_kernel(s.d.n_inputs)) {
      others.push_back(a);
      continue;
    }
    BatchEntry b{};
    b.a = a;
    b.ngroups = (s.d.n_chans + s.k->cpw - 1) / s.k->cpw;
    items.push_back(b);
  }
  int split = p->batch_split;
  if (split == 0) {
    double best = cut_items(p, n_time, 0, items);
    for (int sp : {1, 2, 4, 8}) {
      const double us = cut_items(p, n_time, sp, items);
      if (us < best) best = us, split = sp;
    }
  }
  cut_items(p, n_time, split, items);
  std::stable_sort(items.begin(), items.end(),
                   [](const BatchEntry& x, const BatchEntry& y) { return x.item_us > y.item_us; });
  std::vector<ArrayState*> to_init;
  for (const BatchEntry& b : items) {
    ArrayState& s = p->arrays[b.a];
    if (b.nchunks > 1 && needs_init(s)) to_init.push_back(&s);
  }
  if (!to_init.empty()) {
    const int st = init_for_atomics(p, to_init);
    if (st != XENG_OK) return st;
  }
  for (size_t i = 0; i < items.size();) {
    xeng::batch::Params bp{};
    bp.counters = p->counters;
    int64_t n_items = 0;
    for (; i < items.size() && bp.n_arrays < xeng::batch::MAX_ARRAYS; ++i) {
      const BatchEntry& b = items[i];
      const ArrayState& s = p->arrays[b.a];
      const int64_t more = (int64_t)b.ngroups * b.nchunks;
      if (bp.n_arrays && n_items + more > xeng::batch::MAX_ITEMS) break;  // (the next launch's)
      const int k = bp.n_arrays++;
      bp.arr[k] = base_args(s, s.k, v[b.a], n_time[b.a]);
      bp.arr[k].t_chunk = b.t_chunk;
      bp.arr[k].mode = b.nchunks > 1 ? xeng::EPI_ATOMIC : (s.clean ? xeng::EPI_STORE : xeng::EPI_ADD);
      bp.ngroups[k] = b.ngroups;
      bp.nchunks[k] = b.nchunks;
      n_items += more;
    }
    if (n_items > xeng::batch::MAX_ITEMS) return fail(p, XENG_EINVAL, "array of %lld items", (long long)n_items);
    const int grid = (int)n_items;
    ++p->stats.launches;
    if (p->trace)
      fprintf(stderr, "xeng: plan %p batch launch arrays=%d items=%d\n", (void*)p, bp.n_arrays, grid);
    hipError_t e = xeng::batch::launch(grid, p->stream, bp);
    if (e != hipSuccess) return hip_fail(p, e, "batch kernel launch");
  }
  for (int32_t a : others) {
    const int st = launch_plain(p, p->arrays[a], v[a], n_time[a]);
    if (st != XENG_OK) return st;
  }
  return XENG_OK;
}

// Record the batched call into a graph on the plan's stream (stream capture),
// then launch it.  Instantiated graphs are kept in a ring and updated in place
// for later calls (hipGraphExecUpdate; a fresh instantiation if the update is
// refused); a graph is updated only after its previous launch has completed,
// so a launch in flight never sees new parameters.
int run_batched(xeng_plan_t* p, const uint8_t* const* v, const int64_t* n_time) {
  bool any = false;
  for (int32_t a = 0; a < (int32_t)p->arrays.size(); ++a) any = any || (p->arrays[a].active && n_time[a] > 0);
  if (!any) return XENG_OK;  // nothing to launch
  const int slot = p->next_graph;
  p->next_graph = (slot + 1) % xeng_plan_s::GRAPH_RING;
  hipError_t e;
  if (!p->done[slot]) {
    e = hipEventCreateWithFlags(&p->done[slot], hipEventDisableTiming);
    if (e != hipSuccess) return hip_fail(p, e, "graph event");
  } else {
    e = hipEventSynchronize(p->done[slot]);
    if (e != hipSuccess) return hip_fail(p, e, "graph event wait");
  }
  e = hipStreamBeginCapture(p->stream, hipStreamCaptureModeRelaxed);
  if (e != hipSuccess) return hip_fail(p, e, "begin capture");
  const int st = record_batched(p, v, n_time);
  hipGraph_t graph = nullptr;
  e = hipStreamEndCapture(p->stream, &graph);
  if (st != XENG_OK) {
    if (graph) (void)hipGraphDestroy(graph);
    return st;
  }
  if (e != hipSuccess) return hip_fail(p, e, "end capture");
  if (p->exec[slot]) {
    hipGraphNode_t err_node = nullptr;
    hipGraphExecUpdateResult res;
    if (hipGraphExecUpdate(p->exec[slot], graph, &err_node, &res) != hipSuccess ||
        res != hipGraphExecUpdateSuccess) {
      (void)hipGetLastError();
      (void)hipGraphExecDestroy(p->exec[slot]);
      p->exec[slot] = nullptr;
    }
  }
  if (!p->exec[slot]) {
    e = hipGraphInstantiate(&p->exec[slot], graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
      p->exec[slot] = nullptr;
      (void)hipGraphDestroy(graph);
      return hip_fail(p, e, "graph instantiate");
    }
  }
  (void)hipGraphDestroy(graph);
  e = hipGraphLaunch(p->exec[slot], p->stream);
  if (e != hipSuccess) return hip_fail(p, e, "graph launch");
  e = hipEventRecord(p->done[slot], p->stream);
  if (e != hipSuccess) return hip_fail(p, e, "graph event record");
  return XENG_OK;
}

int zero_accumulators(xeng_plan_t* p) {
  for (ArrayState& s : p->arrays) {
    if (!s.active) continue;
    hipError_t e = hipMemsetAsync(s.acc, 0, s.acc_bytes, p->stream);
    if (e != hipSuccess) return hip_fail(p, e, "accumulator clear");
    s.clean = s.zeroed = true;
    s.n_integrated = 0;
  }
  return XENG_OK;
}

int validate_call(xeng_plan_t* p, const uint8_t* const* d_voltages, const int64_t* n_time) {
  for (int32_t a = 0; a < (int32_t)p->arrays.size(); ++a) {
    const ArrayState& s = p->arrays[a];
    const int64_t T = n_time[a];
    if (!s.active) {
      if (T != 0) return fail(p, XENG_EINVAL, "slot %d holds no array but n_time is %lld", a, (long long)T);
      continue;
    }
    if (T < 0 || T > s.d.max_time_per_call)
      return fail(p, XENG_EINVAL, "array %d: n_time %lld outside [0, %lld]", a, (long long)T,
                  (long long)s.d.max_time_per_call);
    if (T > 0 && (!d_voltages || !d_voltages[a] || !aligned16(d_voltages[a])))
      return fail(p, XENG_EINVAL, "array %d: voltage pointer null or not 16-byte aligned", a);
    if (s.n_integrated + T > XENG_MAX_INTEGRATION)
      return fail(p, XENG_EOVERFLOW, "array %d: %lld + %lld samples exceed %lld", a,
                  (long long)s.n_integrated, (long long)T, (long long)XENG_MAX_INTEGRATION);
  }
  return XENG_OK;
}

int correlate_unchecked(xeng_plan_t* p, const uint8_t* const* d_voltages, const int64_t* n_time) {
  if (p->batched) {
    const int st = run_batched(p, d_voltages, n_time);
    if (st != XENG_OK) return st;
  } else {
    for (int32_t a = 0; a < (int32_t)p->arrays.size(); ++a) {
      if (!p->arrays[a].active || n_time[a] == 0) continue;
      const int st = launch_plain(p, p->arrays[a], d_voltages[a], n_time[a]);
      if (st != XENG_OK) return st;
    }
  }
  ++p->stats.calls;
  for (int32_t a = 0; a < (int32_t)p->arrays.size(); ++a) {
    ArrayState& s = p->arrays[a];
    if (!s.active || n_time[a] == 0) continue;
    s.n_integrated += n_time[a];
    s.clean = s.zeroed = false;
    p->stats.samples += n_time[a];
    p->stats.cmacs += n_time[a] * (int64_t)s.d.n_chans * nbl_of(s.d.n_inputs);
    p->stats.bytes_in += n_time[a] * (int64_t)s.d.n_chans * s.d.n_inputs;
  }
  return XENG_OK;
}

}  // namespace

extern "C" {

int64_t xeng_nbaselines(int32_t n) { return n < 0 ? -1 : nbl_of(n); }

int64_t xeng_baseline_index(int32_t i, int32_t j) {
  if (i < 0 || j < 0 || j > i) return -1;
  return (int64_t)i * (i + 1) / 2 + j;
}

const char* xeng_strerror(int status) {
  switch (status) {
    case XENG_OK: return "ok";
    case XENG_EINVAL: return "invalid argument";
    case XENG_ENOMEM: return "out of memory";
    case XENG_EOVERFLOW: return "integration would overflow int32";
    case XENG_EDEVICE: return "HIP device error";
    case XENG_ESTATE: return "plan unusable after an earlier device error";
    default: return "unknown status";
  }
}

const char* xeng_last_error(const xeng_plan_t* p) { return p ? p->err.c_str() : ""; }

int64_t xeng_integrated(const xeng_plan_t* p, int32_t array) {
  if (!p || array < 0 || array >= (int32_t)p->arrays.size() || !p->arrays[array].active) return -1;
  return p->arrays[array].n_integrated;
}

int32_t xeng_slots(const xeng_plan_t* p) { return p ? (int32_t)p->arrays.size() : -1; }

int64_t xeng_accumulator_bytes(int32_t n_inputs, int32_t n_chans) {
  if (n_inputs < 1 || n_chans < 1) return -1;
  return (int64_t)n_chans * nbl_of(n_inputs) * 2 * (int64_t)sizeof(int32_t);
}

int xeng_plan(xeng_plan_t** out, const xeng_array_desc* arrays, int32_t n_arrays, uint32_t flags,
              void* hip_stream) {
  if (!out || n_arrays < 0 || (n_arrays > 0 && !arrays) || (flags & ~(uint32_t)XENG_PLAN_BATCH))
    return XENG_EINVAL;
  if (n_arrays == 0 && !(flags & XENG_PLAN_BATCH)) return XENG_EINVAL;
  *out = nullptr;
  for (int32_t a = 0; a < n_arrays; ++a)
    if (!valid_desc(arrays[a])) return XENG_EINVAL;
  xeng_plan_t* p = new (std::nothrow) xeng_plan_t();
  if (!p) return XENG_ENOMEM;
  p->batched = n_arrays > 1 || (flags & XENG_PLAN_BATCH);
  {
    const char* t = getenv("XENG_TRACE");
    p->trace = t && *t && strcmp(t, "0") != 0;
  }
  hipError_t e = hipGetDevice(&p->device);
  if (e != hipSuccess) {
    delete p;
    return XENG_EDEVICE;
  }
  int ncu = 0;
  if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, p->device) == hipSuccess &&
      ncu > 0)
    p->n_cu = ncu;
  {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, p->device) == hipSuccess) {
      p->arch = prop.gcnArchName;
      const size_t colon = p->arch.find(':');
      if (colon != std::string::npos) p->arch.resize(colon);
    }
  }
  if (hip_stream) {
    p->stream = reinterpret_cast<hipStream_t>(hip_stream);
  } else {
    e = hipStreamCreateWithFlags(&p->stream, hipStreamNonBlocking);
    if (e != hipSuccess) {
      delete p;
      return XENG_EDEVICE;
    }
    p->own_stream = true;
  }
  if (p->batched) {
    const size_t cbytes = (xeng::batch::QUEUES + 1) * sizeof(int32_t);
    e = hipMalloc(&p->counters, cbytes);
    if (e == hipSuccess) e = hipMemsetAsync(p->counters, 0, cbytes, p->stream);
    if (e != hipSuccess) {
      xeng_destroy(p);
      return e == hipErrorOutOfMemory ? XENG_ENOMEM : XENG_EDEVICE;
    }
  }
  p->arrays.resize(n_arrays);
  for (int32_t a = 0; a < n_arrays; ++a) {
    const int st = init_slot(p, p->arrays[a], arrays[a]);
    if (st != XENG_OK) {
      xeng_destroy(p);
      return st;
    }
  }
  if (p->batched) apply_cached_plan(p, n_arrays);
  *out = p;
  return XENG_OK;
}

int xeng_attach(xeng_plan_t* p, const xeng_array_desc* d, int32_t* index) {
  if (!p || !d || !index) return XENG_EINVAL;
  if (p->dead) return XENG_ESTATE;
  if (!p->batched) return fail(p, XENG_EINVAL, "attach needs a batched plan");
  if (!valid_desc(*d)) return fail(p, XENG_EINVAL, "bad array descriptor");
  int32_t slot = 0;
  while (slot < (int32_t)p->arrays.size() && p->arrays[slot].active) ++slot;
  if (slot == (int32_t)p->arrays.size()) p->arrays.emplace_back();
  const int st = init_slot(p, p->arrays[slot], *d);
  if (st != XENG_OK) {
    if (p->arrays[slot].acc) (void)hipFree(p->arrays[slot].acc);
    p->arrays[slot] = ArrayState{};
    return st;
  }
  *index = slot;
  return XENG_OK;
}

int xeng_detach(xeng_plan_t* p, int32_t index) {
  if (!p) return XENG_EINVAL;
  if (p->dead) return XENG_ESTATE;
  if (index < 0 || index >= (int32_t)p->arrays.size() || !p->arrays[index].active)
    return fail(p, XENG_EINVAL, "slot %d holds no array", index);
  hipError_t e = hipStreamSynchronize(p->stream);
  if (e != hipSuccess) return hip_fail(p, e, "detach synchronize");
  e = hipFree(p->arrays[index].acc);
  p->arrays[index] = ArrayState{};
  if (e != hipSuccess) return hip_fail(p, e, "accumulator free");
  return XENG_OK;
}

int xeng_correlate(xeng_plan_t* p, const uint8_t* const* d_voltages, const int64_t* n_time) {
  if (!p || !n_time) return XENG_EINVAL;
  if (p->dead) return XENG_ESTATE;
  const int st = validate_call(p, d_voltages, n_time);
  if (st != XENG_OK) return st;
  return correlate_unchecked(p, d_voltages, n_time);
}

int xeng_correlate_dump(xeng_plan_t* p, const uint8_t* const* d_voltages, const int64_t* n_time,
                        int32_t* const* d_dst, int64_t* n_integrated) {
  if (!p || !n_time || !d_dst) return XENG_EINVAL;
  if (p->dead) return XENG_ESTATE;
  int st = validate_call(p, d_voltages, n_time);
  if (st != XENG_OK) return st;
  const int32_t na = (int32_t)p->arrays.size();
  for (int32_t a = 0; a < na; ++a) {
    if (!p->arrays[a].active || !d_dst[a]) continue;
    if ((reinterpret_cast<uintptr_t>(d_dst[a]) & 7u) != 0)
      return fail(p, XENG_EINVAL, "array %d: destination not 8-byte aligned", a);
    hipPointerAttribute_t attr{};
    if (hipPointerGetAttributes(&attr, d_dst[a]) != hipSuccess || attr.type != hipMemoryTypeDevice) {
      (void)hipGetLastError();
      return fail(p, XENG_EINVAL, "array %d: destination is not device memory", a);
    }
  }
  // Arrays dumped without new samples: a plain dump each.
  for (int32_t a = 0; a < na; ++a) {
    if (!p->arrays[a].active || !d_dst[a] || n_time[a] != 0) continue;
    int32_t* dst[1] = {d_dst[a]};
    st = xeng_dump(p, a, dst, 0, n_integrated ? n_integrated + a : nullptr);
    if (st != XENG_OK) return st;
  }
  // The others integrate straight into their destination, from nothing or
  // from the accumulator's earlier samples.
  struct Saved {
    int32_t a;
    int32_t* acc;
    bool clean, zeroed;
    int64_t n;
  };
  std::vector<Saved> redirected;
  for (int32_t a = 0; a < na; ++a) {
    ArrayState& s = p->arrays[a];
    if (!s.active || !d_dst[a] || n_time[a] == 0) continue;
    redirected.push_back(Saved{a, s.acc, s.clean, s.zeroed, s.n_integrated});
    s.prev = s.clean ? nullptr : s.acc;
    s.acc = d_dst[a];
    s.zeroed = false;  // clean (empty) destinations hold unknown values
  }
  st = correlate_unchecked(p, d_voltages, n_time);
  for (const Saved& r : redirected) {
    ArrayState& s = p->arrays[r.a];
    s.acc = r.acc;
    s.prev = nullptr;
    if (st != XENG_OK) {
      s.clean = r.clean;
      s.zeroed = r.zeroed;
      s.n_integrated = r.n;
      continue;
    }
    if (n_integrated) n_integrated[r.a] = r.n + n_time[r.a];
    ++p->stats.dumps;
    p->stats.bytes_out += (int64_t)s.acc_bytes;
    // the integration restarts; an accumulator that was empty was not written
    s.n_integrated = 0;
    s.clean = true;
    s.zeroed = r.clean && r.zeroed;
  }
  return st;
}

int xeng_autotune(xeng_plan_t* p, const uint8_t* const* d_voltages, const int64_t* n_time,
                  int32_t reps, float* best_ms) {
  if (!p || !n_time || reps < 1) return XENG_EINVAL;
  if (p->dead) return XENG_ESTATE;
  for (const ArrayState& s : p->arrays)
    if (s.active && s.n_integrated != 0)
      return fail(p, XENG_EINVAL, "autotune needs every accumulator freshly dumped");
  int st = validate_call(p, d_voltages, n_time);
  if (st != XENG_OK) return st;

  hipEvent_t t0, t1;
  if (hipEventCreate(&t0) != hipSuccess) return fail(p, XENG_EDEVICE, "event");
  if (hipEventCreate(&t1) != hipSuccess) {
    (void)hipEventDestroy(t0);
    return fail(p, XENG_EDEVICE, "event");
  }
  // one trial: reps calls from clean accumulators, timed on the stream
  auto trial = [&](float& ms) -> int {
    int r = zero_accumulators(p);
    if (r != XENG_OK) return r;
    r = correlate_unchecked(p, d_voltages, n_time);  // warm-up (also builds the graph)
    if (r != XENG_OK) return r;
    if (hipEventRecord(t0, p->stream) != hipSuccess) return fail(p, XENG_EDEVICE, "event record");
    // (the sums of these calls are thrown away, so the overflow guard is not applied)
    for (int i = 0; i < reps && r == XENG_OK; ++i) r = correlate_unchecked(p, d_voltages, n_time);
    if (r != XENG_OK) return r;
    if (hipEventRecord(t1, p->stream) != hipSuccess || hipEventSynchronize(t1) != hipSuccess)
      return fail(p, XENG_EDEVICE, "event wait");
    return hipEventElapsedTime(&ms, t0, t1) == hipSuccess ? XENG_OK : fail(p, XENG_EDEVICE, "timing");
  };

  float best = 0;
  if (p->batched) {
    // work-item granularity of the batch launch (0: modelled for each call)
    int pick = p->batch_split;
    for (int cand : {0, 1, 2, 4, 8}) {
      if (st != XENG_OK) break;
      p->batch_split = cand;
      float ms = 0;
      st = trial(ms);
      if (st == XENG_OK && (best == 0 || ms < best)) {
        best = ms;
        pick = cand;
      }
    }
    p->batch_split = pick;
    // Per array, largest work first: items of the batch launch (16-row
    // tiles), or a plain launch of its own inside the same graph with the
    // tile shape and time split that suit it best; kept when the whole call
    // gets faster by more than 1%.
    std::vector<int32_t> order;
    for (int32_t a = 0; a < (int32_t)p->arrays.size(); ++a)
      if (p->arrays[a].active && n_time[a] > 0) order.push_back(a);
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
      const ArrayState &sx = p->arrays[x], &sy = p->arrays[y];
      return n_time[x] * sx.d.n_chans * nbl_of(sx.d.n_inputs) > n_time[y] * sy.d.n_chans * nbl_of(sy.d.n_inputs);
    });
    for (int32_t a : order) {
      if (st != XENG_OK) break;
      ArrayState& s = p->arrays[a];
      const ArrayState keep = s;
      ArrayState choice = s;
      for (int kind : {KIND_X16, KIND_X32, KIND_STAGE}) {
        const KernelInfo* k = kernel_of(kind, s.d);
        if (!kernel_fits(k, s.d) || (kind == KIND_X32 && s.d.n_inputs % 16 != 0)) continue;
        for (int split : {1, 2}) {
          set_kernel(s, k, split);
          s.own_launch = true;
          float ms = 0;
          st = trial(ms);
          if (st != XENG_OK) break;
          if (ms < 0.99f * best) {
            best = ms;
            choice = s;
          }
        }
        if (st != XENG_OK) break;
      }
      const bool own = choice.own_launch;
      s = keep;
      if (own) {
        set_kernel(s, choice.k, choice.split);
        s.own_launch = true;
      }
    }
    for (int32_t a : order) record_choice(p, p->arrays[a], n_time[a]);
    {
      std::lock_guard<std::mutex> lock(g_tune_mu);
      g_tune[plan_key(p, (int32_t)p->arrays.size())] = TuneVal{KIND_X16, p->batch_split, 0};
    }
  } else {
    // per array: tile shape (32-row tiles of the ring kernel or 16-row tiles
    // of the staging kernel) and workgroups per CU of the time split, each
    // timed with the chunk room that a new plan with that choice would have
    for (ArrayState& s : p->arrays) {
      if (!s.active) continue;
      std::vector<const KernelInfo*> kernels;
      if (kernel_fits(kernel_of(KIND_X16, s.d), s.d)) kernels.push_back(kernel_of(KIND_X16, s.d));
      if (s.d.n_inputs % 16 == 0) kernels.push_back(xeng::x32_kernel(s.d.n_inputs));
      kernels.push_back(xeng::stage_kernel((s.d.n_inputs + 15) / 16));
      std::vector<std::pair<const KernelInfo*, int>> cands;
      for (const KernelInfo* k : kernels)
        for (int split : {0, 1, 2, 4})
          if (k && (split != 0 || k->split == 0)) cands.emplace_back(k, split);  // (0: only where modelled)
      const std::pair<const KernelInfo*, int> first{s.k, s.split};
      int32_t* const own = s.part;  // kept until the plan goes: calls captured by the caller may name it
      const int own_chunks = s.part_room;
      int most = 0;
      for (const auto& c : cands) {
        set_kernel(s, c.first, c.second);
        most = std::max(most, room_chunks(p, s));
      }
      int32_t* trial_room = nullptr;
      if (most > own_chunks && hipMalloc(&trial_room, most * s.acc_bytes) != hipSuccess) {
        (void)hipGetLastError();
        trial_room = nullptr;
      }
      auto take = [&](const std::pair<const KernelInfo*, int>& c) {
        set_kernel(s, c.first, c.second);
        const int chunks = room_chunks(p, s);
        s.part = chunks > own_chunks && trial_room ? trial_room : own;
        s.part_chunks = std::min(chunks, s.part == trial_room ? most : own_chunks);
      };
      std::pair<const KernelInfo*, int> pick = first;
      float arr_best = 0;
      for (const auto& c : cands) {
        take(c);
        float ms = 0;
        st = trial(ms);
        if (st != XENG_OK) break;
        if (arr_best == 0 || ms < arr_best) {
          arr_best = ms;
          pick = c;
        }
      }
      take(pick);
      if (trial_room && s.part == trial_room) {
        s.part_room = most;
        s.old_part = own;
      } else if (trial_room) {
        (void)hipFree(trial_room);
      }
      best += arr_best;
      if (st != XENG_OK) break;
      if (n_time[&s - &p->arrays[0]] > 0) record_choice(p, s, n_time[&s - &p->arrays[0]]);
    }
  }
  const int z = zero_accumulators(p);
  if (st == XENG_OK) st = z;
  if (st == XENG_OK && hipStreamSynchronize(p->stream) != hipSuccess) st = fail(p, XENG_EDEVICE, "sync");
  (void)hipEventDestroy(t0);
  (void)hipEventDestroy(t1);
  if (st == XENG_OK && best_ms) *best_ms = best / (float)reps;
  return st;
}

int xeng_tune_cache_save(const char* path) {
  if (!path) return XENG_EINVAL;
  FILE* f = fopen(path, "w");
  if (!f) return XENG_EINVAL;
  fprintf(f, "# xeng tuning cache: arch batched N log2F log2T kernel(0=16-row,1=32-row,2=staging) split own\n");
  {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    for (const auto& kv : g_tune)
      fprintf(f, kv.first.phases > 1 ? "%s %d %d %d %d %d %d %d %d\n" : "%s %d %d %d %d %d %d %d\n",
              kv.first.arch.c_str(), kv.first.batched, kv.first.n, kv.first.fb, kv.first.tb, kv.second.kind,
              kv.second.split, kv.second.own, kv.first.phases);
  }
  return fclose(f) == 0 ? XENG_OK : XENG_EINVAL;
}

int xeng_tune_cache_load(const char* path) {
  if (!path) return XENG_EINVAL;
  FILE* f = fopen(path, "r");
  if (!f) return XENG_EINVAL;
  char line[512];
  int st = XENG_OK;
  std::lock_guard<std::mutex> lock(g_tune_mu);
  while (fgets(line, sizeof line, f)) {
    if (line[0] == '#' || line[0] == '\n') continue;
    char arch[128];
    int b, n, fb, tb, kind, split, own, phases = 1;
    if (sscanf(line, "%127s %d %d %d %d %d %d %d %d", arch, &b, &n, &fb, &tb, &kind, &split, &own, &phases) < 8 ||
        n < 0 || n > XENG_MAX_INPUTS || (n == 0 && !b) || kind < KIND_X16 || kind > KIND_STAGE ||
        split < (kind != KIND_X16 ? 1 : 0) || split > 64 || phases < 1) {  // 0: modelled, on the ring kernel and in a batch
      st = XENG_EINVAL;  // malformed line: skipped, reported
      continue;
    }
    g_tune[TuneKey{arch, b ? 1 : 0, n, fb, tb, phases}] = TuneVal{kind, split, own ? 1 : 0};
  }
  fclose(f);
  return st;
}

int xeng_tune_cache_clear(void) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  g_tune.clear();
  return XENG_OK;
}

int xeng_dump(xeng_plan_t* p, int32_t array, int32_t* const* dst, uint32_t flags,
              int64_t* n_integrated) {
  if (!p || !dst) return XENG_EINVAL;
  if (p->dead) return XENG_ESTATE;
  if (flags & ~(uint32_t)(XENG_DUMP_KEEP | XENG_DUMP_TO_HOST)) return XENG_EINVAL;
  const int32_t na = (int32_t)p->arrays.size();
  if (array < -1 || array >= na) return fail(p, XENG_EINVAL, "array index %d out of range", array);
  if (array >= 0 && !p->arrays[array].active) return fail(p, XENG_EINVAL, "slot %d holds no array", array);
  const int32_t a0 = array < 0 ? 0 : array, a1 = array < 0 ? na : array + 1;
  for (int32_t a = a0; a < a1; ++a)
    if (p->arrays[a].active && !dst[a - a0])
      return fail(p, XENG_EINVAL, "dump destination %d is null", a - a0);
  const bool to_host = (flags & XENG_DUMP_TO_HOST) != 0;
  const bool keep = (flags & XENG_DUMP_KEEP) != 0;
  // An empty integration whose memory still holds an earlier dump's sums
  // (clean, not zeroed) is dumped as zeros.  Without KEEP the accumulator is
  // not cleared here: it is marked empty, and the next launch overwrites it.
  xeng::DumpParams dp{};
  int64_t most = 0;
  auto flush = [&]() -> int {
    if (dp.count == 0) return XENG_OK;
    const int64_t blocks = std::min<int64_t>((most + 1023) / 1024, 8LL * p->n_cu);
    hipError_t e = xeng::dump_launch((int)std::max<int64_t>(1, blocks), p->stream, dp);
    dp.count = 0;
    most = 0;
    return e == hipSuccess ? XENG_OK : hip_fail(p, e, "dump kernel");
  };
  for (int32_t a = a0; a < a1; ++a) {
    ArrayState& s = p->arrays[a];
    if (!s.active) continue;
    int32_t* d = dst[a - a0];
    const bool stale = s.clean && !s.zeroed;
    if (!to_host && (reinterpret_cast<uintptr_t>(d) & 7u) == 0) {
      // device destination: one dump kernel copies every array
      dp.acc[dp.count] = stale ? nullptr : reinterpret_cast<const int2*>(s.acc);
      dp.dst[dp.count] = reinterpret_cast<int2*>(d);
      dp.n[dp.count] = (int64_t)(s.acc_bytes / sizeof(int2));
      most = std::max(most, dp.n[dp.count]);
      if (++dp.count == xeng::DUMP_MAX) {
        const int st = flush();
        if (st != XENG_OK) return st;
      }
    } else {
      if (stale) {
        const int st = init_for_atomics(p, {&s});
        if (st != XENG_OK) return st;
      }
      hipError_t e = hipMemcpyAsync(d, s.acc, s.acc_bytes,
                                    to_host ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice, p->stream);
      if (e != hipSuccess) return hip_fail(p, e, "dump copy");
    }
    if (n_integrated) n_integrated[a - a0] = s.n_integrated;
    ++p->stats.dumps;
    p->stats.bytes_out += (int64_t)s.acc_bytes;
    if (!keep) {
      s.n_integrated = 0;
      s.clean = true;
    }
  }
  const int st = flush();
  if (st != XENG_OK) return st;
  if (to_host) {
    hipError_t e = hipStreamSynchronize(p->stream);
    if (e != hipSuccess) return hip_fail(p, e, "dump synchronize");
  }
  return XENG_OK;
}

int xeng_stats(const xeng_plan_t* p, xeng_stats_t* out) {
  if (!p || !out) return XENG_EINVAL;
  *out = p->stats;
  return XENG_OK;
}

int xeng_load_acc(xeng_plan_t* p, int32_t array, const int32_t* src, int64_t n_integrated) {
  if (!p || !src) return XENG_EINVAL;
  if (p->dead) return XENG_ESTATE;
  if (array < 0 || array >= (int32_t)p->arrays.size() || !p->arrays[array].active)
    return fail(p, XENG_EINVAL, "slot %d holds no array", array);
  if (n_integrated < 0 || n_integrated > XENG_MAX_INTEGRATION)
    return fail(p, XENG_EINVAL, "n_integrated %lld outside [0, %lld]", (long long)n_integrated,
                (long long)XENG_MAX_INTEGRATION);
  ArrayState& s = p->arrays[array];
  hipError_t e = hipMemcpyAsync(s.acc, src, s.acc_bytes, hipMemcpyDefault, p->stream);
  if (e != hipSuccess) return hip_fail(p, e, "accumulator load");
  s.n_integrated = n_integrated;
  s.clean = false;   // the next launch adds to the loaded sums
  s.zeroed = false;
  return XENG_OK;
}

void xeng_destroy(xeng_plan_t* p) {
  if (!p) return;
  if (p->stream) (void)hipStreamSynchronize(p->stream);
  for (int i = 0; i < xeng_plan_s::GRAPH_RING; ++i) {
    if (p->exec[i]) (void)hipGraphExecDestroy(p->exec[i]);
    if (p->done[i]) (void)hipEventDestroy(p->done[i]);
  }
  for (ArrayState& s : p->arrays) {
    if (s.acc) (void)hipFree(s.acc);
    if (s.part) (void)hipFree(s.part);
    if (s.old_part) (void)hipFree(s.old_part);
  }
  if (p->counters) (void)hipFree(p->counters);
  if (p->own_stream && p->stream) (void)hipStreamDestroy(p->stream);
  delete p;
}

}  // extern "C"
