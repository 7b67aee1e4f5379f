// Streaming evaluation kernels (Algorithm 1, Sec. IV) for gfx950.
//
// Every workgroup copies the table's image to LDS once - the records (or
// their values and slopes), the knots (NaN padded) and the uniform index map,
// which the build leaves in memory as they stand in LDS - and then streams
// its share of the points with 16-byte non-temporal loads and stores, U
// vectors per thread in flight.  The path is a memory-bound gather (8 bytes
// per point forward, 16 fused forward and backward), so there is no
// matrix-core work: the only per-point work is the map lookup, a short knot
// compare loop in LDS, one record read and one FMA.  The backward accumulates
// dL/dv in LDS with FP64 atomics and writes one column of per-workgroup
// partial sums, which k_dv_reduce adds.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pwl_internal.h"
#include "pwl_locate.h"
#include "pwl_stream.h"

namespace pwl {

namespace {

constexpr size_t kLdsPerCU = 160 * 1024;
constexpr int kXcds = 8;             // MI355X accelerator complex dies; workgroups go to them round-robin
constexpr int64_t kMinPointsPerWG = int64_t(1) << 15;   // streaming grids: points per workgroup, at least
constexpr int64_t kMaxPointsPerWG = 57344;              // (forward, N <= 2048) no more asked for by the staged bytes
constexpr int64_t kPointsPerStagedByte = 2;             // and per byte of table the workgroup stages
constexpr int kWordsPerThread = 3;                      // tables staged through registers: records per thread

using namespace stream;

// A launch's flags; from bit kBlockBit on, the workgroup's size.
constexpr int kVec = 1;      // the arrays are 4-byte aligned: 16-byte accesses
constexpr int kSearch = 2;   // PWL_LOCATE_SEARCH
constexpr int kBlockBit = 8;

template <int U, bool WORDS, class S>
__device__ __forceinline__ void eval_fwd_body(const EvalTable& t, const float* __restrict__ vo, const S& s,
                                              const float* __restrict__ x, float* __restrict__ y, int64_t n,
                                              int flags) {
  const int nt = flags >> kBlockBit;
  const int64_t blk = blockIdx.x, nblk = gridDim.x;
  const bool vec = (flags & kVec) != 0;
  if constexpr (WORDS)
    stage_words(t, vo, nt, s);
  else
    stage_table(t, vo, nt, s);
  staged();
  lds_barrier();
  if (flags & kSearch) {
    fwd_range<U, -1>(t, s, x, y, 0, n, vec, blk, nblk, nt);
    return;
  }
  switch (t.meta[1]) {
    case 0:
    case 1: fwd_range<U, 1>(t, s, x, y, 0, n, vec, blk, nblk, nt); break;
    case 2: fwd_range<U, 2>(t, s, x, y, 0, n, vec, blk, nblk, nt); break;
    case 3: fwd_range<U, 3>(t, s, x, y, 0, n, vec, blk, nblk, nt); break;
    case 4: fwd_range<U, 4>(t, s, x, y, 0, n, vec, blk, nblk, nt); break;
    default: fwd_range<U, 0>(t, s, x, y, 0, n, vec, blk, nblk, nt); break;
  }
}

// REC is the arrangement of the per-segment data in LDS (pwl_set_records):
// packed records, structure of arrays, or value/slope pairs; WORDS: an image
// of at most kWordsPerThread records per thread, staged through registers.  What keeps the two stagings apart is the
// streaming loop, whose schedule and registers the compiler decides for the
// whole kernel: beside the register staging it takes 84 - 90 registers and starts
// half of its lookups before the last loads arrive, beside the copy 102 - 104.  In
// us, registers / copy: Gaussian N = 1024, 2^28 points 332 / 341; 2^27 points
// Lorentzian N = 1024 178.8 / 183.9, 2000 182.5 / 187.2, 2500 188.9 / 194.5,
// 4096 195.9 / 195.0; J0 N = 1500 169.9 / 174.8, 4096 183.6 / 181.4.  Packed
// records, Gaussian N = 1024, 2^28 points 335.8 / 340.3, by binary search
// 1411 / 1458; pairs 347.2 / 349.0 and 1386 / 1449.
template <int U, int REC, bool WORDS>
__global__ __launch_bounds__(1024) void k_eval_fwd(EvalTable t, const float* __restrict__ vo,
                                                   const float* __restrict__ x,
                                                   float* __restrict__ y, int64_t n, int flags) {
  extern __shared__ float4 lds_f4[];
  if constexpr (REC == PWL_RECORDS_SOA)
    eval_fwd_body<U, WORDS>(t, vo, carve_soa(lds_f4, t.N), x, y, n, flags);
  else if constexpr (REC == PWL_RECORDS_PAIRS)
    eval_fwd_body<U, WORDS>(t, vo, carve_pairs(lds_f4, t.N), x, y, n, flags);
  else
    eval_fwd_body<U, WORDS>(t, vo, carve(lds_f4, t.N, t.K, false), x, y, n, flags);
}

template <int U, bool WY, bool WDX, bool WDV>
__global__ __launch_bounds__(1024) void k_eval_bwd(EvalTable t, const float* __restrict__ vo,
                                                   const float* __restrict__ x,
                                                   const float* __restrict__ g,
                                                   float* __restrict__ y, float* __restrict__ dx,
                                                   float* __restrict__ part, int64_t n, int flags) {
  extern __shared__ float4 lds_f4[];
  const Smem s = carve(lds_f4, t.N, t.K, WDV);
  const int nt = flags >> kBlockBit;
  stage_table(t, vo, nt, s);
  if (WDV)
    for (int k = threadIdx.x; k < (t.N + 1) * s.dvc; k += nt) s.dv[k] = 0.0;
  staged();
  lds_barrier();
  using B = Bwd<U, WY, WDX, WDV>;
  const int64_t blk = blockIdx.x, nblk = gridDim.x;
  const bool vec = (flags & kVec) != 0;
  switch (t.meta[1]) {
    case 0:
    case 1: B::template range<1>(t, s, x, g, y, dx, 0, n, vec, blk, nblk, nt); break;
    case 2: B::template range<2>(t, s, x, g, y, dx, 0, n, vec, blk, nblk, nt); break;
    case 3: B::template range<3>(t, s, x, g, y, dx, 0, n, vec, blk, nblk, nt); break;
    case 4: B::template range<4>(t, s, x, g, y, dx, 0, n, vec, blk, nblk, nt); break;
    default: B::template range<0>(t, s, x, g, y, dx, 0, n, vec, blk, nblk, nt); break;
  }
  if (WDV) {
    // This workgroup's dL/dv becomes column `col` of the partial sums
    // part[k][col] (no atomics: k_dv_reduce adds each row in a fixed order).
    // Workgroups are dealt to the 8 XCDs round-robin, so the columns are
    // ordered XCD by XCD: the workgroups of one XCD fill whole cache lines
    // in their own L2.
    lds_barrier();
    const int G = gridDim.x, b = blockIdx.x;
    const int col = (G % kXcds == 0) ? (b % kXcds) * (G / kXcds) + b / kXcds : b;
    for (int k = threadIdx.x; k <= t.N; k += nt) {
      double acc = s.dv[k * s.dvc];
      for (int j = 1; j < s.dvc; ++j) acc += s.dv[k * s.dvc + j];   // the copies, in a fixed order
      part[(int64_t)k * G + col] = (float)acc;
    }
  }
}

// dL/dv[k] = the sum of row k of part[k][0..G), in FP64 and a fixed order:
// one wave per row, lane l adding columns l, l + 64, ... (coalesced 256-byte
// loads, all issued before the first add), then a butterfly over the lanes.
constexpr int kReduceThreads = 256;
__global__ __launch_bounds__(kReduceThreads) void k_dv_reduce(const float* __restrict__ part, int G, int N1,
                                                              float* __restrict__ dv) {
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.x * (kReduceThreads / 64) + (threadIdx.x >> 6);
  if (k >= N1) return;   // whole waves leave together
  const float* row = part + (int64_t)k * G;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  int c = lane;
  for (; c + 192 < G; c += 256) {
    s0 += (double)row[c];
    s1 += (double)row[c + 64];
    s2 += (double)row[c + 128];
    s3 += (double)row[c + 192];
  }
  for (; c < G; c += 64) s0 += (double)row[c];
  double s = (s0 + s1) + (s2 + s3);
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
  if (lane == 0) dv[k] = (float)s;
}

// Segment indices through the same locate the evaluation kernels run: the
// unrolled compare depth chosen from meta[1] (or the binary search), so the
// indices this returns are the ones k_eval_fwd, k_eval_bwd and the batched
// kernels use.
template <int MAXC>
__device__ __forceinline__ void locate_all(const EvalTable& t, const Smem& s, const float* __restrict__ x,
                                           int32_t* __restrict__ seg, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    seg[i] = locate<MAXC>(x[i], t, s);
}

__global__ __launch_bounds__(1024) void k_locate(EvalTable t, const float* __restrict__ x,
                                                 int32_t* __restrict__ seg, int64_t n, int flags) {
  extern __shared__ float4 lds_f4[];
  const Smem s = carve(lds_f4, t.N, t.K, false);
  stage_table(t, nullptr, blockDim.x, s);
  staged();
  lds_barrier();
  if (flags & kSearch) {
    locate_all<-1>(t, s, x, seg, n);
    return;
  }
  switch (t.meta[1]) {
    case 0:
    case 1: locate_all<1>(t, s, x, seg, n); break;
    case 2: locate_all<2>(t, s, x, seg, n); break;
    case 3: locate_all<3>(t, s, x, seg, n); break;
    case 4: locate_all<4>(t, s, x, seg, n); break;
    default: locate_all<0>(t, s, x, seg, n); break;
  }
}

__global__ void k_fill_zero(float* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0f;
}

// The vector path takes arrays at any 4-byte alignment: its vectors sit on
// the 16-byte boundaries of an array that is written, and the hardware reads
// (and writes the other one) across those of the rest.
inline bool word_aligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }

// Launch shape of a streaming evaluation kernel: workgroups of `block`
// threads, each thread handling `unroll` float4 vectors per iteration, on a
// grid of up to `wg_per_cu` workgroups per CU.  The grid may be many times
// what the CUs hold at once (register use caps residency at one 1024-thread
// workgroup per CU): workgroups are then dispatched as CUs free up, so CUs
// and XCDs that stream faster take more of the points, where a grid of one
// resident round waits for its slowest CU.  Each workgroup stages the whole
// table, so the grid is cut back, a whole workgroup per CU at a time (a
// partial last round leaves CUs idle), until a workgroup streams enough
// points, but never below one workgroup per CU (nor above one per iteration
// of work).  The defaults are the autotuner's choice on MI355X: forward at
// 2^28 points, four vectors per thread in 1024-thread workgroups, up to 32
// per CU; fused backward at 2^26 points, two vectors per thread (the dL/dv
// LDS atomics favour a smaller register footprint) in one 768-thread
// workgroup per CU - every further workgroup there adds a dL/dv flush and a
// column to reduce.  The batched kernels take 1024-thread workgroups and
// four vectors per thread: the forward a persistent grid of 3 per CU, the
// fused backward 32 per CU (about one slice per workgroup, in rounds; its
// four-vector body spills a little and still measured 3% faster than two
// vectors in 3 per CU).  pwl_set_launch overrides them.
//
// Enough points, forward: 2^15, and 2.75 per byte of the image up to 57344.
// At 2^28 points N = 16 takes 32 per CU (328 us; 18: 334) and N = 1024 18
// (333 us; 25: 335); at 2^27 the Lorentzian with N = 2000 9 (182.5 us; 6:
// 184.0, 4: 187.1).  Above N = 2048 the map is not widened where knots crowd,
// such tables compare three knots per point and a third round of lookups
// competes with the staging: 2 points per byte (N = 4096, 2^27 points: 3 per
// CU, Lorentzian 195.0 us and J0 181.4; 9 per CU 208.7 and 177.5).
//
// A launch too small to give every CU a workgroup of the tuned shape spreads
// over the CUs instead, in smaller workgroups with fewer vectors per thread.
// Forward: one vector per thread up to 1024 per CU, two up to 2048; of 256,
// 512 and 1024 threads the fewest whose workgroups stage at most 48 KB per
// CU together (or are alone on it; twice that from 4096 vectors per CU).  Kernel times in us, the tuned shape -> this one:
// N = 64, 2^20 points 6.2 -> 3.9; N = 1024, 2^14 6.9 -> 3.1, 2^20 7.5 -> 4.7
// (256 threads 5.0); N = 4096, 2^20 8.0 -> 5.2 (512 threads 7.0).  Up to one
// and a half workgroups per CU, workgroups of fewer threads still fill the
// last round better where the table is small: 5 * 10^6 points N = 64 11.2 ->
// 8.8, N = 1024 11.7 -> 10.3 (8 * 10^6 points N = 1024 13.8 -> 15.1).
// Backward: one vector per thread in 256 threads (512 for N above 1024) up
// to 512 vectors per CU, then two in 512 threads up to 1024: with the dL/dv
// reduction N = 64, 2^17 points 8.5 -> 7.0; N = 4096, 2^17 12.6 -> 11.7.
constexpr LaunchConfig kDefaultLaunch[4] = {{4, 1024, 32}, {2, 768, 1}, {4, 1024, 3}, {4, 1024, 32}};
LaunchConfig g_launch[4] = {kDefaultLaunch[0], kDefaultLaunch[1], kDefaultLaunch[2], kDefaultLaunch[3]};
int g_locate = PWL_LOCATE_MAP;
int g_records = PWL_RECORDS_PACKED;

// The tuned shape on the grid it earns: at least min_points points per workgroup.
LaunchShape stream_shape(const LaunchConfig& c, size_t lds, int64_t min_points, int64_t n4, int64_t n, int num_cu) {
  const int block = c.block;
  const int64_t per_wg = (int64_t)block * c.unroll;
  const int64_t work = (n4 > 0) ? (n4 + per_wg - 1) / per_wg : (n + block - 1) / block;
  // whole workgroups per CU: a last partial round would leave CUs idle
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(c.wg_per_cu, n / (min_points * num_cu)));
  const int64_t grid = std::max<int64_t>(1, std::min<int64_t>((int64_t)num_cu * per_cu, work));
  return LaunchShape{block, (int)grid, lds, c.unroll};
}

// A small launch: `unroll` vectors per thread in workgroups of `block`
// threads (at most the tuned ones'), as many as there is work for.
LaunchShape small_shape(const LaunchConfig& c, int unroll, int block, size_t lds, int64_t n4, int num_cu) {
  unroll = std::min(unroll, c.unroll);
  block = std::min(block, c.block);
  const int64_t per_wg = (int64_t)block * unroll;
  const int64_t grid = std::min<int64_t>((int64_t)num_cu * c.wg_per_cu, (n4 + per_wg - 1) / per_wg);
  return LaunchShape{block, (int)grid, lds, unroll};
}

bool is_small(const LaunchConfig& c, int64_t n4, int num_cu) {
  return n4 > 0 && n4 < (int64_t)num_cu * c.block * c.unroll;
}

LaunchShape forward_shape(int N, size_t lds, int64_t n4, int64_t n, int num_cu) {
  const LaunchConfig c = g_launch[PWL_KERNEL_FORWARD];
  const int64_t v = (n4 + num_cu - 1) / num_cu;   // vectors per CU
  const bool small = is_small(c, n4, num_cu);
  if (small || is_small(c, n4 * 2 / 3, num_cu)) {
    const int unroll = v <= 1024 ? 1 : (v <= 2048 ? 2 : 4);
    const int64_t staged = 48 * 1024 * std::max<int64_t>(1, v / 2048);
    int block = 256;
    while (block < 1024) {
      const int64_t wgs = (v + (int64_t)block * unroll - 1) / ((int64_t)block * unroll);
      if (wgs == 1 || wgs * (int64_t)lds <= staged) break;
      block *= 2;
    }
    if (small || block < 1024) return small_shape(c, unroll, block, lds, n4, num_cu);
  }
  const int64_t staged = N <= kWideMapMaxN ? std::min<int64_t>(kMaxPointsPerWG, 11 * (int64_t)lds / 4)
                                           : kPointsPerStagedByte * (int64_t)lds;
  return stream_shape(c, lds, std::max(kMinPointsPerWG, staged), n4, n, num_cu);
}

}  // namespace

hipError_t set_launch(int kernel, int unroll, int block, int wg_per_cu) {
  if (kernel < 0 || kernel > 3) return hipErrorInvalidValue;
  if (unroll == 0 && block == 0 && wg_per_cu == 0) {
    g_launch[kernel] = kDefaultLaunch[kernel];
    return hipSuccess;
  }
  if (!(unroll == 1 || unroll == 2 || unroll == 4)) return hipErrorInvalidValue;
  if (block < 64 || block > 1024 || (block % 64) != 0) return hipErrorInvalidValue;
  if (wg_per_cu < 1 || wg_per_cu > 32) return hipErrorInvalidValue;
  g_launch[kernel] = LaunchConfig{unroll, block, wg_per_cu};
  return hipSuccess;
}

LaunchConfig get_launch(int kernel) { return g_launch[kernel]; }

hipError_t set_locate(int mode) {
  if (mode != PWL_LOCATE_MAP && mode != PWL_LOCATE_SEARCH) return hipErrorInvalidValue;
  g_locate = mode;
  return hipSuccess;
}

int get_locate() { return g_locate; }

hipError_t set_records(int layout) {
  if (layout != PWL_RECORDS_PACKED && layout != PWL_RECORDS_SOA && layout != PWL_RECORDS_PAIRS)
    return hipErrorInvalidValue;
  g_records = layout;
  return hipSuccess;
}

int get_records() { return g_records; }

hipError_t launch_eval(const EvalTable& t, const float* vo, const float* x, float* y, int64_t n,
                       int num_cu, hipStream_t s) {
  const bool vec = word_aligned(x) && word_aligned(y);
  const int rec = g_records;
  const size_t lds = rec == PWL_RECORDS_SOA     ? eval_lds_bytes_soa(t.N, t.K)
                     : rec == PWL_RECORDS_PAIRS ? eval_lds_bytes_pairs(t.N, t.K)
                                                : eval_lds_bytes(t.N, t.K, false);
  const LaunchShape ls = forward_shape(t.N, lds, vec ? n / 4 : 0, n, num_cu);
  const int v = (vec ? kVec : 0) | (g_locate == PWL_LOCATE_SEARCH ? kSearch : 0) | (ls.block << kBlockBit);
#define PWL_FWD(UU, RR, OO) \
  hipLaunchKernelGGL((k_eval_fwd<UU, RR, OO>), dim3(ls.grid), dim3(ls.block), ls.lds, s, t, vo, x, y, n, v)
#define PWL_FWD_U(RR, OO)                   \
  switch (ls.unroll) {                      \
    case 1: PWL_FWD(1, RR, OO); break;      \
    case 2: PWL_FWD(2, RR, OO); break;      \
    default: PWL_FWD(4, RR, OO); break;     \
  }
#define PWL_FWD_R(RR)                       \
  if (t.N <= kWordsPerThread * ls.block) {  \
    PWL_FWD_U(RR, true)                     \
  } else {                                  \
    PWL_FWD_U(RR, false)                    \
  }
  if (rec == PWL_RECORDS_SOA) {
    PWL_FWD_R(PWL_RECORDS_SOA)
  } else if (rec == PWL_RECORDS_PAIRS) {
    PWL_FWD_R(PWL_RECORDS_PAIRS)
  } else {
    PWL_FWD_R(PWL_RECORDS_PACKED)
  }
#undef PWL_FWD_R
#undef PWL_FWD_U
#undef PWL_FWD
  return hipGetLastError();
}

template <int U>
void launch_bwd_u(const LaunchShape& ls, int key, const EvalTable& t, const float* vo, const float* x,
                  const float* g, float* y, float* dx, float* part, int64_t n, int vec, hipStream_t s) {
#define PWL_BWD_CASE(K, A, B, C)                                                                 \
  case K:                                                                                        \
    hipLaunchKernelGGL((k_eval_bwd<U, A, B, C>), dim3(ls.grid), dim3(ls.block), ls.lds, s, t, vo, \
                       x, g, y, dx, part, n, vec);                                               \
    break;
  switch (key) {
    PWL_BWD_CASE(1, false, false, true)
    PWL_BWD_CASE(2, false, true, false)
    PWL_BWD_CASE(3, false, true, true)
    PWL_BWD_CASE(4, true, false, false)
    PWL_BWD_CASE(5, true, false, true)
    PWL_BWD_CASE(6, true, true, false)
    PWL_BWD_CASE(7, true, true, true)
    default: break;
  }
#undef PWL_BWD_CASE
}

LaunchShape backward_shape(const EvalTable& t, const float* x, const float* g, const float* y, const float* dx,
                           bool wdv, int64_t n, int num_cu) {
  const bool vec = word_aligned(x) && word_aligned(g) && word_aligned(y) && word_aligned(dx);
  const LaunchConfig c = g_launch[PWL_KERNEL_BACKWARD];
  const size_t lds = eval_lds_bytes(t.N, t.K, wdv);
  const int64_t n4 = vec ? n / 4 : 0, v = (n4 + num_cu - 1) / num_cu;   // v: vectors per CU
  // (one workgroup per CU whatever the tuned shape allows: a small launch
  // needs no more partial sums than that)
  const LaunchConfig one{c.unroll, c.block, 1};
  if (is_small(c, n4, num_cu) && v <= 512)
    return small_shape(one, 1, (v <= 256 && t.N <= 1024) ? 256 : 512, lds, n4, num_cu);
  if (is_small(c, n4, num_cu) && v <= 1024) return small_shape(one, 2, 512, lds, n4, num_cu);
  return stream_shape(c, lds, std::max<int64_t>(kMinPointsPerWG, kPointsPerStagedByte * (int64_t)lds), n4, n, num_cu);
}

size_t backward_workspace_floats(const EvalTable& t, const float* x, const float* g, const float* y,
                                 const float* dx, int64_t n, int num_cu) {
  const LaunchShape ls = backward_shape(t, x, g, y, dx, true, n, num_cu);
  return (size_t)ls.grid * (size_t)(t.N + 1);
}

hipError_t launch_eval_backward(const EvalTable& t, const float* vo, const float* x, const float* g,
                                float* y, float* dx, float* dv, float* part, int64_t n, int num_cu,
                                hipStream_t s) {
  const bool vec = word_aligned(x) && word_aligned(g) && word_aligned(y) && word_aligned(dx);
  const bool wdv = dv != nullptr;
  const LaunchShape ls = backward_shape(t, x, g, y, dx, wdv, n, num_cu);
  const int key = (y != nullptr ? 4 : 0) | (dx != nullptr ? 2 : 0) | (wdv ? 1 : 0);
  if (key == 0) return hipErrorInvalidValue;
  if (wdv && n == 0) {   // no points: dL/dv = 0
    hipLaunchKernelGGL(k_fill_zero, dim3(1), dim3(256), 0, s, dv, (int64_t)t.N + 1);
    return hipGetLastError();
  }
  if (wdv && part == nullptr) return hipErrorInvalidValue;
  const int v = (vec ? kVec : 0) | (ls.block << kBlockBit);
  switch (ls.unroll) {
    case 1: launch_bwd_u<1>(ls, key, t, vo, x, g, y, dx, part, n, v, s); break;
    case 2: launch_bwd_u<2>(ls, key, t, vo, x, g, y, dx, part, n, v, s); break;
    default: launch_bwd_u<4>(ls, key, t, vo, x, g, y, dx, part, n, v, s); break;
  }
  if (wdv) {
    const int n1 = t.N + 1, rows_per_wg = kReduceThreads / 64;
    hipLaunchKernelGGL(k_dv_reduce, dim3((n1 + rows_per_wg - 1) / rows_per_wg), dim3(kReduceThreads), 0, s,
                       part, ls.grid, n1, dv);
  }
  return hipGetLastError();
}


hipError_t launch_locate(const EvalTable& t, const float* x, int32_t* seg, int64_t n, int num_cu,
                         hipStream_t s) {
  const size_t lds = eval_lds_bytes(t.N, t.K, false);
  const LaunchShape ls = stream_shape(g_launch[PWL_KERNEL_FORWARD], lds,
                                      std::max<int64_t>(kMinPointsPerWG, kPointsPerStagedByte * (int64_t)lds), 0, n,
                                      num_cu);
  const int v = (g_locate == PWL_LOCATE_SEARCH) ? kSearch : 0;
  hipLaunchKernelGGL(k_locate, dim3(ls.grid), dim3(ls.block), ls.lds, s, t, x, seg, n, v);
  return hipGetLastError();
}

hipError_t configure_eval_kernels(int max_lds) {
  const int lim = max_lds < (int)kLdsPerCU ? max_lds : (int)kLdsPerCU;
  hipError_t e = hipSuccess;
#define PWL_ATTR(K)                                                                           \
  e = hipFuncSetAttribute((const void*)K, hipFuncAttributeMaxDynamicSharedMemorySize, lim);    \
  if (e != hipSuccess) return e;
  PWL_ATTR(k_locate)
#define PWL_ATTR_R(RR, OO)                   \
  PWL_ATTR((k_eval_fwd<1, RR, OO>))          \
  PWL_ATTR((k_eval_fwd<2, RR, OO>))          \
  PWL_ATTR((k_eval_fwd<4, RR, OO>))
  PWL_ATTR_R(PWL_RECORDS_PACKED, false)
  PWL_ATTR_R(PWL_RECORDS_PACKED, true)
  PWL_ATTR_R(PWL_RECORDS_SOA, false)
  PWL_ATTR_R(PWL_RECORDS_SOA, true)
  PWL_ATTR_R(PWL_RECORDS_PAIRS, false)
  PWL_ATTR_R(PWL_RECORDS_PAIRS, true)
#undef PWL_ATTR_R
#define PWL_ATTR_U(U)                            \
  PWL_ATTR((k_eval_bwd<U, false, false, true>))  \
  PWL_ATTR((k_eval_bwd<U, false, true, false>))  \
  PWL_ATTR((k_eval_bwd<U, false, true, true>))   \
  PWL_ATTR((k_eval_bwd<U, true, false, false>))  \
  PWL_ATTR((k_eval_bwd<U, true, false, true>))   \
  PWL_ATTR((k_eval_bwd<U, true, true, false>))   \
  PWL_ATTR((k_eval_bwd<U, true, true, true>))
  PWL_ATTR_U(1)
  PWL_ATTR_U(2)
  PWL_ATTR_U(4)
#undef PWL_ATTR_U
#undef PWL_ATTR
  return hipSuccess;
}

}  // namespace pwl
