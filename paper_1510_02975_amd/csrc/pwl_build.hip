// Table construction on the GPU.
//
//   optimal partition (Sec. III-B1):
//     k_density_totals   FP64 |f''|^(2/5) on the fine grid, trapezoid sum per workgroup
//     k_invert_knots     FP64 prefix of those sums, targets i S_M / N, linear inversion;
//                        per knot also, for the interpolant, f(x_i)
//   every table:
//     k_finalize         uniform knots (Sec. IV) when asked, the uniform index map,
//                        the knot-collapse check, for the projection (Sec. II-B2)
//                        FP32 Gauss-Legendre integrals of f against the hats and the
//                        FP64 solve of M c = b (parallel cyclic reduction), and the
//                        table's images in memory
#include <hip/hip_runtime.h>

#include "pwl_func.h"
#include "pwl_internal.h"
#include "pwl_locate.h"
#include "pwl_stream.h"

namespace pwl {

namespace {

constexpr int kScanThreads = 1024;      // density workgroup size (one cell per thread)
constexpr int kScanWaves = kScanThreads / 64;

// Inclusive sums over the workgroup of one non-negative value per thread: a
// butterfly of shifted adds inside each wave, then the earlier waves' sums
// in order.  s_w: kScanWaves doubles, free to reuse after the next barrier.
// Contraction is off so that every operation is one IEEE-rounded FP64
// operation; all workgroups that scan the same values get the same sums.
__device__ double block_scan(double v, double* s_w) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double u = __shfl_up(v, d, 64);
    if (lane >= d) v = v + u;
  }
  if (lane == 63) s_w[wave] = v;
  __syncthreads();
  double before = 0.0;
#pragma unroll
  for (int w = 0; w < kScanWaves - 1; ++w) before = before + (w < wave ? s_w[w] : 0.0);
  return before + v;
}

// Inclusive maxima over the workgroup, likewise.
__device__ double block_max_scan(double v, double* s_w) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double u = __shfl_up(v, d, 64);
    if (lane >= d) v = fmax(v, u);
  }
  if (lane == 63) s_w[wave] = v;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kScanWaves - 1; ++w)
    if (w < wave) v = fmax(v, s_w[w]);
  return v;
}

// The density at the corners of workgroup blk's cells, one FP64 sample per
// thread (s_d, valid after the next barrier).  Cell j (1-based) spans
// [t_{j-1}, t_j], t_j = a + j dt.
__device__ void sample_block(const BuildParams& bp, int blk, double* s_d) {
#pragma clang fp contract(off)
  constexpr int C = kDensityCellsPerBlock;
  const double dt = (bp.b - bp.a) / (double)bp.M;
  for (int s = threadIdx.x; s <= C; s += kScanThreads) {
    const int j = blk * C + s;
    s_d[s] = (j <= bp.M) ? knot_density(bp.f, bp.a + (double)j * dt) : 0.0;
  }
}

// This thread's cell's trapezoid, (d_{j-1} + d_j) dt / 2.
__device__ double block_cell(const BuildParams& bp, int blk, const double* s_d) {
#pragma clang fp contract(off)
  const int tid = threadIdx.x;
  const double hdt = (bp.b - bp.a) / (double)bp.M / 2.0;
  return (blk * kDensityCellsPerBlock + tid + 1 <= bp.M) ? (s_d[tid] + s_d[tid + 1]) * hdt : 0.0;
}
static_assert(kScanThreads == kDensityCellsPerBlock, "one cell per thread");
static_assert(kMaxDensityBlocks <= kScanThreads, "one block total per thread");

__global__ __launch_bounds__(kScanThreads) void k_density_totals(BuildParams bp, TableDev td) {
  __shared__ double s_d[kDensityCellsPerBlock + 1];
  __shared__ double s_w[kScanWaves];
  sample_block(bp, blockIdx.x, s_d);
  __syncthreads();
  const double sum = block_scan(block_cell(bp, blockIdx.x, s_d), s_w);
  if (threadIdx.x == kScanThreads - 1) td.totals[blockIdx.x] = sum;
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    td.status[0] = 0u;
    td.status[1] = 0u;
  }
}

__device__ double uniform_knot(const BuildParams& bp, int k) {
#pragma clang fp contract(off)
  double x = bp.a + ((bp.b - bp.a) * (double)k) / (double)bp.N;
  if (k == 0) x = bp.a;
  if (k == bp.N) x = bp.b;
  return x;
}

// Everything a knot needs once its position is known: FP64 and FP32 copies
// and, for the interpolant, f at the FP32 knot.
__device__ void emit_knot(const BuildParams& bp, const TableDev& td, int k, double x) {
  const float x32 = (float)x;
  td.knots64[k] = x;
  td.knots[k] = x32;
  if (bp.values == PWL_INTERP) td.values[k] = f_value32(bp.f, x32);
}

__global__ __launch_bounds__(kScanThreads) void k_invert_knots(BuildParams bp, TableDev td) {
#pragma clang fp contract(off)
  constexpr int C = kDensityCellsPerBlock;
  __shared__ double s_d[C + 1];
  __shared__ double s_S[C];
  __shared__ double s_w[3][kScanWaves];
  __shared__ double s_off[3];   // offset of this block, offset of the next, S_M
  const int tid = threadIdx.x;
  const int blk = blockIdx.x;
  // Prefix of the workgroup totals, made non-decreasing: the offset of block
  // b + 1 is the end of block b in every workgroup, so each target falls to
  // exactly one of them.
  // (The samples are taken while the totals arrive.)
  const double tot = tid < bp.G ? td.totals[tid] : 0.0;
  sample_block(bp, blk, s_d);
  const double sum = block_scan(tot, s_w[0]);
  const double run = block_max_scan(sum, s_w[1]);   // (fmax passes NaN over: S_M keeps the sum's)
  if (tid == 0 && blk == 0) s_off[0] = 0.0;
  if (tid == blk - 1) s_off[0] = run;
  if (tid == blk) s_off[1] = run;
  if (tid == bp.G - 1) s_off[2] = (sum == sum) ? run : sum;
  s_S[tid] = block_scan(block_cell(bp, blk, s_d), s_w[2]);
  __syncthreads();
  const double off = s_off[0], next = s_off[1], total = s_off[2];
  if (!(total > 0.0) || !isfinite(total)) {
    // f'' vanishes on the whole grid (or overflowed): uniform fallback.
    if (blk == 0) {
      for (int k = tid; k <= bp.N; k += kScanThreads) emit_knot(bp, td, k, uniform_knot(bp, k));
      if (tid == 0) td.status[0] = isfinite(total) ? PWL_FLAG_DEGENERATE : PWL_FLAG_NONFINITE;
    }
    return;
  }
  // the targets i S_M / N in (off, next], and one more to either side for
  // the rounding of the bounds (S_M is far from denormal: the least density
  // is 4.9e-324^(2/5) on cells of an FP32 domain)
  const int i0 = max(1, (int)(off / total * (double)bp.N) - 1);
  const int i1 = min(bp.N - 1, (int)(next / total * (double)bp.N) + 1);
  const double dt = (bp.b - bp.a) / (double)bp.M;
  const double snap = 1e-12 * (bp.b - bp.a);
  for (int i = i0 + tid; i <= i1; i += kScanThreads) {
    const double tau = ((double)i * total) / (double)bp.N;
    if (!(off < tau && tau <= next)) continue;
    // the target inside the block, at most its last sum (which the rounding
    // of the offsets may pass), and the smallest cell whose sum reaches it
    const double t = fmin(tau - off, s_S[C - 1]);
    int lo = 0, hi = C - 1;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (s_S[mid] >= t) hi = mid; else lo = mid + 1;
    }
    const double Sj = s_S[lo];
    const double Sp = (lo > 0) ? s_S[lo - 1] : 0.0;
    const int j = blk * C + lo + 1;                    // 1-based cell number
    const double frac = (Sj > Sp) ? (t - Sp) / (Sj - Sp) : 0.0;
    double x = (bp.a + (double)(j - 1) * dt) + frac * dt;
    if (fabs(x) <= snap) x = 0.0;
    emit_knot(bp, td, i, x);
  }
  if (blk == 0 && tid == 0) {
    emit_knot(bp, td, 0, bp.a);
    emit_knot(bp, td, bp.N, bp.b);
  }
}

constexpr int kFinalizeThreads = 256;
// The projection's solve.  Every row of the Gram matrix has off-diagonal sum
// rho = 1/2 of its diagonal, and a step of parallel cyclic reduction takes
// rho to at most rho^2 in every row (the eliminated terms leave the diagonal
// and the couplings by the same amount): after six steps the couplings are
// below 2^-64 of the diagonal, so the system is diagonal in FP64 whatever N.
// Six steps also reach only 63 rows to either side, so a workgroup can solve
// kFinalizeRows rows by itself from them and kSolveHalo rows on each side.
constexpr int kSolveSteps = 6;
constexpr int kSolveHalo = 64;
constexpr int kFinalizeRows = 124;
// The map is written in rounds of kOwnCells cells per segment by the
// segments' own threads until kLongSegments or fewer per wave have cells left;
// these the whole wave fills, one after the other.  Knots crowd where f
// curves, so a tail can be one segment of hundreds of cells, at 18 ns each by
// one thread: a rebuild of the Gaussian of width 0.6 on [-5, 5] took 45.3 us
// at N = 1024 and 113 at 4096, and takes 27.1 and 52.4 (width 1: 26.5 and 50.5
// either way).  Filling every segment of more than 16 cells by the wave costs
// the Lorentzian, whose tails have many of them, 27 -> 33 us; two or four
// segments left instead of eight 0 - 4 us.
constexpr int kOwnCells = 16;
constexpr int kLongSegments = 8;

// 1 / d for a normal d: the hardware's estimate and two Newton steps, each
// one exact residual and one correction (last bit aside, the quotient an IEEE
// division gives, in half the dependent operations).
__device__ __forceinline__ double reciprocal(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  return fma(fma(-d, r, 1.0), r, r);
}

// Everything after the knots.  Workgroup g owns rows (knots) and segments
// [g kFinalizeRows, (g + 1) kFinalizeRows):
//  1. all knots into LDS: x_k = a + (b - a) k / N for a uniform partition,
//     otherwise the ones the inversion wrote; the knot-collapse check;
//     workgroup 0 also finds the deepest map cell (the evaluator's unrolled
//     compare depth);
//  2. (projection) <f, phi_k> by 16-point Gauss-Legendre per segment and the
//     FP64 solve of M c = b, one thread per row of the workgroup's window;
//  3. per owned segment k: its cells of the uniform index map lo[u] =
//     #{interior knots with cell < u} - segment k owns (cell(x_k),
//     cell(x_{k+1})], with cell(x_0) = -1 and cell(x_N) = K - 1, so each cell
//     is written once when the knots increase - and its record {x_k, v_k,
//     slope_k, x_{k+1}} (NaN for a collapsed table, whose map is all zero:
//     the evaluators never leave the table through it), in both images.
// What bounds it is latency: one workgroup did all of it in 18.5 us at
// N = 1024 and 50 us at N = 4096 (11 and 13 reduction steps with two barriers
// each); spread so, with one branch on the function per segment instead of
// one per node and the deepest cell found in passes of independent reads, it
// takes 9.8 and 10.8 us.
__global__ __launch_bounds__(kFinalizeThreads) void k_finalize(BuildParams bp, TableDev td) {
  __shared__ __align__(16) float X[PWL_MAX_N + 4];   // FP32 knots
  __shared__ double sA[2][kFinalizeThreads], sC[2][kFinalizeThreads], sD[2][kFinalizeThreads],
      sR[2][kFinalizeThreads];                       // the solve's rows, R the reciprocal diagonal
  __shared__ int s_maxc;
  const int N = bp.N, tid = threadIdx.x;
  const int r0 = blockIdx.x * kFinalizeRows;         // first owned row
  const int i = r0 - kSolveHalo + tid;               // this thread's row and segment
  const bool row = i >= 0 && i <= N, seg = i >= 0 && i < N;
  const bool own = tid >= kSolveHalo && tid < kSolveHalo + kFinalizeRows && row;
  const bool uniform = bp.partition == PWL_UNIFORM;

  // 1. knots, collapse, deepest cell
  if (tid == 0) s_maxc = 0;
  if (uniform) {
    for (int k = tid; k <= N; k += kFinalizeThreads) X[k] = (float)uniform_knot(bp, k);
  } else {
    stream::stage_copy(td.knots, (N + 4) / 4, kFinalizeThreads, X);   // whole words; the array is padded
    stream::staged();
  }
  __syncthreads();
  int bad = 0;
#pragma unroll 4
  for (int k = tid; k < N; k += kFinalizeThreads) bad |= (X[k + 1] > X[k]) ? 0 : 1;
  const bool collapsed = __syncthreads_or(bad) != 0;
  auto cell = [&](int k) { return map_cell(X[k], bp.a32, bp.scale32, bp.K); };
  if (blockIdx.x == 0) {
    // deeper than r if interior knot k + r shares the cell of knot k, for any
    // k: a pass per depth of independent reads; past four (the evaluators
    // take any such depth alike, and it may be thousands) run by run
    int depth = N >= 2 ? 1 : 0, more = depth;
    while (more && depth <= kMaxUnrolledCount) {
      int same = 0;
#pragma unroll 4
      for (int k = 1 + tid; k < N - depth; k += kFinalizeThreads) same |= (cell(k) == cell(k + depth)) ? 1 : 0;
      more = __syncthreads_or(same);
      if (more) ++depth;
    }
    int run = depth;
    for (int k = 1 + tid; more && k < N; k += kFinalizeThreads) {
      const int u = cell(k);
      if (k > 1 && cell(k - 1) == u) continue;       // not the first interior knot of its cell
      int r = 1;
      while (k + r <= N - 1 && cell(k + r) == u) ++r;
      run = max(run, r);
    }
    if (run > 0) atomicMax(&s_maxc, run);
  }

  // 2. vertex values
  double val = 0.0;
  if (bp.values == PWL_PROJ) {
    // one thread per segment: its 16 Gauss-Legendre nodes in order
    double left = 0.0, right = 0.0;                  // <f, phi_i>, <f, phi_{i+1}> on segment i
    if (seg) {
      const float xk = X[i];
      const float h = X[i + 1] - xk;
      float sl = 0.0f, sr = 0.0f;
      with_func(bp.f, [&](auto func) {
        constexpr int F = decltype(func)::value;
        // the cheap functions' evaluations all in flight together
        constexpr int kUnroll = (F == PWL_F_BESSEL_J0 || F == PWL_F_SAMPLED) ? 2 : kGaussPoints;
#pragma unroll kUnroll
        for (int q = 0; q < kGaussPoints; ++q) {
          const float t = bp.gl.t[q];
          const float fq = bp.gl.w[q] * f_value32_of<F>(bp.f, fmaf(h, t, xk));
          sl = fmaf(1.0f - t, fq, sl);
          sr = fmaf(t, fq, sr);
        }
      });
      left = (double)(h * sl);
      right = (double)(h * sr);
    }
    sR[1][tid] = right;
    __syncthreads();
    // Gram matrix of the hat basis from the element matrix (h/6)[[2,1],[1,2]]
    // (half hats at both ends), right-hand side b_i = <f, phi_i>
    double a = 0.0, c = 0.0, d = 1.0, b = 0.0;
    if (row) {
      const double xi = (double)X[i];
      const double hl = (i > 0) ? xi - (double)X[i - 1] : 0.0;
      const double hr = (i < N) ? (double)X[i + 1] - xi : 0.0;
      b = ((i > 0 && tid > 0) ? sR[1][tid - 1] : 0.0) + left;
      a = hl / 6.0;
      c = hr / 6.0;
      d = 2.0 * a + 2.0 * c;
    }
    sA[0][tid] = a; sC[0][tid] = c; sD[0][tid] = b; sR[0][tid] = reciprocal(d);
    __syncthreads();
    // Parallel cyclic reduction: at stride s every row eliminates its
    // couplings to rows i - s and i + s.  No pivoting is needed.  Rows next
    // to the window's ends miss a neighbour; none of them reaches an owned row.
#pragma unroll
    for (int step = 0; step < kSolveSteps; ++step) {
      const int s = 1 << step, p = step & 1;
      double an = 0.0, cn = 0.0;
      if (row && i - s >= 0 && tid - s >= 0) {
        const int q = tid - s;
        const double al = -a * sR[p][q];
        an = al * sA[p][q];
        d += al * sC[p][q];
        b += al * sD[p][q];
      }
      if (row && i + s <= N && tid + s < kFinalizeThreads) {
        const int q = tid + s;
        const double ga = -c * sR[p][q];
        cn = ga * sC[p][q];
        d += ga * sA[p][q];
        b += ga * sD[p][q];
      }
      a = an;
      c = cn;
      if (step + 1 < kSolveSteps) {
        sA[1 - p][tid] = a; sC[1 - p][tid] = c; sD[1 - p][tid] = b; sR[1 - p][tid] = reciprocal(d);
        __syncthreads();
      }
    }
    val = b / d;
    __syncthreads();
  } else if (row) {
    val = (double)(uniform ? f_value32(bp.f, X[i]) : td.values[i]);
  }
  sD[0][tid] = val;
  __syncthreads();

  // 3. values, flags and both images
  const int fw = image_soa_field_words(N), nkw = image_knot_words(N), nmw = image_map_words(bp.K);
  float* soa_k = td.soa + 8 * fw;                                         // the copies of kimg and lo
  uint16_t* soa_lo = reinterpret_cast<uint16_t*>(soa_k + 4 * nkw);
  if (own) {
    if (uniform) {
      td.knots64[i] = uniform_knot(bp, i);
      td.knots[i] = X[i];
    }
    td.values64[i] = val;
    td.values[i] = (float)val;
  }
  int u = 0, u1 = -1;                                // this segment's cells u .. u1
  if (own && seg) {
    const float x0 = X[i], x1 = X[i + 1], f0 = (float)val, f1 = (float)sD[0][tid + 1];
    float4 r;
    r.x = x0;
    r.y = f0;
    r.z = (float)(((double)f1 - (double)f0) / ((double)x1 - (double)x0));
    r.w = x1;
    if (collapsed) {
      r.y = __builtin_nanf("");
      r.z = __builtin_nanf("");
    }
    td.rec[i] = r;
    td.soa[i] = r.y;
    td.soa[4 * fw + i] = r.z;
    td.kimg[i] = x0;
    soa_k[i] = x0;
    if (!collapsed) {
      u = (i == 0) ? 0 : cell(i) + 1;
      u1 = (i + 1 == N) ? bp.K - 1 : cell(i + 1);
    }
  }
  uint64_t left;
  do {
    for (const int e = min(u1, u + kOwnCells - 1); u <= e; ++u) td.lo[u] = soa_lo[u] = (uint16_t)i;
    left = __ballot(u <= u1);
  } while (__popcll(left) > kLongSegments);
  for (; left; left &= left - 1) {
    const int src = __ffsll((unsigned long long)left) - 1;
    const int end = __shfl(u1, src, 64), k = __shfl(i, src, 64);
    for (int w = __shfl(u, src, 64) + (tid & 63); w <= end; w += 64) td.lo[w] = soa_lo[w] = (uint16_t)k;
  }
  if (collapsed)
    for (int u = blockIdx.x * kFinalizeThreads + tid; u < bp.K; u += gridDim.x * kFinalizeThreads)
      td.lo[u] = soa_lo[u] = 0;
  if (blockIdx.x == 0) {
    for (int k = N + tid; k < 4 * nkw; k += kFinalizeThreads) td.kimg[k] = soa_k[k] = __builtin_nanf("");
    for (int u = bp.K + tid; u < 8 * nmw; u += kFinalizeThreads)
      td.lo[u] = soa_lo[u] = (u == bp.K) ? (uint16_t)(N - 1) : (uint16_t)0;
    if (tid == 0) {
      // the density kernels may have raised DEGENERATE / NONFINITE
      uint32_t st = uniform ? 0u : td.status[0];
      if (collapsed) st |= PWL_FLAG_KNOTS_COLLAPSED;
      td.status[0] = st;
      td.status[1] = (uint32_t)s_maxc;
    }
  }
}

// ---- error-prediction integrals (choice of N for a target error) ----------
constexpr int kNormThreads = 1024;

// Block b of the fine grid t_j = a + j (b - a) / Q, j = 0..Q: trapezoid
// weights times |f''|^(2/5) and f''^2, and max |f''|, reduced in FP64 in a
// fixed order (a tree over the block's threads).
__global__ __launch_bounds__(kNormThreads) void k_norms(FuncDesc f, double a, double b, int Q,
                                                        double* __restrict__ part) {
  __shared__ double s_d[kNormThreads], s_q[kNormThreads], s_m[kNormThreads];
  const int tid = threadIdx.x;
  const int64_t j = (int64_t)blockIdx.x * kNormThreads + tid;
  const double dt = (b - a) / (double)Q;
  double d = 0.0, q = 0.0, m = 0.0;
  if (j <= Q) {
    const double x = a + (double)j * dt;
    const double f2 = f_second64(f, x);
    const double w = (j == 0 || j == Q) ? 0.5 * dt : dt;
    d = w * knot_density(f, x);
    q = w * f2 * f2;
    m = fabs(f2);
  }
  s_d[tid] = d;
  s_q[tid] = q;
  s_m[tid] = m;
  __syncthreads();
  for (int h = kNormThreads / 2; h >= 1; h >>= 1) {
    if (tid < h) {
      s_d[tid] += s_d[tid + h];
      s_q[tid] += s_q[tid + h];
      s_m[tid] = fmax(s_m[tid], s_m[tid + h]);
    }
    __syncthreads();
  }
  if (tid == 0) {
    part[3 * blockIdx.x] = s_d[0];
    part[3 * blockIdx.x + 1] = s_q[0];
    part[3 * blockIdx.x + 2] = s_m[0];
  }
}

// One thread adds the G block results in order: out = {int |f''|^(2/5),
// int f''^2, max |f''|}.
__global__ void k_norms_final(const double* __restrict__ part, int G, double* __restrict__ out) {
  if (threadIdx.x != 0) return;
  double d = 0.0, q = 0.0, m = 0.0;
  for (int g = 0; g < G; ++g) {
    d += part[3 * g];
    q += part[3 * g + 1];
    m = fmax(m, part[3 * g + 2]);
  }
  out[0] = d;
  out[1] = q;
  out[2] = m;
}

}  // namespace

int norm_blocks(int Q) { return Q / kNormThreads + 1; }

hipError_t launch_norms(const FuncDesc& f, double a, double b, int Q, double* scratch, hipStream_t s) {
  const int G = norm_blocks(Q);
  hipLaunchKernelGGL(k_norms, dim3(G), dim3(kNormThreads), 0, s, f, a, b, Q, scratch);
  hipLaunchKernelGGL(k_norms_final, dim3(1), dim3(64), 0, s, scratch, G, scratch + 3 * G);
  return hipGetLastError();
}

hipError_t launch_build(const BuildParams& bp, const TableDev& td, hipStream_t s) {
  if (bp.partition == PWL_OPTIMAL) {
    hipLaunchKernelGGL(k_density_totals, dim3(bp.G), dim3(kScanThreads), 0, s, bp, td);
    hipLaunchKernelGGL(k_invert_knots, dim3(bp.G), dim3(kScanThreads), 0, s, bp, td);
  }
  hipLaunchKernelGGL(k_finalize, dim3((bp.N + kFinalizeRows) / kFinalizeRows), dim3(kFinalizeThreads), 0, s, bp, td);
  return hipGetLastError();
}

}  // namespace pwl
