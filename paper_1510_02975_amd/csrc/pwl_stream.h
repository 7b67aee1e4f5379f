// Device building blocks of the streaming evaluators (single-table and
// batched): the LDS image of a table, the segment locate, one point of
// Algorithm 1 and of its derivative, and one grid-stride iteration over U
// float4 vectors per thread.
#pragma once

#include <hip/hip_runtime.h>

#include "pwl_internal.h"
#include "pwl_locate.h"

namespace pwl {
namespace stream {

typedef float v4f __attribute__((ext_vector_type(4)));
// The same read from any 4-byte boundary (one 16-byte load either way).
typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kWaitVm0 = 0x0F70;   // s_waitcnt vmcnt(0), the other counters not waited for

// Packed records: one 16-byte word per segment (a segment's lookup is one
// LDS read of 12 or 16 bytes).
struct Smem {
  float4* rec;      // [N]           {x_k, v_k, slope_k, x_{k+1}}
  float* knot;      // [N + pad]     knot[0] = a, knot[k] = x_k for 1 <= k <= N-1, NaN from N on
  uint16_t* lo;     // [K + 1]       lo[u] = #{interior knots in cells < u}; lo[K] = N - 1
  double* dv;       // [(N + 1) dvc] backward only: this workgroup's dL/dv, entry k of copy c at k dvc + c
  int dvc;          //               copies of dL/dv (a power of two; lane l adds into copy l mod dvc)
  __device__ __forceinline__ float4 record(int k) const { return rec[k]; }
};

// Structure-of-arrays records: v_k and slope_k in arrays of N floats, x_k in
// the knot array (no compare reads its entry 0).  A lookup reads the three fields separately, 4 bytes each.  Forward
// evaluation only.
struct SmemSoA {
  float* knot;      // [N + pad]  knot[0] = a, knot[k] = x_k for 1 <= k <= N-1, NaN from N on
  float* rv;        // [N] v_k
  float* rs;        // [N] slope_k
  uint16_t* lo;
  __device__ __forceinline__ float4 record(int k) const { return make_float4(knot[k], rv[k], rs[k], 0.0f); }
};

// Value/slope pairs: one 8-byte pair {v_k, slope_k} per segment, with x_k
// read from the knot array: a point reads its map cell, the knots of its cell
// with the one before them (the segment's own knot among them; adjacent, so one paired
// read for a cell of one knot) and one pair.  Forward evaluation only.
struct SmemPairs {
  float2* vs;       // [N]        {v_k, slope_k}
  float* knot;      // [N + pad]  knot[0] = a, knot[k] = x_k for 1 <= k <= N-1, NaN from N on
  uint16_t* lo;
};

// Sections of a table image (see image_words).  Every pointer is an offset
// from `base` itself: a pointer rebuilt from an integer would lose its
// address space, and LDS accesses (the dL/dv atomics above all) would go
// through the flat path.
__device__ __forceinline__ Smem carve(void* base, int N, int K, bool backward) {
  Smem s;
  s.rec = reinterpret_cast<float4*>(base);
  s.knot = reinterpret_cast<float*>(s.rec + N);
  s.lo = reinterpret_cast<uint16_t*>(reinterpret_cast<float4*>(s.knot) + image_knot_words(N));
  s.dv = backward ? reinterpret_cast<double*>(reinterpret_cast<float4*>(s.lo) + image_map_words(K)) : nullptr;
  s.dvc = backward ? dv_copies(N) : 1;
  return s;
}

// The structure-of-arrays image: values, slopes, knots, map.
__device__ __forceinline__ SmemSoA carve_soa(void* base, int N) {
  SmemSoA s;
  const int fw = image_soa_field_words(N);
  float4* b4 = reinterpret_cast<float4*>(base);
  s.rv = reinterpret_cast<float*>(b4);
  s.rs = reinterpret_cast<float*>(b4 + fw);
  s.knot = reinterpret_cast<float*>(b4 + 2 * fw);
  s.lo = reinterpret_cast<uint16_t*>(b4 + 2 * fw + image_knot_words(N));
  return s;
}

// The pairs image: the pairs (two per 16-byte word), then the knots and the
// map as in carve.
__device__ __forceinline__ SmemPairs carve_pairs(void* base, int N) {
  SmemPairs s;
  float4* b4 = reinterpret_cast<float4*>(base);
  s.vs = reinterpret_cast<float2*>(b4);
  s.knot = reinterpret_cast<float*>(b4 + image_pair_words(N));
  s.lo = reinterpret_cast<uint16_t*>(reinterpret_cast<float4*>(s.knot) + image_knot_words(N));
  return s;
}

// Record w, with v_override its value and slope re-derived as
// (v_{k+1} - v_k) / (x_{k+1} - x_k) in FP32.
__device__ __forceinline__ float4 record_word(const EvalTable& t, const float* __restrict__ vo, int w) {
  float4 r = t.rec[w];
  if (vo != nullptr) {
    const float v0 = vo[w], v1 = vo[w + 1];
    r.y = v0;
    r.z = (v1 - v0) / (r.w - r.x);
  }
  return r;
}

// Staging.  nt is the workgroup's size, passed as an argument (blockDim is a
// memory load at the head of every kernel that reads it).

// Words 0 .. n-1, word(w) put to LDS by put(w, .), four per thread per
// round: a round's loads are all issued before its first write (indices
// clamped: a load under a per-thread condition would be waited for before
// the next).
template <class Word, class Put>
__device__ __forceinline__ void stage_rounds(int n, int nt, const Word& word, const Put& put) {
  const int tid = threadIdx.x;
  for (int k0 = 0; k0 < n; k0 += 4 * nt) {
    float4 w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = word(min(k0 + j * nt + tid, n - 1));
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (k0 + j * nt + tid < n) put(k0 + j * nt + tid, w[j]);
  }
}

__device__ __forceinline__ int wave_first() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x) & ~63; }

// Copies n words from global memory to LDS without a register in between:
// all of a wave's loads are in flight at once (lane l's word lands at its
// wave's base + l).  The copy has arrived after staged().
__device__ __forceinline__ void stage_copy(const void* __restrict__ src, int n, int nt, void* dst) {
  const float4* __restrict__ s4 = reinterpret_cast<const float4*>(src);
  float4* d4 = reinterpret_cast<float4*>(dst);
  const int lane = threadIdx.x & 63;
  for (int w0 = wave_first(); w0 < n; w0 += nt) {
    if (w0 + lane < n)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(s4 + w0 + lane),
                                       (__attribute__((address_space(3))) void*)(d4 + w0), 16, 0, 0);
  }
}

// Waits for the wave's own part of the staging (and its other loads in
// flight); a barrier then makes the whole image visible.
__device__ __forceinline__ void staged() { __builtin_amdgcn_s_waitcnt(kWaitVm0); }

// Copies the table's image to LDS; with v_override the values and slopes are
// re-derived on the way.  staged() ends the copy.  (The override's path ends
// its own loads: pending ones would make the compiler wait for the copy
// where the paths join.)
__device__ __forceinline__ void stage_table(const EvalTable& t, const float* __restrict__ vo, int nt, const Smem& s) {
  const int nkm = image_knot_words(t.N) + image_map_words(t.K);
  if (vo == nullptr) {
    stage_copy(t.rec, t.N + nkm, nt, s.rec);
  } else {
    stage_copy(t.knots, nkm, nt, s.knot);
    stage_rounds(t.N, nt, [&](int w) { return record_word(t, vo, w); }, [&](int w, float4 r) { s.rec[w] = r; });
    staged();
  }
}

__device__ __forceinline__ void stage_table(const EvalTable& t, const float* __restrict__ vo, int nt,
                                            const SmemSoA& s) {
  const int fw = image_soa_field_words(t.N), nkm = image_knot_words(t.N) + image_map_words(t.K);
  if (vo == nullptr) {
    stage_copy(t.soa, 2 * fw + nkm, nt, s.rv);
  } else {
    stage_copy(t.soa + 8 * fw, nkm, nt, s.knot);
    stage_rounds(t.N, nt, [&](int w) { return record_word(t, vo, w); }, [&](int w, float4 r) {
      s.rv[w] = r.y;
      s.rs[w] = r.z;
    });
    staged();
  }
}

// A workgroup barrier that orders LDS accesses only: global loads and
// stores a wave still has in flight are not waited for (__syncthreads
// would).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The pairs image: word w holds the pairs of segments 2w and 2w + 1 (zero
// past N - 1).
__device__ __forceinline__ float4 pair_word(const EvalTable& t, const float* __restrict__ vo, int w) {
  const float4 r0 = record_word(t, vo, 2 * w);
  float4 r1 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (2 * w + 1 < t.N) r1 = record_word(t, vo, 2 * w + 1);
  return make_float4(r0.y, r0.z, r1.y, r1.z);
}

__device__ __forceinline__ void stage_table(const EvalTable& t, const float* __restrict__ vo, int nt,
                                            const SmemPairs& s) {
  stage_copy(t.knots, image_knot_words(t.N) + image_map_words(t.K), nt, s.knot);
  float4* pair4 = reinterpret_cast<float4*>(s.vs);
  stage_rounds(image_pair_words(t.N), nt, [&](int w) { return pair_word(t, vo, w); },
               [&](int w, float4 p) { pair4[w] = p; });
  staged();
}

// A forward image's record section by words: how many, a word's load and its
// place.
__device__ __forceinline__ int section_words(const EvalTable& t, const Smem&) { return t.N; }
__device__ __forceinline__ int section_words(const EvalTable& t, const SmemSoA&) { return t.N; }
__device__ __forceinline__ int section_words(const EvalTable& t, const SmemPairs&) { return image_pair_words(t.N); }
template <class S>
__device__ __forceinline__ float4 section_word(const EvalTable& t, const float* __restrict__ vo, int w, const S&) {
  return record_word(t, vo, w);
}
__device__ __forceinline__ float4 section_word(const EvalTable& t, const float* __restrict__ vo, int w,
                                               const SmemPairs&) {
  return pair_word(t, vo, w);
}
__device__ __forceinline__ void put_word(const Smem& s, int w, float4 r) { s.rec[w] = r; }
__device__ __forceinline__ void put_word(const SmemSoA& s, int w, float4 r) {
  s.rv[w] = r.y;
  s.rs[w] = r.z;
}
__device__ __forceinline__ void put_word(const SmemPairs& s, int w, float4 p) {
  reinterpret_cast<float4*>(s.vs)[w] = p;
}

// An image through registers where it is not much larger than the workgroup:
// every thread loads its first word of each section before it writes any, and
// the rest follows (staged() ends it).
template <class S>
__device__ __forceinline__ void stage_words(const EvalTable& t, const float* __restrict__ vo, int nt, const S& s) {
  const int tid = threadIdx.x;
  const int nrw = section_words(t, s), nkw = image_knot_words(t.N), nmw = image_map_words(t.K);
  float4* knot4 = reinterpret_cast<float4*>(s.knot);
  float4* map4 = reinterpret_cast<float4*>(s.lo);
  const bool hr = tid < nrw, hk = tid < nkw, hm = tid < nmw;
  float4 r = make_float4(0.0f, 0.0f, 0.0f, 0.0f), k = r, m = r;
  if (hr) r = section_word(t, vo, tid, s);
  if (hk) k = reinterpret_cast<const float4*>(t.knots)[tid];
  if (hm) m = reinterpret_cast<const float4*>(t.lo)[tid];
  if (hr) put_word(s, tid, r);
  if (hk) knot4[tid] = k;
  if (hm) map4[tid] = m;
  for (int w = tid + nt; w < nrw; w += nt) put_word(s, w, section_word(t, vo, w, s));
  if (nkw > nt) stage_copy(t.knots + 4 * nt, nkw - nt, nt, knot4 + nt);
  if (nmw > nt) stage_copy(t.lo + 8 * nt, nmw - nt, nt, map4 + nt);
}

__device__ __forceinline__ float clamp_nan(float x, float a, float b) {
  return (x < a) ? a : ((x > b) ? b : x);   // NaN passes through
}

// Segment of x when no map cell holds more than MAXC knots: compare x with
// the MAXC knots that follow lo[cell(x)].  Knots beyond the cell's own are
// greater than x (they lie in later cells) and the sentinels are NaN, so the
// extra compares are false; the count of true compares is exact.
template <int MAXC, class S>
__device__ __forceinline__ int locate_fixed(float x, const TableShape& t, const S& s) {
  const int u = map_cell(x, t.a32, t.scale32, t.K);
  const int lo = s.lo[u];
  int seg = lo;
#pragma unroll
  for (int j = 1; j <= MAXC; ++j) seg += (x >= s.knot[lo + j]) ? 1 : 0;
  return seg;
}

// Any number of knots per cell: the count is lo[u+1] - lo[u].
template <class S>
__device__ __forceinline__ int locate_any(float x, const TableShape& t, const S& s) {
  const int u = map_cell(x, t.a32, t.scale32, t.K);
  const int lo = s.lo[u];
  const int cnt = (int)s.lo[u + 1] - lo;
  int seg = lo;
  for (int j = 1; j <= cnt; ++j) seg += (x >= s.knot[lo + j]) ? 1 : 0;
  return seg;
}

// The paper's GPU locate (Sec. IV-V): a branch-free binary search over the
// knots, here the interior knots in LDS.  It counts the interior knots <= x
// (so x_i <= x < x_{i+1}; NaN x compares false and gives 0), halving a
// power-of-two step from the largest one below N.
template <class S>
__device__ __forceinline__ int locate_search(float x, const TableShape& t, const S& s) {
  int lo = 0;
  for (int half = (t.N > 1) ? (1 << (31 - __builtin_clz(t.N - 1))) : 0; half >= 1; half >>= 1) {
    const int k = lo + half;
    lo = (k < t.N && s.knot[k] <= x) ? k : lo;
  }
  return lo;
}

// MAXC > 0: map + MAXC unrolled compares; 0: map + counted compares;
// -1: binary search without the map.
template <int MAXC, class S>
__device__ __forceinline__ int locate(float x, const TableShape& t, const S& s) {
  if (MAXC > 0) return locate_fixed<MAXC>(x, t, s);
  if (MAXC < 0) return locate_search(x, t, s);
  return locate_any(x, t, s);
}

template <int MAXC, class S>
__device__ __forceinline__ float eval_point(float x, const TableShape& t, const S& s) {
  const int seg = locate<MAXC>(x, t, s);
  const float4 r = s.record(seg);
  return fmaf(clamp_nan(x, t.a32, t.b32) - r.x, r.z, r.y);
}

// Algorithm 1 through the pairs image.  With MAXC unrolled compares the
// segment's knot comes out of the compares themselves (the last knot of the
// cell that x reaches, or the knot before the cell), so the knot reads are
// adjacent; otherwise it is read after the locate.  The same operations on
// the same values as eval_point, so the outputs are bit-identical.
template <int MAXC>
__device__ __forceinline__ float eval_point(float x, const TableShape& t, const SmemPairs& s) {
  int seg;
  float xs;
  if (MAXC > 0) {
    const int u = map_cell(x, t.a32, t.scale32, t.K);
    const int lo = s.lo[u];
    seg = lo;
    xs = s.knot[lo];
#pragma unroll
    for (int j = 1; j <= MAXC; ++j) {
      const float kj = s.knot[lo + j];
      const bool c = x >= kj;
      seg += c ? 1 : 0;
      xs = c ? kj : xs;
    }
  } else {
    seg = locate<MAXC>(x, t, s);
    xs = s.knot[seg];
  }
  const float2 p = s.vs[seg];
  return fmaf(clamp_nan(x, t.a32, t.b32) - xs, p.y, p.x);
}

template <int MAXC, bool WY, bool WDX, bool WDV>
__device__ __forceinline__ void backward_point(float x, float g, const TableShape& t, const Smem& s,
                                               float& y, float& dx) {
  const int seg = locate<MAXC>(x, t, s);
  const float4 r = s.rec[seg];
  const float d = clamp_nan(x, t.a32, t.b32) - r.x;
  if (WY) y = fmaf(d, r.z, r.y);
  if (WDX) {
    const bool inside = (x >= t.a32) && (x <= t.b32);
    dx = inside ? g * r.z : ((x != x) ? x : 0.0f);
  }
  if (WDV) {
    if (x == x) {
      // The workgroup's dL/dv lives in LDS as FP64: FP64 LDS atomic adds run
      // at full rate on gfx950 (FP32 ones take a slow path) and keep the
      // per-workgroup sums exact to FP32 output precision.  Workgroup scope,
      // relaxed: no point has to wait for the thread's outstanding stores.
      // Each hat weight comes from its own knot distance, (x_{k+1} - x)/h and
      // (x - x_k)/h, with x_{k+1} from the record: forming (1 - delta) g as
      // g - delta g would cancel when delta is near 1.
      const float xc = clamp_nan(x, t.a32, t.b32);
      const float rh = __builtin_amdgcn_rcpf(r.w - r.x);   // 1/h, within 1 ulp
      const float w0 = ((r.w - xc) * rh) * g;   // (1 - delta) g
      const float w1 = (d * rh) * g;            // delta g
      const int at = seg * s.dvc + ((int)__lane_id() & (s.dvc - 1));
      __hip_atomic_fetch_add(s.dv + at, (double)w0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __hip_atomic_fetch_add(s.dv + at + s.dvc, (double)w1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
}

// Which points of [begin, end) go through 16-byte vectors on the 16-byte
// boundaries of array p (the arrays are then 4-byte aligned: vec):
// [head, 4 vend) is vectorised and the points before `head` and from
// max(head, 4 vend) on are scalar.  p is an array that is written; the
// others are read (a second output written) across their own boundaries,
// which the hardware does for any 4-byte address.  2^23.6 points with x one
// element off y's boundaries: 27.8 us point by point, 19.1 us so.
struct Split {
  int64_t head, vbeg, vend;
};

__device__ __forceinline__ Split split_range(const float* p, int64_t begin, int64_t end, bool vec) {
  Split r;
  if (!vec) {
    r.head = end;
    r.vbeg = r.vend = 0;
    return r;
  }
  // element index whose address is 16-byte aligned, at or after begin
  const int64_t phase = (int64_t)((reinterpret_cast<uintptr_t>(p) >> 2) & 3);
  int64_t h = begin + ((4 - ((phase + begin) & 3)) & 3);
  if (h > end) h = end;
  r.head = h;
  r.vbeg = (phase + h) >> 2;               // in units of the aligned float4 array
  r.vend = (phase + end) >> 2;
  if (r.vend < r.vbeg) r.vend = r.vbeg;
  return r;
}

// Lookups of one vector.
template <int MAXC, class S>
__device__ __forceinline__ v4f eval_vec(const v4f& xv, const TableShape& t, const S& s) {
  v4f yv;
  yv.x = eval_point<MAXC>(xv.x, t, s);
  yv.y = eval_point<MAXC>(xv.y, t, s);
  yv.z = eval_point<MAXC>(xv.z, t, s);
  yv.w = eval_point<MAXC>(xv.w, t, s);
  return yv;
}

// One iteration over U float4 vectors per thread: all loads, then all table
// lookups, then all stores.  Full iterations run unguarded so the compiler
// can count outstanding memory operations exactly (a guarded load makes
// every later wait a wait for all stores); the last, partial iteration of a
// thread is guarded.
template <int U, int MAXC, bool GUARD, class S>
__device__ __forceinline__ void fwd_iter(const TableShape& t, const S& s, const v4fu* __restrict__ x4,
                                         v4f* __restrict__ y4, int64_t base, int64_t bs, int64_t n4) {
  v4f xv[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t i = base + u * bs;
    if (!GUARD || i < n4) xv[u] = __builtin_nontemporal_load(x4 + i);
  }
  v4f yv[U];
#pragma unroll
  for (int u = 0; u < U; ++u) yv[u] = eval_vec<MAXC>(xv[u], t, s);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t i = base + u * bs;
    if (!GUARD || i < n4) __builtin_nontemporal_store(yv[u], y4 + i);
  }
}

// Forward over points [begin, end) by `nblk` cooperating workgroups (this one
// is number `blk`): workgroup blk streams vectors blk*bs*U + u*bs + tid of
// each stride of nblk*bs*U vectors.
template <int U, int MAXC, class S>
__device__ __forceinline__ void fwd_range(const EvalTable& t, const S& s, const float* __restrict__ x,
                                          float* __restrict__ y, int64_t begin, int64_t end, bool vec,
                                          int64_t blk, int64_t nblk, int nt) {
  const Split sp = split_range(y, begin, end, vec);
  const int64_t bs = nt, tid = threadIdx.x;
  const int64_t gtid = blk * bs + tid, gthreads = nblk * bs;
  for (int64_t i = begin + gtid; i < sp.head; i += gthreads) y[i] = eval_point<MAXC>(x[i], t, s);
  if (sp.vend > sp.vbeg) {
    const int64_t phase = (int64_t)((reinterpret_cast<uintptr_t>(y) >> 2) & 3);
    const v4fu* __restrict__ x4 = reinterpret_cast<const v4fu*>(x - phase);
    v4f* __restrict__ y4 = reinterpret_cast<v4f*>(y - phase);
    const int64_t stride = nblk * bs * U;
    int64_t base = sp.vbeg + blk * bs * U + tid;
    for (; base + (U - 1) * bs < sp.vend; base += stride) fwd_iter<U, MAXC, false>(t, s, x4, y4, base, bs, sp.vend);
    if (base < sp.vend) fwd_iter<U, MAXC, true>(t, s, x4, y4, base, bs, sp.vend);
  }
  const int64_t tail = (sp.vend > sp.vbeg) ? 4 * sp.vend - (int64_t)((reinterpret_cast<uintptr_t>(y) >> 2) & 3)
                                           : sp.head;
  for (int64_t i = (tail > sp.head ? tail : sp.head) + gtid; i < end; i += gthreads)
    y[i] = eval_point<MAXC>(x[i], t, s);
}

template <int U, bool WY, bool WDX, bool WDV>
struct Bwd {
  template <int MAXC, bool GUARD>
  __device__ __forceinline__ static void iter(const TableShape& t, const Smem& s, const v4fu* __restrict__ x4,
                                              const v4fu* __restrict__ g4, v4fu* __restrict__ y4,
                                              v4fu* __restrict__ dx4, int64_t base, int64_t bs, int64_t n4) {
    v4f xv[U], gv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = base + u * bs;
      if (!GUARD || i < n4) {
        xv[u] = __builtin_nontemporal_load(x4 + i);
        gv[u] = __builtin_nontemporal_load(g4 + i);
      }
    }
    v4f yv[U], dxv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (GUARD && base + u * bs >= n4) continue;
      float yy = 0.0f, dd = 0.0f;
      backward_point<MAXC, WY, WDX, WDV>(xv[u].x, gv[u].x, t, s, yy, dd); yv[u].x = yy; dxv[u].x = dd;
      backward_point<MAXC, WY, WDX, WDV>(xv[u].y, gv[u].y, t, s, yy, dd); yv[u].y = yy; dxv[u].y = dd;
      backward_point<MAXC, WY, WDX, WDV>(xv[u].z, gv[u].z, t, s, yy, dd); yv[u].z = yy; dxv[u].z = dd;
      backward_point<MAXC, WY, WDX, WDV>(xv[u].w, gv[u].w, t, s, yy, dd); yv[u].w = yy; dxv[u].w = dd;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = base + u * bs;
      if (!GUARD || i < n4) {
        if (WY) __builtin_nontemporal_store((v4fu)yv[u], y4 + i);
        if (WDX) __builtin_nontemporal_store((v4fu)dxv[u], dx4 + i);
      }
    }
  }

  // Fused forward + backward over points [begin, end), cooperating
  // workgroups as in fwd_range.
  template <int MAXC>
  __device__ __forceinline__ static void range(const TableShape& t, const Smem& s,
                                               const float* __restrict__ x, const float* __restrict__ g,
                                               float* __restrict__ y, float* __restrict__ dx, int64_t begin,
                                               int64_t end, bool vec, int64_t blk, int64_t nblk, int nt) {
    const float* aligned = WY ? y : (WDX ? dx : x);
    const Split sp = split_range(aligned, begin, end, vec);
    const int64_t bs = nt, tid = threadIdx.x;
    const int64_t gtid = blk * bs + tid, gthreads = nblk * bs;
    for (int64_t i = begin + gtid; i < sp.head; i += gthreads) scalar<MAXC>(t, s, x, g, y, dx, i);
    const int64_t phase = (int64_t)((reinterpret_cast<uintptr_t>(aligned) >> 2) & 3);
    if (sp.vend > sp.vbeg) {
      const v4fu* __restrict__ x4 = reinterpret_cast<const v4fu*>(x - phase);
      const v4fu* __restrict__ g4 = reinterpret_cast<const v4fu*>(g - phase);
      v4fu* __restrict__ y4 = WY ? reinterpret_cast<v4fu*>(y - phase) : nullptr;
      v4fu* __restrict__ dx4 = WDX ? reinterpret_cast<v4fu*>(dx - phase) : nullptr;
      const int64_t stride = nblk * bs * U;
      int64_t base = sp.vbeg + blk * bs * U + tid;
      for (; base + (U - 1) * bs < sp.vend; base += stride)
        iter<MAXC, false>(t, s, x4, g4, y4, dx4, base, bs, sp.vend);
      if (base < sp.vend) iter<MAXC, true>(t, s, x4, g4, y4, dx4, base, bs, sp.vend);
    }
    const int64_t tail = (sp.vend > sp.vbeg) ? 4 * sp.vend - phase : sp.head;
    for (int64_t i = (tail > sp.head ? tail : sp.head) + gtid; i < end; i += gthreads)
      scalar<MAXC>(t, s, x, g, y, dx, i);
  }

  template <int MAXC>
  __device__ __forceinline__ static void scalar(const TableShape& t, const Smem& s, const float* __restrict__ x,
                                                const float* __restrict__ g, float* __restrict__ y,
                                                float* __restrict__ dx, int64_t i) {
    float yy = 0.0f, dd = 0.0f;
    backward_point<MAXC, WY, WDX, WDV>(x[i], g[i], t, s, yy, dd);
    if (WY) y[i] = yy;
    if (WDX) dx[i] = dd;
  }
};

}  // namespace stream
}  // namespace pwl
