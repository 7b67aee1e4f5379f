// Sample application of the approximation (Sec. VI-A): per-pixel sums of
// Gaussian kernels of a nonparametric background model.  For pixel (y, x)
// of the current frame and every pixel (y', x') of the (2r+1) x (2r+1)
// window (clamped to the image) in each of T reference frames,
//   L(y, x) = 1 / (T (2r+1)^2) * sum prod_{c = R, G, B} g((f_c - h_c) / sigma_c),
// with g(u) = exp(-u^2 / 2) evaluated either through a CPWL table (|u| when
// the table's domain starts at 0) or with expf / __expf - the comparison the
// paper makes for this application.  The sum is accumulated in FP64 so that
// only the kernel evaluations round.
//
// The channels are 8-bit, so g has 511 arguments per channel in a whole
// call: every workgroup evaluates it at all of them once (six evaluations
// per thread against 4800 for the kernel values of its pixels one by one at
// T = 16, r = 2) into an LDS list per channel, and a tap is three LDS reads
// at f_c - h_c, two products and one FP64 addition.  Neighbouring pixels'
// differences are near each other and consecutive list entries lie in
// consecutive banks, so the reads hardly conflict (6% of the LDS cycles).
// What bounds the kernel is VALU issue - 10 instructions per tap in all, two
// of them FP64 - so a thread takes kPx pixels of a row: it extracts the bytes
// of a reference pixel once for all of its pixels that have it in their
// windows, and the next row's loads are in flight while one is summed.
// 1080 x 1920, T = 16, r = 2: a uniform N = 64 table 1491 us with one table
// evaluation per kernel value, 343 us so (0.17 ns per pixel), expf and
// __expf the same; outputs bit-identical where one wave sums all frames.
#include <hip/hip_runtime.h>

#include "pwl_internal.h"
#include "pwl_stream.h"

namespace pwl {

namespace {

using namespace stream;

constexpr int kKdeThreads = 256;
constexpr int kPx = 4;                      // consecutive pixels of a row per thread
constexpr int kTileBits = 4;                // a wave's tile: at most 2^4 lanes along a row (64 x 4 pixels)
constexpr int kWaves = kKdeThreads / 64;
constexpr int kListLen = 512;               // differences -255 .. 255 of one channel

// The table's arrays in global memory: the list of a workgroup needs too few
// evaluations to stage the table's image for.
struct GlobalTable {
  const float4* rec;
  const float* knot;
  const uint16_t* lo;
  __device__ __forceinline__ float4 record(int k) const { return rec[k]; }
};

__device__ __forceinline__ float kernel_g(int mode, float u, const EvalTable& t) {
  if (mode == PWL_KDE_TABLE) {
    const GlobalTable s{t.rec, t.knots, t.lo};
    return eval_point<0>(t.a32 >= 0.0f ? fabsf(u) : u, t, s);
  }
  return mode == PWL_KDE_EXPF ? expf(-0.5f * u * u) : __expf(-0.5f * u * u);
}

// The reference pixels of columns x0 - R .. x0 + kPx - 1 + R of one row,
// clamped to the image.
template <int R>
__device__ __forceinline__ void load_row(const uint32_t* __restrict__ row, int x0, int W, bool inside,
                                         uint32_t (&h)[kPx + 2 * R]) {
  if (inside) {
    __builtin_memcpy(h, row + (x0 - R), sizeof(h));
  } else {
#pragma unroll
    for (int c = 0; c < kPx + 2 * R; ++c) h[c] = row[min(max(x0 - R + c, 0), W - 1)];
  }
}

// One tap: list entries at byte offsets at[c] (that of difference f_c) minus
// 4 h_c.
__device__ __forceinline__ float tap(const char* list, const int (&at)[3], int h0, int h1, int h2) {
  const float g0 = *reinterpret_cast<const float*>(list + (at[0] - h0));
  const float g1 = *reinterpret_cast<const float*>(list + (at[1] - h1));
  const float g2 = *reinterpret_cast<const float*>(list + (at[2] - h2));
  return g0 * g1 * g2;
}

// R >= 0: the window radius; -1: any radius, from r.  A wave's tile has 2^bits
// lanes along a row and the others along y.  S waves of a workgroup share a
// tile, each with its part of the reference frames or, where S does not divide
// their number (ROWS), of the T (2r+1) rows of the windows.
template <int R, int S, bool ROWS>
__global__ __launch_bounds__(kKdeThreads) void k_kde(EvalTable t, int mode, const uint32_t* __restrict__ frame,
                                                     const uint32_t* __restrict__ hist, int H, int W, int T,
                                                     int r, int bits, float is0, float is1, float is2,
                                                     float* __restrict__ out) {
  __shared__ float s_list[3 * kListLen];
  __shared__ double s_part[S > 1 ? kWaves * 64 * kPx : 1];
  const int tid = threadIdx.x;
  for (int i = tid; i < 3 * kListLen; i += kKdeThreads) {
    const int c = i / kListLen, d = i % kListLen - 255;
    s_list[i] = kernel_g(mode, (float)d * (c == 0 ? is0 : (c == 1 ? is1 : is2)), t);
  }
  __syncthreads();
  const int wave = tid >> 6, lane = tid & 63, part = wave % S;
  const int x0 = ((blockIdx.x << bits) + (lane & ((1 << bits) - 1))) * kPx;
  const int y = ((blockIdx.y * (kWaves / S) + wave / S) << (6 - bits)) + (lane >> bits);
  double sum[kPx] = {};
  if (x0 < W && y < H) {
    const char* list = reinterpret_cast<const char*>(s_list);
    int at[kPx][3];
#pragma unroll
    for (int j = 0; j < kPx; ++j) {
      const uint32_t p = frame[(int64_t)y * W + min(x0 + j, W - 1)];
      at[j][0] = 4 * (255 + (int)(p & 255u));
      at[j][1] = 4 * (255 + kListLen + (int)((p >> 8) & 255u));
      at[j][2] = 4 * (255 + 2 * kListLen + (int)((p >> 16) & 255u));
    }
    // ROWS: window rows [i0, i1) of fewer than 2^30, row i being row
    // i % (2r+1) - r of the window in frame i / (2r+1)
    const uint32_t w = R >= 0 ? 2 * R + 1 : 2 * (uint32_t)r + 1;
    const uint32_t n = (uint32_t)T * w, i0 = n * part / S, i1 = n * (part + 1) / S;
    const int k0 = ROWS ? (int)(i0 / w) : (int)((int64_t)T * part / S);
    const int k1 = ROWS ? (int)((i1 + w - 1) / w) : (int)((int64_t)T * (part + 1) / S);
    for (int k = k0; k < k1; ++k) {
      const uint32_t* __restrict__ hk = hist + (int64_t)k * H * W;
      const int dy0 = ROWS && k == k0 ? (int)(i0 - k * w) - r : -r;
      const int dy1 = ROWS && k == k1 - 1 ? (int)(i1 - k * w) - r - 1 : r;   // the last row
      if constexpr (R >= 0) {
        // one row of the window at a time, the next row's loads in flight
        const bool inside = x0 >= R && x0 + kPx + R <= W;
        auto row = [&](int dy) { return hk + (int64_t)min(max(y + dy, 0), H - 1) * W; };
        uint32_t h[kPx + 2 * R], hn[kPx + 2 * R];
        load_row<R>(row(dy0), x0, W, inside, h);
#pragma unroll 1
        for (int dy = dy0; dy <= dy1; ++dy) {
          load_row<R>(row(min(dy + 1, dy1)), x0, W, inside, hn);
#pragma unroll
          for (int c = 0; c < kPx + 2 * R; ++c) {
            const int h0 = 4 * (int)(h[c] & 255u), h1 = 4 * (int)((h[c] >> 8) & 255u),
                      h2 = 4 * (int)((h[c] >> 16) & 255u);
#pragma unroll
            for (int j = 0; j < kPx; ++j)
              if (c >= j && c - j <= 2 * R) sum[j] += (double)tap(list, at[j], h0, h1, h2);
          }
#pragma unroll
          for (int c = 0; c < kPx + 2 * R; ++c) h[c] = hn[c];
        }
      } else {
        for (int dy = dy0; dy <= dy1; ++dy) {
          const uint32_t* __restrict__ row = hk + (int64_t)min(max(y + dy, 0), H - 1) * W;
          for (int c = 0; c < kPx + 2 * r; ++c) {
            const uint32_t h = row[min(max(x0 - r + c, 0), W - 1)];
            const int h0 = 4 * (int)(h & 255u), h1 = 4 * (int)((h >> 8) & 255u), h2 = 4 * (int)((h >> 16) & 255u);
#pragma unroll
            for (int j = 0; j < kPx; ++j)
              if (c >= j && c - j <= 2 * r) sum[j] += (double)tap(list, at[j], h0, h1, h2);
          }
        }
      }
    }
  }
  if constexpr (S > 1) {   // the parts' sums, added in order
#pragma unroll
    for (int j = 0; j < kPx; ++j) s_part[(wave * kPx + j) * 64 + lane] = sum[j];
    __syncthreads();
    if (part != 0) return;
#pragma unroll
    for (int j = 0; j < kPx; ++j)
      for (int q = 1; q < S; ++q) sum[j] += s_part[((wave + q) * kPx + j) * 64 + lane];
  }
  if (x0 >= W || y >= H) return;
  const int w = 2 * r + 1;
#pragma unroll
  for (int j = 0; j < kPx; ++j)
    if (x0 + j < W) out[(int64_t)y * W + x0 + j] = (float)(sum[j] / ((double)T * w * w));
}

template <int R>
void launch_kde_r(const EvalTable& t, int mode, const uint32_t* f, const uint32_t* h, int H, int W, int T, int r,
                  float is0, float is1, float is2, float* out, int num_cu, hipStream_t s) {
  // The widest tile that pads the rows by at most a sixth, since what a tile
  // has beyond the image is computed all the same; one lane along a row (whose
  // lanes each read a row of their own) only where two would pad a seventh more.
  // About 10^6 pixels of uniformly distributed bytes, 64-pixel tiles -> these:
  // T = 16, r = 2, W = 1 4972 -> 864 us, 16 446 -> 222, 33 308 -> 264, 65 442 ->
  // 242, 97 303 -> 248, 200 278 -> 237; T = 2, r = 1, W = 16 27.2 -> 14.5, 65 25.4
  // -> 20.0, but 130 17.0 -> 17.9.  From 330 pixels on it is the widest.
  int bits = kTileBits;
  auto columns = [&](int b) { return ((int64_t)W + (kPx << b) - 1) / (kPx << b); };
  auto padded = [&](int b) { return columns(b) * (kPx << b); };
  while (bits > 0 && padded(bits) > (int64_t)W + W / 6) --bits;
  if (bits == 0 && 7 * padded(1) <= 8 * padded(0)) bits = 1;
  const int th = 64 >> bits;
  const unsigned gx = (unsigned)columns(bits);
  const int64_t tiles = (int64_t)gx * ((H + th - 1) / th);
  auto launch = [&](auto kernel, int S) {
    const int rows = th * kWaves / S;
    hipLaunchKernelGGL(kernel, dim3(gx, (unsigned)((H + rows - 1) / rows)), dim3(kKdeThreads), 0, s, t, mode, f, h, H,
                       W, T, r, bits, is0, is1, is2, out);
  };
  // One wave per tile leaves a small image with few waves, and a mid-sized
  // one with an uneven last round (24 waves fit a CU): the frames, or the rows of
  // all windows, are then split over 2 or 4 waves.  With at least 100 taps per part (16
  // frames, r = 2; one frame, r = 10) it pays up to 60 waves per CU, with fewer
  // up to 16.  One wave per tile -> the split chosen, uniformly distributed
  // bytes: 288 x 352 T = 16, r = 2 67 -> 32 us, T = 1, r = 32 1363 -> 378;
  // 480 x 640 T = 16, r = 2 115 -> 74, T = 1, r = 4 34 -> 23; 720 x 1280 T = 16,
  // r = 2 227 -> 207; past it 1080 x 1920 439 (437 in 4 parts); fewer taps: 480 x
  // 640 T = 2, r = 2 17.6 -> 14.6, past it 720 x 1280 T = 1, r = 1 9.5 (12.4 in
  // 4 parts).
  const int64_t rows_of_all = (int64_t)T * (2 * r + 1), taps = rows_of_all * (2 * r + 1);
  auto splits = [&](int S) {
    return rows_of_all >= S && rows_of_all < (1 << 30) && tiles * S <= (int64_t)num_cu * (taps >= 100 * S ? 60 : 16);
  };
  if (splits(4)) {
    if (T % 4 == 0) launch(k_kde<R, 4, false>, 4); else launch(k_kde<R, 4, true>, 4);
  } else if (splits(2)) {
    if (T % 2 == 0) launch(k_kde<R, 2, false>, 2); else launch(k_kde<R, 2, true>, 2);
  } else {
    launch(k_kde<R, 1, false>, 1);
  }
}

}  // namespace

hipError_t launch_kde(const EvalTable& t, int mode, const void* frame, const void* hist, int H, int W, int T,
                      int r, const float* sigma, float* out, int num_cu, hipStream_t s) {
  const float is0 = 1.0f / sigma[0], is1 = 1.0f / sigma[1], is2 = 1.0f / sigma[2];
  const uint32_t* f = static_cast<const uint32_t*>(frame);
  const uint32_t* h = static_cast<const uint32_t*>(hist);
  switch (r) {
    case 1: launch_kde_r<1>(t, mode, f, h, H, W, T, r, is0, is1, is2, out, num_cu, s); break;
    case 2: launch_kde_r<2>(t, mode, f, h, H, W, T, r, is0, is1, is2, out, num_cu, s); break;
    case 3: launch_kde_r<3>(t, mode, f, h, H, W, T, r, is0, is1, is2, out, num_cu, s); break;
    default: launch_kde_r<-1>(t, mode, f, h, H, W, T, r, is0, is1, is2, out, num_cu, s); break;
  }
  return hipGetLastError();
}

}  // namespace pwl
