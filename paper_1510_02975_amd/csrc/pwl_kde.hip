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
constexpr int kTileLanes = 16;              // lanes along a row; the wave's other 4 along y
constexpr int kTileW = kTileLanes * kPx;    // a wave's tile: 64 x 4 pixels
constexpr int kTileH = 64 / kTileLanes;
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

// R >= 0: the window radius; -1: any radius, from r.  S waves of a workgroup
// share a tile, each with its part of the reference frames.
template <int R, int S>
__global__ __launch_bounds__(kKdeThreads) void k_kde(EvalTable t, int mode, const uint32_t* __restrict__ frame,
                                                     const uint32_t* __restrict__ hist, int H, int W, int T,
                                                     int r, float is0, float is1, float is2,
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
  const int x0 = blockIdx.x * kTileW + (lane % kTileLanes) * kPx;
  const int y = blockIdx.y * (kTileH * kWaves / S) + (wave / S) * kTileH + lane / kTileLanes;
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
    const int k1 = (int)((int64_t)T * (part + 1) / S);
    for (int k = (int)((int64_t)T * part / S); k < k1; ++k) {
      const uint32_t* __restrict__ hk = hist + (int64_t)k * H * W;
      if constexpr (R >= 0) {
        // one row of the window at a time, the next row's loads in flight
        const bool inside = x0 >= R && x0 + kPx + R <= W;
        auto row = [&](int dy) { return hk + (int64_t)min(max(y + dy, 0), H - 1) * W; };
        uint32_t h[kPx + 2 * R], hn[kPx + 2 * R];
        load_row<R>(row(-R), x0, W, inside, h);
#pragma unroll 1
        for (int dy = -R; dy <= R; ++dy) {
          load_row<R>(row(min(dy + 1, R)), x0, W, inside, hn);
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
        for (int dy = -r; dy <= r; ++dy) {
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
  if constexpr (S > 1) {   // the parts' sums, added in frame order
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
  const unsigned gx = (unsigned)((W + kTileW - 1) / kTileW);
  const int64_t tiles = (int64_t)gx * ((H + kTileH - 1) / kTileH);
  auto launch = [&](auto kernel, int S) {
    const int rows = kTileH * kWaves / S;
    hipLaunchKernelGGL(kernel, dim3(gx, (unsigned)((H + rows - 1) / rows)), dim3(kKdeThreads), 0, s, t, mode, f, h, H,
                       W, T, r, is0, is1, is2, out);
  };
  // One wave per tile leaves a small image with few waves, and a mid-sized
  // one with an uneven last round (24 waves fit a CU): the frames are then
  // split over 2 or 4 waves.  With at least 100 taps per part (16 frames,
  // r = 2) it pays up to 60 waves per CU - 288 x 352 62 -> 26 us, 480 x 640
  // 87 -> 56, 900 x 1440 233 -> 205, 720 x 1280 151 -> 147; 1080 x 1920, past
  // it, 295 -> 300 - and with fewer up to 16: 240 x 320 in 4 frames 18.9 ->
  // 11.6 us, but 720 x 1280 in 4 frames at r = 1 22.9 -> 26.9.
  const int64_t taps = (int64_t)T * (2 * r + 1) * (2 * r + 1);
  auto splits = [&](int S) { return T >= S && tiles * S <= (int64_t)num_cu * (taps >= 100 * S ? 60 : 16); };
  if (splits(4))
    launch(k_kde<R, 4>, 4);
  else if (splits(2))
    launch(k_kde<R, 2>, 2);
  else
    launch(k_kde<R, 1>, 1);
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
