// The SIFT-flow data term of section 3.3 on gfx950: dense SIFT "colours"
// reduced by PCA, and the Flow Field search of sections 3.1 and 3.2 with
// that data term.
//
// Colours.  Every pixel's 128-dimensional SIFT vector (Lowe 2004, upright
// and dense as in Liu et al.'s SIFT flow; 4 x 4 cells of 3 px, 8 orientation
// bins, Gaussian window of sigma 6, normalise / clamp at 0.2 / normalise) is
// computed separably: one pass bins the central-difference gradients of the
// CIELab lightness and filters them along x with the four cell-column
// windows (32 values per pixel), a second pass filters along y with the four
// cell-row windows and normalises (fp32 throughout).  The PCA basis of a
// pair and the projection on its first S eigenvectors, quantised to int16
// codes, are in ff_pca.hip.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "ff_device.h"
#include "ff_internal.h"

namespace ff {

constexpr int kSiftReach = 7;                  // |dx| < 2.5 c with c = 3
constexpr int kSiftTaps = 2 * kSiftReach + 1;
constexpr int kSiftMaxS = 32;

// cell-column (and, the same, cell-row) windows: Gaussian times the
// bilinear cell weight, per cell index and offset
struct SiftWin {
  float w[4][kSiftTaps];
};

static SiftWin sift_window() {
  SiftWin s;
  const double c = 3.0, sig = 2.0 * c;
  for (int i = 0; i < 4; ++i)
    for (int t = 0; t < kSiftTaps; ++t) {
      const int d = t - kSiftReach;
      const double b = 1.0 - std::fabs(d / c - (i - 1.5));
      s.w[i][t] = b > 0.0 ? (float)(std::exp(-(double)(d * d) / (2.0 * sig * sig)) * b) : 0.0f;
    }
  return s;
}

// ---------------------------------------------------------------- pass 1: bin and filter along x
// One workgroup = 64 x 4 pixels.  The binned gradients of the tile grown by
// 7 columns each side (zero outside the image) are staged in LDS as 8 bins
// per pixel; each thread then sums its 15 horizontal neighbours into 4 cell
// columns x 8 bins.  Output A: per pixel 32 floats, index i * 8 + o.
constexpr int kHistTW = 64, kHistTH = 4, kHistCols = kHistTW + 2 * kSiftReach;

__global__ __launch_bounds__(256) void k_sift_hist(const uint8_t* __restrict__ L, int W, int H, SiftWin win,
                                                   float* __restrict__ A) {
  __shared__ float hs[kHistTH][kHistCols][8];
  const int x0 = blockIdx.x * kHistTW, y0 = blockIdx.y * kHistTH;
  const float kTwoPi = 6.28318530717958647692f, kInvBin = 1.27323954473516268615f;   // 4 / pi
  for (int e = threadIdx.x; e < kHistTH * kHistCols; e += 256) {
    const int ty = e / kHistCols, tx = e - ty * kHistCols;
    const int x = x0 + tx - kSiftReach, y = y0 + ty;
    float m0 = 0.0f, m1 = 0.0f;
    int o0 = 0;
    if (x >= 0 && x < W && y < H) {
      const uint8_t* row = L + (size_t)y * W;
      const float gx = 0.5f * ((float)row[min(x + 1, W - 1)] - (float)row[max(x - 1, 0)]);
      const float gy = 0.5f * ((float)L[(size_t)min(y + 1, H - 1) * W + x] - (float)L[(size_t)max(y - 1, 0) * W + x]);
      const float m = sqrtf(gx * gx + gy * gy);
      if (m > 0.0f) {
        float th = atan2f(gy, gx);
        if (th < 0.0f) th += kTwoPi;
        const float t = th * kInvBin;
        const float fl = floorf(t);
        const float w1 = t - fl;
        o0 = ((int)fl) & 7;
        m0 = m * (1.0f - w1);
        m1 = m * w1;
      }
    }
    const int o1 = (o0 + 1) & 7;
#pragma unroll
    for (int o = 0; o < 8; ++o) hs[ty][tx][o] = (o == o0 ? m0 : 0.0f) + (o == o1 ? m1 : 0.0f);
  }
  __syncthreads();
  const int tx = threadIdx.x % kHistTW, ty = threadIdx.x / kHistTW;
  const int x = x0 + tx, y = y0 + ty;
  if (x >= W || y >= H) return;
  float acc[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int o = 0; o < 8; ++o) acc[i][o] = 0.0f;
#pragma unroll
  for (int t = 0; t < kSiftTaps; ++t) {
    const float4 h0 = *reinterpret_cast<const float4*>(&hs[ty][tx + t][0]);
    const float4 h1 = *reinterpret_cast<const float4*>(&hs[ty][tx + t][4]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float w = win.w[i][t];
      acc[i][0] = fmaf(w, h0.x, acc[i][0]);
      acc[i][1] = fmaf(w, h0.y, acc[i][1]);
      acc[i][2] = fmaf(w, h0.z, acc[i][2]);
      acc[i][3] = fmaf(w, h0.w, acc[i][3]);
      acc[i][4] = fmaf(w, h1.x, acc[i][4]);
      acc[i][5] = fmaf(w, h1.y, acc[i][5]);
      acc[i][6] = fmaf(w, h1.z, acc[i][6]);
      acc[i][7] = fmaf(w, h1.w, acc[i][7]);
    }
  }
  float4* out = reinterpret_cast<float4*>(A + ((size_t)y * W + x) * 32);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[2 * i] = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
    out[2 * i + 1] = make_float4(acc[i][4], acc[i][5], acc[i][6], acc[i][7]);
  }
}

// ---------------------------------------------------------------- pass 2: filter along y, normalise
// 8 lanes per pixel, 32 pixels per workgroup: lane q owns elements 4q..4q+3
// of the 32 per cell row, for the 4 cell rows j (descriptor element
// j * 32 + i * 8 + o = (4 j + i) 8 + o).  Rows outside the image add nothing.
__global__ __launch_bounds__(256) void k_sift_desc(const float* __restrict__ A, int W, int H, SiftWin win,
                                                   float* __restrict__ D) {
  const int q = threadIdx.x & 7;
  const int pix = blockIdx.x * 32 + (threadIdx.x >> 3);
  const bool ok = pix < W * H;
  const int p = ok ? pix : 0;
  const int x = p % W, y = p / W;
  float acc[4][4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[j][e] = 0.0f;
#pragma unroll
  for (int t = 0; t < kSiftTaps; ++t) {
    const int yy = y + t - kSiftReach;
    if (yy < 0 || yy >= H) continue;
    const float4 a = *reinterpret_cast<const float4*>(A + ((size_t)yy * W + x) * 32 + 4 * q);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float w = win.w[j][t];
      acc[j][0] = fmaf(w, a.x, acc[j][0]);
      acc[j][1] = fmaf(w, a.y, acc[j][1]);
      acc[j][2] = fmaf(w, a.z, acc[j][2]);
      acc[j][3] = fmaf(w, a.w, acc[j][3]);
    }
  }
  float nn = 0.0f;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) nn = fmaf(acc[j][e], acc[j][e], nn);
  nn += __shfl_xor(nn, 1);
  nn += __shfl_xor(nn, 2);
  nn += __shfl_xor(nn, 4);
  if (nn > 0.0f) {
    const float s = 1.0f / sqrtf(nn);
    float n2 = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[j][e] = fminf(acc[j][e] * s, 0.2f);
        n2 = fmaf(acc[j][e], acc[j][e], n2);
      }
    n2 += __shfl_xor(n2, 1);
    n2 += __shfl_xor(n2, 2);
    n2 += __shfl_xor(n2, 4);
    const float s2 = 1.0f / sqrtf(n2);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[j][e] *= s2;
  }
  if (!ok) return;
  float4* out = reinterpret_cast<float4*>(D + (size_t)pix * kSiftDim);
#pragma unroll
  for (int j = 0; j < 4; ++j) out[j * 8 + q] = make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
}

// ---------------------------------------------------------------- colour-stage layout
struct SiftColorLayout {
  size_t off_A, off_D1, off_D2, off_pca, off_out;
  size_t bytes;
};

static SiftColorLayout sift_color_layout(int w1, int h1, int w2, int h2) {
  SiftColorLayout L{};
  const size_t N1 = (size_t)w1 * h1, N2 = (size_t)w2 * h2, Nm = std::max(N1, N2);
  size_t off = 0;
  L.off_A = off;
  off = align_up(off + Nm * 32 * 4, 256);
  L.off_D1 = off;
  off = align_up(off + N1 * kSiftDim * 4, 256);
  L.off_D2 = off;
  off = align_up(off + N2 * kSiftDim * 4, 256);
  L.off_pca = off;
  off = align_up(off + pca_scratch_bytes(), 256);
  L.off_out = off;
  off = align_up(off + (size_t)(2 * kSiftDim + kSiftDim * kSiftDim) * 8, 256);
  L.bytes = off;
  return L;
}

static void enqueue_dense_sift(const uint8_t* L, int W, int H, const SiftWin& win, float* A, float* D,
                               hipStream_t stream) {
  k_sift_hist<<<dim3((W + kHistTW - 1) / kHistTW, (H + kHistTH - 1) / kHistTH), 256, 0, stream>>>(L, W, H, win, A);
  k_sift_desc<<<(unsigned)(((size_t)W * H + 31) / 32), 256, 0, stream>>>(A, W, H, win, D);
}

static bool sift_dims_ok(int w, int h) { return w >= 1 && h >= 1 && w <= kMaxDim && h <= kMaxDim && (int64_t)w * h <= kMaxPoints; }

}  // namespace ff

using namespace ff;

extern "C" {

int32_t ff_sift_pitch(int32_t S) { return S < 1 || S > kSiftMaxS ? 0 : (S + 3) / 4 * 4; }

size_t ff_sift_workspace_bytes(int32_t w1, int32_t h1, int32_t w2, int32_t h2) {
  if (!sift_dims_ok(w1, h1) || !sift_dims_ok(w2, h2)) return 0;
  const size_t colors = sift_color_layout(w1, h1, w2, h2).bytes;
  const size_t levels = std::max(sift_levels_scratch_bytes(w1, h1, kSiftMaxS), sift_levels_scratch_bytes(w2, h2, kSiftMaxS));
  return std::max(colors, align_up(levels, 256));
}

ff_status ff_dense_sift(const uint8_t* L, int32_t width, int32_t height, float* desc, void* workspace,
                        size_t workspace_bytes, hipStream_t stream) {
  if (!L || !desc || !workspace) return FF_ERR_ARG;
  if (width < 1 || height < 1) return FF_ERR_ARG;
  if (!sift_dims_ok(width, height)) return FF_ERR_SIZE;
  if (workspace_bytes < (size_t)width * height * 32 * 4) return FF_ERR_WORKSPACE;
  ff_status st = ensure_init();
  if (st != FF_OK) return st;
  static const SiftWin win = sift_window();
  prof_mark(FF_PROF_SIFT_COLORS, stream, true);
  enqueue_dense_sift(L, width, height, win, static_cast<float*>(workspace), desc, stream);
  prof_mark(FF_PROF_SIFT_COLORS, stream, false);
  return launch_status();
}

ff_status ff_sift_colors(const uint8_t* L1, int32_t w1, int32_t h1, const uint8_t* L2, int32_t w2, int32_t h2,
                         int32_t S, int16_t* codes1, int16_t* codes2, double* pca, float* desc1, float* desc2,
                         void* workspace, size_t workspace_bytes, hipStream_t stream) {
  if (!L1 || !L2 || !codes1 || !codes2 || !workspace) return FF_ERR_ARG;
  if (w1 < 1 || h1 < 1 || w2 < 1 || h2 < 1 || S < 1 || S > kSiftMaxS) return FF_ERR_ARG;
  if (!sift_dims_ok(w1, h1) || !sift_dims_ok(w2, h2)) return FF_ERR_SIZE;
  const SiftColorLayout Lo = sift_color_layout(w1, h1, w2, h2);
  if (workspace_bytes < Lo.bytes) return FF_ERR_WORKSPACE;
  ff_status st = ensure_init();
  if (st != FF_OK) return st;
  static const SiftWin win = sift_window();
  char* ws = static_cast<char*>(workspace);
  float* A = reinterpret_cast<float*>(ws + Lo.off_A);
  float* D1 = desc1 ? desc1 : reinterpret_cast<float*>(ws + Lo.off_D1);
  float* D2 = desc2 ? desc2 : reinterpret_cast<float*>(ws + Lo.off_D2);
  double* P = pca ? pca : reinterpret_cast<double*>(ws + Lo.off_out);
  const int N1 = w1 * h1, N2 = w2 * h2;
  prof_mark(FF_PROF_SIFT_COLORS, stream, true);
  enqueue_dense_sift(L1, w1, h1, win, A, D1, stream);
  enqueue_dense_sift(L2, w2, h2, win, A, D2, stream);
  prof_mark(FF_PROF_SIFT_PCA, stream, true);
  enqueue_pca(D1, N1, D2, N2, reinterpret_cast<double*>(ws + Lo.off_pca), P, stream);
  prof_mark(FF_PROF_SIFT_PCA, stream, false);
  enqueue_project(D1, N1, P, S, codes1, stream);
  enqueue_project(D2, N2, P, S, codes2, stream);
  prof_mark(FF_PROF_SIFT_COLORS, stream, false);
  return launch_status();
}

ff_status ff_sift_levels(const int16_t* codes, int32_t width, int32_t height, int32_t S, int32_t k, int16_t* levels,
                         void* workspace, size_t workspace_bytes, hipStream_t stream) {
  if (!codes || !levels || !workspace) return FF_ERR_ARG;
  if (width < 1 || height < 1 || S < 1 || S > kSiftMaxS || k < 0 || k > 4) return FF_ERR_ARG;
  if (!sift_dims_ok(width, height)) return FF_ERR_SIZE;
  if (workspace_bytes < sift_levels_scratch_bytes(width, height, S)) return FF_ERR_WORKSPACE;
  ff_status st = ensure_init();
  if (st != FF_OK) return st;
  prof_mark(FF_PROF_SIFT_LEVELS, stream, true);
  enqueue_sift_levels(codes, width, height, S, ff_sift_pitch(S), k, levels, static_cast<int32_t*>(workspace), stream);
  prof_mark(FF_PROF_SIFT_LEVELS, stream, false);
  return launch_status();
}

}  // extern "C"
