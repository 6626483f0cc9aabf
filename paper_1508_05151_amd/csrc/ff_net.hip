// Learned coarse-flow proposal: a 6-layer 3x3 convolutional network that maps
// the stacked RGB pair to a 2-channel flow on the 1/8 grid (the seed grid of
// a 3-level hierarchy); its rounded output enters the seed step as one extra
// candidate, so the exact data term still decides every match.
//
// Layers (Cin, Cout, stride, dilation, ReLU): (6,32,2,1,y) (32,32,2,1,y)
// (32,32,2,1,y) (32,32,1,4,y) (32,32,1,8,y) (32,2,1,1,n); padding =
// dilation; flow in px = 32 * output.  Weights and activations are bf16,
// every product sum accumulates in fp32 on the matrix cores
// (gfx950's v_mfma_f32_16x16x32_bf16: 16 x 16 outputs, 32 products each);
// master weights and Adam state are fp32.
//
// All three convolutions are implicit GEMMs on 16x16x32 MFMA tiles:
//   forward        M = Cout, N = output pixels, K = 9 taps x Cin
//   backward-data  M = Cin,  N = input pixels,  K = 9 taps x Cout (stride 2:
//                  per parity of the pixel, the taps that reach it)
//   backward-weight per tap: M = Cout, N = Cin, K = pixels, split over fixed
//                  runs of rows and reduced in a fixed order (deterministic)
// Tensors are NHWC; Cin is padded to 8 (input) or 32 channels so that one
// lane's 8 consecutive K values are 8 contiguous channels of one tap (one
// 16-byte load).  Lane l of a 16x16x32 MFMA holds A[m = l % 16][k = 8 (l / 16)
// .. + 7], B[k = 8 (l / 16) .. + 7][n = l % 16] and D[m = 4 (l / 16) + i][n =
// l % 16], i = 0..3.  A wavefront of the forward and backward-data kernels
// keeps the layer's packed weight fragments in registers and runs 16-pixel
// tiles against them; channels are dealt to the fragments' rows so that a lane
// ends with eight neighbouring ones (one 16-byte store).
//
// A layer's launch is short (0.1 to 1.8 M pixels for 16 pairs of 1024x436), so
// what a step does besides its contractions counts as much: weights and input
// are packed in one launch, and one launch reduces every layer's weight
// gradient and applies Adam.  16 x 1024x436: training step 1.78 -> 0.40 ms, forward
// of two pairs 163 -> 37 us.
#include <math.h>

#include "ff_internal.h"

namespace ff {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kNetLayers = 6;
constexpr int kKStep = 32;      // K per MFMA

struct NetLayer {
  int cin, cout, stride, dil, relu;
  int cinp, coutp;   // padded channel counts of the input / output tensors
};
static const NetLayer kNet[kNetLayers] = {{6, 32, 2, 1, 1, 8, 32},  {32, 32, 2, 1, 1, 32, 32},
                                          {32, 32, 2, 1, 1, 32, 32}, {32, 32, 1, 4, 1, 32, 32},
                                          {32, 32, 1, 8, 1, 32, 32}, {32, 2, 1, 1, 0, 32, 8}};

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// LDS accesses of a wavefront before and after this point stay in order
__device__ __forceinline__ void wave_lds_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}

static int param_offset(int layer) {
  int o = 0;
  for (int l = 0; l < layer; ++l) o += kNet[l].cout * kNet[l].cin * 9 + kNet[l].cout;
  return o;
}
static int param_total() { return param_offset(kNetLayers); }
static int chunks_of(int cinp) { return (9 * cinp + kKStep - 1) / kKStep; }
static int tiles_of(int c) { return (c + 15) / 16; }

// ---------------------------------------------------------------- packing
// What a step reads in another form than its caller has it, in one launch: the
// images, the layers' weight fragments and, for training, the number of
// labelled points (per block, summed by the loss kernel).
//
// Weight fragments, 16 bytes per (chunk, tile, lane): W[chunk c][tile t][g][row
// r][i] for K index k = 32 c + 8 g + i = tap * cpad + channel (zero where out
// of range); row r of tile t is channel 8 (r / 4) + 4 t + r % 4 of two tiles,
// channel r of one.
struct PackLayer {
  int off, cin, cout;   // parameters
  int cpad, tiles;      // padded K channels, row tiles
  int bwd;              // rows are input channels, K runs over output channels
  int end;              // elements up to and including this layer's
  uint16_t* out;
};
struct PackArgs {
  PackLayer l[2 * kNetLayers];
  int n, blocks_in, blocks_w;   // layers; blocks of each role, the rest count labels
  const uint8_t *i1, *i2;
  size_t npx;
  uint16_t* x;
  const float* theta;
  const int32_t* labels;
  size_t nlabels;
  int32_t* counts;
};
constexpr int kCountBlocks = 64;

__global__ __launch_bounds__(256) void k_pack(PackArgs a) {
  __shared__ uint32_t s_tab[256];
  __shared__ uint4 s_px[4][64 * 5];   // four pixels per lane, a fifth place between
  const int blk = blockIdx.x;
  if (blk < a.blocks_in) {
    // u8 RGB pair (B x H x W x 3 each) -> bf16 NHWC with 8 channels:
    // RGB1/255 - 1/2, RGB2/255 - 1/2, 0, 0
    s_tab[threadIdx.x] = f2bf((float)threadIdx.x / 255.0f - 0.5f);
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    auto of = [&](const uint32_t (&c)[6]) {
      uint4 o;
      o.x = s_tab[c[0]] | (s_tab[c[1]] << 16);
      o.y = s_tab[c[2]] | (s_tab[c[3]] << 16);
      o.z = s_tab[c[4]] | (s_tab[c[5]] << 16);
      o.w = 0;
      return o;
    };
    // four pixels, three words of each image, at a time where those are aligned
    const bool words = (((uintptr_t)a.i1 | (uintptr_t)a.i2) & 3) == 0;
    const size_t quads = words ? a.npx / 4 : 0;
    const size_t tid = (size_t)blk * 256 + threadIdx.x, step = (size_t)a.blocks_in * 256;
    for (size_t q0 = tid - lane; q0 < quads; q0 += step) {
      const size_t q = min(q0 + lane, quads - 1);
      uint32_t w1[3], w2[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        w1[k] = reinterpret_cast<const uint32_t*>(a.i1)[q * 3 + k];
        w2[k] = reinterpret_cast<const uint32_t*>(a.i2)[q * 3 + k];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        uint32_t c[6];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const int e = 3 * k + j;
          c[j] = (w1[e >> 2] >> (8 * (e & 3))) & 0xFF;
          c[3 + j] = (w2[e >> 2] >> (8 * (e & 3))) & 0xFF;
        }
        s_px[wave][lane * 5 + k] = of(c);
      }
      // a wavefront's 256 pixels back in order, so that a store is 1 KB
      wave_lds_order();
      const size_t p0 = q0 * 4;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int e = 64 * k + lane;
        if (p0 + e < quads * 4) reinterpret_cast<uint4*>(a.x)[p0 + e] = s_px[wave][(e >> 2) * 5 + (e & 3)];
      }
      wave_lds_order();
    }
    for (size_t p = quads * 4 + tid; p < a.npx; p += step) {
      const uint32_t c[6] = {a.i1[p * 3], a.i1[p * 3 + 1], a.i1[p * 3 + 2], a.i2[p * 3], a.i2[p * 3 + 1], a.i2[p * 3 + 2]};
      reinterpret_cast<uint4*>(a.x)[p] = of(c);
    }
  } else if (blk < a.blocks_in + a.blocks_w) {
    const int at = (blk - a.blocks_in) * 256 + threadIdx.x;
    int li = 0;
    while (li < a.n && at >= a.l[li].end) ++li;
    if (li == a.n) return;
    const PackLayer& L = a.l[li];
    const int e = at - (li ? a.l[li - 1].end : 0);
    const int i = e & 7, r = (e >> 3) & 15, g = (e >> 7) & 3, rest = e >> 9;
    const int t = rest % L.tiles, c = rest / L.tiles;
    const int k = kKStep * c + 8 * g + i, tap = k / L.cpad, kc = k % L.cpad;
    const int rc = L.tiles == 2 ? 8 * (r >> 2) + 4 * t + (r & 3) : r;
    const int ci = L.bwd ? rc : kc, co = L.bwd ? kc : rc;
    float w = 0.f;
    if (tap < 9 && ci < L.cin && co < L.cout) w = a.theta[L.off + (co * L.cin + ci) * 9 + tap];
    L.out[e] = f2bf(w);
  } else {
    const int b = blk - a.blocks_in - a.blocks_w;
    int c = 0;
    for (size_t i = (size_t)b * 256 + threadIdx.x; i < a.nlabels; i += (size_t)kCountBlocks * 256) c += a.labels[i] != kEmpty;
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if ((threadIdx.x & 63) == 0) s_tab[threadIdx.x >> 6] = (uint32_t)c;
    __syncthreads();
    if (threadIdx.x == 0) a.counts[b] = (int32_t)(s_tab[0] + s_tab[1] + s_tab[2] + s_tab[3]);
  }
}

__device__ __forceinline__ bf16x8 bf16x8_of(uint4 u) { return __builtin_bit_cast(bf16x8, u); }
__device__ __forceinline__ f32x4 mfma32(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// eight floats as bf16, in order
__device__ __forceinline__ uint4 pack8(const float (&v)[8]) {
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = f2bf(v[2 * k]) | ((uint32_t)f2bf(v[2 * k + 1]) << 16);
  return make_uint4(w[0], w[1], w[2], w[3]);
}
// v * 1 where the bf16 activation is above zero, v * 0 elsewhere
__device__ __forceinline__ void mask8(float (&v)[8], uint4 act) {
  const uint32_t w[4] = {act.x, act.y, act.z, act.w};
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] *= bf2f((uint16_t)(w[k >> 1] >> (16 * (k & 1)))) > 0.f ? 1.f : 0.f;
}
// flow in px / 32 to packed 1/Q px (nearest even), clamped to int16
__device__ __forceinline__ int32_t to_proposal(float x, float y, float q) {
  const float fx = fminf(fmaxf(rintf(x * 32.f * q), -32767.f), 32767.f);
  const float fy = fminf(fmaxf(rintf(y * 32.f * q), -32767.f), 32767.f);
  return packf((int)fx, (int)fy);
}

// ---------------------------------------------------------------- forward, backward-data at stride 1
// y[p] = sum over taps of W[tap] x[p * stride + (tap - centre) * dil], one
// wavefront per run of 16-pixel tiles of output rows (p = 16 pixels of a row),
// the next tile's loads in flight while one is multiplied.  Backward-data at
// stride 1 is the same sum with -dil, and the producing layer's ReLU: stored
// gradient = sum * (activation > 0).
// Bound: at 0.4 M pixels and more the bytes, below them one round trip and the
// launch.  A 14,080-pixel layer took 25 us with its weights staged through LDS
// and four tiles of nine loads one after another; now 4 us.
struct ConvArgs {
  const uint16_t* x;
  const uint4* wb;
  const float* bias;       // forward
  const uint16_t* aprev;   // backward: the activation at y's pixels
  uint16_t* y;
  float *yf, *flow;        // last layer: output as fp32, and a caller's copy
  int32_t* prop;           // and its rounding
  float q;
  int rows, H, W, Ho, Wo, stride, dil, relu, cout;   // rows = batch * Ho
};
template <int CINP, int NT, bool BWD>
__global__ __launch_bounds__(256) void k_conv(ConvArgs a) {
  constexpr int NC = (9 * CINP + kKStep - 1) / kKStep;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = lane & 15, g = lane >> 4;
  const int nxt = (a.Wo + 15) >> 4, ntile = a.rows * nxt, step = gridDim.x * 4;
  int tile = blockIdx.x * 4 + wave;
  if (tile >= ntile) return;
  uint4 wf[NC][NT];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int t = 0; t < NT; ++t) wf[c][t] = a.wb[(c * NT + t) * 64 + lane];
  float bias[4 * NT];
#pragma unroll
  for (int k = 0; k < 4 * NT; ++k) {
    const int co = NT == 2 ? 8 * g + k : 4 * g + k;
    bias[k] = !BWD && co < a.cout ? a.bias[co] : 0.f;
  }
  struct Tile {
    uint4 v[NC], act;
    uint32_t ok;   // taps inside the image
    int row, ox;
  };
  auto load = [&](int t) {
    Tile T;
    T.row = t / nxt;
    T.ox = (t - T.row * nxt) * 16 + m;
    const int b = T.row / a.Ho, oy = T.row - b * a.Ho;
    const uint16_t* img = a.x + (size_t)b * a.H * a.W * CINP;
    T.ok = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int tap = CINP == 32 ? c : 4 * c + g;
      const int iy = oy * a.stride + (tap / 3 - 1) * a.dil, ix = T.ox * a.stride + (tap % 3 - 1) * a.dil;
      const bool ok = tap < 9 && (uint32_t)iy < (uint32_t)a.H && (uint32_t)ix < (uint32_t)a.W;
      T.ok |= ok ? 1u << c : 0u;
      const int cy = clampi(iy, 0, a.H - 1), cx = clampi(ix, 0, a.W - 1);
      const uint16_t* at = CINP == 32 ? img + (size_t)cy * a.W * CINP + (uint32_t)(cx * CINP + 8 * g)
                                      : img + (size_t)((uint32_t)cy * (uint32_t)a.W + (uint32_t)cx) * CINP;
      T.v[c] = *reinterpret_cast<const uint4*>(at);
    }
    if (BWD) T.act = *reinterpret_cast<const uint4*>(a.aprev + ((size_t)T.row * a.Wo + min(T.ox, a.Wo - 1)) * 32 + 8 * g);
    return T;
  };
  Tile T = load(tile);
  for (;;) {
    const int next = tile + step;
    Tile N;
    if (next < ntile) N = load(next);
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      uint4 v = T.v[c];
      if (!((T.ok >> c) & 1)) v = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = mfma32(bf16x8_of(wf[c][t]), bf16x8_of(v), acc[t]);
    }
    if (T.ox < a.Wo) {
      const size_t p = (size_t)T.row * a.Wo + T.ox;
      if constexpr (NT == 2) {
        // channels 8 g + 4 t + i
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          v[k] = acc[k >> 2][k & 3];
          if (!BWD) v[k] += bias[k];
          if (!BWD && a.relu) v[k] = fmaxf(v[k], 0.f);
        }
        if (BWD) mask8(v, T.act);
        *reinterpret_cast<uint4*>(a.y + p * 32 + 8 * g) = pack8(v);
      } else if (g == 0) {
        // the last layer's two channels
        float v[2] = {acc[0][0] + bias[0], acc[0][1] + bias[1]};
        if (a.relu) v[0] = fmaxf(v[0], 0.f), v[1] = fmaxf(v[1], 0.f);
        a.yf[p * 2] = v[0];
        a.yf[p * 2 + 1] = v[1];
        if (a.flow) {
          a.flow[p * 2] = v[0];
          a.flow[p * 2 + 1] = v[1];
        }
        if (a.prop) a.prop[p] = to_proposal(v[0], v[1], a.q);
      }
    }
    if (next >= ntile) break;
    T = N;
    tile = next;
  }
}

// ---------------------------------------------------------------- backward-data at stride 2
// dX of the 2x2 input pixels around G's pixel (cy, cx), dilation 1: pixel
// (2 cy + dy, 2 cx + dx) is reached by tap row 1 of G row cy where dy = 0, by
// tap rows 0 of cy + 1 and 2 of cy where dy = 1, columns likewise: nine taps
// for four pixels, where a sum over all nine for each multiplies three zeros
// in four.  Then the producing layer's ReLU.  Bound: bytes.
// 16 x 1024x436, 32 channels into 1.8 M pixels: 194 -> 52 us.
__global__ __launch_bounds__(256) void k_conv_bwd2(const uint16_t* __restrict__ G, int rows, int Ho, int Wo, int H, int W,
                                                   const uint4* __restrict__ wbt, const uint16_t* __restrict__ aprev,
                                                   uint16_t* __restrict__ gprev) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = lane & 15, g = lane >> 4;
  const int nxt = (Wo + 15) >> 4, ntile = rows * nxt, step = gridDim.x * 4;
  int tile = blockIdx.x * 4 + wave;
  if (tile >= ntile) return;
  uint4 wf[9][2];
#pragma unroll
  for (int c = 0; c < 9; ++c)
#pragma unroll
    for (int t = 0; t < 2; ++t) wf[c][t] = wbt[(c * 2 + t) * 64 + lane];
  struct Tile {
    uint4 v[4], act[4];   // G at (cy + k / 2, cx + k % 2); activations at (2 cy + k / 2, 2 cx + k % 2)
    int b, cy, cx;
  };
  auto load = [&](int t) {
    Tile T;
    const int row = t / nxt;
    T.cx = (t - row * nxt) * 16 + m;
    T.b = row / Ho;
    T.cy = row - T.b * Ho;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int y = min(T.cy + (k >> 1), Ho - 1), x = min(T.cx + (k & 1), Wo - 1);
      T.v[k] = *reinterpret_cast<const uint4*>(G + ((size_t)(T.b * Ho + y) * Wo + x) * 32 + 8 * g);
      const int py = min(2 * T.cy + (k >> 1), H - 1), px = min(2 * T.cx + (k & 1), W - 1);
      T.act[k] = *reinterpret_cast<const uint4*>(aprev + ((size_t)(T.b * H + py) * W + px) * 32 + 8 * g);
    }
    return T;
  };
  Tile T = load(tile);
  for (;;) {
    const int next = tile + step;
    Tile N;
    if (next < ntile) N = load(next);
    const uint4 zero = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (((k & 1) && T.cx + 1 >= Wo) || ((k & 2) && T.cy + 1 >= Ho)) T.v[k] = zero;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int dy = k >> 1, dx = k & 1;
      f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int ty = dy ? 0 : 1; ty < 3; ty += dy ? 2 : 3)
#pragma unroll
        for (int tx = dx ? 0 : 1; tx < 3; tx += dx ? 2 : 3) {
          const int src = (dy && ty == 0 ? 2 : 0) + (dx && tx == 0 ? 1 : 0), tap = 3 * ty + tx;
#pragma unroll
          for (int t = 0; t < 2; ++t) acc[t] = mfma32(bf16x8_of(wf[tap][t]), bf16x8_of(T.v[src]), acc[t]);
        }
      const int py = 2 * T.cy + dy, px = 2 * T.cx + dx;
      if (py < H && px < W) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = acc[e >> 2][e & 3];
        mask8(v, T.act[k]);
        *reinterpret_cast<uint4*>(gprev + ((size_t)(T.b * H + py) * W + px) * 32 + 8 * g) = pack8(v);
      }
    }
    if (next >= ntile) break;
    T = N;
    tile = next;
  }
}

// ---------------------------------------------------------------- backward-weight
// dW[tap][co][ci] = sum_p G[p][co] X[p_in(p, tap)][ci] with K = pixels, bias
// gradient sum_p G[p][co].  A workgroup takes a run of 32-pixel pieces of
// output rows.  A lane's operand is eight pixels (g, g + 4, ..) of one channel:
// it loads channels 2m, 2m + 1 of its eight pixels (a wavefront's load is four
// neighbouring pixels, 64 bytes each), and the low and the high halves make the
// fragments of the even and of the odd channels -- the transposition costs four
// byte permutes per fragment and no LDS.  Sums stay in registers over the run;
// the wavefronts' are added pairwise in a fixed order at its end.
// 32-channel X: three wavefronts per piece, one per tap row (a third of the
// sums each: three to four wavefronts per SIMD instead of two), the next
// piece's loads in flight while one is multiplied.
// Eight-channel X (the images): four taps of eight channels fill the 16
// columns; a pixel is 16 bytes, so its rows are staged in LDS, 65 pixels of
// three rows per piece and wavefront, by 16-byte loads that are in flight over
// the piece before, and read there in words.
// Bound: bytes, and loads in flight at the small layers.
// 16 x 1024x436, against staging 64 pixels of all taps through LDS with 2-byte
// writes: first layer 205 -> 60 us, second 107 -> 43, the rest 34 -> 14 each.
// Partials: [run][fragment (slot, mt, nt)][lane][4], slot = tap, or four taps.
template <int CINP, int GCH>
struct WGrad {
  static constexpr int slots = CINP == 32 ? 9 : 3, mts = GCH == 32 ? 2 : 1;
  static constexpr int frags = slots * mts * 2;
};
constexpr int kWGroups = 4;    // pieces at once in a workgroup, 32-channel X
constexpr int kWWaves0 = 8;    // and eight-channel X

// the low (the high) halves of eight words, in order
constexpr uint32_t kLowHalf = 0x05040100u, kHighHalf = 0x07060302u;
__device__ __forceinline__ bf16x8 halves(const uint32_t (&w)[8], uint32_t sel) {
  return bf16x8_of(make_uint4(__builtin_amdgcn_perm(w[1], w[0], sel), __builtin_amdgcn_perm(w[3], w[2], sel),
                              __builtin_amdgcn_perm(w[5], w[4], sel), __builtin_amdgcn_perm(w[7], w[6], sel)));
}
// G's channels 2m, 2m + 1 (eight-channel G: 0 and 1) of pixels 32 xb + g + 4 j
// of a row, zero past its end
template <int GCH>
__device__ __forceinline__ void load_g(const uint16_t* G, int row, int xb, int Wo, int m, int g, uint32_t (&gd)[8]) {
  const uint16_t* gr = G + (size_t)row * Wo * GCH + (GCH == 32 ? 2 * m : 0);
  const int ox = 32 * xb + g;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t w = *reinterpret_cast<const uint32_t*>(gr + (uint32_t)(min(ox + 4 * j, Wo - 1) * GCH));
    gd[j] = ox + 4 * j < Wo && (GCH == 32 || m < 2) ? w : 0u;
  }
}
template <int GCH, int MTS>
__device__ __forceinline__ void g_frags(const uint32_t (&gd)[8], int m, bf16x8 (&A)[MTS]) {
  if constexpr (GCH == 32) {
    A[0] = halves(gd, kLowHalf);
    A[1] = halves(gd, kHighHalf);
  } else {
    A[0] = halves(gd, m == 0 ? kLowHalf : kHighHalf);
  }
}

template <int GCH, int STRIDE>
__global__ __launch_bounds__(64 * 3 * kWGroups) void k_conv_bwd_w(const uint16_t* __restrict__ G,
                                                                 const uint16_t* __restrict__ X, int rows, int Ho, int Wo,
                                                                 int H, int W, int dil, float4* __restrict__ part,
                                                                 float* __restrict__ partb) {
  using S = WGrad<32, GCH>;
  constexpr int FR = S::frags / 3;   // of one tap row
  __shared__ f32x4 s_red[kWGroups / 2][3][FR * 64];
  __shared__ float s_b[kWGroups][32];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave / 3, ky = wave - 3 * grp;
  const int m = lane & 15, g = lane >> 4;
  const int nxb = (Wo + 31) >> 5;
  const int64_t units = (int64_t)rows * nxb;
  const int u0 = (int)(units * blockIdx.x / gridDim.x), u1 = (int)(units * (blockIdx.x + 1) / gridDim.x);
  f32x4 acc[3][S::mts][2];
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int mt = 0; mt < S::mts; ++mt)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) acc[s][mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float bs[2] = {0.f, 0.f};
  struct Piece {
    uint32_t gd[8], xd[3][8];
    uint32_t ok[3];   // pixels of each tap inside the image (bit j)
  };
  auto load = [&](int u) {
    Piece P;
    const int row = u / nxb, xb = u - row * nxb, b = row / Ho, oy = row - b * Ho;
    load_g<GCH>(G, row, xb, Wo, m, g, P.gd);
    const int iy = oy * STRIDE + (ky - 1) * dil;
    const bool in = (uint32_t)iy < (uint32_t)H;
    const uint16_t* xr = X + ((size_t)b * H + clampi(iy, 0, H - 1)) * W * 32 + 2 * m;
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
      const int ix0 = (32 * xb + g) * STRIDE + (kx - 1) * dil;
      P.ok[kx] = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int ix = ix0 + 4 * j * STRIDE;
        P.xd[kx][j] = *reinterpret_cast<const uint32_t*>(xr + (uint32_t)(clampi(ix, 0, W - 1) * 32));
        P.ok[kx] |= in && (uint32_t)ix < (uint32_t)W ? 1u << j : 0u;
      }
    }
    return P;
  };
  int u = u0 + grp;
  Piece P;
  if (u < u1) P = load(u);
  while (u < u1) {
    const int next = u + kWGroups;
    Piece N;
    if (next < u1) N = load(next);
    bf16x8 A[S::mts];
    g_frags<GCH>(P.gd, m, A);
    if (ky == 0) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        bs[0] += bf2f((uint16_t)P.gd[j]);
        bs[1] += bf2f((uint16_t)(P.gd[j] >> 16));
      }
    }
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
      if (__ballot(P.ok[kx] != 0xFFu)) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (!((P.ok[kx] >> j) & 1)) P.xd[kx][j] = 0;
      }
      const bf16x8 B[2] = {halves(P.xd[kx], kLowHalf), halves(P.xd[kx], kHighHalf)};
#pragma unroll
      for (int mt = 0; mt < S::mts; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) acc[kx][mt][nt] = mfma32(A[mt], B[nt], acc[kx][mt][nt]);
    }
    P = N;
    u = next;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    bs[k] += __shfl_xor(bs[k], 16);
    bs[k] += __shfl_xor(bs[k], 32);
    if (ky == 0 && lane < 16) s_b[grp][2 * lane + k] = GCH == 32 || lane == 0 ? bs[k] : 0.f;
  }
  for (int half = kWGroups / 2; half > 0; half >>= 1) {
    if (grp >= half && grp < 2 * half) {
#pragma unroll
      for (int f = 0; f < FR; ++f) s_red[grp - half][ky][f * 64 + lane] = acc[f / (2 * S::mts)][(f >> 1) % S::mts][f & 1];
    }
    __syncthreads();
    if (grp < half) {
#pragma unroll
      for (int f = 0; f < FR; ++f) acc[f / (2 * S::mts)][(f >> 1) % S::mts][f & 1] += s_red[grp][ky][f * 64 + lane];
    }
    __syncthreads();
  }
  if (grp == 0) {
    f32x4* const o = reinterpret_cast<f32x4*>(part) + ((size_t)blockIdx.x * 3 + ky) * FR * 64;
#pragma unroll
    for (int f = 0; f < FR; ++f) o[f * 64 + lane] = acc[f / (2 * S::mts)][(f >> 1) % S::mts][f & 1];
  }
  if (threadIdx.x < 32) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < kWGroups; ++k) t += s_b[k][threadIdx.x];
    partb[(size_t)blockIdx.x * 32 + threadIdx.x] = t;
  }
}

// the first layer: X of eight channels, 32-channel G, stride 2, dilation 1
__global__ __launch_bounds__(64 * kWWaves0) void k_conv_bwd_w0(const uint16_t* __restrict__ G,
                                                              const uint16_t* __restrict__ X, int rows, int Ho, int Wo,
                                                              int H, int W, float4* __restrict__ part,
                                                              float* __restrict__ partb) {
  using S = WGrad<8, 32>;
  constexpr int kCols = 65, kQuads = 3 * kCols, kLoads = (kQuads + 63) / 64;
  union Smem {
    uint4 x[kWWaves0][kQuads];                    // rows 2 oy - 1 .., columns 64 xb - 1 ..
    f32x4 red[kWWaves0 / 2][S::frags * 64];
  };
  __shared__ Smem s;
  __shared__ float s_b[kWWaves0][32];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = lane & 15, g = lane >> 4;
  const int nxb = (Wo + 31) >> 5;
  const int64_t units = (int64_t)rows * nxb;
  const int u0 = (int)(units * blockIdx.x / gridDim.x), u1 = (int)(units * (blockIdx.x + 1) / gridDim.x);
  f32x4 acc[S::slots][2][2];
#pragma unroll
  for (int i = 0; i < S::slots; ++i)
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) acc[i][mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float bs[2] = {0.f, 0.f};
  // this lane's words: tap 4 i + m / 4, channels 2 (m % 4), + 1
  const uint32_t* word[S::slots];
  bool tapok[S::slots];
#pragma unroll
  for (int i = 0; i < S::slots; ++i) {
    const int tap = 4 * i + (m >> 2);
    tapok[i] = tap < 9;
    word[i] = reinterpret_cast<const uint32_t*>(&s.x[wave][min(tap, 8) / 3 * kCols + min(tap, 8) % 3 + 2 * g]) + (m & 3);
  }
  struct Piece {
    uint32_t gd[8];
    uint4 x[kLoads];
  };
  auto load = [&](int u) {
    Piece P;
    const int row = u / nxb, xb = u - row * nxb, b = row / Ho, oy = row - b * Ho;
    load_g<32>(G, row, xb, Wo, m, g, P.gd);
    const uint16_t* img = X + (size_t)b * H * W * 8;
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const int e = lane + 64 * k, r = e / kCols, iy = 2 * oy - 1 + r, ix = 64 * xb - 1 + e - r * kCols;
      const uint4 v = *reinterpret_cast<const uint4*>(
          img + (size_t)((uint32_t)clampi(iy, 0, H - 1) * (uint32_t)W + (uint32_t)clampi(ix, 0, W - 1)) * 8);
      P.x[k] = (uint32_t)iy < (uint32_t)H && (uint32_t)ix < (uint32_t)W ? v : make_uint4(0, 0, 0, 0);
    }
    return P;
  };
  int u = u0 + wave;
  Piece P;
  if (u < u1) P = load(u);
  while (u < u1) {
    // this wavefront's own rows: no other one reads them
#pragma unroll
    for (int k = 0; k < kLoads; ++k)
      if (lane + 64 * k < kQuads) s.x[wave][lane + 64 * k] = P.x[k];
    wave_lds_order();
    const int next = u + kWWaves0;
    Piece N;
    if (next < u1) N = load(next);
    bf16x8 A[2];
    g_frags<32>(P.gd, m, A);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      bs[0] += bf2f((uint16_t)P.gd[j]);
      bs[1] += bf2f((uint16_t)(P.gd[j] >> 16));
    }
#pragma unroll
    for (int i = 0; i < S::slots; ++i) {
      uint32_t xd[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {   // pixel g + 4 j, its tap's column 2 (g + 4 j) + kx
        const uint32_t w = word[i][j * 8 * 4];
        xd[j] = tapok[i] ? w : 0u;
      }
      const bf16x8 B[2] = {halves(xd, kLowHalf), halves(xd, kHighHalf)};
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) acc[i][mt][nt] = mfma32(A[mt], B[nt], acc[i][mt][nt]);
    }
    wave_lds_order();
    P = N;
    u = next;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    bs[k] += __shfl_xor(bs[k], 16);
    bs[k] += __shfl_xor(bs[k], 32);
    if (lane < 16) s_b[wave][2 * lane + k] = bs[k];
  }
  for (int half = kWWaves0 / 2; half > 0; half >>= 1) {
    if (wave >= half && wave < 2 * half) {
#pragma unroll
      for (int f = 0; f < S::frags; ++f) s.red[wave - half][f * 64 + lane] = acc[f / 4][(f >> 1) & 1][f & 1];
    }
    __syncthreads();
    if (wave < half) {
#pragma unroll
      for (int f = 0; f < S::frags; ++f) acc[f / 4][(f >> 1) & 1][f & 1] += s.red[wave][f * 64 + lane];
    }
    __syncthreads();
  }
  if (wave == 0) {
    f32x4* const o = reinterpret_cast<f32x4*>(part) + (size_t)blockIdx.x * S::frags * 64;
#pragma unroll
    for (int f = 0; f < S::frags; ++f) o[f * 64 + lane] = acc[f / 4][(f >> 1) & 1][f & 1];
  }
  if (threadIdx.x < 32) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < kWWaves0; ++k) t += s_b[k][threadIdx.x];
    partb[(size_t)blockIdx.x * 32 + threadIdx.x] = t;
  }
}

// ---------------------------------------------------------------- gradient sums, Adam
// Every layer's gradient from its partials, and the update: 64 elements per
// workgroup, a sixteenth of the partials per wavefront, added in a fixed order;
// the last workgroup sums the loss.  Bound: the partials' bytes (49 MB at
// 16 x 1024x436, 12 us).  One launch per layer with one thread per element took
// 107 us each: a chain of 512 loads on 36 workgroups.
struct StepLayer {
  const float *part, *partb;
  int runs, frags;      // partials; fragments of 256 floats in each
  int off, cin, cout;   // parameters
  int cinp, mts;
  int end;              // workgroups up to and including this layer's
};
struct StepArgs {
  StepLayer l[kNetLayers];
  float *theta, *m, *v;   // m, v null: no update
  float* grad_out;        // may be null, as loss_out
  const float* lpart;
  int lparts;
  float* loss_out;
  float lr, b1, b2, eps, c1, c2;
};
constexpr int kStepTpb = 1024;

__global__ __launch_bounds__(kStepTpb) void k_grad_step(StepArgs a) {
  __shared__ float s_sum[kStepTpb / 64][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = kStepTpb / 64;
  int li = 0;
  while (li < kNetLayers && (int)blockIdx.x >= a.l[li].end) ++li;
  const float* src = a.lpart;
  int n = a.lparts, pitch = 1, at = -1;   // terms, their distance, the parameter
  float s = 0.f;
  if (li == kNetLayers) {
    for (int i = threadIdx.x; i < n; i += kStepTpb) s += src[i];
  } else {
    const StepLayer& L = a.l[li];
    const int e = ((int)blockIdx.x - (li ? a.l[li - 1].end : 0)) * 64 + lane, nf = L.frags * 256;
    n = L.runs;
    if (e < nf) {
      const int i = e & 3, fl = (e >> 2) & 63, f = e >> 8;
      const int row = 4 * (fl >> 4) + i, col = fl & 15, nt = f & 1, mt = (f >> 1) % L.mts, slot = (f >> 1) / L.mts;
      const int co = L.mts == 2 ? 2 * row + mt : row;
      const int ci = L.cinp == 32 ? 2 * col + nt : 2 * (col & 3) + nt;
      const int tap = L.cinp == 32 ? slot : 4 * slot + (col >> 2);
      if (tap < 9 && co < L.cout && ci < L.cin) at = L.off + (co * L.cin + ci) * 9 + tap;
      src = L.part + e;
      pitch = nf;
    } else {
      const int co = e - nf;
      if (co < L.cout) at = L.off + L.cout * L.cin * 9 + co;
      src = L.partb + (co & 31);
      pitch = 32;
    }
#pragma unroll 8
    for (int c = w; c < n; c += nw) s += src[(size_t)c * pitch];
  }
  s_sum[w][lane] = s;
  __syncthreads();
  if (w) return;
  float t = 0.f;
#pragma unroll
  for (int k = 0; k < kStepTpb / 64; ++k) t += s_sum[k][lane];
  if (li == kNetLayers) {
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
    if (lane == 0 && a.loss_out) *a.loss_out = t;
    return;
  }
  if (at < 0) return;
  if (a.grad_out) a.grad_out[at] = t;
  if (a.m) {
    const float mi = a.b1 * a.m[at] + (1.f - a.b1) * t;
    const float vi = a.b2 * a.v[at] + (1.f - a.b2) * t * t;
    a.m[at] = mi;
    a.v[at] = vi;
    a.theta[at] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
  }
}

// ---------------------------------------------------------------- loss
// masked L1 on the 1/8 grid: labels in 1/Q px (FF_EMPTY = none), output in
// px / 32: per-element gradient sign(out - t) / count into the bf16 gradient
// tensor (8 channels), and per-block loss partials summed in a fixed order.
__global__ __launch_bounds__(256) void k_loss_grad(const float* __restrict__ out, const int32_t* __restrict__ labels,
                                                   size_t n, float inv_q, const int32_t* __restrict__ counts,
                                                   uint16_t* __restrict__ g6, float* __restrict__ lpart) {
  __shared__ float red[256];
  int count = counts[threadIdx.x & (kCountBlocks - 1)];
  static_assert(kCountBlocks == 64, "one count per lane");
  for (int o = 32; o > 0; o >>= 1) count += __shfl_xor(count, o);
  const float inv_n = 1.f / (float)max(count, 1);
  float ls = 0.f;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    const int32_t lb = labels[i];
    float gx = 0.f, gy = 0.f;
    if (lb != kEmpty) {
      const float tx = (float)fx_of(lb) * inv_q / 32.f, ty = (float)fy_of(lb) * inv_q / 32.f;
      const float dx = out[i * 2] - tx, dy = out[i * 2 + 1] - ty;
      ls = fabsf(dx) + fabsf(dy);
      gx = (dx > 0.f ? 1.f : (dx < 0.f ? -1.f : 0.f)) * inv_n;
      gy = (dy > 0.f ? 1.f : (dy < 0.f ? -1.f : 0.f)) * inv_n;
    }
    reinterpret_cast<uint4*>(g6)[i] = make_uint4(f2bf(gx) | ((uint32_t)f2bf(gy) << 16), 0, 0, 0);
  }
  red[threadIdx.x] = ls;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) lpart[blockIdx.x] = red[0] * inv_n;
}

// ---------------------------------------------------------------- workspace plan
struct NetPlan {
  int H[kNetLayers + 1], W[kNetLayers + 1];   // tensor sizes: [0] input, [l+1] output of layer l
  size_t off_x[kNetLayers + 1];               // activations (bf16, padded channels); [6] = fp32 output
  size_t off_g[kNetLayers + 1];               // gradients w.r.t. pre-activation outputs (bf16)
  size_t off_wb[kNetLayers], off_wbt[kNetLayers];
  size_t off_part[kNetLayers], off_partb[kNetLayers], off_lpart, off_count;
  int runs[kNetLayers], frags[kNetLayers];    // weight-gradient partials, fragments of each
  size_t lparts;
  size_t bytes;
};

static NetPlan net_plan(int Bn, int W, int H) {
  NetPlan P{};
  P.H[0] = H;
  P.W[0] = W;
  for (int l = 0; l < kNetLayers; ++l) {
    P.H[l + 1] = (P.H[l] + kNet[l].stride - 1) / kNet[l].stride;
    P.W[l + 1] = (P.W[l] + kNet[l].stride - 1) / kNet[l].stride;
  }
  size_t off = 0;
  auto take = [&](size_t bytes) {
    off = align_up(off, 256);
    const size_t o = off;
    off += bytes;
    return o;
  };
  for (int l = 0; l <= kNetLayers; ++l) {
    const size_t px = (size_t)Bn * P.H[l] * P.W[l];
    const int ch = l == 0 ? 8 : kNet[l - 1].coutp;
    P.off_x[l] = take(l == kNetLayers ? px * 2 * 4 : px * ch * 2);
    P.off_g[l] = l == 0 ? 0 : take(px * (l == kNetLayers ? 8 : ch) * 2);
  }
  for (int l = 0; l < kNetLayers; ++l) {
    P.off_wb[l] = take((size_t)chunks_of(kNet[l].cinp) * tiles_of(kNet[l].cout) * 64 * 16);
    P.off_wbt[l] = take((size_t)chunks_of(kNet[l].coutp) * tiles_of(kNet[l].cin) * 64 * 16);
    // runs of a weight gradient: two workgroups per CU at the first layer, whose
    // partials are a third of the others', one at those (fixed for a given
    // size: run-to-run identical sums)
    const int64_t units = (int64_t)Bn * P.H[l + 1] * ((P.W[l + 1] + 31) / 32);
    P.runs[l] = l == 0 ? (int)std::min<int64_t>((units + kWWaves0 - 1) / kWWaves0, 512)
                       : (int)std::min<int64_t>((units + kWGroups - 1) / kWGroups, 256);
    P.frags[l] = l == 0                ? WGrad<8, 32>::frags
                 : l == kNetLayers - 1 ? WGrad<32, 8>::frags
                                       : WGrad<32, 32>::frags;
    P.off_part[l] = take((size_t)P.runs[l] * P.frags[l] * 256 * 4);
    P.off_partb[l] = take((size_t)P.runs[l] * 32 * 4);
  }
  const size_t nout = (size_t)Bn * P.H[kNetLayers] * P.W[kNetLayers];
  P.lparts = (nout + 255) / 256;
  P.off_lpart = take(P.lparts * 4);
  P.off_count = take(kCountBlocks * 4);
  P.bytes = align_up(off, 256);
  return P;
}

// grid of a convolution launch: a wavefront per tile, and at most as many as
// the chip holds (per_cu workgroups on a CU, by registers)
static unsigned conv_blocks(int rows, int Wo, int per_cu) {
  const int64_t tiles = (int64_t)rows * ((Wo + 15) / 16);
  return (unsigned)std::min<int64_t>((tiles + 3) / 4, 256 * per_cu);
}

// everything up to the network's output (fp32; flow, prop: see ConvArgs).
// labels: of a training step, or null
static void enqueue_forward(const NetPlan& P, int Bn, const float* theta, const uint8_t* i1, const uint8_t* i2, char* ws,
                            const int32_t* labels, float* flow, int32_t* prop, float q, hipStream_t s) {
  PackArgs a{};
  a.i1 = i1;
  a.i2 = i2;
  a.npx = (size_t)Bn * P.H[0] * P.W[0];
  a.x = reinterpret_cast<uint16_t*>(ws + P.off_x[0]);
  a.theta = theta;
  int end = 0;
  for (int bwd = 0; bwd < (labels ? 2 : 1); ++bwd)
    for (int l = bwd; l < kNetLayers; ++l) {   // the first layer's input needs no gradient
      const NetLayer& L = kNet[l];
      const int cpad = bwd ? L.coutp : L.cinp, tiles = tiles_of(bwd ? L.cin : L.cout);
      end += chunks_of(cpad) * tiles * 64 * 8;
      a.l[a.n++] = {param_offset(l), L.cin, L.cout, cpad, tiles, bwd, end,
                    reinterpret_cast<uint16_t*>(ws + (bwd ? P.off_wbt[l] : P.off_wb[l]))};
    }
  a.blocks_in = (int)std::min<size_t>((a.npx + 1023) / 1024, 8192);
  a.blocks_w = (end + 255) / 256;
  a.labels = labels;
  a.nlabels = (size_t)Bn * P.H[kNetLayers] * P.W[kNetLayers];
  a.counts = reinterpret_cast<int32_t*>(ws + P.off_count);
  k_pack<<<a.blocks_in + a.blocks_w + (labels ? kCountBlocks : 0), 256, 0, s>>>(a);
  for (int l = 0; l < kNetLayers; ++l) {
    const NetLayer& L = kNet[l];
    ConvArgs c{};
    c.x = reinterpret_cast<const uint16_t*>(ws + P.off_x[l]);
    c.wb = reinterpret_cast<const uint4*>(ws + P.off_wb[l]);
    c.bias = theta + param_offset(l) + L.cout * L.cin * 9;
    c.rows = Bn * P.H[l + 1];
    c.H = P.H[l];
    c.W = P.W[l];
    c.Ho = P.H[l + 1];
    c.Wo = P.W[l + 1];
    c.stride = L.stride;
    c.dil = L.dil;
    c.relu = L.relu;
    c.cout = L.cout;
    const unsigned blocks = conv_blocks(c.rows, c.Wo, l == 0 ? 5 : l + 1 == kNetLayers ? 3 : 2);
    if (l + 1 == kNetLayers) {
      c.yf = reinterpret_cast<float*>(ws + P.off_x[l + 1]);
      c.flow = flow;
      c.prop = prop;
      c.q = q;
      k_conv<32, 1, false><<<blocks, 256, 0, s>>>(c);
    } else {
      c.y = reinterpret_cast<uint16_t*>(ws + P.off_x[l + 1]);
      if (l == 0) k_conv<8, 2, false><<<blocks, 256, 0, s>>>(c);
      else k_conv<32, 2, false><<<blocks, 256, 0, s>>>(c);
    }
  }
}

static ff_status check_net(int Bn, int W, int H) {
  if (Bn < 1 || Bn > 256 || W < 8 || H < 8 || W > kMaxDim || H > kMaxDim) return FF_ERR_ARG;
  if ((int64_t)Bn * W * H > (int64_t)1 << 30) return FF_ERR_SIZE;
  return FF_OK;
}

}  // namespace ff

using namespace ff;

extern "C" {

int32_t ff_net_param_count(void) { return param_total(); }

size_t ff_net_workspace_bytes(int32_t batch, int32_t width, int32_t height) {
  if (check_net(batch, width, height) != FF_OK) return 0;
  return net_plan(batch, width, height).bytes;
}

ff_status ff_proposal_forward(const float* params, const uint8_t* img1, const uint8_t* img2, int32_t batch,
                              int32_t width, int32_t height, int32_t subpel, int32_t* proposal, float* flow_out,
                              void* workspace, size_t workspace_bytes, hipStream_t stream) {
  if (!params || !img1 || !img2 || !proposal || !workspace) return FF_ERR_ARG;
  if (subpel != 1 && subpel != 2 && subpel != 4 && subpel != 8) return FF_ERR_ARG;
  ff_status st = check_net(batch, width, height);
  if (st != FF_OK) return st;
  const NetPlan P = net_plan(batch, width, height);
  if (workspace_bytes < P.bytes) return FF_ERR_WORKSPACE;
  char* ws = static_cast<char*>(workspace);
  prof_mark(FF_PROF_PROPOSAL, stream, true);
  enqueue_forward(P, batch, params, img1, img2, ws, nullptr, flow_out, proposal, (float)subpel, stream);
  prof_mark(FF_PROF_PROPOSAL, stream, false);
  return launch_status();
}

ff_status ff_proposal_train_step(float* params, float* adam_m, float* adam_v, int32_t step, float lr,
                                 const uint8_t* img1, const uint8_t* img2, const int32_t* labels, int32_t batch,
                                 int32_t width, int32_t height, int32_t subpel, float* grad_out, float* loss_out,
                                 void* workspace, size_t workspace_bytes, hipStream_t stream) {
  if (!params || !img1 || !img2 || !labels || !workspace) return FF_ERR_ARG;
  if (subpel != 1 && subpel != 2 && subpel != 4 && subpel != 8) return FF_ERR_ARG;
  const bool update = adam_m && adam_v;
  if ((adam_m != nullptr) != (adam_v != nullptr) || (update && step < 1)) return FF_ERR_ARG;
  ff_status st = check_net(batch, width, height);
  if (st != FF_OK) return st;
  const NetPlan P = net_plan(batch, width, height);
  if (workspace_bytes < P.bytes) return FF_ERR_WORKSPACE;
  char* ws = static_cast<char*>(workspace);
  prof_mark(FF_PROF_TRAIN, stream, true);
  enqueue_forward(P, batch, params, img1, img2, ws, labels, nullptr, nullptr, 0.f, stream);
  // loss and dL/d(out)
  const size_t n6 = (size_t)batch * P.H[kNetLayers] * P.W[kNetLayers];
  float* lpart = reinterpret_cast<float*>(ws + P.off_lpart);
  k_loss_grad<<<(unsigned)P.lparts, 256, 0, stream>>>(reinterpret_cast<const float*>(ws + P.off_x[kNetLayers]), labels,
                                                     n6, 1.f / (float)subpel, reinterpret_cast<int32_t*>(ws + P.off_count),
                                                     reinterpret_cast<uint16_t*>(ws + P.off_g[kNetLayers]), lpart);
  // backward, last layer first
  StepArgs a{};
  int end = 0;
  for (int l = 0; l < kNetLayers; ++l) {
    const NetLayer& L = kNet[l];
    end += (P.frags[l] * 256 + 32 + 63) / 64;
    a.l[l] = {reinterpret_cast<const float*>(ws + P.off_part[l]), reinterpret_cast<const float*>(ws + P.off_partb[l]),
              P.runs[l], P.frags[l], param_offset(l), L.cin, L.cout, L.cinp, l + 1 == kNetLayers ? 1 : 2, end};
  }
  for (int l = kNetLayers - 1; l >= 0; --l) {
    const NetLayer& L = kNet[l];
    const uint16_t* G = reinterpret_cast<const uint16_t*>(ws + P.off_g[l + 1]);
    const uint16_t* X = reinterpret_cast<const uint16_t*>(ws + P.off_x[l]);
    const int H = P.H[l], W = P.W[l], Ho = P.H[l + 1], Wo = P.W[l + 1], rows = batch * Ho;
    float4* part = reinterpret_cast<float4*>(ws + P.off_part[l]);
    float* partb = reinterpret_cast<float*>(ws + P.off_partb[l]);
    constexpr int tpb = 64 * 3 * kWGroups;
    if (l == 0) k_conv_bwd_w0<<<P.runs[l], 64 * kWWaves0, 0, stream>>>(G, X, rows, Ho, Wo, H, W, part, partb);
    else if (l + 1 == kNetLayers)
      k_conv_bwd_w<8, 1><<<P.runs[l], tpb, 0, stream>>>(G, X, rows, Ho, Wo, H, W, L.dil, part, partb);
    else if (L.stride == 2)
      k_conv_bwd_w<32, 2><<<P.runs[l], tpb, 0, stream>>>(G, X, rows, Ho, Wo, H, W, L.dil, part, partb);
    else
      k_conv_bwd_w<32, 1><<<P.runs[l], tpb, 0, stream>>>(G, X, rows, Ho, Wo, H, W, L.dil, part, partb);
    if (l == 0) break;
    uint16_t* gprev = reinterpret_cast<uint16_t*>(ws + P.off_g[l]);
    const uint4* wbt = reinterpret_cast<const uint4*>(ws + P.off_wbt[l]);
    if (L.stride == 2) {   // dilation 1
      k_conv_bwd2<<<conv_blocks(rows, Wo, 3), 256, 0, stream>>>(G, rows, Ho, Wo, H, W, wbt, X, gprev);
      continue;
    }
    ConvArgs c{};
    c.x = G;
    c.wb = wbt;
    c.aprev = X;
    c.y = gprev;
    c.rows = rows;
    c.H = c.Ho = H;
    c.W = c.Wo = W;
    c.stride = 1;
    c.dil = -L.dil;
    if (l + 1 == kNetLayers) k_conv<8, 2, true><<<conv_blocks(rows, W, 5), 256, 0, stream>>>(c);
    else k_conv<32, 2, true><<<conv_blocks(rows, W, 2), 256, 0, stream>>>(c);
  }
  a.grad_out = grad_out;
  a.loss_out = loss_out;
  a.lpart = lpart;
  a.lparts = (int)P.lparts;
  if (update) {
    a.theta = params;
    a.m = adam_m;
    a.v = adam_v;
    a.lr = lr;
    a.b1 = 0.9f;
    a.b2 = 0.999f;
    a.eps = 1e-8f;
    a.c1 = 1.f - powf(a.b1, (float)step);
    a.c2 = 1.f - powf(a.b2, (float)step);
  }
  k_grad_step<<<end + 1, kStepTpb, 0, stream>>>(a);
  prof_mark(FF_PROF_TRAIN, stream, false);
  return launch_status();
}

}  // extern "C"
