// The Flow Field search of sections 3.1 and 3.2 with the SIFT-flow data term
// of section 3.3, for a batch of fields in one call.
//
// Data term E^n_r(p, f): over the (2r+1)^2 samples at stride n, the L2
// distance of the first S colours of the level's smoothed colour images,
// the target side bilinear in the four neighbours of floor(m / Q) + n delta
// at the subpixel phase m mod Q (m = pQ + f; the +1 neighbours clamp), the
// source side scaled by Q^2: floor(sqrt(sum_s d_s^2 * 256 / Q^4)) per sample
// (1/16 code units at every Q), summed; lookups clamp to the image; f is
// invalid ("infinite") unless m lies in the image.  All integer, so every
// decision of the search is exact.
//
// Stages: kd-tree seeds over the CIELab WHT vectors (section 3.1; the tree
// build of the census search), re-ranked by this data term on the 2^k grid
// (Eq. 4); per level the alternating propagation sweeps (Eq. 2) and random
// searches (R_n = R n), coarse flows seeding the next level.
//
// Propagation: the sweep's tiles are solved in any order and again when a
// border value changes (ff_relax.h), one workgroup per tile, one wavefront
// per four tile rows.  A candidate is costed with a sliding window: its
// predecessor's cost minus the row (column) leaving the patch plus the one
// entering it, 2 (2r+1) samples.
#include <algorithm>
#include <vector>

#include "ff_device.h"
#include "ff_internal.h"
#include "ff_relax.h"

namespace ff {

constexpr int kSLanes = 16;   // lanes per point (entry): one DPP row
constexpr int kSiftRecsPerWrite = 12;
constexpr int kSiftStatusBytes = 256;

struct SiftRec {
  const int16_t* src;    // colour levels: (levels) x Hs x Ws x P int16
  const int16_t* dst;
  const int32_t* Vsrc;   // source WHT vectors of radius r (seed queries)
  int32_t* flow;         // outputs (the level-1 grid)
  int32_t* cost;
  char* ws;              // field region: kd-tree, grids of levels 2..2^k, handoff words
  int32_t Ws, Hs, Wd, Hd;
  int32_t P, S, r, vstride;
  uint32_t k0, k1, c3, t_nodes;
  uint32_t o_dim, o_split, o_perm;
  // as in FieldRec; border words per level, two buffers that the level's
  // sweeps alternate, each right columns then bottom rows
  uint32_t o_alt, o_seen, clear_words, ones_words;
  uint32_t o_grid[5], o_st[5], o_x[5];
  int32_t t0[5];
};

struct SCtx {
  const int16_t* src;
  const int16_t* dst;
  int Ws, Hs, Wd, Hd, P, S, r, n, Q, qshift;
};

__device__ __forceinline__ SCtx sctx_of(const SiftRec& f, int lev, int qshift) {
  SCtx c;
  c.src = f.src + (size_t)lev * f.Ws * f.Hs * f.P;
  c.dst = f.dst + (size_t)lev * f.Wd * f.Hd * f.P;
  c.Ws = f.Ws;
  c.Hs = f.Hs;
  c.Wd = f.Wd;
  c.Hd = f.Hd;
  c.P = f.P;
  c.S = f.S;
  c.r = f.r;
  c.n = 1 << lev;
  c.Q = 1 << qshift;
  c.qshift = qshift;
  return c;
}

__device__ __forceinline__ int32_t* sgrid_flow(const SiftRec& f, int lev, int buf) {
  if (buf) return reinterpret_cast<int32_t*>(f.ws + f.o_alt);
  return lev == 0 ? f.flow : reinterpret_cast<int32_t*>(f.ws + f.o_grid[lev]);
}
__device__ __forceinline__ int32_t* sgrid_cost(const SiftRec& f, int lev, int buf) {
  if (!buf && lev == 0) return f.cost;
  const int n = 1 << lev;
  return sgrid_flow(f, lev, buf) + ((f.Ws + n - 1) >> lev) * ((f.Hs + n - 1) >> lev);
}

__device__ __forceinline__ bool svalid(const SCtx& c, int px, int py, int32_t f) {
  const int mx = px * c.Q + fx_of(f), my = py * c.Q + fy_of(f);
  return mx >= 0 && my >= 0 && mx <= (c.Wd - 1) * c.Q && my <= (c.Hd - 1) * c.Q;
}

// SG groups of four colours of one pixel, as packed int16 pairs
template <int SG>
struct Col {
  uint32_t w[2 * SG];
};
template <int SG>
__device__ __forceinline__ Col<SG> load_col(const int16_t* p) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(8)));
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  Col<SG> r;
#pragma unroll
  for (int g = 0; g + 2 <= SG; g += 2) {
    const u4 x = *(__attribute__((address_space(1))) const u4*)(p + 4 * g);
#pragma unroll
    for (int i = 0; i < 4; ++i) r.w[2 * g + i] = x[i];
  }
  if (SG & 1) {
    const u2 x = *(__attribute__((address_space(1))) const u2*)(p + 4 * (SG - 1));
    r.w[2 * SG - 2] = x[0];
    r.w[2 * SG - 1] = x[1];
  }
  return r;
}

typedef short short2_t __attribute__((ext_vector_type(2)));
// w * (the low or the high half of v) + acc, w in the matching half of wv
__device__ __forceinline__ int32_t mad16(uint32_t v, uint32_t wv, int32_t acc) {
  return __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, v), __builtin_bit_cast(short2_t, wv), acc, false);
}

// floor(sqrt(v)) of N values v < 2^46.  Below 2^40 (codes up to 2047, which is
// what the projection gives) the hardware root of the rounded v is off by less
// than one, so one step either way corrects it; above (a caller's own codes)
// by up to three.  The root is below 2^23, so its squares are full-rate 24-bit
// products.
__device__ __forceinline__ uint64_t sq24(uint32_t x) {
  const uint32_t y = x & 0xFFFFFFu;   // no-op here: x < 2^24
  return (uint64_t)y * y;
}
template <int N>
__device__ __forceinline__ void isqrt46(const uint64_t (&v)[N], uint32_t (&k)[N]) {
  uint32_t top = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float fv = fmaf((float)(uint32_t)(v[i] >> 32), 4294967296.0f, (float)(uint32_t)v[i]);
    k[i] = (uint32_t)__builtin_amdgcn_sqrtf(fv);
    k[i] -= sq24(k[i]) > v[i] ? 1u : 0u;
    k[i] += sq24(k[i] + 1) <= v[i] ? 1u : 0u;
    top |= (uint32_t)(v[i] >> 32);
  }
  if (top >= 256) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      while (sq24(k[i]) > v[i]) --k[i];
      while (sq24(k[i] + 1) <= v[i]) ++k[i];
    }
  }
}

// int16 offset of pixel (x, y) in a plane of width w and pitch P: below
// 2^27 (pixels < 2^22, P <= 32), so 32-bit full-rate 24-bit products
__device__ __forceinline__ uint32_t pix_off(int x, int y, int w, int P) {
  return __umul24(__umul24((uint32_t)y, (uint32_t)w) + (uint32_t)x, (uint32_t)P);
}

// the five weights of a sample, negated for the target's four: source,
// (0, 0), (1, 0), (0, 1), (1, 1); used in the low half, and shifted to the high
struct Weights {
  uint32_t w[5];
};
__device__ __forceinline__ Weights weights_of(const SCtx& c, int mx, int my) {
  const int a = mx & (c.Q - 1), b = my & (c.Q - 1);
  return {{(uint32_t)(c.Q * c.Q), (uint32_t)(uint16_t)(-(c.Q - a) * (c.Q - b)), (uint32_t)(uint16_t)(-a * (c.Q - b)),
           (uint32_t)(uint16_t)(-(c.Q - a) * b), (uint32_t)(uint16_t)(-a * b)}};
}

// one sample's five pixels: offset (dx, dy) from the source point and from
// the target centre alike
template <int SG>
struct Sample {
  Col<SG> p[5];
};
template <int SG>
__device__ __forceinline__ Sample<SG> load_sample(const SCtx& c, int px, int py, int Mx, int My, int dx, int dy) {
  const int X = clampi(Mx + dx, 0, c.Wd - 1), Y = clampi(My + dy, 0, c.Hd - 1);
  const int X1 = min(X + 1, c.Wd - 1), Y1 = min(Y + 1, c.Hd - 1);
  Sample<SG> s;
  s.p[0] = load_col<SG>(c.src + pix_off(clampi(px + dx, 0, c.Ws - 1), clampi(py + dy, 0, c.Hs - 1), c.Ws, c.P));
  s.p[1] = load_col<SG>(c.dst + pix_off(X, Y, c.Wd, c.P));
  s.p[2] = load_col<SG>(c.dst + pix_off(X1, Y, c.Wd, c.P));
  s.p[3] = load_col<SG>(c.dst + pix_off(X, Y1, c.Wd, c.P));
  s.p[4] = load_col<SG>(c.dst + pix_off(X1, Y1, c.Wd, c.P));
  return s;
}

// its squared distance, sum_s d_s^2 * 256 / Q^4: a colour pair is weighted and
// summed by one packed dot product per weight
template <int SG>
__device__ __forceinline__ uint64_t sample_sq(const SCtx& c, const Sample<SG>& s, const Weights& wl) {
  int64_t ss = 0;
#pragma unroll
  for (int g = 0; g < SG; ++g)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int32_t e = 0;
#pragma unroll
      for (int t = 0; t < 5; ++t) e = mad16(s.p[t].w[2 * g + (i >> 1)], i & 1 ? wl.w[t] << 16 : wl.w[t], e);
      // the last group's channels past S (only there: 4 SG - S < 4)
      if (g == SG - 1 && i > 0) e = 4 * g + i < c.S ? e : 0;
      ss += (int64_t)e * e;
    }
  return c.qshift <= 2 ? (uint64_t)ss << (8 - 4 * c.qshift) : (uint64_t)ss >> 4;
}

// f(the field's own group count, 1 .. SG, as a constant)
template <int SG, typename F>
__device__ __forceinline__ void with_groups(int sg, F&& f) {
  if constexpr (SG > 1) {
    if (sg < SG) return with_groups<SG - 1>(sg, static_cast<F&&>(f));
  }
  f(std::integral_constant<int, SG>{});
}

// this lane's share (samples lane, lane + L, ...) of E for candidate fl
template <int SG>
__device__ __forceinline__ int32_t sift_partial(const SCtx& c, int px, int py, int32_t fl, int lane, int L) {
  const int mx = px * c.Q + fx_of(fl), my = py * c.Q + fy_of(fl);
  const Weights wl = weights_of(c, mx, my);
  const int Sd = 2 * c.r + 1;
  int32_t sum = 0;
  for (int k = lane; k < Sd * Sd; k += L) {
    const int iy = k / Sd, ix = k - iy * Sd;
    const Sample<SG> s =
        load_sample<SG>(c, px, py, mx >> c.qshift, my >> c.qshift, (ix - c.r) * c.n, (iy - c.r) * c.n);
    const uint64_t v[1] = {sample_sq<SG>(c, s, wl)};
    uint32_t d[1];
    isqrt46(v, d);
    sum += (int32_t)d[0];
  }
  return sum;
}

// ---------------------------------------------------------------- table, clears
struct SiftChunk {
  SiftRec r[kSiftRecsPerWrite];
};
struct TreeChunk {
  FieldRec r[kSiftRecsPerWrite];
};

__global__ void k_sift_write_table(SiftChunk chunk, int n, SiftRec* __restrict__ out) {
  if ((int)threadIdx.x < n) out[threadIdx.x] = chunk.r[threadIdx.x];
}
__global__ void k_tree_write_table(TreeChunk chunk, int n, FieldRec* __restrict__ out) {
  if ((int)threadIdx.x < n) out[threadIdx.x] = chunk.r[threadIdx.x];
}

// every field's request counters to zero, its border words to all ones
// (empty); grid: chunks x fields
__global__ void k_sift_clear(const SiftRec* __restrict__ table) {
  const SiftRec& f = table[blockIdx.y];
  int32_t* x = reinterpret_cast<int32_t*>(f.ws + f.o_st[0]);
  const size_t n0 = f.clear_words, nw = n0 + f.ones_words;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nw; i += (size_t)gridDim.x * blockDim.x)
    x[i] = i < n0 ? 0 : -1;
}

// ---------------------------------------------------------------- seeds (Eq. 1 / Eq. 4)
// One wavefront per coarse grid point: descend the kd-tree with the source
// WHT vector, re-rank the leaf (ascending pixel index) by the data term;
// the first minimum wins.  grid: (points / 4, fields)
template <int SG>
__global__ __launch_bounds__(256) void k_sift_seed(const SiftRec* __restrict__ table, int lev, int qshift, int buf) {
  const SiftRec& f = table[blockIdx.y];
  const SCtx c = sctx_of(f, lev, qshift);
  const int Gw = (f.Ws + c.n - 1) >> lev, Gh = (f.Hs + c.n - 1) >> lev;
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (wave >= Gw * Gh) return;
  const int gx = wave % Gw, gy = wave / Gw;
  const int px = gx * c.n, py = gy * c.n;
  const int32_t* node_dim = reinterpret_cast<const int32_t*>(f.ws + f.o_dim);
  const int32_t* node_split = reinterpret_cast<const int32_t*>(f.ws + f.o_split);
  const int32_t* perm = reinterpret_cast<const int32_t*>(f.ws + f.o_perm);
  const int Nd = f.Wd * f.Hd;
  const int32_t* q = f.Vsrc + ((size_t)py * f.Ws + px) * f.vstride;
  int node = 0, start = 0, cnt = Nd;
  for (;;) {
    const int dim = node_dim[node];
    if (dim < 0 || 2 * node + 2 >= (int)f.t_nodes) break;
    const int h = cnt >> 1;
    if (q[dim] >= node_split[node]) {
      node = 2 * node + 2;
      start += h;
      cnt -= h;
    } else {
      node = 2 * node + 1;
      cnt = h;
    }
  }
  int32_t bestF = kEmpty, bestC = kInf;
  with_groups<SG>((c.S + 3) >> 2, [&](auto G) {
    for (int i = 0; i < cnt && start + i < Nd; ++i) {
      const int id = perm[start + i];
      const int32_t fl = packf((id % f.Wd - px) * c.Q, (id / f.Wd - py) * c.Q);
      const int32_t e = wave_sum(sift_partial<decltype(G)::value>(c, px, py, fl, lane, 64));
      if (e < bestC) {
        bestC = e;
        bestF = fl;
      }
    }
  });
  if (lane == 0) {
    sgrid_flow(f, lev, buf)[(size_t)gy * Gw + gx] = bestF;
    sgrid_cost(f, lev, buf)[(size_t)gy * Gw + gx] = bestC;
  }
}

// ---------------------------------------------------------------- level entry
// Section 3.2: the coarser grid's points keep their flow, re-costed with
// this level's patch; new points start empty.  16 lanes per coarse point,
// which also write the three new points it covers.
template <int SG>
__global__ __launch_bounds__(256) void k_sift_entry(const SiftRec* __restrict__ table, int lev, int qshift, int buf) {
  const SiftRec& f = table[blockIdx.y];
  const SCtx c = sctx_of(f, lev, qshift);
  const int Gw = (f.Ws + c.n - 1) >> lev, Gh = (f.Hs + c.n - 1) >> lev;
  const int Gwc = (f.Ws + 2 * c.n - 1) >> (lev + 1), Ghc = (f.Hs + 2 * c.n - 1) >> (lev + 1);
  const int cid = (blockIdx.x * blockDim.x + threadIdx.x) / kSLanes;
  const int lane = threadIdx.x % kSLanes;
  if (cid >= Gwc * Ghc) return;
  const int gx = 2 * (cid % Gwc), gy = 2 * (cid / Gwc);
  const int32_t fl = sgrid_flow(f, lev + 1, 0)[cid];   // a finished level ends in buffer 0
  int32_t e = kInf;
  if (fl != kEmpty)
    with_groups<SG>((c.S + 3) >> 2, [&](auto G) {
      e = row16_sum(sift_partial<decltype(G)::value>(c, gx * c.n, gy * c.n, fl, lane, kSLanes));
    });
  if (lane < 4) {
    const int x = gx + (lane & 1), y = gy + (lane >> 1);
    if (x < Gw && y < Gh) {
      sgrid_flow(f, lev, buf)[(size_t)y * Gw + x] = lane == 0 ? fl : kEmpty;
      sgrid_cost(f, lev, buf)[(size_t)y * Gw + x] = lane == 0 ? e : kInf;
    }
  }
}

// ---------------------------------------------------------------- random search
// One offset per point, per axis an integer in [-nRQ, nRQ] 1/Q px from
// Philox keyed by the seed with counter (pixel, level, step, field | pair
// << 2); replace only on a strictly lower cost.
// A workgroup covers 32 x its points, a wavefront 8 x its of them: it draws
// all its candidates at once, one per lane, and costs a row of eight at a
// time, eight lanes per point, a sample per lane and round; a candidate whose
// sum reaches the point's cost is out.  Runs of adjacent tiles go to one XCD.
// Bound: the texture path and integer work alike (200 bytes and 200
// instructions a sample).  Against 16 lanes per point, 8-byte loads and 24-bit
// multiplies: 1242x375 gray (F, B1, B2) level 0 810 -> 436 us per launch, all
// twelve launches 3.7 -> 2.2 ms.
template <int SG>
__device__ __forceinline__ void rs_rows(const SCtx& c, int32_t* F, int32_t* C, int Gw, int gx0, int gy0, int its,
                                        int32_t cands, int32_t bounds) {
  const int lane = threadIdx.x & 63, i = lane >> 3, j = lane & 7;
  const int Sd = 2 * c.r + 1, n2 = Sd * Sd;
  const uint32_t inv = 65536u / (uint32_t)Sd + 1;   // k / Sd = k inv >> 16 for k < 31 * 31
  for (int it = 0; it < its; ++it) {
    const int32_t cand = __shfl(cands, it * 8 + i), bound = __shfl(bounds, it * 8 + i);
    bool use = bound >= 0;
    const int px = (gx0 + i) * c.n, py = (gy0 + it) * c.n;
    const int mx = px * c.Q + fx_of(cand), my = py * c.Q + fy_of(cand);
    const Weights wl = weights_of(c, mx, my);
    int32_t total = 0;
    for (int k0 = 0; k0 < n2 && __ballot(use) != 0; k0 += 8) {
      if (use) {
        const int k = min(k0 + j, n2 - 1), iy = (int)(__umul24((uint32_t)k, inv) >> 16), ix = k - iy * Sd;
        const Sample<SG> s =
            load_sample<SG>(c, px, py, mx >> c.qshift, my >> c.qshift, (ix - c.r) * c.n, (iy - c.r) * c.n);
        const uint64_t v[1] = {sample_sq<SG>(c, s, wl)};
        uint32_t root[1];
        isqrt46(v, root);
        int32_t d = k0 + j < n2 ? (int32_t)root[0] : 0;
        // over the point's eight lanes
        d += __builtin_amdgcn_update_dpp(0, d, 0xB1, 0xF, 0xF, false);    // quad_perm [1,0,3,2]
        d += __builtin_amdgcn_update_dpp(0, d, 0x4E, 0xF, 0xF, false);    // quad_perm [2,3,0,1]
        d += __builtin_amdgcn_update_dpp(0, d, 0x141, 0xF, 0xF, false);   // row_half_mirror
        total += d;
        use = total < bound;
      }
    }
    if (use && j == 0) {
      const int p = (gy0 + it) * Gw + gx0 + i;
      F[p] = cand;
      C[p] = total;
    }
  }
}

template <int SG>
__global__ __launch_bounds__(256) void k_sift_rs(const SiftRec* __restrict__ table, int lev, int qshift, int step,
                                                 int R, int buf, int its) {
  const SiftRec& f = table[blockIdx.y];
  const SCtx c = sctx_of(f, lev, qshift);
  const int Gw = (f.Ws + c.n - 1) >> lev, Gh = (f.Hs + c.n - 1) >> lev;
  const int tilesX = (Gw + 31) >> 5, nt = tilesX * ((Gh + its - 1) / its);
  const int per = (nt + 7) >> 3, tile = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || tile >= nt) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int gx0 = tile % tilesX * 32 + wave * 8, gy0 = tile / tilesX * its;
  int32_t* F = sgrid_flow(f, lev, buf);
  int32_t* C = sgrid_cost(f, lev, buf);
  // this lane's point
  const int gx = gx0 + (lane & 7), gy = gy0 + (lane >> 3);
  int32_t cand = 0, bound = -1;
  if (lane < 8 * its && gx < Gw && gy < Gh) {
    const int32_t fl = F[gy * Gw + gx];
    if (fl != kEmpty) {
      const int px = gx * c.n, py = gy * c.n;
      uint32_t u0, u1;
      philox2((uint32_t)(py * f.Ws + px), (uint32_t)lev, (uint32_t)step, f.c3, f.k0, f.k1, u0, u1);
      const int rad = c.n * R * c.Q;
      const uint64_t span = (uint64_t)(2 * rad + 1);
      cand = packf(fx_of(fl) + (int)((u0 * span) >> 32) - rad, fy_of(fl) + (int)((u1 * span) >> 32) - rad);
      if (svalid(c, px, py, cand)) bound = C[gy * Gw + gx];
    }
  }
  with_groups<SG>((c.S + 3) >> 2,
                  [&](auto G) { rs_rows<decltype(G)::value>(c, F, C, Gw, gx0, gy0, its, cand, bound); });
}

// ---------------------------------------------------------------- propagation (Eq. 2)
// Sweep (sx, sy): 1: (+,+), 2: (-,-), 3: (-,+), 4: (+,-); predecessors at
// -sx (horizontal) and -sy (vertical).  Candidate order of Eq. 2: current,
// vertical, horizontal, replaced only on a strictly lower cost; a candidate
// equal to the current flow is not evaluated (it cannot win).
//
// One workgroup per tile, 16 lanes per row: four lanes for each of the lines
// of samples that a step needs -- the row leaving and the row entering the
// patch of the vertical candidate, the column leaving and the column entering
// for the horizontal one: E(p, F(q)) = C(q) - leaving + entering, exact
// because every lookup clamps per coordinate.  In the sweep direction
// (sx, sy) the entering row is at sy r and the leaving one at -sy (r + 1)
// (columns likewise with sx).  A lane takes samples q, q + 4 of its line (more
// for r > 3), their five pixels' loads all in flight together; rows hand
// results down through LDS, one barrier per step.
// Bound: at level 0 the loads and integer work of the visits (2.7 visits per
// tile), on coarser levels the chain of visits.  A colour pair is weighted
// and summed by one packed dot product per weight.  Measured on the 1242x375
// gray pair (F, B1, B2 in one launch): level-0 sweep 0.69 ms where bands of
// 4 rows, each waiting for the one above, took 5.1; all 16 sweeps 5.8 ms
// against 34.  By the tiles alone the pair took 19.3 for 46.0 ms and a 161x119
// pair 5.6 for 9.1; with the searches, PCA and workgroup counts since, 10.9 and
// 2.5.

// Signed share of a lane in its line's sum: samples q, q + 4, ... of the line
// whose sample k lies at p + (dx0 + k kx, dy0 + k ky) around the source point
// and the target centre alike.
template <int SG>
__device__ __forceinline__ int32_t slide_line(const SCtx& c, int px, int py, int mx, int my, int dx0, int dy0,
                                              int kx, int ky, int q) {
  const int Mx = mx >> c.qshift, My = my >> c.qshift;
  const Weights wl = weights_of(c, mx, my);
  const int Sd = 2 * c.r + 1;
  int32_t sum = 0;
  for (int k0 = q; k0 < Sd; k0 += 8) {
    Sample<SG> p[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int k = min(k0 + 4 * s, Sd - 1);
      p[s] = load_sample<SG>(c, px, py, Mx, My, dx0 + k * kx, dy0 + k * ky);
    }
    uint64_t v[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) v[s] = sample_sq<SG>(c, p[s], wl);
    uint32_t d[2];
    isqrt46(v, d);
    sum += (int32_t)(d[0] + (k0 + 4 < Sd ? d[1] : 0u));
  }
  return sum;
}

struct STile {
  int2 own[kTileH * (kTileW + 1)];   // own values
  int2 res[kTileH * (kTileW + 1)];   // results, on entry those of the visit before
  int2 left[kTileH], top[kTileW + 2];   // border values: flow, 2 cost + changed
  int2 step[2][kTileH];              // rows' results of a step, by its parity
};

// the 16 steps of a visit (as the census sweep's: row i at column u0 + t - i)
template <int SG>
__device__ __forceinline__ void sift_steps(const SCtx& c, STile& s, int lev, int sx, int sy, int u0, int v0, int Gw,
                                           int Gh, bool first) {
  const int i = threadIdx.x >> 4, l = threadIdx.x & 15, line = l >> 2, q = l & 3;
  const bool horiz = line >= 2, enter = (line & 1) != 0;
  const int nQshift = lev + c.qshift;
  const int gy = sy > 0 ? v0 + i : Gh - 1 - (v0 + i), py = gy * c.n;
  const int gx0 = sx > 0 ? u0 - i : Gw - 1 - (u0 - i);
  const uint32_t maxMx = (uint32_t)((c.Wd - 1) * c.Q), maxMy = (uint32_t)((c.Hd - 1) * c.Q);
  const int across = (horiz ? sx : sy) * (enter ? c.r : -c.r - 1) * c.n, back = -c.r * c.n;
  const int dx0 = horiz ? across : back, dy0 = horiz ? back : across;
  const int kx = horiz ? 0 : c.n, ky = horiz ? c.n : 0;
  int uL = v0 + i < Gh ? u0 - i : -(1 << 20);
  int2 h = s.left[i], v = i == 0 ? s.top[0] : s.left[i > 0 ? i - 1 : 0];
  constexpr int kPO = kTileW + 1;
  for (int t = 0; t < kTileW; ++t) {
    const int2 own = s.own[i * kPO + t], old = s.res[i * kPO + t];
    const int px = (gx0 + sx * t) * c.n;
    // this lane's candidate
    const int2 cand = horiz ? h : v;
    const int mx = (px << c.qshift) + fx_of(cand.x), my = (gy << nQshift) + fy_of(cand.x);
    // a point none of whose inputs changed keeps its result; EMPTY lies outside
    const bool in = ((uint32_t)uL < (uint32_t)Gw) & (((v.y | h.y) & 1) != 0);
    // A cost depends on the point and the flow alone, so a candidate is read
    // only if nothing tells its cost yet: not the horizontal one with the
    // vertical one's flow; not the flow the last visit ended with; and not,
    // where that was the point's own, an unchanged candidate, which lost then.
    // 1242x375: 15.6 -> 15.1 ms a pair.  The census sweep has no such test:
    // its steps are short of latency, not of bandwidth, and the longer chain
    // cost a 128x96 pair 3 % for 0.6 % of eight pairs.
    const bool use = in & (cand.x != own.x) & ((uint32_t)mx <= maxMx) & ((uint32_t)my <= maxMy) &
                     !((old.x == own.x) & !(cand.y & 1)) & !(horiz & (h.x == v.x));
    const bool ev = use & (cand.x != old.x);
    int32_t e = use ? old.y : kInf;
    if (__ballot(ev)) {
      int32_t d = 0;
      if (ev) d = slide_line<SG>(c, px, py, mx, my, dx0, dy0, kx, ky, q);
      d = enter ? d : -d;
      // over the candidate's eight lanes
      d += __builtin_amdgcn_update_dpp(0, d, 0xB1, 0xF, 0xF, false);    // quad_perm [1,0,3,2]
      d += __builtin_amdgcn_update_dpp(0, d, 0x4E, 0xF, 0xF, false);    // quad_perm [2,3,0,1]
      d += __builtin_amdgcn_update_dpp(0, d, 0x141, 0xF, 0xF, false);   // row_half_mirror
      if (ev) e = (int32_t)((uint32_t)cand.y >> 1) + d;
    }
    const int32_t oe = __builtin_amdgcn_update_dpp(0, e, 0x128, 0xF, 0xF, false);        // row_ror:8
    const int32_t ofl = __builtin_amdgcn_update_dpp(0, cand.x, 0x128, 0xF, 0xF, false);
    const int32_t eV = horiz ? oe : e, eH = horiz ? e : oe;
    const int32_t fV = horiz ? ofl : cand.x, fH = horiz ? cand.x : ofl;
    int2 res = in ? own : old;
    if (eV < res.y) res = make_int2(fV, eV);
    if (eH < res.y) res = make_int2(fH, eH);
    h = make_int2(res.x, (int)((uint32_t)res.y << 1) | (first || res.x != old.x ? 1 : 0));
    if (l == 0) {
      s.res[i * kPO + t] = res;
      s.step[t & 1][i] = h;
    }
    lds_barrier();
    v = i == 0 ? s.top[t + 1] : s.step[t & 1][i > 0 ? i - 1 : 0];
    ++uL;
  }
}
struct SiftSweepArgs {
  int nf, lev, qshift, sx, sy;
  int base;    // of the request counters (ff_relax.h)
  int par;     // border word buffer in use; the other one is emptied
  int inbuf;   // grid buffer read; the other one is written
};

// Workgroups of a sweep, at most: those that the chip holds at once (three per
// CU by registers, two with the widest pixels).  More only start when others
// leave, with tiles whose neighbours have long been solved: 1242x375, all
// sweeps of a pair with 256 / 512 / 768 / 1,024 / 2,048 of them: the pair takes
// 13.9 / 11.9 / 11.7 / 12.1 / 12.9 ms.
template <int SG>
constexpr int kSiftSweepGrid = SG <= 5 ? 768 : 512;

// SG: groups of four colours of the widest field of the call
template <int SG>
__global__ __launch_bounds__(256, SG <= 5 ? 3 : 2) void k_sift_sweep(const SiftRec* __restrict__ table, SiftSweepArgs a, RelaxQ q) {
  __shared__ STile s;
  __shared__ int s_next, s_first;
  const int tid = threadIdx.x, lev = a.lev, n = 1 << lev, sx = a.sx, sy = a.sy;
  const bool wave0 = __builtin_amdgcn_readfirstlane(tid >> 6) == 0;
  constexpr int kPO = kTileW + 1;
  RelaxWg w{};   // the first wavefront's
  if (wave0) w = relax_begin(q, blockIdx.x);
  int gt = blockIdx.x;
  bool first = true;   // no earlier visit of this tile in this launch
  do {
    // the tile's field: the last one whose first tile is not above it
    int fi = 0;
    for (int b = 0; b < a.nf; b += 64) {
      const int k = b + (tid & 63);
      const bool le = k < a.nf && table[k].t0[lev] <= gt;
      fi += __popcll(__ballot(le));
    }
    fi = __builtin_amdgcn_readfirstlane(fi - 1);
    const SiftRec& f = table[fi];
    const int Gw = (f.Ws + n - 1) >> lev, Gh = (f.Hs + n - 1) >> lev;
    const int g0 = f.t0[lev], tile = gt - g0;
    const int nu = tiles_x(Gw), nv = tiles_y(Gh);
    const int tv = tile / nu, tu = tile - tv * nu;
    const int u0 = tu * kTileW, v0 = tv * kTileH;
    int32_t* const cnt = reinterpret_cast<int32_t*>(f.ws + f.o_st[lev]);
    const int have = ld_coh(cnt + tile) - a.base;   // requests this visit answers
    const int32_t* const inF = sgrid_flow(f, lev, a.inbuf);
    const int32_t* const inC = sgrid_cost(f, lev, a.inbuf);
    int32_t* const outF = sgrid_flow(f, lev, a.inbuf ^ 1);
    int32_t* const outC = sgrid_cost(f, lev, a.inbuf ^ 1);
    auto pidx = [&](int u, int v) { return (sy > 0 ? v : Gh - 1 - v) * Gw + (sx > 0 ? u : Gw - 1 - u); };
    // one point per thread: its own value, and its result if the tile was visited before
    const int pi = tid >> 4, pt = tid & 15, pu = u0 + pt - pi, pv = v0 + pi;
    const bool pok = pu >= 0 && pu < Gw && pv < Gh;
    const int pp = pidx(clampi(pu, 0, Gw - 1), min(pv, Gh - 1));
    int2 own = make_int2(gp(inF)[pp], gp(inC)[pp]), old = own;
    if (!first) old = make_int2(ld_coh(outF + pp), ld_coh(outC + pp));
    if (!pok) own = old = make_int2(kEmpty, kInf);
    s.own[pi * kPO + pt] = own;
    s.res[pi * kPO + pt] = old;
    // border words: right columns (tile column major), bottom rows; the
    // first 32 threads hold the column left of the tile and the row above it
    const size_t xwords = (size_t)nu * Gh + (size_t)nv * Gw;
    uint64_t* const xr = reinterpret_cast<uint64_t*>(f.ws + f.o_x[lev]) + (a.par ? xwords : 0);
    uint64_t* const xb = xr + (size_t)nu * Gh;
    int32_t* const was = reinterpret_cast<int32_t*>(f.ws + f.o_seen) + tile * 32;
    const bool isl = tid < 16;
    const int bl = tid & 15;
    const int hu = isl ? u0 - bl - 1 : u0 + bl, hv = isl ? v0 + bl : v0 - 1;
    const int ou = isl ? u0 + 15 - bl : u0 + bl - 15, ov = isl ? v0 + bl : v0 + 15;
    const bool ook = tid < 32 && ou >= 0 && ou < Gw && ov < Gh && (isl ? tu + 1 < nu : tv + 1 < nv);
    const ptrdiff_t oat = isl ? (ptrdiff_t)((size_t)tu * Gh + ov) : (ptrdiff_t)((size_t)nu * Gh + (size_t)tv * Gw + ou);
    const int handled = __builtin_amdgcn_readfirstlane(have);
    int32_t hf = kEmpty, hc = kInf;
    if (wave0) {
      mem_wait();   // the request counter is read before the borders
      if (tid < 32) {
        int32_t wasF = 0;
        if (!first) wasF = ld_coh(was + tid);
        if (hu >= 0 && hu < Gw && hv >= 0 && hv < Gh) {
          const uint64_t w = ld_coh(isl ? xr + (size_t)(tu - 1) * Gh + hv : xb + (size_t)(tv - 1) * Gw + hu);
          hf = gp(inF)[pidx(hu, hv)];
          hc = gp(inC)[pidx(hu, hv)];
          if (w != ~0ull) {
            hf = (int32_t)(uint32_t)w;
            hc = (int32_t)(uint32_t)(w >> 32);
          }
        }
        // cost doubled, the low bit marks a value this tile has not seen
        // (costs stay below 2^31; EMPTY's is never used)
        const int2 b = make_int2(hf, (int)((uint32_t)hc << 1) | (first || hf != wasF ? 1 : 0));
        if (isl)
          s.left[bl] = b;
        else
          s.top[bl] = b;
      }
      if (tid == 32) s.top[kTileW] = make_int2(kEmpty, 0);
    }
    __syncthreads();
    // what the readers of this tile's border hold so far
    const int oidx = isl ? bl * kPO + 15 : 15 * kPO + bl;
    int32_t seen = s.res[oidx < kTileH * kPO ? oidx : 0].x;
    asm volatile("" : "+v"(seen));
    __syncthreads();
    const SCtx c = sctx_of(f, lev, a.qshift);
    with_groups<SG>((f.S + 3) >> 2,
                    [&](auto G) { sift_steps<decltype(G)::value>(c, s, lev, sx, sy, u0, v0, Gw, Gh, first); });
    __syncthreads();
    // ---- results out, changed border words published
    if (pok) {
      const int2 x = s.res[pi * kPO + pt];
      st_coh(outF + pp, x.x);
      st_coh(outC + pp, x.y);
    }
    uint64_t cm = 0;
    if (wave0) {
      const int2 now = s.res[oidx < kTileH * kPO ? oidx : 0];
      const bool chg = ook && now.x != seen;
      if (tid < 32) {
        st_coh(was + tid, hf);
        // the buffer of the level's next sweep starts empty
        if (first && ook) st_coh(reinterpret_cast<uint64_t*>(f.ws + f.o_x[lev]) + (a.par ? 0 : xwords) + oat, (uint64_t)~0ull);
      }
      if (chg) st_coh(xr + oat, ((uint64_t)(uint32_t)now.y << 32) | (uint32_t)now.x);
      cm = __ballot(chg);
    }
    mem_wait();
    __syncthreads();
    if (wave0) {
      const int own = relax_done(q, cnt, a.base, tile, nu, g0, handled, (cm & 0xFFFFu) != 0, (cm & 0x7FFF0000u) != 0,
                                 (cm & 0x80000000u) != 0, w);
      bool fresh;
      const int next = relax_next(q, w, own, fresh);
      if (tid == 0) {
        s_next = next;
        s_first = fresh;
      }
    }
    __syncthreads();
    gt = __builtin_amdgcn_readfirstlane(s_next);
    first = s_first != 0;
    __syncthreads();
  } while (gt >= 0);
}

// write the grid of level lev into the full-resolution outputs (inspection
// stops); grid: (W / 256, H, fields)
__global__ void k_sift_write_grid(const SiftRec* __restrict__ table, int lev, int buf) {
  const SiftRec& f = table[blockIdx.z];
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= f.Ws || y >= f.Hs) return;
  const int n = 1 << lev;
  const int Gw = (f.Ws + n - 1) >> lev;
  const size_t o = (size_t)y * f.Ws + x;
  if ((x % n) == 0 && (y % n) == 0) {
    f.flow[o] = sgrid_flow(f, lev, buf)[(size_t)(y / n) * Gw + x / n];
    f.cost[o] = sgrid_cost(f, lev, buf)[(size_t)(y / n) * Gw + x / n];
  } else {
    f.flow[o] = kEmpty;
    f.cost[o] = kInf;
  }
}

// ---------------------------------------------------------------- host
struct SiftFieldPlan {
  TreeLayout tree;
  size_t off_grid[5], off_st[5], off_x[5];
  size_t off_alt, off_seen;
  size_t clear_words, ones_words;   // from off_st[0]: request counters, then border words
  size_t bytes;
};

static SiftFieldPlan sift_field_plan(const ff_sift_job& j, const ff_match_params* p) {
  SiftFieldPlan P{};
  const int Ws = j.src->width, Hs = j.src->height;
  P.tree = tree_layout(j.dst->width * j.dst->height, p->leaf, 0);
  size_t off = P.tree.bytes;
  auto grid_of = [](int size, int lev) { return (size + (1 << lev) - 1) >> lev; };
  for (int lev = 1; lev <= p->k; ++lev) {
    off = align_up(off, 256);
    P.off_grid[lev] = off;
    off += (size_t)grid_of(Ws, lev) * grid_of(Hs, lev) * 8;
  }
  off = align_up(off, 256);
  const size_t clear0 = off;
  for (int lev = 0; lev <= p->k; ++lev) {
    P.off_st[lev] = off;
    off += (size_t)tiles_x(grid_of(Ws, lev)) * tiles_y(grid_of(Hs, lev)) * 4;
  }
  off = align_up(off, 8);
  P.clear_words = (off - clear0) / 4;
  for (int lev = 0; lev <= p->k; ++lev) {
    const int Gw = grid_of(Ws, lev), Gh = grid_of(Hs, lev);
    P.off_x[lev] = off;
    off += 2 * ((size_t)tiles_x(Gw) * Gh + (size_t)tiles_y(Gh) * Gw) * 8;
  }
  P.ones_words = (off - clear0) / 4 - P.clear_words;
  P.off_seen = off;
  off += (size_t)tiles_x(Ws) * tiles_y(Hs) * 32 * 4;
  // the second grid buffer: what the tree build needs beside the finished
  // tree is free once the tree stands, if the source fits there
  const size_t alt = (size_t)Ws * Hs * 8;
  if (P.tree.bytes - P.tree.off_perm2 >= alt) {
    P.off_alt = P.tree.off_perm2;
  } else {
    P.off_alt = off = align_up(off, 256);
    off += alt;
  }
  P.bytes = align_up(off, 256);
  return P;
}

struct SiftBatchLayout {
  size_t off_ctl, off_ring, off_table, off_ttable;   // scheduler words of every launch, the queue they share
  size_t ctl_words;                                  // from off_ctl, cleared per call
  int launches, cap;
  std::vector<size_t> off_field;
  size_t bytes;
};

static SiftBatchLayout sift_batch_layout(const ff_sift_job* jobs, int n, const ff_match_params* p) {
  SiftBatchLayout B{};
  size_t off = kSiftStatusBytes;
  B.off_ctl = off;
  B.launches = (p->k + 1) * p->n_prop;
  off += (size_t)B.launches * sizeof(RelaxCtl);
  B.off_ring = off;
  for (int i = 0; i < n; ++i) B.cap += tiles_x(jobs[i].src->width) * tiles_y(jobs[i].src->height);
  off += (size_t)B.cap * 4;
  B.ctl_words = (off - B.off_ctl) / 4;
  off = align_up(off, 256);
  B.off_table = off;
  off = align_up(off + (size_t)n * sizeof(SiftRec), 256);
  B.off_ttable = off;
  off = align_up(off + (size_t)n * sizeof(FieldRec), 256);
  B.off_field.resize(n);
  for (int i = 0; i < n; ++i) {
    B.off_field[i] = off;
    off = align_up(off + sift_field_plan(jobs[i], p).bytes, 256);
  }
  B.bytes = off;
  return B;
}

static ff_status check_sift_job(const ff_sift_job& j, const ff_match_params* p) {
  if (!j.src || !j.dst || !j.src_blob || !j.dst_blob || !j.src_levels || !j.dst_levels || !j.flow || !j.cost)
    return FF_ERR_ARG;
  const ff_desc* s = j.src;
  const ff_desc* d = j.dst;
  if (s->subpel != d->subpel) return FF_ERR_ARG;
  if (j.radius < 1 || j.radius > kMaxRadius) return FF_ERR_ARG;
  if (j.pitch < 4 || j.pitch > 32 || (j.pitch & 3) || j.channels < 1 || j.channels > j.pitch) return FF_ERR_ARG;
  if (p->k < 0 || p->k > j.levels || j.levels > 4) return FF_ERR_ARG;
  if (j.field_id > 3) return FF_ERR_ARG;
  if (!wht_block(s, j.src_blob, j.radius) || !wht_block(d, j.dst_blob, j.radius)) return FF_ERR_ARG;
  return FF_OK;
}

static ff_status check_sift_params(const ff_match_params* p) {
  if (!p) return FF_ERR_ARG;
  if (p->k < 0 || p->k > 4) return FF_ERR_ARG;
  if (p->R < 0 || p->R > 64 || p->n_prop < 0 || p->n_prop > 64 || p->n_rs < 0 || p->n_rs > p->n_prop) return FF_ERR_ARG;
  if (p->use_kdtree != 1) return FF_ERR_UNSUPPORTED;   // seeds come from the kd-tree only
  if (p->leaf < 2 || p->leaf > kMaxLeaf) return FF_ERR_ARG;
  if (p->watchdog_us < 0) return FF_ERR_ARG;
  return FF_OK;
}

static SiftRec make_sift_rec(const ff_sift_job& j, const SiftFieldPlan& P, char* fws) {
  SiftRec r{};
  r.src = j.src_levels;
  r.dst = j.dst_levels;
  r.Vsrc = wht_block(j.src, j.src_blob, j.radius);
  r.flow = j.flow;
  r.cost = j.cost;
  r.ws = fws;
  r.Ws = j.src->width;
  r.Hs = j.src->height;
  r.Wd = j.dst->width;
  r.Hd = j.dst->height;
  r.P = j.pitch;
  r.S = j.channels;
  r.r = j.radius;
  r.vstride = j.src->wht_stride;
  r.k0 = (uint32_t)(j.seed & 0xFFFFFFFFu);
  r.k1 = (uint32_t)(j.seed >> 32);
  r.c3 = j.field_id | (j.pair_id << 2);
  r.t_nodes = (uint32_t)P.tree.nodes;
  r.o_dim = (uint32_t)P.tree.off_dim;
  r.o_split = (uint32_t)P.tree.off_split;
  r.o_perm = (uint32_t)P.tree.off_perm;
  r.o_alt = (uint32_t)P.off_alt;
  r.o_seen = (uint32_t)P.off_seen;
  r.clear_words = (uint32_t)P.clear_words;
  r.ones_words = (uint32_t)P.ones_words;
  for (int l = 0; l < 5; ++l) {
    r.o_grid[l] = (uint32_t)P.off_grid[l];
    r.o_st[l] = (uint32_t)P.off_st[l];
    r.o_x[l] = (uint32_t)P.off_x[l];
  }
  return r;
}

// the record the kd-tree build reads: the target's WHT vectors and the tree
// offsets in the field region
static FieldRec make_tree_rec(const ff_sift_job& j, const SiftFieldPlan& P, char* fws) {
  FieldRec r{};
  r.Vdst = wht_block(j.dst, j.dst_blob, j.radius);
  r.Ws = j.src->width;
  r.Hs = j.src->height;
  r.Wd = j.dst->width;
  r.Hd = j.dst->height;
  r.r = j.radius;
  r.D = j.dst->wht_dims;
  r.vstride = j.dst->wht_stride;
  r.ws = fws;
  r.t_nodes = P.tree.nodes;
  r.t_top = P.tree.top;
  r.o_dim = (uint32_t)P.tree.off_dim;
  r.o_split = (uint32_t)P.tree.off_split;
  r.o_perm = (uint32_t)P.tree.off_perm;
  r.o_perm2 = (uint32_t)P.tree.off_perm2;
  r.o_mm = (uint32_t)P.tree.off_minmax;
  r.o_hist = (uint32_t)P.tree.off_hist;
  r.o_cnt = (uint32_t)P.tree.off_cnt;
  r.o_key = (uint32_t)P.tree.off_key;
  return r;
}

template <int SG>
static ff_status run_sift_batch(const ff_sift_job* jobs, int n, const ff_match_params* p, char* ws,
                                const SiftBatchLayout& B, hipStream_t stream) {
  int32_t* status = reinterpret_cast<int32_t*>(ws);
  RelaxCtl* ctl = reinterpret_cast<RelaxCtl*>(ws + B.off_ctl);
  SiftRec* table = reinterpret_cast<SiftRec*>(ws + B.off_table);
  FieldRec* ttable = reinterpret_cast<FieldRec*>(ws + B.off_ttable);
  std::vector<SiftRec> recs(n);
  std::vector<FieldRec> trecs(n);
  int maxW = 0, maxH = 0, maxN = 0, maxTop = 0;
  auto tiles_of = [](const SiftRec& f, int lev) {
    const int m = (1 << lev) - 1;
    return tiles_x((f.Ws + m) >> lev) * tiles_y((f.Hs + m) >> lev);
  };
  for (int i = 0; i < n; ++i) {
    const SiftFieldPlan P = sift_field_plan(jobs[i], p);
    recs[i] = make_sift_rec(jobs[i], P, ws + B.off_field[i]);
    trecs[i] = make_tree_rec(jobs[i], P, ws + B.off_field[i]);
    maxW = std::max(maxW, recs[i].Ws);
    maxH = std::max(maxH, recs[i].Hs);
    maxN = std::max(maxN, recs[i].Wd * recs[i].Hd);
    maxTop = std::max(maxTop, trecs[i].t_top);
    for (int lev = 0; lev <= p->k && i > 0; ++lev) recs[i].t0[lev] = recs[i - 1].t0[lev] + tiles_of(recs[i - 1], lev);
  }
  const int qshift = ilog2i(jobs[0].src->subpel);
  const int k = p->k;
  fill_i32(status, 1, 0, stream);
  fill_i32(reinterpret_cast<int32_t*>(ctl), B.ctl_words, 0, stream);
  for (int i = 0; i < n; i += kSiftRecsPerWrite) {
    SiftChunk sc{};
    TreeChunk tc{};
    const int m = std::min(kSiftRecsPerWrite, n - i);
    for (int q = 0; q < m; ++q) {
      sc.r[q] = recs[i + q];
      tc.r[q] = trecs[i + q];
    }
    k_sift_write_table<<<1, kSiftRecsPerWrite, 0, stream>>>(sc, m, table + i);
    k_tree_write_table<<<1, kSiftRecsPerWrite, 0, stream>>>(tc, m, ttable + i);
  }
  k_sift_clear<<<dim3(64, n), 256, 0, stream>>>(table);
  prof_mark(FF_PROF_TREE, stream, true);
  ff_status st = enqueue_tree_build(ttable, n, maxN, maxTop, p->leaf, stream);
  prof_mark(FF_PROF_TREE, stream, false);
  if (st != FF_OK) return st;
  auto pts = [&](int lev) { return ((maxW + (1 << lev) - 1) >> lev) * ((maxH + (1 << lev) - 1) >> lev); };
  auto groups = [&](int npts) { return (unsigned)(((size_t)npts * kSLanes + 255) / 256); };
  // the grid buffer in use: every sweep reads one and writes the other, and a
  // level's last one ends in buffer 0
  const int buf0 = p->n_prop & 1;
  int steps = 0, cur_lev = k, buf = buf0;
  auto stop = [&]() { return p->max_steps >= 0 && steps >= p->max_steps; };
  auto finish = [&]() -> ff_status {
    if (cur_lev > 0 || buf)
      k_sift_write_grid<<<dim3((maxW + 255) / 256, maxH, n), 256, 0, stream>>>(table, cur_lev, buf);
    return launch_status();
  };
  k_sift_seed<SG><<<dim3((pts(k) + 3) / 4, n), 256, 0, stream>>>(table, k, qshift, buf);
  ++steps;
  if (stop()) return finish();
  const uint64_t timeout = p->watchdog_us > 0 ? (uint64_t)p->watchdog_us * 100u : 200000000ull;
  auto sx_of = [](int i) { return ((i & 3) == 0 || (i & 3) == 3) ? 1 : -1; };
  auto sy_of = [](int i) { return ((i & 3) == 0 || (i & 3) == 2) ? 1 : -1; };
  int launch = 0;
  for (int lev = k; lev >= 0; --lev) {
    cur_lev = lev;
    if (lev < k) {
      buf = buf0;
      k_sift_entry<SG><<<dim3(groups(pts(lev + 1)), n), 256, 0, stream>>>(table, lev, qshift, buf);
      ++steps;
      if (stop()) return finish();
    }
    for (int i = 0; i < p->n_prop; ++i) {
      const SiftSweepArgs a{n, lev, qshift, sx_of(i), sy_of(i), -(i + 1), i & 1, buf};
      RelaxQ q{};
      q.ctl = ctl + launch;
      q.ring = reinterpret_cast<int32_t*>(ws + B.off_ring);
      q.cap = B.cap;
      q.T = recs[n - 1].t0[lev] + tiles_of(recs[n - 1], lev);
      q.G = std::min(q.T, kSiftSweepGrid<SG>);
      q.status = status;
      q.timeout = timeout;
      prof_mark(FF_PROF_SIFT_PROPAGATE, stream, true);
      k_sift_sweep<SG><<<q.G, 256, 0, stream>>>(table, a, q);
      prof_mark(FF_PROF_SIFT_PROPAGATE, stream, false);
      buf ^= 1;
      ++launch;
      ++steps;
      if (stop()) return finish();
      if (i < p->n_rs) {
        const int Gw = (maxW + (1 << lev) - 1) >> lev, Gh = (maxH + (1 << lev) - 1) >> lev, wide = (Gw + 31) / 32;
        // rows of points per wavefront: eight, fewer where that leaves the
        // chip short of wavefronts (16 per CU)
        int its = 8;
        while (its > 1 && (int64_t)wide * 4 * ((Gh + its - 1) / its) * n < 4096) its >>= 1;
        const unsigned tiles = (unsigned)(wide * ((Gh + its - 1) / its));
        k_sift_rs<SG><<<dim3((tiles + 7) / 8 * 8, n), 256, 0, stream>>>(table, lev, qshift, i, p->R, buf, its);
        ++steps;
        if (stop()) return finish();
      }
    }
  }
  return finish();
}

}  // namespace ff

using namespace ff;

extern "C" {

size_t ff_match_sift_workspace_bytes(const ff_sift_job* jobs, int32_t n_jobs, const ff_match_params* p) {
  if (!jobs || n_jobs < 1 || check_sift_params(p) != FF_OK) return 0;
  for (int i = 0; i < n_jobs; ++i)
    if (check_sift_job(jobs[i], p) != FF_OK) return 0;
  return sift_batch_layout(jobs, n_jobs, p).bytes;
}

ff_status ff_match_sift(const ff_sift_job* jobs, int32_t n_jobs, const ff_match_params* p, void* workspace,
                        size_t workspace_bytes, hipStream_t stream) {
  if (!jobs || n_jobs < 1 || !workspace) return FF_ERR_ARG;
  ff_status st = check_sift_params(p);
  if (st != FF_OK) return st;
  for (int i = 0; i < n_jobs; ++i) {
    st = check_sift_job(jobs[i], p);
    if (st != FF_OK) return st;
    if (jobs[i].src->subpel != jobs[0].src->subpel) return FF_ERR_ARG;
  }
  const SiftBatchLayout B = sift_batch_layout(jobs, n_jobs, p);
  if (workspace_bytes < B.bytes) return FF_ERR_WORKSPACE;
  st = ensure_init();
  if (st != FF_OK) return st;
  prof_mark(FF_PROF_SIFT_MATCH, stream, true);
  int sg = 1;
  for (int i = 0; i < n_jobs; ++i) sg = std::max(sg, (jobs[i].channels + 3) / 4);
  char* w = static_cast<char*>(workspace);
  // instances by what their registers allow: a field's own group count picks
  // the code inside
  st = sg <= 3   ? run_sift_batch<3>(jobs, n_jobs, p, w, B, stream)
       : sg <= 5 ? run_sift_batch<5>(jobs, n_jobs, p, w, B, stream)
                 : run_sift_batch<8>(jobs, n_jobs, p, w, B, stream);
  prof_mark(FF_PROF_SIFT_MATCH, stream, false);
  return st;
}

}  // extern "C"
