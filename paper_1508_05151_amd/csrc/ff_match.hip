// The Flow Field search of one field (sections 3.1, 3.2): kd-tree seeds on
// the coarsest grid, then per level the alternating propagation sweeps and
// random searches, coarse flows seeding the next level.
//
// Data term E^n_r(p, f) (Eq. 1/3/4 with the census of section 3.3): the sum
// over the (2r+1)^2 samples at stride n of popcount(D1 ^ D2), D1 from the
// source's phase-(0,0) plane of level n at p + n d, D2 from the target's
// plane of the subpixel phase of m = pQ + f at floor(m/Q) + n d; lookups
// clamp to the image; f is invalid ("infinite") unless m lies in the image.
//
// Propagation (Eq. 2): the raster-order sweep is the one solution of "every
// point holds the best of its own value and its two predecessors' new
// values", so its tiles may be solved in any order as long as they are solved
// again whenever a border value changes (ff_relax.h).  Propagated candidates
// are costed with sliding windows: E(p, F(q)) = C(q) - (row or column leaving
// the patch) + (row or column entering it), 2(2r+1) terms instead of
// (2r+1)^2, exact because every sample lookup clamps per coordinate.
#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "ff_device.h"
#include "ff_internal.h"
#include "ff_relax.h"

namespace ff {

constexpr int kLanesPt = 16;      // lanes per point in recost / random search
constexpr int kStatusBytes = 256;
constexpr int kRecsPerWrite = 12; // table records per writer launch (kernel argument size)

// ---------------------------------------------------------------- per-field cost context
struct CostCtx {
  const uint32_t* src;   // source plane, level n, phase (0,0)
  const uint32_t* dst;   // target planes of level n (phase i at dst + i * pw)
  const uint32_t* srcT;  // the same, transposed (x-major, pitch Hs / Hd)
  const uint32_t* dstT;
  uint32_t pw;           // target plane words
  int Ws, Hs, Wd, Hd;
  int qshift, qmask, Q;
  int n, r;
};

__device__ __forceinline__ CostCtx ctx_of(const FieldRec& f, int lev, int qshift) {
  CostCtx c;
  const int Q = 1 << qshift;
  c.src = f.src + (size_t)lev * Q * Q * f.pws;
  c.srcT = f.srcT + (size_t)lev * Q * Q * f.pws;
  c.dst = f.dst + (size_t)lev * Q * Q * f.pwd;
  c.dstT = f.dstT + (size_t)lev * Q * Q * f.pwd;
  c.pw = f.pwd;
  c.Ws = f.Ws;
  c.Hs = f.Hs;
  c.Wd = f.Wd;
  c.Hd = f.Hd;
  c.Q = Q;
  c.qshift = qshift;
  c.qmask = Q - 1;
  c.n = 1 << lev;
  c.r = f.r;
  return c;
}

// level grids: buffer 0 of n = 1 is the output pair itself; buffer 1 is one
// region of the workspace for every level
__device__ __forceinline__ int32_t* grid_flow(const FieldRec& f, int lev, int buf) {
  if (buf) return reinterpret_cast<int32_t*>(f.ws + f.o_alt);
  return lev == 0 ? f.flow : reinterpret_cast<int32_t*>(f.ws + f.o_grid[lev]);
}
__device__ __forceinline__ int32_t* grid_cost(const FieldRec& f, int lev, int buf) {
  if (!buf && lev == 0) return f.cost;
  const int n = 1 << lev;
  return grid_flow(f, lev, buf) + ((f.Ws + n - 1) >> lev) * ((f.Hs + n - 1) >> lev);
}

__device__ __forceinline__ bool centre_valid(const CostCtx& c, int px, int py, int fx, int fy) {
  const int mx = px * c.Q + fx, my = py * c.Q + fy;
  return mx >= 0 && my >= 0 && mx <= (c.Wd - 1) * c.Q && my <= (c.Hd - 1) * c.Q;
}

// partial patch sum over this lane's share (terms lane, lane+L, ...)
__device__ __forceinline__ int32_t patch_partial(const CostCtx& c, int px, int py, int fx, int fy, int lane, int L) {
  const int mx = px * c.Q + fx, my = py * c.Q + fy;
  const int Mx = mx >> c.qshift, My = my >> c.qshift;
  const uint32_t* D2 = c.dst + (size_t)c.pw * (size_t)(((my & c.qmask) << c.qshift) + (mx & c.qmask));
  const int S = 2 * c.r + 1;
  int dy = lane / S, dx = lane - dy * S;
  const int stepy = L / S, stepx = L - stepy * S;
  int32_t sum = 0;
#pragma unroll 4
  for (int t = lane; t < S * S; t += L) {
    const int oy = (dy - c.r) * c.n, ox = (dx - c.r) * c.n;
    const uint32_t a = c.src[(size_t)clampi(py + oy, 0, c.Hs - 1) * c.Ws + clampi(px + ox, 0, c.Ws - 1)];
    const uint32_t b = D2[(size_t)clampi(My + oy, 0, c.Hd - 1) * c.Wd + clampi(Mx + ox, 0, c.Wd - 1)];
    sum += __popc(a ^ b);
    dx += stepx;
    dy += stepy;
    if (dx >= S) { dx -= S; ++dy; }
  }
  return sum;
}

template <int L>
__device__ __forceinline__ int32_t group_sum(int32_t v) {
  static_assert(L == 16 || L == 64, "rows of 16 lanes");
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);    // lane ^ 1
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);    // lane ^ 2
  v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);   // 7 - lane, within eight
  v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);   // 15 - lane
#pragma unroll
  for (int o = 16; o < L; o <<= 1) v += __shfl_xor(v, o, L);
  return v;
}

// Census distance of two S x S patches at stride 1 by a group of 16 lanes
// (partial sums, one per lane): lane l < min(S, 16) sums patch column l over
// all S rows, so each load of a wavefront reads 64 consecutive bytes per
// point rather than one row segment per lane; column 16 (S = 17) spreads its
// rows over the lanes.  Each side is given as the address of the patch's
// column 0 in plane row 0 (sb, tb), its row pitch in words and the plane row
// of patch row 0 (sy0, ty0); rows clamp to [0, ymax], columns are not
// clamped, so the caller guarantees that both S-word row segments lie inside
// their planes.
typedef __attribute__((address_space(1))) const uint32_t g_u32;

template <int S>
__device__ __forceinline__ int32_t cols_sum_n1(g_u32* sb, int spw, int sy0, int symax, g_u32* tb, int tpw, int ty0,
                                               int tymax, int lane) {
  int32_t sum = 0;
  if (lane < S) {
#pragma unroll
    for (int row = 0; row < S; ++row)
      sum += __popc(sb[clampi(sy0 + row, 0, symax) * spw + lane] ^ tb[clampi(ty0 + row, 0, tymax) * tpw + lane]);
  }
  for (int row = lane; S > 16 && row < S; row += 16)
    sum += __popc(sb[clampi(sy0 + row, 0, symax) * spw + 16] ^ tb[clampi(ty0 + row, 0, tymax) * tpw + 16]);
  return sum;
}

// ---------------------------------------------------------------- field table
struct RecChunk {
  FieldRec r[kRecsPerWrite];
};

__global__ void k_write_table(RecChunk chunk, int n, FieldRec* __restrict__ out) {
  if ((int)threadIdx.x < n) out[threadIdx.x] = chunk.r[threadIdx.x];
}

// zero every field's border words and request counters (grid: chunks x fields)
__global__ void k_clear_borders(const FieldRec* __restrict__ table) {
  const FieldRec& f = table[blockIdx.y];
  int32_t* x = reinterpret_cast<int32_t*>(f.ws + f.o_st[0]);
  const size_t nw = f.clear_words;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nw; i += (size_t)gridDim.x * blockDim.x) x[i] = 0;
}

// ---------------------------------------------------------------- seeds (Eq. 1 / Eq. 4)
// One wavefront per coarse grid point: descend the kd-tree with the source
// patch's WHT vector, then re-rank the leaf (ascending pixel index) and the
// optional proposal by the data term; the first minimum wins.
// grid: (points / 4, fields)
__global__ __launch_bounds__(256) void k_seed(const FieldRec* __restrict__ table, int lev, int qshift, int use_tree,
                                                int buf) {
  const FieldRec& f = table[blockIdx.y];
  const CostCtx c = ctx_of(f, lev, qshift);
  const int Gw = (f.Ws + c.n - 1) >> lev, Gh = (f.Hs + c.n - 1) >> lev;
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (wave >= Gw * Gh) return;
  const int gx = wave % Gw, gy = wave / Gw;
  const int px = gx * c.n, py = gy * c.n;
  int32_t bestF = kEmpty, bestC = kInf;
  if (use_tree) {
    const int32_t* node_dim = reinterpret_cast<const int32_t*>(f.ws + f.o_dim);
    const int32_t* node_split = reinterpret_cast<const int32_t*>(f.ws + f.o_split);
    const int32_t* perm = reinterpret_cast<const int32_t*>(f.ws + f.o_perm);
    const int Nd = f.Wd * f.Hd;
    const int32_t* q = f.Vsrc + ((size_t)py * c.Ws + px) * f.vstride;
    int node = 0, start = 0, cnt = Nd;
    for (;;) {
      const int dim = node_dim[node];
      if (dim < 0 || 2 * node + 2 >= f.t_nodes) break;
      const int h = cnt >> 1;
      if (q[dim] >= node_split[node]) { node = 2 * node + 2; start += h; cnt -= h; }
      else { node = 2 * node + 1; cnt = h; }
    }
    for (int i = 0; i < cnt && start + i < Nd; ++i) {
      const int id = perm[start + i];
      const int fx = (id % c.Wd - px) * c.Q, fy = (id / c.Wd - py) * c.Q;
      const int32_t e = group_sum<64>(patch_partial(c, px, py, fx, fy, lane, 64));
      if (e < bestC) { bestC = e; bestF = packf(fx, fy); }
    }
  }
  if (f.proposal) {
    const int32_t fp = f.proposal[(size_t)gy * Gw + gx];
    if (fp != kEmpty && centre_valid(c, px, py, fx_of(fp), fy_of(fp))) {
      const int32_t e = group_sum<64>(patch_partial(c, px, py, fx_of(fp), fy_of(fp), lane, 64));
      if (e < bestC) { bestC = e; bestF = fp; }
    }
  }
  if (lane == 0) {
    grid_flow(f, lev, buf)[(size_t)gy * Gw + gx] = bestF;
    grid_cost(f, lev, buf)[(size_t)gy * Gw + gx] = bestC;
  }
}

// ---------------------------------------------------------------- level entry
// Section 3.2: points of the coarser grid keep their flow and are re-costed
// with this level's patch; new points start empty.  One group of L lanes per
// coarse point (the fine points of even coordinates), which also writes the
// three new points it covers.  grid: (coarse pts L / 256, fields)
template <int L>
__global__ __launch_bounds__(256) void k_level_entry(const FieldRec* __restrict__ table, int lev, int qshift, int buf) {
  static_assert(L == 16, "the row path assumes 16 lanes per point");
  const FieldRec& f = table[blockIdx.y];
  const CostCtx c = ctx_of(f, lev, qshift);
  const int Gw = (f.Ws + c.n - 1) >> lev, Gh = (f.Hs + c.n - 1) >> lev;
  const int Gwc = (f.Ws + 2 * c.n - 1) >> (lev + 1), Ghc = (f.Hs + 2 * c.n - 1) >> (lev + 1);
  const int cid = (blockIdx.x * blockDim.x + threadIdx.x) / L;
  const int lane = threadIdx.x % L;
  if (cid >= Gwc * Ghc) return;
  const int cx = cid % Gwc, cy = cid / Gwc;
  const int gx = 2 * cx, gy = 2 * cy;
  const int32_t fl = grid_flow(f, lev + 1, 0)[cid];   // a finished level ends in buffer 0
  int32_t e = kInf;
  if (fl != kEmpty) {
    const int px = gx * c.n, py = gy * c.n, fx = fx_of(fl), fy = fy_of(fl);
    const int mx = px * c.Q + fx, my = py * c.Q + fy;
    const int Mx = mx >> c.qshift, My = my >> c.qshift;
    int32_t part;
    if (lev == 0 && (c.r == 8 || c.r == 6) && px >= c.r && px + c.r < c.Ws && Mx >= c.r && Mx + c.r < c.Wd) {
      // stride 1, no column clamp on either side: whole columns per lane
      const uint32_t* D2 = c.dst + (size_t)c.pw * (size_t)(((my & c.qmask) << c.qshift) + (mx & c.qmask));
      g_u32* sb = (g_u32*)(c.src + (px - c.r));
      g_u32* tb = (g_u32*)(D2 + (Mx - c.r));
      part = c.r == 8 ? cols_sum_n1<17>(sb, c.Ws, py - 8, c.Hs - 1, tb, c.Wd, My - 8, c.Hd - 1, lane)
                      : cols_sum_n1<13>(sb, c.Ws, py - 6, c.Hs - 1, tb, c.Wd, My - 6, c.Hd - 1, lane);
    } else {
      part = patch_partial(c, px, py, fx, fy, lane, L);
    }
    e = group_sum<L>(part);
  }
  int32_t* F = grid_flow(f, lev, buf);
  int32_t* C = grid_cost(f, lev, buf);
  if (lane < 4) {
    const int x = gx + (lane & 1), y = gy + (lane >> 1);
    if (x < Gw && y < Gh) {
      F[(size_t)y * Gw + x] = lane == 0 ? fl : kEmpty;
      C[(size_t)y * Gw + x] = lane == 0 ? e : kInf;
    }
  }
  (void)Ghc;
}

typedef __attribute__((address_space(1))) const char g_byte;

// clamp to [0, hi] in one instruction (the compiler emits max then min when
// the upper bound is not a constant)
__device__ __forceinline__ uint32_t clamp0(int v, int hi) {
  int r;
  asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(v), "v"(hi));
  return (uint32_t)r;
}
// target word at a 32-bit word offset from a uniform base: the byte offset is
// formed in 32 bits so the load takes the scalar-base + 32-bit-offset form
// (ff_desc_init refuses layouts whose largest offset would not fit)
__device__ __forceinline__ uint32_t tword(g_byte* base, uint32_t w) {
  return *reinterpret_cast<__attribute__((address_space(1))) const uint32_t*>(base + (w << 2));
}

// CW words of a line from byte offset at: consecutive (WIDE, one load) or every fourth sample
template <int CW, bool WIDE, int LEV>
__device__ __forceinline__ void load_line(g_byte* tgt, uint32_t at, int lev, uint32_t (&w)[CW]) {
  g_byte* const p = tgt + at;
  typedef uint32_t vec __attribute__((ext_vector_type(CW == 3 ? 4 : CW), aligned(4)));
  if (WIDE && CW == 4) {
    const vec x = *reinterpret_cast<__attribute__((address_space(1))) const vec*>(p);
#pragma unroll
    for (int m = 0; m < CW; ++m) w[m] = x[m];
  } else {
#pragma unroll
    for (int m = 0; m < CW; ++m)
      w[m] = *reinterpret_cast<__attribute__((address_space(1))) const uint32_t*>(
          p + (WIDE ? 4 * m : (16 * m) << (LEV >= 0 ? LEV : lev)));
  }
}

// ---------------------------------------------------------------- random search
// Section 3.1 / 3.2: one uniform offset per point, per axis an integer in
// [-nRQ, nRQ] 1/Q px, from Philox keyed by the seed with counter (pixel, level,
// step, field | pair << 2); replace only on a strictly lower cost.
// Bound: the texture addresser.  A candidate's rows lie at unrelated addresses,
// so a patch is S cache lines or more however it is read, and three of four
// candidates lose: both kernels add the patch up in thirds and drop a
// candidate once its sum reaches the point's cost.
//
// All levels and radii: one workgroup = 16 consecutive points of one grid row,
// 16 lanes per point.  Their source patches overlap: the union (grid-aligned
// samples clamped to the image) is staged in LDS once.  A point's terms go
// round its lanes, those of a third all in flight at once (S_ > 0).
// 1024x436, levels 1-3: 28 us per launch with the patch in one go, 24 us in
// thirds; eight pairs of 641x479 and below 295 and 270 us.
constexpr int kSearchPts = 16;
struct SearchSmem {
  uint32_t src[(2 * kMaxRadius + 1) * (2 * kMaxRadius + kSearchPts + 1)];
  int32_t f[kSearchPts], c[kSearchPts];
};
template <int S_>
__device__ __forceinline__ void search_row(const FieldRec& f, SearchSmem& sm, int lev, int qshift, int step, int R, int buf) {
  constexpr int L = 16, PTS = kSearchPts;
  uint32_t* const stile = sm.src;
  const CostCtx c = ctx_of(f, lev, qshift);
  const int Gw = (f.Ws + c.n - 1) >> lev, Gh = (f.Hs + c.n - 1) >> lev;
  const int tilesX = (Gw + PTS - 1) / PTS;
  const int gy = blockIdx.x / tilesX, gx0 = (blockIdx.x % tilesX) * PTS;
  if (gy >= Gh) return;   // whole workgroup
  // tile rows: S patch rows of an odd pitch
  const int r = S_ ? S_ / 2 : c.r, S = 2 * r + 1, TWs = S - 1 + PTS, TP = TWs | 1;
  int32_t* F = grid_flow(f, lev, buf);
  int32_t* C = grid_cost(f, lev, buf);
  const int py = gy * c.n;
  // each point's flow and cost, loaded before the tile so that the two
  // round trips overlap
  const int gq = gx0 + (int)threadIdx.x;
  int32_t fl = kEmpty, cq = 0;
  if (threadIdx.x < PTS && gq < Gw) {
    fl = gp(F)[gy * Gw + gq];
    cq = gp(C)[gy * Gw + gq];
  }
  auto stage = [&](int e) {
    const int yy = e / TWs, xx = e - yy * TWs;
    const int sy = clampi((gy + yy - r) * c.n, 0, c.Hs - 1), sx = clampi((gx0 + xx - r) * c.n, 0, c.Ws - 1);
    stile[yy * TP + xx] = gp(c.src)[sy * c.Ws + sx];
  };
  if (S_) {
#pragma unroll
    for (int k = 0; k < (S_ * (S_ - 1 + PTS) + 255) / 256; ++k)
      if ((int)threadIdx.x + 256 * k < S * TWs) stage(threadIdx.x + 256 * k);
  } else {
    for (int e = threadIdx.x; e < S * TWs; e += 256) stage(e);
  }
  // each point's candidate, once per point (one lane of the first wavefront
  // per point: the Philox rounds are quarter-rate multiplies)
  if (threadIdx.x < PTS) {
    int32_t fq = 0, bound = -1;
    if (fl != kEmpty) {
      const int pxq = gq * c.n;
      const int rad = c.n * R * c.Q;
      uint32_t u0, u1;
      philox2((uint32_t)(py * c.Ws + pxq), (uint32_t)lev, (uint32_t)step, f.c3, f.k0, f.k1, u0, u1);
      const uint64_t span = (uint64_t)(2 * rad + 1);
      const int fx = fx_of(fl) + (int)((u0 * span) >> 32) - rad, fy = fy_of(fl) + (int)((u1 * span) >> 32) - rad;
      fq = packf(fx, fy);
      if (centre_valid(c, pxq, py, fx, fy)) bound = cq;
    }
    sm.f[threadIdx.x] = fq;
    sm.c[threadIdx.x] = bound;
  }
  __syncthreads();
  const int i = threadIdx.x / L, lane = threadIdx.x % L;
  const int32_t bound = sm.c[i];
  if (bound < 0) return;   // no such point, nothing to search around, or outside the image
  const int gx = gx0 + i, px = gx * c.n;
  const int32_t cand = sm.f[i];
  const int mx = px * c.Q + fx_of(cand), my = py * c.Q + fy_of(cand);
  const int Mx = mx >> c.qshift, My = my >> c.qshift;
  const uint32_t plane = __umul24(c.pw, (uint32_t)(((my & c.qmask) << c.qshift) + (mx & c.qmask)));
  g_byte* const tgt = (g_byte*)c.dst;
  const uint32_t* sp = stile + i;
  int32_t sum = 0;
  // term t = lane + 16 k of the patch, at (dx, dy)
  int dy = lane / S, dx = lane - dy * S;
  const int stepy = L / S, stepx = L - stepy * S;
  auto at = [&] {
    return plane + __umul24(clamp0(My + (dy - r) * c.n, c.Hd - 1), (uint32_t)c.Wd) +
           clamp0(Mx + (dx - r) * c.n, c.Wd - 1);
  };
  auto next = [&] {
    dx += stepx;
    dy += stepy;
    if (dx >= S) { dx -= S; ++dy; }
  };
  if (S_) {
    // a third of the terms at a time; a candidate whose sum reaches the
    // point's cost is out
    constexpr int K = (S_ * S_ + L - 1) / L, T = S_ ? (K + 2) / 3 : 1;
    int32_t total = 0;
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += T) {
      uint32_t w[T], a[T];
#pragma unroll
      for (int k = 0; k < T; ++k) {   // past the patch for some lanes at the end: read (rows clamp), not summed
        if (k0 + k >= K) break;
        w[k] = tword(tgt, at());
        a[k] = sp[min(dy, S - 1) * TP + dx];
        next();
      }
#pragma unroll
      for (int k = 0; k < T; ++k)
        if (k0 + k < K) sum += lane + L * (k0 + k) < S * S ? __popc(w[k] ^ a[k]) : 0;
      total = group_sum<L>(sum);
      if (total >= bound) return;
    }
    sum = total;
  } else {
    for (int t = lane; t < S * S; t += L) {
      sum += __popc(tword(tgt, at()) ^ sp[dy * TP + dx]);
      next();
    }
  }
  if (!S_) sum = group_sum<L>(sum);
  if (lane == 0 && sum < bound) {
    gp(F)[gy * Gw + gx] = cand;
    gp(C)[gy * Gw + gx] = sum;
  }
}

__global__ __launch_bounds__(256) void k_random_search(const FieldRec* __restrict__ table, int lev, int qshift, int step,
                                                       int R, int buf) {
  __shared__ SearchSmem sm;
  const FieldRec& f = table[blockIdx.y];
  if (f.r == 8) search_row<17>(f, sm, lev, qshift, step, R, buf);
  else if (f.r == 6) search_row<13>(f, sm, lev, qshift, step, R, buf);
  else search_row<0>(f, sm, lev, qshift, step, R, buf);
}

// Level 0, r = 8 and 6: workgroups of 16 x 16 points.  A wavefront draws 64
// candidates, one per lane, and costs them 16 at a time, four lanes per
// point: a row of the patch is one load per lane (four words, or three of one
// word), neighbouring lanes on neighbouring words, so that an instruction
// reads whole row segments of 16 points; the row's last word is left to the
// lane whose turn it is.  Row and word offsets are uniform and go into the
// scalar base of the load.  Runs of adjacent tiles go to one XCD, whose L2
// then serves their overlap.
// Against 16 lanes per point, whole patches: eight pairs (641x479 and below)
// 1,390 -> 793 us per launch; all four levels of eight pairs 6.9 -> 4.8 ms, of
// 1024x436 0.56 -> 0.40 ms a field.  At levels 1-3 most patches clamp and
// their samples lie 2 to 8 words apart, so that no row is one load, and the
// grids are too small for four rounds per wavefront: this kernel took 59 us a
// launch there (1024x436) against 24, and they keep the one above.
struct TileSmem {
  uint32_t src[32 * 32];
  int32_t f[256], bound[256];
};
template <int S>
__device__ __forceinline__ void search_tile(const FieldRec& f, TileSmem& sm, int qshift, int step, int R, int buf) {
  constexpr int r = S / 2, CW = S / 4, TP = 16 + 2 * r;
  static_assert(S % 4 == 1 && TP <= 32, "row split");
  uint32_t* const s_src = sm.src;
  int32_t *const s_f = sm.f, *const s_bound = sm.bound;
  const CostCtx c = ctx_of(f, 0, qshift);
  const int Gw = f.Ws, Gh = f.Hs;
  const int tilesX = (Gw + 15) >> 4, nt = tilesX * ((Gh + 15) >> 4);
  const int per = (nt + 7) >> 3, tile = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || tile >= nt) return;   // whole workgroup
  const int gy0 = tile / tilesX * 16, gx0 = tile % tilesX * 16;
  int32_t* F = grid_flow(f, 0, buf);
  int32_t* C = grid_cost(f, 0, buf);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // this lane's point: its flow and cost, loaded before the tile so that the
  // round trips overlap
  const int pgx = gx0 + (lane & 15), pgy = gy0 + wave * 4 + (lane >> 4);
  int32_t fl = kEmpty, bound = -1;
  if (pgx < Gw && pgy < Gh) {
    fl = gp(F)[pgy * Gw + pgx];
    bound = gp(C)[pgy * Gw + pgx];
  }
  {
    // rows lane / 16 + 4 wave + 16 k, columns lane % 16 + 16 j
    constexpr int NK = (TP + 15) / 16;
    uint32_t w[NK][NK];
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
      for (int j = 0; j < NK; ++j) {
        const int y = wave * 4 + (lane >> 4) + 16 * k, x = (lane & 15) + 16 * j;
        w[k][j] = gp(c.src)[clampi(gy0 + y - r, 0, c.Hs - 1) * c.Ws + clampi(gx0 + x - r, 0, c.Ws - 1)];
      }
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
      for (int j = 0; j < NK; ++j) {
        const int y = wave * 4 + (lane >> 4) + 16 * k, x = (lane & 15) + 16 * j;
        if (y < TP && x < TP) s_src[y * TP + x] = w[k][j];
      }
  }
  {
    int32_t cand = 0;
    if (fl != kEmpty) {
      const int rad = R * c.Q;
      uint32_t u0, u1;
      philox2((uint32_t)(pgy * c.Ws + pgx), 0u, (uint32_t)step, f.c3, f.k0, f.k1, u0, u1);
      const uint64_t span = (uint64_t)(2 * rad + 1);
      const int fx = fx_of(fl) + (int)((u0 * span) >> 32) - rad, fy = fy_of(fl) + (int)((u1 * span) >> 32) - rad;
      cand = packf(fx, fy);
      if (!centre_valid(c, pgx, pgy, fx, fy)) bound = -1;
    } else {
      bound = -1;   // nothing to search around
    }
    s_f[threadIdx.x] = cand;
    s_bound[threadIdx.x] = bound;
  }
  __syncthreads();
  const int i = lane >> 2, j = lane & 3;
  const int Wm = c.Wd - 1, Hm = c.Hd - 1;
  const bool room = Wm >= 2 * r && Hm >= 2 * r;
  g_byte* const tgt = (g_byte*)c.dst;
  const uint32_t Wd = (uint32_t)c.Wd;
  for (int it = 0; it < 4; ++it) {
    const int q = wave * 64 + it * 16 + i, ly = wave * 4 + it;
    const int32_t cand = s_f[q], bnd = s_bound[q];
    bool use = bnd >= 0;
    if (__ballot(use) == 0) continue;
    const int mx = ((gx0 + i) << c.qshift) + fx_of(cand), my = ((gy0 + ly) << c.qshift) + fy_of(cand);
    const int Mx = mx >> c.qshift, My = my >> c.qshift;
    const uint32_t plane = __umul24(c.pw, (uint32_t)(((my & c.qmask) << c.qshift) + (mx & c.qmask)));
    const uint32_t* sp = s_src + ly * TP + i;
    int32_t sum = 0;
    auto quad = [&](int32_t v) {   // over the point's four lanes
      v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
      return v + __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    };
    const bool clamps = ((uint32_t)(Mx - r) > (uint32_t)(Wm - 2 * r)) | ((uint32_t)(My - r) > (uint32_t)(Hm - 2 * r));
    if (room && __ballot(use & clamps) == 0) {
      // a third of the rows at a time; a candidate whose sum reaches the
      // point's cost is out
      const uint32_t at = plane + __umul24((uint32_t)(My - r), Wd) + (uint32_t)(Mx - r);
      const uint32_t o = (at + (uint32_t)(CW * j)) << 2, ot = (at + __umul24((uint32_t)j, Wd)) << 2;
      const size_t rowB = (size_t)c.Wd * 4;
      constexpr int kThird = (S + 2) / 3;
      int32_t total = 0;
#pragma unroll
      for (int y0 = 0; y0 < S; y0 += kThird) {
        if (use) {
          uint32_t w[kThird][CW], wt[(kThird + 3) / 4];
#pragma unroll
          for (int y = 0; y < kThird; ++y)
            if (y0 + y < S) load_line<CW, true, 0>(tgt + (y0 + y) * rowB, o, 0, w[y]);
#pragma unroll
          for (int t = 0; t < kThird; t += 4)   // row y0 + t + j
            if (t + 3 < kThird && y0 + t + 3 < S ? true : t + j < kThird && y0 + t + j < S)
              wt[t / 4] = *reinterpret_cast<__attribute__((address_space(1))) const uint32_t*>(tgt + (y0 + t) * rowB +
                                                                                              (S - 1) * 4 + ot);
          sum = 0;
#pragma unroll
          for (int y = 0; y < kThird; ++y)
            if (y0 + y < S) {
#pragma unroll
              for (int m = 0; m < CW; ++m) sum += __popc(w[y][m] ^ sp[(y0 + y) * TP + CW * j + m]);
            }
#pragma unroll
          for (int t = 0; t < kThird; t += 4)
            if (t + 3 < kThird && y0 + t + 3 < S ? true : t + j < kThird && y0 + t + j < S)
              sum += __popc(wt[t / 4] ^ sp[(y0 + t + j) * TP + S - 1]);
          total += quad(sum);
          use = total < bnd;
        }
        if (y0 + kThird < S && __ballot(use) == 0) break;
      }
      sum = total;
    } else if (use) {
      // columns and rows clamp one by one; a lane takes every fourth word
      uint32_t xo[CW];
#pragma unroll
      for (int m = 0; m < CW; ++m) xo[m] = plane + clamp0(Mx + j + 4 * m - r, Wm);
      const uint32_t xt = plane + clamp0(Mx + r, Wm);
      uint32_t w[S][CW], wt[(S + 3) / 4];
#pragma unroll
      for (int y = 0; y < S; ++y) {
        const uint32_t row = __umul24(clamp0(My + y - r, Hm), Wd);
#pragma unroll
        for (int m = 0; m < CW; ++m) w[y][m] = tword(tgt, row + xo[m]);
      }
#pragma unroll
      for (int t = 0; t < (S + 3) / 4; ++t)   // row 4 t + j (past the last one for some lanes: read, not summed)
        wt[t] = tword(tgt, __umul24(clamp0(My + 4 * t + j - r, Hm), Wd) + xt);
#pragma unroll
      for (int y = 0; y < S; ++y)
#pragma unroll
        for (int m = 0; m < CW; ++m) sum += __popc(w[y][m] ^ sp[y * TP + j + 4 * m]);
#pragma unroll
      for (int t = 0; t < (S + 3) / 4; ++t)
        if (4 * t + j < S) sum += __popc(wt[t] ^ sp[(4 * t + j) * TP + S - 1]);
      sum = quad(sum);
    }
    if (j == 0 && use && sum < bnd) {
      const int p = (gy0 + ly) * Gw + gx0 + i;
      gp(F)[p] = cand;
      gp(C)[p] = sum;
    }
  }
}

__global__ __launch_bounds__(256) void k_random_search_tile(const FieldRec* __restrict__ table, int qshift, int step, int R,
                                                            int buf) {
  __shared__ TileSmem sm;
  const FieldRec& f = table[blockIdx.y];
  if (f.r == 8) search_tile<17>(f, sm, qshift, step, R, buf);
  else search_tile<13>(f, sm, qshift, step, R, buf);
}

// ---------------------------------------------------------------- propagation (Eq. 2)
// Sweep direction (sx, sy): 1: (+,+), 2: (-,-), 3: (-,+), 4: (+,-); the
// predecessors of a point lie at -sx (horizontal) and -sy (vertical).  In
// the transformed coordinates u = sx > 0 ? gx : Gw-1-gx (same for v) every
// sweep runs right and down.
//
// One wavefront visits one tile at a time (ff_relax.h has the scheduling and
// why the order does not matter).  At step t row i of the tile is at column
// u0 + t - i, on four lanes.  A step costs both candidates of its 16 points:
// per point the row leaving and the row entering the patch (vertical
// candidate) and the column leaving and entering it (horizontal), S = 2r+1
// census words each, a quarter of every line per lane -- neighbouring lanes
// read neighbouring words, so that a load instruction touches 16 lines, not
// 64.  Source lines come from the tile's source census in LDS, held
// row-major and column-major so that both kinds of line are contiguous.
//
// Bound: memory latency.  A step is one dependent chain (result, addresses,
// loads, sums); neighbouring flows differ by subpixel steps, so its 64 lines
// lie in different phase planes and mostly miss both caches: 0.62 us per step
// with the chip idle, 1.3 us with every CU at work, of which instructions are
// 0.25 us.  A visit is 16 steps and about 4 us around them.  Measured on
// 1024x436 (three fields at once) the four level-1 sweeps take 0.63, 0.32, 0.23
// and 0.19 ms where one wavefront per band of 16 rows, every band waiting for
// the one above, took 1.15 ms each.  By this alone a pair took 6.2 ms for 10.3,
// one 641x479 field 2.7 for 6.7, eight mixed pairs in one call 31.8 for 41.4;
// with the searches, trees and launch counts since, 5.4 to 5.6, 2.5 and 26.
// 64 mixed pairs (a full chip throughout): 209 -> 194 ms with all of it.
// Tile size (modelled from the visits each needs on that pair): 16 x 8, 8 x 16
// and 8 x 8 points need 1.5 to 2 times the visits for the same chain, 16 x 32
// has a longer one.
struct SweepArgs {
  int f0, nf;        // fields of this launch
  int lev, qshift;
  int sx, sy;
  uint32_t tag;      // of this launch, in the border words
  int base;          // of the request counters (ff_relax.h)
  int inbuf;         // grid buffer read; the other one is written
};

// LDS of a sweep's workgroup.  RM: the largest radius; even pitches: the rows
// of a step lie a pitch -+ 1 apart, so their words fall in different banks.
template <int RM>
struct SweepPitch {
  static constexpr int row = kTileW + kTileH + 2 * RM, col = (kTileH + 2 * RM + 4) & ~1;
};
constexpr int kPitchOwn = kTileW + 1;
template <int RM>
struct SweepSmem {
  uint32_t row[(kTileH + 2 * RM + 1) * SweepPitch<RM>::row];       // source census, row-major
  uint32_t col[(kTileW + kTileH + 2 * RM) * SweepPitch<RM>::col];  // and column-major
  int2 own[kTileH * kPitchOwn];                                    // own values
  int2 res[kTileH * kPitchOwn];                                    // results, on entry those of the visit before
  int2 left[kTileH], top[kTileW + 2];                              // border values: flow, 2 cost + changed
};

// One visit of tile gt (number in the launch) of field f; returns the next
// tile this workgroup owns, or -1.  S = 2r+1, or 0: the field's own (up to 31);
// LEV: the level, or -1: any.  first: no earlier visit of this tile in this
// launch.
template <int S, int LEV, int RMS>
__device__ __forceinline__ int sweep_visit(const FieldRec& f, const SweepArgs& a, const RelaxQ& q, SweepSmem<RMS>& sm,
                                           int gt, bool first, RelaxWg& w) {
  constexpr int RM = S ? S / 2 : kMaxRadius;
  static_assert(RM <= RMS, "the workgroup's LDS");
  constexpr int CW = S ? S / 4 : 1;      // words of a line per lane, one more word per line left over (S = 4 CW + 1)
  constexpr bool kWide = S && LEV == 0;  // consecutive words
  static_assert(S == 0 || S % 4 == 1, "line split");
  constexpr int P1 = SweepPitch<RM>::row, P2 = SweepPitch<RM>::col;
  uint32_t *const s_row = sm.row, *const s_col = sm.col;
  int2 *const s_own = sm.own, *const s_res = sm.res, *const s_left = sm.left, *const s_top = sm.top;
  const int lane = threadIdx.x;
  const int lev = LEV >= 0 ? LEV : a.lev;
  const int n = 1 << lev;
  const int sx = a.sx, sy = a.sy;
  const CostCtx c = ctx_of(f, lev, a.qshift);
  const int r = S ? S / 2 : c.r;
  const int Sd = 2 * r + 1;
  const int Q = c.Q;
  const int Gw = (f.Ws + n - 1) >> lev, Gh = (f.Hs + n - 1) >> lev;
  const int g0 = f.t0[lev], tile = gt - g0;
  const int nu = tiles_x(Gw), nv = tiles_y(Gh);
  const int tv = tile / nu, tu = tile - tv * nu;
  const int u0 = tu * kTileW, v0 = tv * kTileH;
  int32_t* const cnt = reinterpret_cast<int32_t*>(f.ws + f.o_st[lev]);
  const int have = ld_coh(cnt + tile) - a.base;   // requests this visit answers
  const int32_t* const inF = grid_flow(f, lev, a.inbuf);
  const int32_t* const inC = grid_cost(f, lev, a.inbuf);
  auto gx_of = [&](int u) { return sx > 0 ? u : Gw - 1 - u; };
  auto gy_of = [&](int v) { return sy > 0 ? v : Gh - 1 - v; };
  auto pidx = [&](int u, int v) { return gy_of(v) * Gw + gx_of(u); };
  // own values, four points per lane (points outside the grid: EMPTY)
  const int lx = lane & 15, ly = lane >> 4;
  int32_t of[4], oc[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int p = pidx(clampi(u0 + lx - k * 4 - ly, 0, Gw - 1), min(v0 + k * 4 + ly, Gh - 1));
    of[k] = gp(inF)[p];
    oc[k] = gp(inC)[p];
  }
  // a tile visited before: its results, and the border flows they came from
  int32_t* const outF = grid_flow(f, lev, a.inbuf ^ 1);
  int32_t* const outC = grid_cost(f, lev, a.inbuf ^ 1);
  int32_t* const was = reinterpret_cast<int32_t*>(f.ws + f.o_seen) + tile * 32;
  int32_t pf[4], pc[4], wasF = 0;
  if (!first) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int p = pidx(clampi(u0 + lx - k * 4 - ly, 0, Gw - 1), min(v0 + k * 4 + ly, Gh - 1));
      pf[k] = ld_coh(outF + p);
      pc[k] = ld_coh(outC + p);
    }
    wasF = ld_coh(was + (lane & 31));
  }
  // the source census under the tile's patches, in ascending grid
  // coordinates from (gxm, gym), clamped to the image in pixels; lane
  // (ly, lx) takes the samples at rows ly + 4 k, columns lx + 16 j
  const int TH = kTileH + 2 * r + 1, TW = kTileW + kTileH + 2 * r;
  constexpr int NK = (kTileH + 2 * RM + 1 + 3) / 4, NJ = (kTileW + kTileH + 2 * RM + 15) / 16;
  const int gxm = sx > 0 ? u0 - kTileH - r : Gw - kTileW - u0 - r;
  const int gym = sy > 0 ? v0 - r - 1 : Gh - kTileH - v0 - r;
  int scol[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) scol[j] = clampi((gxm + lx + 16 * j) * n, 0, c.Ws - 1);
  auto stage = [&](auto K0, auto K1) {
    uint32_t w[K1.value - K0.value][NJ];
#pragma unroll
    for (int k = K0.value; k < K1.value; ++k) {
      const int row = clampi((gym + ly + 4 * k) * n, 0, c.Hs - 1) * c.Ws;
#pragma unroll
      for (int j = 0; j < NJ; ++j) w[k - K0.value][j] = gp(c.src)[row + scol[j]];
    }
#pragma unroll
    for (int k = K0.value; k < K1.value; ++k)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int y = ly + 4 * k, x = lx + 16 * j;
        if (y < TH && x < TW) {
          s_row[y * P1 + x] = w[k - K0.value][j];
          s_col[x * P2 + y] = w[k - K0.value][j];
        }
      }
  };
  stage(std::integral_constant<int, 0>{}, std::integral_constant<int, NK / 2>{});
  // the neighbours' border values: lanes 0..15 the column left of row
  // `lane`, lanes 16..31 the row above; and this tile's own border words,
  // its right column and its bottom row.  Read after the request counter.
  uint64_t* const xr = reinterpret_cast<uint64_t*>(f.ws + f.o_xr);
  uint64_t* const xb = reinterpret_cast<uint64_t*>(f.ws + f.o_xb);
  const bool isl = lane < 16;
  const int bl = lane & 15;
  const int hu = isl ? u0 - bl - 1 : u0 + bl, hv = isl ? v0 + bl : v0 - 1;
  const bool hok = lane < 32 && hu >= 0 && hu < Gw && hv >= 0 && hv < Gh;
  const int ou = isl ? u0 + 15 - bl : u0 + bl - 15, ov = isl ? v0 + bl : v0 + 15;
  const bool ook = lane < 32 && ou >= 0 && ou < Gw && ov < Gh && (isl ? tu + 1 < nu : tv + 1 < nv);
  const int handled = __builtin_amdgcn_readfirstlane(have);
  mem_wait();
  uint64_t hw = 0;
  int32_t hf = kEmpty, hc = kInf;
  if (hok) {
    hw = ld_coh(isl ? xr + (size_t)(tu - 1) * Gh + hv : xb + (size_t)(tv - 1) * Gw + hu);
    hf = gp(inF)[pidx(hu, hv)];
    hc = gp(inC)[pidx(hu, hv)];
  }
  stage(std::integral_constant<int, NK / 2>{}, std::integral_constant<int, NK>{});
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int u = u0 + lx - k * 4 - ly;
    const bool ok = u >= 0 && u < Gw && v0 + k * 4 + ly < Gh;
    const int2 own = ok ? make_int2(of[k], oc[k]) : make_int2(kEmpty, kInf);
    s_own[(k * 4 + ly) * kPitchOwn + lx] = own;
    s_res[(k * 4 + ly) * kPitchOwn + lx] = first || !ok ? own : make_int2(pf[k], pc[k]);
  }
  if ((uint32_t)(hw >> 48) == a.tag) {
    const uint32_t c16 = (uint32_t)(hw >> 32) & 0xFFFFu;
    hf = (int32_t)(uint32_t)hw;
    hc = c16 == 0xFFFFu ? kInf : (int32_t)c16;
  }
  // cost doubled, the low bit marks a value that this tile has not seen
  // (EMPTY's cost is never used)
  if (lane < 32) (isl ? s_left : s_top)[bl] = make_int2(hf, (int)((uint32_t)hc << 1) | (first || hf != wasF ? 1 : 0));
  if (lane == 32) s_top[kTileW] = make_int2(kEmpty, 0);
  __syncthreads();
  // what the readers of this tile's border hold so far
  const int oidx = isl ? bl * kPitchOwn + 15 : 15 * kPitchOwn + bl;
  int2 seen = s_res[oidx];
  asm volatile("" : "+v"(seen.x), "+v"(seen.y));   // read before the steps overwrite it
  // ---- the steps
  const int i = lane >> 2, j = lane & 3;
  g_byte* const tgt = (g_byte*)(c.dst);
  const uint32_t dT = (uint32_t)(c.dstT - c.dst);   // transposed planes after the row-major ones
  const int Wm = c.Wd - 1, Hm = c.Hd - 1;
  const uint32_t Wd = (uint32_t)c.Wd, Hd = (uint32_t)c.Hd;
  const uint32_t maxMx = (uint32_t)(Wm * Q), maxMy = (uint32_t)(Hm * Q);
  const int rn = r * n;
  const int offX0 = -sx * (r + 1) * n, offX1 = sx * rn, offY0 = -sy * (r + 1) * n, offY1 = sy * rn;
  const int vi = v0 + i, gyi = gy_of(vi), gx0 = gx_of(u0 - i);
  const int js = kWide ? CW * j : j;                // the lane's first word of a line
  const int jt = (kWide ? CW * j : j * n) - rn;     // and its place in the target's
  const uint32_t* spv = s_row + (gyi - sy * (r + 1) - gym) * P1 + (gx0 - r - gxm) + js;
  const uint32_t* sph = s_col + (gx0 - sx * (r + 1) - gxm) * P2 + (gyi - r - gym) + js;
  const int eV = sy * Sd * P1, eH = sx * Sd * P2;   // from a leaving line to the entering one
  // the last word of line j (S = 4 CW + 1)
  const uint32_t* spt = (j < 2 ? spv + (j & 1) * eV : sph + (j & 1) * eH) + (S - 1 - js);
  const int32_t tmul = (j & 1 ? 1 : -1) * (j >= 2 ? 65536 : 1);
  const int tailOff = (S - 1) * n - rn - jt;
  const int nQshift = lev + c.qshift;
  const int pyq = gyi << nQshift;
  int pxq = gx0 << nQshift;
  int uL = vi < Gh ? u0 - i : -(1 << 20);
  int2 h = s_left[i], v = i == 0 ? s_top[0] : s_left[i > 0 ? i - 1 : 0];
  // LDS values are read a step ahead of their use
  int2 ownN = s_own[i * kPitchOwn], oldN = s_res[i * kPitchOwn], topN = s_top[1];
  const bool roomX = Wm >= 2 * rn, roomY = Hm >= 2 * rn;   // else every line clamps
#pragma unroll 1
  for (int t = 0; t < kTileW; ++t) {
    const int2 own = ownN, old = oldN, top = topN;
    ownN = s_own[i * kPitchOwn + t + 1];
    oldN = s_res[i * kPitchOwn + t + 1];
    topN = s_top[t + 2];
    const int mxv = pxq + fx_of(v.x), myv = pyq + fy_of(v.x), mxh = pxq + fx_of(h.x), myh = pyq + fy_of(h.x);
    // EMPTY (-32768, -32768) lies outside, so this rejects it too
    // a point none of whose inputs changed keeps its result
    const bool in = ((uint32_t)uL < (uint32_t)Gw) & (((v.y | h.y) & 1) != 0);
    const bool useV = in & (v.x != own.x) & ((uint32_t)mxv <= maxMx) & ((uint32_t)myv <= maxMy);
    const bool useH = in & (h.x != own.x) & ((uint32_t)mxh <= maxMx) & ((uint32_t)myh <= maxMy);
    int2 res = in ? own : old;
    if (__ballot(useV || useH)) {
      const int Mxv = mxv >> c.qshift, Myv = myv >> c.qshift, Mxh = mxh >> c.qshift, Myh = myh >> c.qshift;
      // every product has both factors below 2^24 (plane words <= 2^22,
      // phase < 64, coordinates and pitches < 8192)
      const uint32_t plv = __umul24(c.pw, (uint32_t)(((myv & c.qmask) << c.qshift) + (mxv & c.qmask)));
      const uint32_t plh = dT + __umul24(c.pw, (uint32_t)(((myh & c.qmask) << c.qshift) + (mxh & c.qmask)));
      uint32_t l0 = plv + __umul24(clamp0(Myv + offY0, Hm), Wd), l1 = plv + __umul24(clamp0(Myv + offY1, Hm), Wd);
      uint32_t l2 = plh + __umul24(clamp0(Mxh + offX0, Wm), Hd), l3 = plh + __umul24(clamp0(Mxh + offX1, Wm), Hd);
      uint32_t lea = 0, ent = 0, leaH = 0, entH = 0, tail = 0;
      const bool clampV = (uint32_t)(Mxv - rn) > (uint32_t)(Wm - 2 * rn);
      const bool clampH = (uint32_t)(Myh - rn) > (uint32_t)(Hm - 2 * rn);
      if (S && roomX && roomY && __ballot((useV & clampV) | (useH & clampH)) == 0) {
        // no sample of a candidate in use clamps; the lanes of a candidate
        // that is not read word 0
        l0 = useV ? l0 + (uint32_t)(Mxv + jt) : 0;
        l1 = useV ? l1 + (uint32_t)(Mxv + jt) : 0;
        l2 = useH ? l2 + (uint32_t)(Myh + jt) : 0;
        l3 = useH ? l3 + (uint32_t)(Myh + jt) : 0;
        const uint32_t lt = j < 2 ? (j & 1 ? l1 : l0) : (j & 1 ? l3 : l2);
        uint32_t w0[CW], w1[CW], w2[CW], w3[CW];
        load_line<CW, kWide, LEV>(tgt, l0 << 2, lev, w0);
        load_line<CW, kWide, LEV>(tgt, l1 << 2, lev, w1);
        load_line<CW, kWide, LEV>(tgt, l2 << 2, lev, w2);
        load_line<CW, kWide, LEV>(tgt, l3 << 2, lev, w3);
        const uint32_t wt = tword(tgt, lt + (uint32_t)((j < 2 ? useV : useH) ? tailOff : 0));
#pragma unroll
        for (int m = 0; m < CW; ++m) {
          const int k = kWide ? m : 4 * m;
          lea += __popc(w0[m] ^ spv[k]);
          ent += __popc(w1[m] ^ spv[eV + k]);
          leaH += __popc(w2[m] ^ sph[k]);
          entH += __popc(w3[m] ^ sph[eH + k]);
        }
        tail = __popc(wt ^ *spt);
        asm volatile("" : "+v"(tail));   // keeps this branch's loads in it
      } else {
        if (S) {
          // all loads first: one round trip
          uint32_t x[4][CW];
#pragma unroll
          for (int m = 0; m < CW; ++m) {
            const int o = (js + (kWide ? m : 4 * m)) * n - rn;
            const uint32_t xv = clamp0(Mxv + o, Wm), yh = clamp0(Myh + o, Hm);
            x[0][m] = tword(tgt, l0 + xv);
            x[1][m] = tword(tgt, l1 + xv);
            x[2][m] = tword(tgt, l2 + yh);
            x[3][m] = tword(tgt, l3 + yh);
          }
          const uint32_t lt = j < 2 ? (j & 1 ? l1 : l0) : (j & 1 ? l3 : l2);
          const uint32_t wt = tword(tgt, lt + clamp0((j < 2 ? Mxv : Myh) + rn, j < 2 ? Wm : Hm));
#pragma unroll
          for (int m = 0; m < CW; ++m) {
            const int k = kWide ? m : 4 * m;
            lea += __popc(x[0][m] ^ spv[k]);
            ent += __popc(x[1][m] ^ spv[eV + k]);
            leaH += __popc(x[2][m] ^ sph[k]);
            entH += __popc(x[3][m] ^ sph[eH + k]);
          }
          tail = __popc(wt ^ *spt);
        } else {
          for (int k = 0; k < Sd - js; k += 4) {
            const int o = (js + k) * n - rn;
            const uint32_t xv = clamp0(Mxv + o, Wm), yh = clamp0(Myh + o, Hm);
            lea += __popc(tword(tgt, l0 + xv) ^ spv[k]);
            ent += __popc(tword(tgt, l1 + xv) ^ spv[eV + k]);
            leaH += __popc(tword(tgt, l2 + yh) ^ sph[k]);
            entH += __popc(tword(tgt, l3 + yh) ^ sph[eH + k]);
          }
        }
      }
      // vertical sum in the low half, horizontal in the high half
      // (|sums| < 2^15), over the row's four lanes
      int32_t d = (int32_t)(ent - lea) + (int32_t)((entH - leaH) << 16) + __mul24((int32_t)tail, tmul);
      d += __builtin_amdgcn_update_dpp(0, d, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
      d += __builtin_amdgcn_update_dpp(0, d, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
      const int32_t dV = (int32_t)(int16_t)(uint16_t)((uint32_t)d & 0xFFFFu), dH = (d - dV) >> 16;
      // candidate order of Eq. 2: current, vertical, horizontal; strict <
      const int costV = (v.y >> 1) + dV, costH = (h.y >> 1) + dH;
      if (useV && costV < res.y) res = make_int2(v.x, costV);
      if (useH && costH < res.y) res = make_int2(h.x, costH);
    }
    s_res[i * kPitchOwn + t] = res;
    // next step's candidates: horizontal the row's own result, vertical the
    // result of the row above (four lanes down; across a 16-lane DPP row
    // its last lane's value; the top row from the border)
    h = make_int2(res.x, (int)((uint32_t)res.y << 1) | (first || res.x != old.x ? 1 : 0));
    v.x = __builtin_amdgcn_update_dpp(top.x, h.x, 0x114, 0xF, 0xF, false);   // row_shr:4
    v.y = __builtin_amdgcn_update_dpp(top.y, h.y, 0x114, 0xF, 0xF, false);
    v.x = __builtin_amdgcn_update_dpp(v.x, h.x, 0x142, 0xE, 0x1, false);     // row_bcast:15
    v.y = __builtin_amdgcn_update_dpp(v.y, h.y, 0x142, 0xE, 0x1, false);
    pxq += sx * (1 << nQshift);
    spv += sx;
    sph += sx * P2;
    spt += j < 2 ? sx : sx * P2;
    ++uL;
  }
  __syncthreads();
  // ---- results out, changed border words published
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int u = u0 + lx - k * 4 - ly, v = v0 + k * 4 + ly;
    if (u >= 0 && u < Gw && v < Gh) {
      const int2 x = s_res[(k * 4 + ly) * kPitchOwn + lx];
      st_coh(outF + pidx(u, v), x.x);
      st_coh(outC + pidx(u, v), x.y);
    }
  }
  if (lane < 32) st_coh(was + lane, hf);
  const int2 now = s_res[oidx];
  const bool chg = ook && now.x != seen.x;
  if (chg) st_coh(isl ? xr + (size_t)tu * Gh + ov : xb + (size_t)tv * Gw + ou, xch_pack(now.x, now.y, a.tag));
  const uint64_t cm = __ballot(chg);
  mem_wait();
  __syncthreads();
  return relax_done(q, cnt, a.base, tile, nu, g0, handled, (cm & 0xFFFFu) != 0, (cm & 0x7FFF0000u) != 0,
                    (cm & 0x80000000u) != 0, w);
}

// The visits of a workgroup: its first visits, dealt out in turn, then queued
// tiles.
template <typename Visit>
__device__ __forceinline__ void sweep_tiles(const FieldRec* __restrict__ table, const SweepArgs& a, const RelaxQ& q, int lev,
                                            Visit visit) {
  const int lane = threadIdx.x;
  RelaxWg w = relax_begin(q, blockIdx.x);
  int gt = w.mine;
  bool first = true;
  do {
    // the tile's field: the last one whose first tile is not above it
    int fi = a.f0 + (a.nf == 1 ? 1 : 0);
    for (int b = 0; b < a.nf && a.nf > 1; b += 64) {
      const int k = b + lane;
      const bool le = k < a.nf && table[a.f0 + k].t0[lev] <= gt;
      fi += __popcll(__ballot(le));
    }
    fi = __builtin_amdgcn_readfirstlane(fi - 1);
    gt = relax_next(q, w, visit(table[fi], gt, first, w), first);
  } while (gt >= 0);
}

// fields of one radius
template <int S, int LEV>
__global__ __launch_bounds__(64) void k_sweep(const FieldRec* __restrict__ table, SweepArgs a, RelaxQ q) {
  constexpr int RM = S ? S / 2 : kMaxRadius;
  __shared__ SweepSmem<RM> sm;
  sweep_tiles(table, a, q, LEV >= 0 ? LEV : a.lev, [&](const FieldRec& f, int gt, bool first, RelaxWg& w) {
    return sweep_visit<S, LEV, RM>(f, a, q, sm, gt, first, w);
  });
}

// Fields of r = 8 and of r = 6 in one launch: one chain of revisits at its end
// instead of two (eight mixed pairs 29.5 -> 26.5 ms).
template <int LEV>
__global__ __launch_bounds__(64) void k_sweep_mixed(const FieldRec* __restrict__ table, SweepArgs a, RelaxQ q) {
  __shared__ SweepSmem<8> sm;
  sweep_tiles(table, a, q, LEV >= 0 ? LEV : a.lev, [&](const FieldRec& f, int gt, bool first, RelaxWg& w) {
    return f.r == 8 ? sweep_visit<17, LEV, 8>(f, a, q, sm, gt, first, w)
                    : sweep_visit<13, LEV, 8>(f, a, q, sm, gt, first, w);
  });
}

// write the grid of level lev into the full-resolution outputs (inspection
// stops); grid: (W / 256, H, fields)
__global__ void k_write_grid(const FieldRec* __restrict__ table, int lev, int buf) {
  const FieldRec& f = table[blockIdx.z];
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= f.Ws || y >= f.Hs) return;
  const int n = 1 << lev;
  const int Gw = (f.Ws + n - 1) >> lev;
  const size_t o = (size_t)y * f.Ws + x;
  if ((x % n) == 0 && (y % n) == 0) {
    f.flow[o] = grid_flow(f, lev, buf)[(size_t)(y / n) * Gw + x / n];
    f.cost[o] = grid_cost(f, lev, buf)[(size_t)(y / n) * Gw + x / n];
  } else {
    f.flow[o] = kEmpty;
    f.cost[o] = kInf;
  }
}

template <int S>
static void launch_sweep_s(const FieldRec* table, const SweepArgs& a, const RelaxQ& q, hipStream_t stream) {
  switch (a.lev) {
    case 0: k_sweep<S, 0><<<q.G, 64, 0, stream>>>(table, a, q); break;
    case 1: k_sweep<S, 1><<<q.G, 64, 0, stream>>>(table, a, q); break;
    case 2: k_sweep<S, 2><<<q.G, 64, 0, stream>>>(table, a, q); break;
    case 3: k_sweep<S, 3><<<q.G, 64, 0, stream>>>(table, a, q); break;
    default: k_sweep<S, -1><<<q.G, 64, 0, stream>>>(table, a, q); break;
  }
}

static void launch_sweep_mixed(const FieldRec* table, const SweepArgs& a, const RelaxQ& q, hipStream_t stream) {
  switch (a.lev) {
    case 0: k_sweep_mixed<0><<<q.G, 64, 0, stream>>>(table, a, q); break;
    case 1: k_sweep_mixed<1><<<q.G, 64, 0, stream>>>(table, a, q); break;
    case 2: k_sweep_mixed<2><<<q.G, 64, 0, stream>>>(table, a, q); break;
    case 3: k_sweep_mixed<3><<<q.G, 64, 0, stream>>>(table, a, q); break;
    default: k_sweep_mixed<-1><<<q.G, 64, 0, stream>>>(table, a, q); break;
  }
}

// The paper's radii (r = 8, r2 = 6) have instances of their own, and go in one
// launch; r, rl: of the launch's first and last field.
static bool sweep_together(int r0, int r1) { return r0 == r1 || (r0 == 8 && r1 == 6) || (r0 == 6 && r1 == 8); }
// Workgroups of such a launch that the chip holds, by LDS (160 KB per CU): eight
// per CU with 17.9 KB (r = 8; r = 6 alone has less, and no use for more), five
// of the instance for any radius, which has LDS for the largest one.
constexpr int kSweepGrid = 256 * 8;
static int sweep_places(int r0, int r1) {
  return (r0 == 8 || r0 == 6) && (r1 == 8 || r1 == 6) ? kSweepGrid : 256 * 5;
}
static void launch_sweep(int r, int rl, const FieldRec* table, const SweepArgs& a, const RelaxQ& q, hipStream_t stream) {
  if (r != rl) launch_sweep_mixed(table, a, q, stream);
  else if (r == 8) launch_sweep_s<17>(table, a, q, stream);
  else if (r == 6) launch_sweep_s<13>(table, a, q, stream);
  else k_sweep<0, -1><<<q.G, 64, 0, stream>>>(table, a, q);
}

// ---------------------------------------------------------------- host plans
struct FieldPlan {
  bool has_tree;
  TreeLayout tree;        // offsets relative to the field region
  size_t off_grid[5], off_st[5];
  size_t off_alt, off_xr, off_xb, off_seen;
  size_t clear_words;     // from off_st[0]: counters and border words
  size_t alt_past;        // what the buffer at off_alt needs past the tree's region
  size_t bytes;
};

static FieldPlan field_plan(const ff_desc* src, const ff_desc* dst, const ff_match_params* p) {
  FieldPlan P{};
  size_t off = 0;
  P.has_tree = p->use_kdtree != 0;
  if (P.has_tree) {
    P.tree = tree_layout(dst->width * dst->height, p->leaf, 0);
    off = P.tree.bytes;
  }
  // the second grid buffer: what the tree build needs beside the finished
  // tree (which seeding reads) is free once the tree stands; a source too
  // large for it reaches past its end
  P.off_alt = P.has_tree ? P.tree.off_perm2 : 0;
  const size_t alt_end = align_up(P.off_alt + (size_t)src->width * src->height * 8, 256);
  P.alt_past = alt_end > off ? alt_end - off : 0;
  off += P.alt_past;
  for (int lev = 1; lev <= p->k; ++lev) {
    const int n = 1 << lev;
    const size_t G = (size_t)((src->width + n - 1) / n) * ((src->height + n - 1) / n);
    off = align_up(off, 256);
    P.off_grid[lev] = off;
    off += G * 8;
  }
  off = align_up(off, 256);
  const size_t clear0 = off;
  for (int lev = 0; lev <= p->k; ++lev) {
    const int n = 1 << lev;
    P.off_st[lev] = off;
    off += (size_t)tiles_x((src->width + n - 1) / n) * tiles_y((src->height + n - 1) / n) * 4;
  }
  off = align_up(off, 256);
  P.off_xr = off;
  off += (size_t)tiles_x(src->width) * src->height * 8;
  P.off_xb = off;
  off += (size_t)tiles_y(src->height) * src->width * 8;
  P.clear_words = (off - clear0) / 4;
  P.off_seen = off;
  off += (size_t)tiles_x(src->width) * tiles_y(src->height) * 32 * 4;
  P.bytes = align_up(off, 256);
  return P;
}

static ff_status check_params(const ff_desc* src, const ff_desc* dst, int radius, const ff_match_params* p) {
  if (!src || !dst || !p) return FF_ERR_ARG;
  if (src->channels != dst->channels || src->subpel != dst->subpel) return FF_ERR_ARG;
  if (p->k < 0 || p->k > src->k || p->k > dst->k) return FF_ERR_ARG;
  if (radius < 1 || radius > kMaxRadius) return FF_ERR_ARG;
  if (p->R < 0 || p->R > 64 || p->n_prop < 0 || p->n_prop > 64 || p->n_rs < 0 || p->n_rs > p->n_prop) return FF_ERR_ARG;
  if (p->field_id > 3) return FF_ERR_ARG;
  if (p->band_rows != 0 && p->band_rows != 8 && p->band_rows != 16 && p->band_rows != 32) return FF_ERR_ARG;
  if (p->pipeline != 0 && p->pipeline != 1) return FF_ERR_ARG;
  if (p->watchdog_us < 0) return FF_ERR_ARG;
  if (p->use_kdtree < 0 || p->use_kdtree > 2) return FF_ERR_ARG;
  if (p->use_kdtree) {
    if (p->leaf < 2 || p->leaf > kMaxLeaf) return FF_ERR_ARG;
    bool hs = false, hd = false;
    for (int i = 0; i < src->n_radii; ++i) hs |= src->radii[i] == radius;
    for (int i = 0; i < dst->n_radii; ++i) hd |= dst->radii[i] == radius;
    if (!hs || !hd) return FF_ERR_ARG;
  }
  return FF_OK;
}

static ff_status check_job(const ff_field_job& j, const ff_match_params* p) {
  ff_match_params q = *p;
  q.field_id = j.field_id;
  ff_status st = check_params(j.src, j.dst, j.radius, &q);
  if (st != FF_OK) return st;
  if (!j.src_blob || !j.dst_blob || !j.flow || !j.cost) return FF_ERR_ARG;
  if (!p->use_kdtree && !j.proposal) return FF_ERR_ARG;
  return FF_OK;
}

// Per-job host arrays of a call: held inline for a single job (so that the
// single-field entry points touch no host heap either), on the heap for more.
template <class T>
struct JobArray {
  T one{};
  std::vector<T> many;
  int n = 0;
  void resize(int k) {
    n = k;
    if (k > 1) many.assign((size_t)k, T{});
  }
  T& operator[](int i) { return n > 1 ? many[(size_t)i] : one; }
  const T& operator[](int i) const { return n > 1 ? many[(size_t)i] : one; }
};

struct BatchLayout {
  size_t off_ctl, off_ring, off_table;   // scheduler words of every launch, the queue they share
  size_t ctl_words;                      // from off_ctl, cleared per call
  int launches, cap;
  JobArray<size_t> off_field;   // per table entry
  JobArray<int> order;          // table entry -> job index (grouped by radius)
  size_t bytes;
};

static BatchLayout batch_layout(const ff_field_job* jobs, int n, const ff_match_params* p) {
  BatchLayout B{};
  B.order.resize(n);
  for (int i = 0; i < n; ++i) B.order[i] = i;
  if (n > 1)
    std::stable_sort(B.order.many.begin(), B.order.many.end(),
                     [&](int a, int b) { return jobs[a].radius > jobs[b].radius; });
  int groups = 0;
  for (int i = 0; i < n; ++i)
    if (i == 0 || jobs[B.order[i]].radius != jobs[B.order[i - 1]].radius) ++groups;
  // the fields come before what depends on the number of sweeps: a tree left in
  // the workspace is found there by a call with another k or n_prop as well
  size_t off = kStatusBytes;
  B.off_table = off;
  off = align_up(off + (size_t)n * sizeof(FieldRec), 256);
  B.off_field.resize(n);
  for (int i = 0; i < n; ++i) {
    const ff_field_job& j = jobs[B.order[i]];
    B.off_field[i] = off;
    off = align_up(off + field_plan(j.src, j.dst, p).bytes, 256);
  }
  B.off_ctl = off;
  B.launches = (p->k + 1) * p->n_prop * groups;
  off += (size_t)B.launches * sizeof(RelaxCtl);
  B.off_ring = off;
  for (int i = 0; i < n; ++i)   // tiles of the finest level over all fields: every launch has fewer
    B.cap += tiles_x(jobs[i].src->width) * tiles_y(jobs[i].src->height);
  off += (size_t)B.cap * 4;
  B.ctl_words = (off - B.off_ctl) / 4;
  B.bytes = align_up(off, 256);
  return B;
}

static FieldRec make_rec(const ff_field_job& j, const ff_match_params* p, char* fws) {
  const ff_desc* s = j.src;
  const ff_desc* d = j.dst;
  const FieldPlan P = field_plan(s, d, p);
  FieldRec r{};
  r.src = census_plane(s, j.src_blob, 0, 0, 0);
  r.srcT = census_plane_t(s, j.src_blob, 0, 0, 0);
  r.dst = census_plane(d, j.dst_blob, 0, 0, 0);
  r.dstT = census_plane_t(d, j.dst_blob, 0, 0, 0);
  r.Vsrc = p->use_kdtree ? wht_block(s, j.src_blob, j.radius) : nullptr;
  r.Vdst = p->use_kdtree ? wht_block(d, j.dst_blob, j.radius) : nullptr;
  r.proposal = j.proposal;
  r.flow = j.flow;
  r.cost = j.cost;
  r.ws = fws;
  r.pws = (uint32_t)(s->width * s->height);
  r.pwd = (uint32_t)(d->width * d->height);
  r.Ws = s->width;
  r.Hs = s->height;
  r.Wd = d->width;
  r.Hd = d->height;
  r.r = j.radius;
  r.D = d->wht_dims;
  r.vstride = d->wht_stride;
  r.k0 = (uint32_t)(j.seed & 0xFFFFFFFFu);
  r.k1 = (uint32_t)(j.seed >> 32);
  r.c3 = j.field_id | (j.pair_id << 2);
  if (P.has_tree) {
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
  }
  for (int l = 0; l < 5; ++l) {
    r.o_grid[l] = (uint32_t)P.off_grid[l];
    r.o_st[l] = (uint32_t)P.off_st[l];
  }
  r.o_alt = (uint32_t)P.off_alt;
  r.o_xr = (uint32_t)P.off_xr;
  r.o_xb = (uint32_t)P.off_xb;
  r.o_seen = (uint32_t)P.off_seen;
  r.clear_words = (uint32_t)P.clear_words;
  return r;
}

static void write_table(const JobArray<FieldRec>& recs, int nrec, FieldRec* dev, hipStream_t stream) {
  for (int i = 0; i < nrec; i += kRecsPerWrite) {
    RecChunk ch{};
    const int n = std::min(kRecsPerWrite, nrec - i);
    for (int k = 0; k < n; ++k) ch.r[k] = recs[i + k];
    k_write_table<<<1, kRecsPerWrite, 0, stream>>>(ch, n, dev + i);
  }
}

// The whole search for a batch of fields.  Every stage is one launch over
// all fields (propagation: one launch per patch radius).
// tree_only: the call's set-up and the kd-tree build, nothing after (the
// tree stays in the workspace for a later call with use_kdtree = 2)
static ff_status run_batch(const ff_field_job* jobs, int n, const ff_match_params* p, char* ws, const BatchLayout& B,
                           hipStream_t stream, bool tree_only = false) {
  int32_t* status = reinterpret_cast<int32_t*>(ws);
  RelaxCtl* ctl = reinterpret_cast<RelaxCtl*>(ws + B.off_ctl);
  FieldRec* table = reinterpret_cast<FieldRec*>(ws + B.off_table);
  JobArray<FieldRec> recs;
  recs.resize(n);
  bool paper_radii = true;
  int maxW = 0, maxH = 0, maxN = 0, maxTop = 0;
  const int k = p->k;
  auto grid_of = [](int size, int lev) { return (size + (1 << lev) - 1) >> lev; };
  auto tiles_of = [&](const FieldRec& f, int lev) {
    return tiles_x(grid_of(f.Ws, lev)) * tiles_y(grid_of(f.Hs, lev));
  };
  for (int i = 0; i < n; ++i) {
    const ff_field_job& j = jobs[B.order[i]];
    recs[i] = make_rec(j, p, ws + B.off_field[i]);
    paper_radii &= recs[i].r == 8 || recs[i].r == 6;
    maxW = std::max(maxW, recs[i].Ws);
    maxH = std::max(maxH, recs[i].Hs);
    maxN = std::max(maxN, recs[i].Wd * recs[i].Hd);
    maxTop = std::max(maxTop, recs[i].t_top);
    if (i > 0 && sweep_together(recs[i - 1].r, recs[i].r))
      for (int lev = 0; lev <= k; ++lev) recs[i].t0[lev] = recs[i - 1].t0[lev] + tiles_of(recs[i - 1], lev);
  }
  const int qshift = ilog2i(jobs[0].dst->subpel);
  fill_i32(status, 1, 0, stream);
  fill_i32(reinterpret_cast<int32_t*>(ctl), B.ctl_words, 0, stream);
  write_table(recs, n, table, stream);
  k_clear_borders<<<dim3(64, n), 256, 0, stream>>>(table);
  if (p->use_kdtree == 1 || tree_only) {
    prof_mark(FF_PROF_TREE, stream, true);
    ff_status st = enqueue_tree_build(table, n, maxN, maxTop, p->leaf, stream);
    prof_mark(FF_PROF_TREE, stream, false);
    if (st != FF_OK) return st;
  }
  if (tree_only) return launch_status();
  auto pts = [&](int lev) { return grid_of(maxW, lev) * grid_of(maxH, lev); };
  // the grid buffer in use: every sweep reads one and writes the other, and a
  // level's last one ends in buffer 0
  const int buf0 = p->n_prop & 1;
  int steps = 0, cur_lev = k, buf = buf0;
  auto stop = [&]() { return p->max_steps >= 0 && steps >= p->max_steps; };
  auto finish = [&]() -> ff_status {
    if (cur_lev > 0 || buf)
      k_write_grid<<<dim3((maxW + 255) / 256, maxH, n), 256, 0, stream>>>(table, cur_lev, buf);
    return launch_status();
  };
  prof_mark(FF_PROF_SEED, stream, true);
  k_seed<<<dim3((pts(k) + 3) / 4, n), 256, 0, stream>>>(table, k, qshift, p->use_kdtree ? 1 : 0, buf);
  prof_mark(FF_PROF_SEED, stream, false);
  ++steps;
  if (stop()) return finish();
  // watchdog of the sweeps' waits: 2 s of the 100 MHz clock
  const uint64_t timeout = p->watchdog_us > 0 ? (uint64_t)p->watchdog_us * 100u : 200000000ull;
  int launch = 0;
  auto sx_of = [](int i) { return ((i & 3) == 0 || (i & 3) == 3) ? 1 : -1; };
  auto sy_of = [](int i) { return ((i & 3) == 0 || (i & 3) == 2) ? 1 : -1; };
  // sweep i of a level, one launch per patch radius (r = 8 and 6 together)
  auto sweep = [&](int lev, int i) {
    prof_mark(FF_PROF_PROPAGATE, stream, true);
    for (int f0 = 0; f0 < n;) {
      int f1 = f0;
      while (f1 < n && (f1 == f0 || sweep_together(recs[f1 - 1].r, recs[f1].r))) ++f1;
      // request counters start at -(i + 1): every sweep of a level leaves
      // them where the next one's first visits are owed
      const SweepArgs a{f0, f1 - f0, lev, qshift, sx_of(i), sy_of(i), (uint32_t)(launch + 1), -(i + 1), buf};
      RelaxQ q{};
      q.ctl = ctl + launch;
      q.ring = reinterpret_cast<int32_t*>(ws + B.off_ring);
      q.cap = B.cap;
      q.T = recs[f1 - 1].t0[lev] + tiles_of(recs[f1 - 1], lev);
      // One field: a pair's three fields are matched side by side on streams
      // of their own, so each takes a third of the places of the r = 8 and 6
      // instances (1024x436 6.23 -> 5.74 ms a pair, 1920x1080 21.6 -> 19.2; a
      // 641x479 field alone 2.30 -> 2.34).  As many with any other radius: with
      // a third of that instance's places a pair of r = 5 and 3 takes 5.30 for
      // 5.45 ms (641x479) and 7.18 for 7.27 (1024x436), but a field of r = 5
      // alone 4.07 for 4.03 and 5.25 for 5.08.
      // Several in one call: all places (eight fields of 641x479: r = 3 8.8,
      // r = 5 10.4, r = 15 22.9 ms; with the 2,048 of the others 10.0, 11.7 and
      // 25.3: workgroups that start late hold first visits back).
      q.G = std::min(q.T, f1 - f0 == 1 ? kSweepGrid / 3 : sweep_places(recs[f0].r, recs[f1 - 1].r));
      q.status = status;
      q.timeout = timeout;
      launch_sweep(recs[f0].r, recs[f1 - 1].r, table, a, q, stream);
      ++launch;
      f0 = f1;
    }
    buf ^= 1;
    prof_mark(FF_PROF_PROPAGATE, stream, false);
  };
  for (int lev = k; lev >= 0; --lev) {
    cur_lev = lev;
    if (lev < k) {
      buf = buf0;
      // one group of lanes per point of the coarser grid
      const unsigned gpts = (unsigned)(((size_t)pts(lev + 1) * kLanesPt + 255) / 256);
      prof_mark(FF_PROF_LEVEL_ENTRY, stream, true);
      k_level_entry<kLanesPt><<<dim3(gpts, n), 256, 0, stream>>>(table, lev, qshift, buf);
      prof_mark(FF_PROF_LEVEL_ENTRY, stream, false);
      ++steps;
      if (stop()) return finish();
    }
    for (int i = 0; i < p->n_prop; ++i) {
      sweep(lev, i);
      ++steps;
      if (stop()) return finish();
      if (i < p->n_rs) {
        prof_mark(FF_PROF_RANDOM_SEARCH, stream, true);
        const unsigned Gw = (unsigned)grid_of(maxW, lev), Gh = (unsigned)grid_of(maxH, lev), wide = (Gw + 15) / 16;
        if (lev == 0 && paper_radii)   // 16 x 16 points per workgroup, in eight runs of tiles
          k_random_search_tile<<<dim3((wide * ((Gh + 15) / 16) + 7) / 8 * 8, n), 256, 0, stream>>>(table, qshift, i, p->R, buf);
        else
          k_random_search<<<dim3((Gw + kSearchPts - 1) / kSearchPts * Gh, n), 256, 0, stream>>>(table, lev, qshift, i, p->R, buf);
        prof_mark(FF_PROF_RANDOM_SEARCH, stream, false);
        ++steps;
        if (stop()) return finish();
      }
    }
  }
  return finish();
}

// ---------------------------------------------------------------- no-allocation scratch
// The limit of ff_match_field_noalloc counts neither what the second grid
// buffer needs past the tree's region nor, of the scheduler words, the ones that
// count the started workgroups.  The latter have room of their own; with the
// former the limit is still kept: a source so large leaves the tree little of
// it (64.0 MiB at most, over sizes, leaves and depths that the limit lets by).
constexpr size_t kUncountedWords = sizeof(RelaxCtl) - 3 * 128;
constexpr size_t kNoallocWords = 5 * 64 * kUncountedWords;   // levels x sweeps, at most
constexpr size_t kNoallocBytes = FF_NOALLOC_SCRATCH_BYTES + kNoallocWords;
// ff_match_field_noalloc keeps what ff_match_field keeps in its workspace
// (status word, scheduler words, field table, kd-tree, level grids, border
// words) in this one static array per device.  On the host its name
// is only a stand-in symbol, not a device address: host code uses the address
// hipGetSymbolAddress returns for the current device, looked up once per
// device (at ff_init, else at the entry point's first call there).
static __device__ __align__(256) char scratch[kNoallocBytes];

namespace {
std::mutex g_scratch_mu;
char* g_scratch_ptr[64];
}  // namespace

ff_status noalloc_scratch(char** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return FF_ERR_HIP;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return FF_ERR_HIP;
    g_scratch_ptr[dev] = static_cast<char*>(ptr);
  }
  if (out) *out = g_scratch_ptr[dev];
  return FF_OK;
}

__global__ void k_copy_status(const int32_t* __restrict__ from, int32_t* __restrict__ to) { *to = *from; }

}  // namespace ff

using namespace ff;

extern "C" {

void ff_default_params(ff_match_params* p) {
  if (!p) return;
  *p = ff_match_params{};
  p->k = 3;
  p->R = 1;
  p->leaf = 8;
  p->n_prop = 4;
  p->n_rs = 3;
  p->use_kdtree = 1;
  p->max_steps = -1;
  p->band_rows = 16;
  p->pipeline = 1;
}

size_t ff_match_batch_workspace_bytes(const ff_field_job* jobs, int32_t n_jobs, const ff_match_params* p) {
  if (!jobs || !p || n_jobs < 1 || n_jobs > 4096) return 0;
  for (int i = 0; i < n_jobs; ++i) {
    ff_match_params q = *p;
    q.field_id = jobs[i].field_id;
    if (!jobs[i].src || !jobs[i].dst || check_params(jobs[i].src, jobs[i].dst, jobs[i].radius, &q) != FF_OK) return 0;
    if (jobs[i].dst->subpel != jobs[0].dst->subpel) return 0;
  }
  return batch_layout(jobs, n_jobs, p).bytes;
}

ff_status ff_match_batch(const ff_field_job* jobs, int32_t n_jobs, const ff_match_params* p, void* workspace,
                         size_t workspace_bytes, hipStream_t stream) {
  if (!jobs || !p || !workspace || n_jobs < 1 || n_jobs > 4096) return FF_ERR_ARG;
  // a tree left in the workspace by ff_match_field_tree belongs to one field
  if (p->use_kdtree == 2 && n_jobs != 1) return FF_ERR_ARG;
  for (int i = 0; i < n_jobs; ++i) {
    if (!jobs[i].src || !jobs[i].dst) return FF_ERR_ARG;
    ff_status st = check_job(jobs[i], p);
    if (st != FF_OK) return st;
    if (jobs[i].dst->subpel != jobs[0].dst->subpel) return FF_ERR_ARG;
  }
  const BatchLayout B = batch_layout(jobs, n_jobs, p);
  if (workspace_bytes < B.bytes) return FF_ERR_WORKSPACE;
  ff_status st = ensure_init();
  if (st != FF_OK) return st;
  return run_batch(jobs, n_jobs, p, static_cast<char*>(workspace), B, stream);
}

static ff_field_job single_job(const ff_desc* src, const void* src_blob, const ff_desc* dst, const void* dst_blob,
                               int32_t radius, const ff_match_params* p, const int32_t* proposal, int32_t* flow,
                               int32_t* cost) {
  ff_field_job j{};
  j.src = src;
  j.src_blob = src_blob;
  j.dst = dst;
  j.dst_blob = dst_blob;
  j.radius = radius;
  j.field_id = p ? p->field_id : 0;
  j.pair_id = p ? p->pair_id : 0;
  j.seed = p ? p->seed : 0;
  j.proposal = proposal;
  j.flow = flow;
  j.cost = cost;
  return j;
}

size_t ff_match_workspace_bytes(const ff_desc* src, const ff_desc* dst, int32_t radius, const ff_match_params* p) {
  if (check_params(src, dst, radius, p) != FF_OK) return 0;
  const ff_field_job j = single_job(src, nullptr, dst, nullptr, radius, p, nullptr, nullptr, nullptr);
  return batch_layout(&j, 1, p).bytes;
}

ff_status ff_match_field(const ff_desc* src, const void* src_blob, const ff_desc* dst, const void* dst_blob,
                         int32_t radius, const ff_match_params* p, const int32_t* proposal, int32_t* flow,
                         int32_t* cost, void* workspace, size_t workspace_bytes, hipStream_t stream) {
  if (!p) return FF_ERR_ARG;
  const ff_field_job j = single_job(src, src_blob, dst, dst_blob, radius, p, proposal, flow, cost);
  return ff_match_batch(&j, 1, p, workspace, workspace_bytes, stream);
}

ff_status ff_match_field_tree(const ff_desc* src, const void* src_blob, const ff_desc* dst, const void* dst_blob,
                              int32_t radius, const ff_match_params* p, void* workspace, size_t workspace_bytes,
                              hipStream_t stream) {
  if (!p || !workspace || !p->use_kdtree) return FF_ERR_ARG;
  ff_status st = check_params(src, dst, radius, p);
  if (st != FF_OK) return st;
  const ff_field_job j = single_job(src, src_blob, dst, dst_blob, radius, p, nullptr, nullptr, nullptr);
  if (!src_blob || !dst_blob) return FF_ERR_ARG;
  const BatchLayout B = batch_layout(&j, 1, p);
  if (workspace_bytes < B.bytes) return FF_ERR_WORKSPACE;
  st = ensure_init();
  if (st != FF_OK) return st;
  return run_batch(&j, 1, p, static_cast<char*>(workspace), B, stream, true);
}

ff_status ff_match_field_noalloc(const ff_desc* src, const void* src_blob, const ff_desc* dst, const void* dst_blob,
                                 int32_t radius, const ff_match_params* p, const int32_t* proposal, int32_t* flow,
                                 int32_t* cost, int32_t* status, hipStream_t stream) {
  // the library's scratch never holds a tree built ahead by ff_match_field_tree
  if (!p || p->use_kdtree == 2) return FF_ERR_ARG;
  ff_status st = check_params(src, dst, radius, p);
  if (st != FF_OK) return st;
  const ff_field_job j = single_job(src, src_blob, dst, dst_blob, radius, p, proposal, flow, cost);
  const BatchLayout B = batch_layout(&j, 1, p);
  const size_t counted = B.bytes - field_plan(src, dst, p).alt_past - B.launches * kUncountedWords;
  if (counted > FF_NOALLOC_SCRATCH_BYTES || B.bytes > kNoallocBytes) return FF_ERR_SIZE;
  st = check_job(j, p);
  if (st != FF_OK) return st;
  st = ensure_init();
  if (st != FF_OK) return st;
  char* ws = nullptr;
  st = noalloc_scratch(&ws);
  if (st != FF_OK) return st;
  st = run_batch(&j, 1, p, ws, B, stream);
  if (st != FF_OK) return st;
  if (status) {
    k_copy_status<<<1, 1, 0, stream>>>(reinterpret_cast<const int32_t*>(ws), status);
    return launch_status();
  }
  return FF_OK;
}

ff_status ff_read_status(const void* workspace, int32_t* status_host) {
  if (!workspace || !status_host) return FF_ERR_ARG;
  if (hipMemcpy(status_host, workspace, 4, hipMemcpyDeviceToHost) != hipSuccess) return FF_ERR_HIP;
  return FF_OK;
}

ff_status ff_build_kdtree(const ff_desc* d, const void* blob, int32_t radius, int32_t leaf, int32_t* node_dim,
                          int32_t* node_split, int32_t* perm, void* workspace, size_t workspace_bytes,
                          hipStream_t stream) {
  if (!d || !blob || !node_dim || !node_split || !perm || !workspace) return FF_ERR_ARG;
  if (leaf < 2 || leaf > kMaxLeaf) return FF_ERR_ARG;
  if (!wht_block(d, blob, radius)) return FF_ERR_ARG;
  ff_match_params p;
  ff_default_params(&p);
  p.k = 0;
  p.leaf = leaf;
  const ff_field_job j = single_job(d, blob, d, blob, radius, &p, nullptr, node_dim, node_split);
  const BatchLayout B = batch_layout(&j, 1, &p);
  if (workspace_bytes < B.bytes) return FF_ERR_WORKSPACE;
  ff_status st = ensure_init();
  if (st != FF_OK) return st;
  char* ws = static_cast<char*>(workspace);
  JobArray<FieldRec> recs;
  recs.resize(1);
  recs[0] = make_rec(j, &p, ws + B.off_field[0]);
  FieldRec* table = reinterpret_cast<FieldRec*>(ws + B.off_table);
  write_table(recs, 1, table, stream);
  st = enqueue_tree_build(table, 1, d->width * d->height, recs[0].t_top, leaf, stream);
  if (st != FF_OK) return st;
  const char* fws = ws + B.off_field[0];
  const int N = d->width * d->height;
  if (hipMemcpyAsync(node_dim, fws + recs[0].o_dim, (size_t)recs[0].t_nodes * 4, hipMemcpyDeviceToDevice, stream) !=
          hipSuccess ||
      hipMemcpyAsync(node_split, fws + recs[0].o_split, (size_t)recs[0].t_nodes * 4, hipMemcpyDeviceToDevice,
                     stream) != hipSuccess ||
      hipMemcpyAsync(perm, fws + recs[0].o_perm, (size_t)N * 4, hipMemcpyDeviceToDevice, stream) != hipSuccess)
    return FF_ERR_HIP;
  return FF_OK;
}

}  // extern "C"

// ---------------------------------------------------------------- load-latency probe
// One wavefront follows a cycle of indices through global memory (every
// lane the same one): every hop is one load whose address is the previous
// load's value, so a hop costs one dependent round trip to wherever the
// cycle's lines live.  A visit of a sweep's tile is such a chain (a step's
// result decides the next step's target addresses), so a visit takes at least
// this round trip times its steps.
namespace ff {
__global__ void k_chase(const int32_t* __restrict__ next, int32_t mask, int32_t warm, int32_t hops,
                        int64_t* __restrict__ out) {
  const __attribute__((address_space(1))) int32_t* p = gp(next);
  // a lane-varying start (0 in every lane of the one wavefront launched)
  // keeps the walk in vector registers, so every hop is a vector-memory load
  // through the vector L1 and the L2, the path of the sweep's target loads,
  // not a scalar-cache load
  int32_t i = (int32_t)(threadIdx.x >> 6);
  for (int h = 0; h < warm; ++h) i = p[i] & mask;
  // the clock is read once the warm walk's last load has returned, and again
  // once the timed walk's has (the asm consumes the index in a register)
  asm volatile("" ::"v"(i));
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  for (int h = 0; h < hops; ++h) i = p[i] & mask;
  asm volatile("" ::"v"(i));
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  const uint64_t t1 = __builtin_amdgcn_s_memrealtime();
  if (threadIdx.x == 0) {
    out[0] = (int64_t)(t1 - t0);
    out[1] = i;
  }
}
}  // namespace ff

extern "C" ff_status ff_probe_load_latency(const int32_t* next, int32_t n, int32_t warm, int32_t hops, int64_t* out,
                                           hipStream_t stream) {
  if (!next || !out || n < 2 || n > (1 << 28) || (n & (n - 1)) != 0) return FF_ERR_ARG;
  // at most 2^22 hops per walk: a few seconds even if every hop went to HBM
  if (hops < 1 || hops > (1 << 22) || warm < 0 || warm > (1 << 22)) return FF_ERR_ARG;
  k_chase<<<1, 64, 0, stream>>>(next, n - 1, warm, hops, out);
  return launch_status();
}
