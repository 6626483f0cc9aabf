// PCA of the SIFT vectors (section 3.3) on gfx950, fp64 throughout.
//
// Covariance: per-wavefront Gram sums on the fp64 matrix cores (upper half
// only), a fixed-order reduction, E[d d^T] - mean mean^T.
//
// Eigen-decomposition of the 128 x 128 covariance C.  One workgroup reduces C
// to tridiagonal form by Householder reflections with C in its registers
// (k_eig_tri); one wavefront per eigenvalue then brackets it by 64-way
// multisection of the Sturm count, takes its vector from the twisted
// factorisation (Fernando, "On computing an eigenvector of a tridiagonal
// matrix", 1997; Parlett and Dhillon, "Fernando's solution to Wilkinson's
// problem", 1997) and reflects it back (k_eig_vec); one step of the first-order
// correction of Ogita and Aishima ("Iterative refinement for symmetric
// eigenvalue decomposition", 2018) makes the basis orthogonal and the vectors
// accurate to rounding (k_eig_w, k_eig_s, k_eig_correct).  The step squares
// the basis' error, and its own size says whether that is enough: if a
// correction exceeds 1e-8 -- eigenvalues that coincide to rounding, where the
// vectors of the tridiagonal form are not even independent -- the one-sided
// Jacobi solver decides (k_sift_eig; it returns at once otherwise).
//
// Bound: the chains of one workgroup (126 reflections) and of a wavefront (the
// Sturm counts).  Measured: 0.26 + 0.13 + 0.06 ms where the Jacobi solver alone
// took 3.04 (12 sweeps of 127 rounds); the basis of a 640x480 pair is
// orthonormal to 9e-16 against 1e-13.
#include <algorithm>
#include <cmath>

#include "ff_device.h"
#include "ff_internal.h"

namespace ff {

constexpr double kCodeScale = 1024.0;
constexpr int kCodeMax = 2047;
constexpr int kDim = kSiftDim;
typedef double d4_t __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- covariance
// Rows of the two images' vectors stacked (image 1 first), four at a time: a
// lane holds columns 16 b + l % 16 of row l / 16 for the eight 16-column
// blocks b, which serve as both operands of the 36 products of the upper
// half (v_mfma_f64_16x16x4: 4 k-rows per instruction).  Two wavefronts share
// a run of rows, 18 tiles each (36 would not fit a wavefront's registers); a
// workgroup's four runs are summed in LDS.
// part: per workgroup 36 x 256 sums and the 128 column sums.
// Bound: the fp64 matrix rate.  Measured for 614,400 rows: 0.26 ms,
// 44 TFLOP/s of the upper half (both halves in vector instructions, 0.95 ms).
constexpr int kTilesU = 36;
constexpr int kPartDoubles = kTilesU * 256 + kDim;
constexpr int kGramWgs = 256, kGramRuns = 4;

__device__ __forceinline__ void tile_ij(int t, int& bi, int& bj) {
  bi = 0;
  while (t >= 8 - bi) {
    t -= 8 - bi;
    ++bi;
  }
  bj = bi + t;
}

template <int HALF>
__device__ __forceinline__ void gram_half(const float* __restrict__ D1, int N1, const float* __restrict__ D2, int N2,
                                          int r0, int rows, int run, double* sum) {
  constexpr int B0 = HALF ? 2 : 0, NT = kTilesU / 2;   // tiles 18.. lie in blocks 2..7
  const int lane = threadIdx.x & 63, kr = lane >> 4, col = lane & 15;
  d4_t acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = d4_t{0.0, 0.0, 0.0, 0.0};
  double msum[8];
#pragma unroll
  for (int b = 0; b < 8; ++b) msum[b] = 0.0;
  const int N = N1 + N2, r1 = min(N, r0 + rows);
  auto load = [&](int r, float (&x)[8]) {
    const int row = min(r + kr, N - 1);
    const float* src = row < N1 ? D1 + (size_t)row * kDim : D2 + (size_t)(row - N1) * kDim;
    const bool ok = r + kr < r1;
#pragma unroll
    for (int b = B0; b < 8; ++b) {
      const float v = src[16 * b + col];
      x[b] = ok ? v : 0.0f;
    }
  };
  float nx[8];
  if (r0 < r1) load(r0, nx);
  for (int r = r0; r < r1; r += 4) {
    double x[8];
#pragma unroll
    for (int b = B0; b < 8; ++b) x[b] = (double)nx[b];
    if (r + 4 < r1) load(r + 4, nx);
    int t = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = i; j < 8; ++j) {
        if (t / NT == HALF) acc[t % NT] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i], x[j], acc[t % NT], 0, 0, 0);
        ++t;
      }
    if (!HALF) {
#pragma unroll
      for (int b = 0; b < 8; ++b) msum[b] += x[b];
    }
  }
  // the runs in turn, so the order of the sums is fixed
  for (int w = 0; w < kGramRuns; ++w) {
    if (run == w) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          double* p = sum + (HALF * NT + t) * 256 + e * 64 + lane;
          *p = w == 0 ? acc[t][e] : *p + acc[t][e];
        }
      if (!HALF) {
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          double m = msum[b];   // rows 0..3 of this column: lanes 16 apart
          m += __shfl_xor(m, 16);
          m += __shfl_xor(m, 32);
          if (lane < 16) {
            double* p = sum + kTilesU * 256 + 16 * b + lane;
            *p = w == 0 ? m : *p + m;
          }
        }
      }
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(128 * kGramRuns) void k_sift_gram(const float* __restrict__ D1, int N1,
                                                               const float* __restrict__ D2, int N2, int rows,
                                                               double* __restrict__ part) {
  __shared__ double sum[kPartDoubles];
  const int wave = threadIdx.x >> 6, run = wave >> 1;
  const int r0 = (blockIdx.x * kGramRuns + run) * rows;
  if (wave & 1)
    gram_half<1>(D1, N1, D2, N2, r0, rows, run, sum);
  else
    gram_half<0>(D1, N1, D2, N2, r0, rows, run, sum);
  double* out = part + (size_t)blockIdx.x * kPartDoubles;
  for (int e = threadIdx.x; e < kPartDoubles; e += 128 * kGramRuns) out[e] = sum[e];
}

// fixed-order sum of the partials over N, into the full matrix E[d d^T]
// (row-major) and the mean after it; 64 sums per workgroup, four groups of
// partials each
__global__ __launch_bounds__(256) void k_sift_gram_reduce(const double* __restrict__ part, int nparts, int N,
                                                          double* __restrict__ raw) {
  __shared__ double s[4][64];
  const int g = threadIdx.x >> 6, l = threadIdx.x & 63, e = blockIdx.x * 64 + l;
  double a = 0.0;
  const int per = (nparts + 3) >> 2, p1 = min(nparts, (g + 1) * per);
#pragma unroll 8
  for (int p = g * per; p < p1; ++p) a += part[(size_t)p * kPartDoubles + e];
  s[g][l] = a;
  __syncthreads();
  if (g) return;
  const double v = (((s[0][l] + s[1][l]) + s[2][l]) + s[3][l]) / (double)N;
  if (e >= kTilesU * 256) {
    raw[kDim * kDim + e - kTilesU * 256] = v;
    return;
  }
  int bi, bj;
  tile_ij(e >> 8, bi, bj);
  // accumulator register q of lane l of a 16 x 16 tile: row l / 16 + 4 q, column l % 16
  const int q = (e >> 6) & 3, i = 16 * bi + (l >> 4) + 4 * q, j = 16 * bj + (l & 15);
  if (bi == bj && i > j) return;   // the lower triangle of a diagonal tile: its mirror writes it
  raw[i * kDim + j] = v;
  raw[j * kDim + i] = v;
}

// ---------------------------------------------------------------- eigen-decomposition
// scratch (doubles): C, reflectors V (row k: the k-th), tau, d, e (128 each),
// X (vectors of the tridiagonal form reflected back, columns descending), W =
// C X, S = X^T C X, R = I - X^T X, X' (corrected), and the largest
// off-diagonal |S|, largest |R| and largest correction (bit patterns of
// non-negative doubles, which order as integers)
constexpr int kMat = kDim * kDim;
struct EigScratch {
  double *C, *V, *tau, *d, *e, *X, *W, *S, *R, *X1;
  unsigned long long* mx;
};
__host__ __device__ inline EigScratch eig_scratch(double* p) {
  EigScratch s;
  s.C = p;
  s.V = s.C + kMat;
  s.X = s.V + kMat;
  s.W = s.X + kMat;
  s.S = s.W + kMat;
  s.R = s.S + kMat;
  s.X1 = s.R + kMat;
  s.tau = s.X1 + kMat;
  s.d = s.tau + kDim;
  s.e = s.d + kDim;
  s.mx = reinterpret_cast<unsigned long long*>(s.e + kDim);
  return s;
}
constexpr int kEigDoubles = 7 * kMat + 3 * kDim + 8;
constexpr double kMaxCorrection = 1e-8;   // its square is below rounding

__device__ __forceinline__ double readlane_f64(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
__device__ __forceinline__ double wave_sum_f64(double v) {
  v = row16_sum_f64(v);
  return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}
// 1 / q by two Newton steps on the hardware estimate (q finite, not 0)
__device__ __forceinline__ double rcp_f64(double q) {
  double y = __builtin_amdgcn_rcp(q);
  y = fma(y, fma(-q, y, 1.0), y);
  return fma(y, fma(-q, y, 1.0), y);
}

// Householder reduction to tridiagonal form.  Thread (r, s) holds row r,
// columns s + 8 m of the matrix in registers; a step's column (a row, the
// matrix being symmetric), the reflector's scalars and the product with it go
// through LDS, three barriers per step.  Step k leaves columns below 8 (k / 8) and rows up to k as
// they are (nothing reads them again): a wavefront whose eight rows are done
// only keeps the barriers.  Bound: the chain of 126 steps.  260 us with
// every column and wavefront in every step and the scalars in each of them,
// 187 without the finished ones, 182 now.
__global__ __launch_bounds__(1024) void k_eig_tri(const double* __restrict__ raw, double* __restrict__ scratch) {
  __shared__ double xs[2][kDim], ps[kDim], part[16], par[2];
  const EigScratch S = eig_scratch(scratch);
  const int tid = threadIdx.x, r = tid >> 3, s = tid & 7, lane = tid & 63;
  const int rlast = __builtin_amdgcn_readfirstlane(r | 7);   // of this wavefront
  const double* mean = raw + kMat;
  if (tid < 3) S.mx[tid] = 0ull;
  double a[16];
  const double mr = mean[r];
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    const int c = s + 8 * m;
    a[m] = raw[r * kDim + c] - mr * mean[c];
    S.C[r * kDim + c] = a[m];
  }
#pragma unroll
  for (int mk = 0; mk < 16; ++mk)
#pragma unroll 1
    for (int sk = 0; sk < 8; ++sk) {
      const int k = 8 * mk + sk;
      double* const x = xs[k & 1];
      if (s == sk) x[r] = a[mk];
      __syncthreads();
      if (k >= kDim - 2) {
        if (tid == kDim * 8 - 64) {
          S.d[k] = x[k];
          S.e[k] = k + 1 < kDim ? x[k + 1] : 0.0;
          S.tau[k] = 0.0;
        }
        continue;
      }
      // the last wavefront, which is on in every step, forms the reflector's
      // scalars once (a root and two quotients, which sixteen wavefronts would
      // queue for)
      if (r >= kDim - 8) {
        const double x0 = x[k + 1], x1 = x[lane], x2 = x[lane + 64];
        const double sig = wave_sum_f64((lane > k + 1 ? x1 * x1 : 0.0) + (lane + 64 > k + 1 ? x2 * x2 : 0.0));
        double beta = x0, tau = 0.0, sc = 0.0;
        if (sig > 0.0) {
          const double nrm = sqrt(fma(x0, x0, sig));
          beta = x0 > 0.0 ? -nrm : nrm;
          tau = (beta - x0) / beta;
          sc = 1.0 / (x0 - beta);
        }
        if (lane == 0) {
          par[0] = tau;
          par[1] = sc;
          S.d[k] = x[k];
          S.e[k] = beta;
          S.tau[k] = tau;
        }
      }
      __syncthreads();
      const double tau = par[0], sc = par[1];   // tau = 0: the column is reduced already
      const bool on = rlast > k && tau != 0.0;
      double vr = 0.0, vc[16], pr = 0.0;
      if (on) {
        auto vof = [&](int i) { return i > k + 1 ? x[i] * sc : (i == k + 1 ? 1.0 : 0.0); };
        vr = vof(r);
        double p = 0.0;
#pragma unroll
        for (int m = mk; m < 16; ++m) {
          vc[m] = vof(s + 8 * m);
          p = fma(a[m], vc[m], p);
        }
        // over the row's eight threads
        p += dpp_f64<0xB1>(p);
        p += dpp_f64<0x4E>(p);
        p += dpp_f64<0x141>(p);
        pr = tau * p;
        if (s == 0) ps[r] = pr;
      }
      // this wavefront's share of p v
      {
        double t = s == 0 ? pr * vr : 0.0;
        t = wave_sum_f64(t);
        if (lane == 0) part[tid >> 6] = t;
      }
      if (s == 0) S.V[k * kDim + r] = vr;
      __syncthreads();
      if (on) {
        const double K = 0.5 * tau * row16_sum_f64(part[lane & 15]);
        const double wr = fma(-K, vr, pr);
#pragma unroll
        for (int m = mk; m < 16; ++m) {
          const double wc = fma(-K, vc[m], ps[s + 8 * m]);
          a[m] = fma(-vr, wc, fma(-wr, vc[m], a[m]));
        }
      }
    }
}

// One wavefront per eigenvalue (ascending index i): 64 shifts per pass, ten
// passes (a 65th of the interval each); then the twisted factorisation of
// T - lambda (from the top in lane 0, from the bottom in lane 1), the vector
// outwards from the row with the smallest twist pivot, and the reflectors in
// reverse.  Column 127 - i of X.
__global__ __launch_bounds__(256) void k_eig_vec(double* __restrict__ scratch) {
  __shared__ double d[kDim], e[kDim];
  __shared__ double2 de[kDim], ed[kDim];   // d_j with e_(j-1)^2, and with e_j^2
  __shared__ double2 sc[kDim];             // de of the scaled form
  __shared__ double qf[4][kDim], qb[4][kDim], z[4][kDim];
  const EigScratch S = eig_scratch(scratch);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (threadIdx.x < kDim) {
    d[threadIdx.x] = S.d[threadIdx.x];
    e[threadIdx.x] = S.e[threadIdx.x];
    const int up = threadIdx.x > 0 ? threadIdx.x - 1 : 0;
    de[threadIdx.x] = make_double2(S.d[threadIdx.x], S.e[up] * S.e[up]);
    ed[threadIdx.x] = make_double2(S.d[threadIdx.x], S.e[threadIdx.x] * S.e[threadIdx.x]);
  }
  __syncthreads();
  const int i = blockIdx.x * 4 + wave;
  // Gershgorin interval
  auto edge = [&](int j) { return (j > 0 ? fabs(e[j - 1]) : 0.0) + (j < kDim - 1 ? fabs(e[j]) : 0.0); };
  double lo = fmin(d[lane] - edge(lane), d[lane + 64] - edge(lane + 64));
  double hi = fmax(d[lane] + edge(lane), d[lane + 64] + edge(lane + 64));
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o));
    hi = fmax(hi, __shfl_xor(hi, o));
  }
  const double wide = 1e-14 * fmax(fabs(lo), fabs(hi));
  lo -= wide;
  hi += wide;
  const double tiny = 1e-290;
  auto guard = [&](double q) { return fabs(q) < tiny ? -tiny : q; };
  // Eigenvalues below x: sign changes of the leading minors' determinants
  // p_j = (d_j - x) p_(j-1) - e_(j-1)^2 p_(j-2), one fused multiply-add of
  // latency per row (the quotients' recurrence has a reciprocal in it: 131 ->
  // 112 us).  T is scaled by a power of two to a radius of one, p every eight
  // rows: eight factors of at most 3, or down to 1e-19, stay in range.
  const double rad = fmax(fabs(lo), fabs(hi));
  const int ex = rad > 0.0 ? __builtin_amdgcn_frexp_exp(rad) : 0;
  lo = ldexp(lo, -ex);
  hi = ldexp(hi, -ex);
  if (threadIdx.x < kDim)
    sc[threadIdx.x] = make_double2(ldexp(de[threadIdx.x].x, -ex), ldexp(de[threadIdx.x].y, -2 * ex));
  __syncthreads();
  for (int pass = 0; pass < 10; ++pass) {
    const double step = (hi - lo) * (1.0 / 65.0), x = fma((double)(lane + 1), step, lo);
    double p0 = 0.0, p1 = 1.0;   // p_(j-2), p_(j-1)
    bool neg = false;            // the sign of p_(j-1); of zero, the opposite of the one before
    int cnt = 0;
#pragma unroll 1
    for (int j = 0; j < kDim; j += 8) {
      double2 t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = sc[j + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double p = fma(t[u].x - x, p1, -(t[u].y * p0));
        const bool n = p < 0.0 || (p == 0.0 && !neg);
        cnt += n != neg ? 1 : 0;
        neg = n;
        p0 = p1;
        p1 = p;
      }
      const double big = fmax(fabs(p0), fabs(p1));
      if (big == 0.0) {
        p1 = neg ? -1.0 : 1.0;
      } else {
        const int e0 = __builtin_amdgcn_frexp_exp(big);
        p0 = ldexp(p0, -e0);
        p1 = ldexp(p1, -e0);
      }
    }
    const uint64_t m = __ballot(cnt > i);
    const int f = m ? __ffsll((unsigned long long)m) - 1 : 64;
    const double nhi = f < 64 ? readlane_f64(x, f & 63) : hi;
    const double nlo = f > 0 ? readlane_f64(x, (f - 1) & 63) : lo;
    lo = nlo;
    hi = nhi;
  }
  const double lam = ldexp(0.5 * (lo + hi), ex);
  if (lane < 2) {
    const bool up = lane == 1;   // from the bottom
    double q = guard((up ? d[kDim - 1] : d[0]) - lam);
    double* const out = up ? qb[wave] : qf[wave];
    out[up ? kDim - 1 : 0] = q;
    const double2* const co = up ? ed : de;
#pragma unroll 1
    for (int t0 = 1; t0 < kDim; t0 += 8) {
      double2 t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = co[up ? max(kDim - 1 - t0 - u, 0) : min(t0 + u, kDim - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (t0 + u == kDim) break;
        q = guard((t[u].x - lam) - t[u].y * rcp_f64(q));
        out[up ? kDim - 1 - t0 - u : t0 + u] = q;
      }
    }
  }
  __syncthreads();
  double g = fabs((qf[wave][lane] + qb[wave][lane]) - (d[lane] - lam));
  int k = lane;
  {
    const double g2 = fabs((qf[wave][lane + 64] + qb[wave][lane + 64]) - (d[lane + 64] - lam));
    if (g2 < g) {
      g = g2;
      k = lane + 64;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const double og = __shfl_xor(g, o);
    const int ok = __shfl_xor(k, o);
    if (og < g || (og == g && ok < k)) {
      g = og;
      k = ok;
    }
  }
  __syncthreads();
  // ratios z_j / z_(j+1) above the twist, z_j / z_(j-1) below it
  for (int j = lane; j < kDim; j += 64) {
    qf[wave][j] = j < k ? -e[j] / qf[wave][j] : 1.0;
    if (j > k) qf[wave][j] = -e[j - 1] / qb[wave][j];
  }
  __syncthreads();
  if (lane < 2) {
    // lane 0 up from row k (the ratio there is 1), lane 1 down from it
    const int dir = lane == 0 ? -1 : 1, n = lane == 0 ? k + 1 : kDim - 1 - k;
    const int at = lane == 0 ? k : k + 1;
    double v = 1.0;
#pragma unroll 1
    for (int t0 = 0; t0 < n; t0 += 8) {
      double f[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) f[u] = qf[wave][at + dir * min(t0 + u, n - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        v *= f[u];
        if (t0 + u < n) z[wave][at + dir * (t0 + u)] = v;
      }
    }
  }
  __syncthreads();
  double z1 = z[wave][lane], z2 = z[wave][lane + 64];
  const double inv = 1.0 / sqrt(wave_sum_f64(fma(z1, z1, z2 * z2)));
  z1 *= inv;
  z2 *= inv;
  // reflect back, kAhead reflectors' loads in flight
  constexpr int kAhead = 14;
  static_assert((kDim - 2) % kAhead == 0, "whole rounds");
  double v1[kAhead], v2[kAhead], tq[kAhead];
  auto fetch = [&](int kk, int b) {
    const int c = kk < 0 ? 0 : kk;
    v1[b] = S.V[c * kDim + lane];
    v2[b] = S.V[c * kDim + 64 + lane];
    tq[b] = kk < 0 ? 0.0 : S.tau[c];
  };
#pragma unroll
  for (int b = 0; b < kAhead; ++b) fetch(kDim - 3 - b, b);
#pragma unroll 1
  for (int kk = kDim - 3; kk >= 0; kk -= kAhead) {
#pragma unroll
    for (int b = 0; b < kAhead; ++b) {
      if (tq[b] != 0.0) {   // uniform; no reflector was stored otherwise
        const double f = tq[b] * wave_sum_f64(fma(v1[b], z1, v2[b] * z2));
        z1 = fma(-f, v1[b], z1);
        z2 = fma(-f, v2[b], z2);
      }
      fetch(kk - kAhead - b, b);
    }
  }
  S.X[lane * kDim + kDim - 1 - i] = z1;
  S.X[(lane + 64) * kDim + kDim - 1 - i] = z2;
}

// 16 x 16 tiles of the products: grid (8, 8), one element per thread
__global__ __launch_bounds__(256) void k_eig_w(double* __restrict__ scratch) {   // W = C X
  __shared__ double A[16][kDim + 1], B[kDim][17];
  const EigScratch S = eig_scratch(scratch);
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4, i0 = 16 * blockIdx.y, j0 = 16 * blockIdx.x;
  for (int t = threadIdx.x; t < 16 * kDim; t += 256) {
    A[t >> 7][t & 127] = S.C[(i0 + (t >> 7)) * kDim + (t & 127)];
    B[t >> 4][t & 15] = S.X[(t >> 4) * kDim + j0 + (t & 15)];
  }
  __syncthreads();
  double w = 0.0;
#pragma unroll 16
  for (int k = 0; k < kDim; ++k) w = fma(A[ty][k], B[k][tx], w);
  S.W[(i0 + ty) * kDim + j0 + tx] = w;
}

__global__ __launch_bounds__(256) void k_eig_s(double* __restrict__ scratch) {   // S = X^T W, R = I - X^T X
  __shared__ double A[kDim][17], B[kDim][17], Y[kDim][17];
  const EigScratch S = eig_scratch(scratch);
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4, i0 = 16 * blockIdx.y, j0 = 16 * blockIdx.x;
  for (int t = threadIdx.x; t < 16 * kDim; t += 256) {
    const int k = t >> 4, c = t & 15;
    A[k][c] = S.X[k * kDim + i0 + c];
    B[k][c] = S.W[k * kDim + j0 + c];
    Y[k][c] = S.X[k * kDim + j0 + c];
  }
  __syncthreads();
  double s = 0.0, x = 0.0;
#pragma unroll 16
  for (int k = 0; k < kDim; ++k) {
    s = fma(A[k][ty], B[k][tx], s);
    x = fma(A[k][ty], Y[k][tx], x);
  }
  const int i = i0 + ty, j = j0 + tx;
  const double rr = (i == j ? 1.0 : 0.0) - x;
  S.S[i * kDim + j] = s;
  S.R[i * kDim + j] = rr;
  if (i != j) atomicMax(S.mx + 0, (unsigned long long)__double_as_longlong(fabs(s)));
  atomicMax(S.mx + 1, (unsigned long long)__double_as_longlong(fabs(rr)));
}

// X' = X + X E; E_ij = R_ij / 2 + (S_ij + (l_i + l_j) / 2 R_ij) / (l_j - l_i),
// the second part antisymmetric (S symmetrised, so exactly) and left out for
// pairs whose eigenvalues are closer than the matrices' errors
__device__ __forceinline__ double ritz(const EigScratch& S, int j) {
  return S.S[j * kDim + j] / (1.0 - S.R[j * kDim + j]);
}
__global__ __launch_bounds__(256) void k_eig_correct(double* __restrict__ scratch) {
  __shared__ double A[16][kDim + 1], E[kDim][17], l[kDim];
  const EigScratch S = eig_scratch(scratch);
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4, i0 = 16 * blockIdx.y, j0 = 16 * blockIdx.x;
  if (threadIdx.x < kDim) l[threadIdx.x] = ritz(S, threadIdx.x);
  __syncthreads();
  double lmax = 0.0;
  for (int k = 0; k < kDim; ++k) lmax = fmax(lmax, fabs(l[k]));
  const double off = __longlong_as_double((long long)S.mx[0]), rmx = __longlong_as_double((long long)S.mx[1]);
  const double near = 2.0 * kDim * (off + lmax * rmx);
  double emx = 0.0;
  bool nan = false;
  for (int t = threadIdx.x; t < 16 * kDim; t += 256) {
    A[t >> 7][t & 127] = S.X[(i0 + (t >> 7)) * kDim + (t & 127)];
    const int i = t >> 4, j = j0 + (t & 15);
    const double rr = S.R[i * kDim + j], gap = l[j] - l[i];
    double x = 0.5 * rr;
    if (i != j && fabs(gap) > near)
      x += (0.5 * (S.S[i * kDim + j] + S.S[j * kDim + i]) + 0.5 * (l[i] + l[j]) * rr) / gap;
    E[i][t & 15] = x;
    emx = fmax(emx, fabs(x));
    nan |= !(fabs(x) < 1.0);
  }
  if (nan) emx = 1.0;
  for (int o = 32; o > 0; o >>= 1) emx = fmax(emx, __shfl_xor(emx, o));
  if ((threadIdx.x & 63) == 0) atomicMax(S.mx + 2, (unsigned long long)__double_as_longlong(emx));
  __syncthreads();
  double x = 0.0;
#pragma unroll 16
  for (int k = 0; k < kDim; ++k) x = fma(A[ty][k], E[k][tx], x);
  S.X1[(i0 + ty) * kDim + j0 + tx] = A[ty][j0 + tx] + x;
}

__device__ __forceinline__ bool eig_corrected(const EigScratch& S) {
  return __longlong_as_double((long long)S.mx[2]) < kMaxCorrection;
}

// mean, eigenvalues descending (ties by index), each vector's
// largest-magnitude component (the first on ties) positive
__global__ __launch_bounds__(1024) void k_eig_out(const double* __restrict__ raw, double* __restrict__ scratch,
                                                  double* __restrict__ out) {
  __shared__ double l[kDim];
  const EigScratch S = eig_scratch(scratch);
  if (!eig_corrected(S)) return;   // the Jacobi solver's
  // eight threads per column
  const int t = threadIdx.x >> 3, q = threadIdx.x & 7;
  if (q == 0) {
    const double v = ritz(S, t);
    l[t] = v > 0.0 ? v : 0.0;   // C is positive semi-definite
    out[t] = raw[kMat + t];
  }
  __syncthreads();
  const double lt = l[t];
  int rank = 0;
  for (int j = q; j < kDim; j += 8) rank += (l[j] > lt || (l[j] == lt && j < t)) ? 1 : 0;
  rank += __shfl_xor(rank, 1);
  rank += __shfl_xor(rank, 2);
  rank += __shfl_xor(rank, 4);
  double best = -1.0, val = 0.0;
  int bm = 0;
  for (int k = q; k < kDim; k += 8) {
    const double x = S.X1[k * kDim + t];
    if (fabs(x) > best) {
      best = fabs(x);
      val = x;
      bm = k;
    }
  }
  for (int o = 1; o < 8; o <<= 1) {
    const double ob = __shfl_xor(best, o), ov = __shfl_xor(val, o);
    const int om = __shfl_xor(bm, o);
    if (ob > best || (ob == best && om < bm)) {
      best = ob;
      val = ov;
      bm = om;
    }
  }
  if (q == 0) out[kDim + rank] = lt;
  for (int k = q; k < kDim; k += 8) {
    const double x = S.X1[k * kDim + t];
    out[2 * kDim + k * kDim + rank] = val < 0.0 ? -x : x;
  }
}

// ---------------------------------------------------------------- one-sided Jacobi eigen-solver
// For covariances whose eigenvalues coincide to rounding (constant images,
// fewer distinct vectors than dimensions).
// The covariance C (128 x 128, positive semi-definite) is orthogonalised by
// one-sided (Hestenes) Jacobi rotations of its columns, M <- M J with M = C
// at the start: a pair of columns (p, q) with norms a = |m_p|^2, b = |m_q|^2
// and product g = m_p . m_q is rotated by the angle that makes them
// orthogonal (zeta = (b - a) / (2 g), t = sign(zeta) / (|zeta| +
// sqrt(1 + zeta^2)), c = 1 / sqrt(1 + t^2), s = t c).  At convergence M = C V
// with orthogonal columns, so C^2 is diagonal in V and column i is
// lambda_i v_i: the eigenvalues are the column norms and the eigenvectors
// the normalised columns -- no rotation product is accumulated, and the
// whole matrix stays in LDS.  A sweep is 127 rounds of the round-robin
// tournament, 64 disjoint pairs per round, 16 lanes per pair (dot products
// by DPP row sums, one barrier per round).  Pairs whose columns are already
// orthogonal to 1e-13 of their norms, or whose rotation angle is below
// 1e-15 (no change beyond rounding), are left alone; sweeps stop when none is
// rotated (or after 30).  Eigenvalues are then ranked descending (ties by
// index), each eigenvector's largest-magnitude component (the first on
// ties) is made positive, and out receives mean (128), eigenvalues (128) and
// the basis (128 x 128, element [k][s] = component k of eigenvector s).
constexpr int kMP = kSiftDim + 2;   // LDS row pitch (doubles): the 4 pairs of a wavefront in different banks
constexpr int kJacobiSweeps = 30;
constexpr double kOrthTol = 1e-13;
constexpr double kMinAngle = 1e-15;

__device__ __forceinline__ void tourney(int round, int k, int& p, int& q) {
  // circle method: player 0 fixed, players 1..127 rotate
  auto pos = [&](int i) { return 1 + (i + round) % 127; };
  if (k == 0) {
    p = 0;
    q = pos(0);
  } else {
    p = pos(k);
    q = pos(127 - k);
  }
}

__global__ __launch_bounds__(1024) void k_sift_eig(const double* __restrict__ raw, double* __restrict__ scratch,
                                                   double* __restrict__ out) {
  __shared__ double Mt[kSiftDim * kMP];   // row i = column i of M
  __shared__ int s_rot[16];
  __shared__ double s_norm[kSiftDim];
  __shared__ int s_rank[kSiftDim];
  if (eig_corrected(eig_scratch(scratch))) return;
  const int t = threadIdx.x;
  const double* mean = raw + kSiftDim * kSiftDim;
  for (int e = t; e < kSiftDim * kSiftDim; e += 1024) {
    const int i = e >> 7, j = e & 127;
    Mt[i * kMP + j] = raw[e] - mean[i] * mean[j];
  }
  __syncthreads();
  const int g = t >> 4, l = t & 15;
  for (int sweep = 0; sweep < kJacobiSweeps; ++sweep) {
    int rotated = 0;
    for (int round = 0; round < 127; ++round) {
      int p, q;
      tourney(round, g, p, q);
      double* mp = Mt + p * kMP;
      double* mq = Mt + q * kMP;
      double x[8], y[8];
      double a = 0.0, b = 0.0, c = 0.0;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        x[i] = mp[l + 16 * i];
        y[i] = mq[l + 16 * i];
        a = fma(x[i], x[i], a);
        b = fma(y[i], y[i], b);
        c = fma(x[i], y[i], c);
      }
      a = row16_sum_f64(a);   // the pair's 16 lanes are one DPP row
      b = row16_sum_f64(b);
      c = row16_sum_f64(c);
      if (fabs(c) > kOrthTol * sqrt(a * b)) {   // the same in all 16 lanes of the pair
        const double zeta = (b - a) / (2.0 * c);
        const double tt = (zeta >= 0.0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
        // a rotation by less than the rounding of the columns changes
        // nothing (pairs with a column at rounding level stay there)
        if (fabs(tt) > kMinAngle) {
          const double cs = 1.0 / sqrt(1.0 + tt * tt), sn = tt * cs;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            mp[l + 16 * i] = cs * x[i] - sn * y[i];
            mq[l + 16 * i] = sn * x[i] + cs * y[i];
          }
          rotated = 1;
        }
      }
      __syncthreads();
    }
    // any rotation in this sweep?
    const int any = __any(rotated) ? 1 : 0;
    if ((t & 63) == 0) s_rot[t >> 6] = any;
    __syncthreads();
    int tot = 0;
    for (int w = 0; w < 16; ++w) tot |= s_rot[w];
    __syncthreads();
    if (!tot) break;
  }
  if (t < kSiftDim) {
    double nn = 0.0;
    for (int k = 0; k < kSiftDim; ++k) nn = fma(Mt[t * kMP + k], Mt[t * kMP + k], nn);
    s_norm[t] = sqrt(nn);
  }
  __syncthreads();
  if (t < kSiftDim) {
    const double li = s_norm[t];
    int rank = 0;
    for (int j = 0; j < kSiftDim; ++j) {
      const double lj = s_norm[j];
      rank += (lj > li || (lj == li && j < t)) ? 1 : 0;
    }
    s_rank[t] = rank;
    out[t] = mean[t];
    out[kSiftDim + rank] = li;
  }
  __syncthreads();
  if (t < kSiftDim) {
    // column t of M becomes basis column s_rank[t]
    const double* v = Mt + t * kMP;
    int m = 0;
    double best = fabs(v[0]);
    for (int k = 1; k < kSiftDim; ++k)
      if (fabs(v[k]) > best) {
        best = fabs(v[k]);
        m = k;
      }
    const double inv = s_norm[t] > 0.0 ? (v[m] < 0.0 ? -1.0 : 1.0) / s_norm[t] : 0.0;
    const int s = s_rank[t];
    for (int k = 0; k < kSiftDim; ++k) out[2 * kSiftDim + k * kSiftDim + s] = v[k] * inv;
  }
}

// ---------------------------------------------------------------- projection to codes
// (d - mean) . basis on the fp64 matrix cores, 16 pixels per wavefront and
// step: lane l holds elements 16 g + 4 (l / 16) + c of pixel l % 16 (one
// 16-byte load per g), so instruction (g, c) takes k-row l / 16 from element
// 16 g + 4 (l / 16) + c on both operands.  The basis columns (NT tiles of 16,
// zeros past S) stay in registers.  Codes round-half-even(1024 c) clamped to
// +-2047, H x W x S int16.
// Bound: the fp64 matrix rate.  Measured for S = 18, 307,200 pixels: 58 us
// (one thread per pixel, its vector read in 32 strided pieces: 185).
template <int NT>
__global__ __launch_bounds__(256) void k_sift_project(const float* __restrict__ D, int N, const double* __restrict__ pca,
                                                      int S, int groups, int16_t* __restrict__ codes) {
  const int lane = threadIdx.x & 63, kr = lane >> 4, col = lane & 15;
  double bs[8][4][NT], mu[8][4];
#pragma unroll
  for (int g = 0; g < 8; ++g)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int k = 16 * g + 4 * kr + c;
      mu[g][c] = pca[k];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int s = 16 * t + col;
        bs[g][c][t] = s < S ? pca[2 * kDim + k * kDim + s] : 0.0;
      }
    }
  const int nw = gridDim.x * 4;
  for (int w = blockIdx.x * 4 + (threadIdx.x >> 6); w < groups; w += nw) {
    const int p = min(w * 16 + col, N - 1);
    const float4* src = reinterpret_cast<const float4*>(D + (size_t)p * kDim) + kr;
    float4 v[8];
#pragma unroll
    for (int g = 0; g < 8; ++g) v[g] = src[4 * g];
    d4_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const float x[4] = {v[g].x, v[g].y, v[g].z, v[g].w};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double a = (double)x[c] - mu[g][c];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bs[g][c][t], acc[t], 0, 0, 0);
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int px = w * 16 + kr + 4 * q, s = 16 * t + col;
        if (px < N && s < S) {
          const double r = rint(acc[t][q] * kCodeScale);
          codes[(size_t)px * S + s] = (int16_t)(r > kCodeMax ? kCodeMax : (r < -kCodeMax ? -kCodeMax : (int)r));
        }
      }
  }
}

void enqueue_project(const float* D, int N, const double* pca, int S, int16_t* codes, hipStream_t stream) {
  const int groups = (N + 15) / 16;
  const unsigned g = (unsigned)std::min((groups + 3) / 4, 256 * 2);
  if (S <= 16)
    k_sift_project<1><<<g, 256, 0, stream>>>(D, N, pca, S, groups, codes);
  else
    k_sift_project<2><<<g, 256, 0, stream>>>(D, N, pca, S, groups, codes);
}

size_t pca_scratch_bytes() { return ((size_t)kGramWgs * kPartDoubles + kMat + kDim + kEigDoubles) * 8; }

void enqueue_pca(const float* D1, int N1, const float* D2, int N2, double* scratch, double* out, hipStream_t stream) {
  double* part = scratch;
  double* raw = part + (size_t)kGramWgs * kPartDoubles;
  double* eig = raw + kMat + kDim;
  const int N = N1 + N2;
  // whole chip, at least eight steps of four rows per run
  const int runs = kGramRuns * kGramWgs;
  const int rows = std::max(32, ((N + runs - 1) / runs + 3) / 4 * 4);
  const int wgs = (N + kGramRuns * rows - 1) / (kGramRuns * rows);
  k_sift_gram<<<wgs, 128 * kGramRuns, 0, stream>>>(D1, N1, D2, N2, rows, part);
  k_sift_gram_reduce<<<kPartDoubles / 64, 256, 0, stream>>>(part, wgs, N, raw);
  k_eig_tri<<<1, 1024, 0, stream>>>(raw, eig);
  k_eig_vec<<<kDim / 4, 256, 0, stream>>>(eig);
  k_eig_w<<<dim3(8, 8), 256, 0, stream>>>(eig);
  k_eig_s<<<dim3(8, 8), 256, 0, stream>>>(eig);
  k_eig_correct<<<dim3(8, 8), 256, 0, stream>>>(eig);
  k_eig_out<<<1, 1024, 0, stream>>>(raw, eig, out);
  k_sift_eig<<<1, 1024, 0, stream>>>(raw, eig, out);
}

}  // namespace ff
