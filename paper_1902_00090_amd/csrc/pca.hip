// Principal-component basis of solution snapshots (Sec. 3, PCA paragraph) and
// the batched projection loss (Sec. 3, eq:proj_loss).
//
// The basis is the leading left singular vectors of the snapshot matrix
// X = [s_1 .. s_M] whose columns are field vectors (uncentred).  With the
// snapshots stored as M rows of D elements, G = X^H X (G_ab = <s_a, s_b>) is
// formed on the device in FP64; its leading eigenpairs (sigma_i^2, w_i) come
// from a Lanczos iteration with full reorthogonalisation (FP64; on the device
// from 128 snapshots on, the small tridiagonal problem on the host); u_i =
// X w_i / sigma_i is formed on the device and the basis is re-orthonormalised by
// one Cholesky QR pass.
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstring>
#include <random>
#include <vector>

#include "common.h"
#include "devbuf.h"
#include "gram.h"

#define DD_MAX_KPCA 64

using cd = std::complex<double>;

// ------------------------------------------------------------ device Gram ----
// G_ab = sum_e conj(S[a][e]) S[b][e] for a square tile of snapshot pairs (only
// tiles on and above the diagonal) over one slice of the elements, on the FP64
// matrix cores: the real part is re^T re + im^T im, the imaginary part re^T im -
// im^T re, four 16x16x4 products for four elements.  Four waves a workgroup, each
// B x B blocks of 16 x 16; 32 elements a stage, the next stage's loads in
// flight during the products.  Bound by the matrix cores: each LDS value feeds
// 16 B products.  Measured for 1000 snapshots of 115,200 elements: 30.2 ms with
// a 2 x 2 block of FP64 vector sums a thread, 8.9 here (0.46 TFLOP; a library
// product of 4096 x 4096 FP64 matrices runs at 64 TFLOP/s).
typedef double v4d __attribute__((ext_vector_type(4)));
#define PE 32
template <int B>
__global__ __launch_bounds__(256) void k_pca_gram(const float2* __restrict__ S, int M, int D,
                                                  int per, double2* __restrict__ part) {
  constexpr int TILE = 32 * B, LD = TILE * PE / 256;
  // tile (ta, tb), tb >= ta, of the triangle's list
  int ta = 0, rest = blockIdx.x;
  const int nta = (M + TILE - 1) / TILE;
  while (rest >= nta - ta) rest -= nta - ta++;
  const int tb = ta + rest;
  const bool diag = ta == tb;
  const int e0 = blockIdx.y * per, e1 = min(D, e0 + per);
  __shared__ float2 sa[TILE][PE + 1], sb[TILE][PE + 1];
  const int t = threadIdx.x, lane = t & 63, wr = (t >> 6) >> 1, wc = (t >> 6) & 1;
  const int li = lane & 15, lk = lane >> 4;
  v4d ar[B][B], ai[B][B];
#pragma unroll
  for (int i = 0; i < B; ++i)
#pragma unroll
    for (int j = 0; j < B; ++j) ar[i][j] = ai[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  float2 na[LD], nb[LD];
  const float2 zero = make_float2(0.f, 0.f);
  auto fetch = [&](int eb) {
#pragma unroll
    for (int q = 0; q < LD; ++q) {
      const int r = (t + 256 * q) / PE, e = eb + (t + 256 * q) % PE;
      const int a = ta * TILE + r, b = tb * TILE + r;
      na[q] = (a < M && e < e1) ? S[(size_t)a * D + e] : zero;
      if (!diag) nb[q] = (b < M && e < e1) ? S[(size_t)b * D + e] : zero;
    }
  };
  fetch(e0);
  const float2(*pb)[PE + 1] = diag ? sa : sb;
  for (int eb = e0; eb < e1; eb += PE) {
#pragma unroll
    for (int q = 0; q < LD; ++q) {
      const int r = (t + 256 * q) / PE, c = (t + 256 * q) % PE;
      sa[r][c] = na[q];
      if (!diag) sb[r][c] = nb[q];
    }
    __syncthreads();
    if (eb + PE < e1) fetch(eb + PE);
#pragma unroll
    for (int kk = 0; kk < PE; kk += 4) {
      double xr[B], xi[B], yr[B], yi[B];
#pragma unroll
      for (int i = 0; i < B; ++i) {
        const float2 x = sa[(wr * B + i) * 16 + li][kk + lk];
        const float2 y = pb[(wc * B + i) * 16 + li][kk + lk];
        xr[i] = x.x; xi[i] = x.y;
        yr[i] = y.x; yi[i] = y.y;
      }
#pragma unroll
      for (int i = 0; i < B; ++i)
#pragma unroll
        for (int j = 0; j < B; ++j) {
          ar[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[i], yr[j], ar[i][j], 0, 0, 0);
          ai[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[i], yi[j], ai[i][j], 0, 0, 0);
          ar[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(xi[i], yi[j], ar[i][j], 0, 0, 0);
          ai[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-xi[i], yr[j], ai[i][j], 0, 0, 0);
        }
    }
    __syncthreads();
  }
  // the row and column of each result value in a 16 x 16 block, from products
  // with the row and column numbers
  const v4d none = {0.0, 0.0, 0.0, 0.0};
  const double one = lk == 0 ? 1.0 : 0.0, num = lk == 0 ? (double)li : 0.0;
  const v4d rows = __builtin_amdgcn_mfma_f64_16x16x4f64(num, one, none, 0, 0, 0);
  const v4d cols = __builtin_amdgcn_mfma_f64_16x16x4f64(one, num, none, 0, 0, 0);
  double2* out = part + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * TILE * TILE;
#pragma unroll
  for (int i = 0; i < B; ++i)
#pragma unroll
    for (int j = 0; j < B; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        out[((wr * B + i) * 16 + (int)rows[v]) * TILE + (wc * B + j) * 16 + (int)cols[v]] =
            make_double2(ar[i][j][v], ai[i][j][v]);
}

// G (M x M, row-major, full Hermitian) from the slice partials in a fixed
// order: 64 entries of a tile a workgroup, four threads an entry (a quarter of
// the slices each, eight loads in flight).  bad (if given): set if a sum is not finite.
__global__ __launch_bounds__(256) void k_pca_gram_reduce(const double2* __restrict__ part, int M,
                                                         int tile, int nslices,
                                                         double2* __restrict__ G,
                                                         int* __restrict__ bad) {
  int ta = 0, rest = blockIdx.x;
  const int nta = (M + tile - 1) / tile, ntiles = nta * (nta + 1) / 2;
  while (rest >= nta - ta) rest -= nta - ta++;
  const int tb = ta + rest, i = blockIdx.y * 64 + (threadIdx.x & 63), q = threadIdx.x >> 6;
  const double2* src = part + (size_t)blockIdx.x * tile * tile + i;
  const size_t ld = (size_t)ntiles * tile * tile;
  double sx = 0.0, sy = 0.0;
  for (int s = q; s < nslices; s += 32) {
    double2 v[8];
#pragma unroll
    for (int r = 0; r < 8; ++r)
      v[r] = (s + 4 * r < nslices) ? src[(size_t)(s + 4 * r) * ld] : make_double2(0.0, 0.0);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      sx += v[r].x;
      sy += v[r].y;
    }
  }
  __shared__ double2 sum[4][64];
  sum[q][threadIdx.x & 63] = make_double2(sx, sy);
  __syncthreads();
  if (q != 0) return;
  const int l = threadIdx.x;
  sx = (sum[0][l].x + sum[1][l].x) + (sum[2][l].x + sum[3][l].x);
  sy = (sum[0][l].y + sum[1][l].y) + (sum[2][l].y + sum[3][l].y);
  const int a = ta * tile + i / tile, b = tb * tile + i % tile;
  if (a >= M || b >= M) return;
  if (bad && (!isfinite(sx) || !isfinite(sy))) atomicOr(bad, 1);
  // a diagonal tile holds both halves; its own lower one is left to the upper
  if (a > b) return;
  G[(size_t)a * M + b] = make_double2(sx, a == b ? 0.0 : sy);
  if (a < b) G[(size_t)b * M + a] = make_double2(sx, -sy);
}

// out[r][e] = sum_m coef[m][r] F[m][e] for R rows (coef: FP64, [M][R]) on the FP64
// matrix cores.  A workgroup takes 32 rows and 128 elements, a wave 32 of them;
// a step is four vectors m.  The fields are read once per 32 rows, 128 bytes a
// vector and half wave, the coefficients from the L2; both straight into the
// operands, two steps at a time.  step, window: rows [s step, (s + 1) step) take
// only the vectors within `window` of s (their other coefficients are zero); step = 0:
// all vectors.  Measured at 115,200 elements: 20 rows from 1000 vectors 1.21 ms
// as FP64 vector sums with 16 rows a thread (2.07 with 24 and scalar loads), 0.64
// here; 320 rows from 17 of 32 vectors each 2.45 ms, 0.15 ms here, of which 0.06 ms
// are the result's bytes.
__global__ __launch_bounds__(256) void k_field_combine(const float2* __restrict__ F, int M, int D,
                                                       const double2* __restrict__ coef, int R,
                                                       int step, int window,
                                                       const int* __restrict__ bad,
                                                       float2* __restrict__ out) {
  // a field that is not finite makes every target so, as its zero coefficients do
  if (bad && *bad) step = 0;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int r0 = blockIdx.y * 32, e0 = blockIdx.x * 128 + (threadIdx.x >> 6) * 32;
  int lo = 0, hi = M;
  if (step > 0) {
    lo = max(0, r0 / step - window);
    hi = min(M, min(r0 + 31, R - 1) / step + window + 1);
  }
  const v4d none = {0.0, 0.0, 0.0, 0.0};
  v4d ar[2][2], ai[2][2];             // [rows][elements]
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) ar[i][j] = ai[i][j] = none;
  int col[2], el[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    col[i] = min(r0 + 16 * i + li, R - 1);
    el[i] = min(e0 + 16 * i + li, D - 1);
  }
  auto fetch = [&](int m0, float2 (&f)[2][2], double2 (&c)[2][2]) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int m = m0 + 4 * u + lk, mc = min(m, hi - 1);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        f[u][i] = F[(size_t)mc * D + el[i]];
        c[u][i] = coef[(size_t)mc * R + col[i]];
      }
      if (m >= hi) c[u][0] = c[u][1] = make_double2(0.0, 0.0);
    }
  };
  float2 f[2][2], fn[2][2];
  double2 c[2][2], cn[2][2];
  fetch(lo, fn, cn);
  for (int m0 = lo; m0 < hi; m0 += 8) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        f[u][i] = fn[u][i];
        c[u][i] = cn[u][i];
      }
    fetch(min(m0 + 8, hi - 1), fn, cn);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const double fx = f[u][j].x, fy = f[u][j].y;
          ar[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[u][i].x, fx, ar[i][j], 0, 0, 0);
          ai[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[u][i].x, fy, ai[i][j], 0, 0, 0);
          ar[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-c[u][i].y, fy, ar[i][j], 0, 0, 0);
          ai[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[u][i].y, fx, ai[i][j], 0, 0, 0);
        }
  }
  // row and column of the result values, as in k_pca_gram
  const double one = lk == 0 ? 1.0 : 0.0, num = lk == 0 ? (double)li : 0.0;
  const v4d rows = __builtin_amdgcn_mfma_f64_16x16x4f64(num, one, none, 0, 0, 0);
  const v4d cols = __builtin_amdgcn_mfma_f64_16x16x4f64(one, num, none, 0, 0, 0);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = r0 + 16 * i + (int)rows[v], e = e0 + 16 * j + (int)cols[v];
        if (r < R && e < D)
          out[(size_t)r * D + e] = make_float2((float)ar[i][j][v], (float)ai[i][j][v]);
      }
}

// Coefficients of local_pca_targets, one workgroup per step s: the eigenvectors of
// the Gram matrix G_ab = <F_a, F_b> / (||F_a|| ||F_b||) of the M <= 32 fields of the
// step's window, by Jacobi rotations in LDS, M / 2 disjoint ones at a time (the
// circle method's rounds).  A round's rotations are formed by one thread each; then
// every thread transforms the 2 x 2 blocks G[{p,q},{r,t}] on both sides, in place,
// and the pairs of columns of W.  Sweeps go on until one meets no element above
// rounding.  With G w_j = theta_j w_j, u_j = sum_m w_mj F_m / (||F_m|| sigma_j) has
// u_j^H F_s / ||F_s|| = sigma_j conj(w_sj), and target j is the combination of the
// fields with coefficients w_mj conj(w_sj) / ||F_m||.  A chain of latencies: about
// 130 rounds of two barriers each for 17 fields, all steps at once; 32 steps 139 us
// (on the host one after the other 520 us, with two copies and waits).
#define PJ_MAX 32
__global__ __launch_bounds__(256) void k_window_coefs(const double2* __restrict__ G0, int S,
                                                      int window, int k,
                                                      double2* __restrict__ coef) {
  __shared__ double2 G[PJ_MAX][PJ_MAX + 1], W[PJ_MAX][PJ_MAX + 1];   // columns over the banks
  __shared__ double2 ph[PJ_MAX / 2];       // conj of the phase of G_pq
  __shared__ double cs[PJ_MAX / 2], sn[PJ_MAX / 2], nrm[PJ_MAX];
  __shared__ int pr[PJ_MAX / 2][2];        // the round's pairs
  __shared__ int again, broken, order[PJ_MAX];
  const int t = threadIdx.x, s = blockIdx.x;
  const int lo = max(0, s - window), hi = min(S, s + window + 1), M = hi - lo, N = (M + 1) & ~1;
  const int kk = min(k, M);
  if (t == 0) broken = 0;
  if (t < M) {
    const double g = G0[(size_t)(lo + t) * S + lo + t].x;
    nrm[t] = sqrt(g < 1e-300 ? 1e-300 : g);
  }
  __syncthreads();
  // an odd M gets a row and a column of zeros, which no rotation touches
  for (int i = t; i < N * N; i += 256) {
    const int a = i / N, b = i - a * N;
    double2 g = make_double2(0.0, 0.0);
    if (a < M && b < M) {
      g = G0[(size_t)(lo + a) * S + lo + b];
      if (!isfinite(g.x) || !isfinite(g.y)) broken = 1;
      const double q = nrm[a] * nrm[b];
      g = make_double2(g.x / q, g.y / q);
    }
    G[a][b] = g;
    W[a][b] = make_double2(a == b ? 1.0 : 0.0, 0.0);
  }
  __syncthreads();
  const double tiny = 0x1p-54 * M;          // against the trace
  const int np = N / 2, n = N - 1;
  // this thread's items of a round: block (u, v) of G, or row u of pair v of W
  constexpr int NIT = (PJ_MAX / 2) * (PJ_MAX / 2 + PJ_MAX) / 256;
  int iu[NIT], iv[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int i = t + 256 * it, l = i - np * np;
    iu[it] = l < 0 ? i / np : l % N;
    iv[it] = l < 0 ? i % np : l / N;
  }
  for (int sweep = 0; sweep < 30 && !broken; ++sweep) {
    if (t == 0) again = 0;
    for (int r = 0; r < n; ++r) {
      __syncthreads();
      if (t < np) {
        // pair t of round r of the circle method on N players
        int p = r + t, q = r - t;
        p = t == 0 ? r : (p >= n ? p - n : p);
        q = t == 0 ? n : (q < 0 ? q + n : q);
        if (p > q) {
          const int x = p;
          p = q;
          q = x;
        }
        const double2 g = G[p][q];
        const double a = sqrt(g.x * g.x + g.y * g.y);
        double c = 1.0, sv = 0.0;
        double2 e = make_double2(1.0, 0.0);
        if (a > 1e-40) {
          if (a > tiny) again = 1;
          const double ia = 1.0 / a, tau = 0.5 * (G[q][q].x - G[p][p].x) * ia;
          const double tn = copysign(1.0, tau) / (fabs(tau) + sqrt(1.0 + tau * tau));
          c = 1.0 / sqrt(1.0 + tn * tn);
          sv = tn * c;
          e = make_double2(g.x * ia, -g.y * ia);
        }
        cs[t] = c;
        sn[t] = sv;
        ph[t] = e;
        pr[t][0] = p;
        pr[t][1] = q;
      }
      __syncthreads();
      // columns: x' = c x - s e y, y' = s x + c e y, with e = conj(phase)
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int i = t + 256 * it, u = iu[it], v = iv[it];
        if (i >= np * np + N * np) break;
        const int a = pr[v][0], b = pr[v][1];
        if (i < np * np) {
          const int p = pr[u][0], q = pr[u][1];
          const double c1 = cs[u], s1 = sn[u], c2 = cs[v], s2 = sn[v];
          const double2 e1 = ph[u], e2 = ph[v];
          double2 z[2][2] = {{G[p][a], G[p][b]}, {G[q][a], G[q][b]}};
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const double2 x = z[h][0], y = make_double2(e2.x * z[h][1].x - e2.y * z[h][1].y,
                                                        e2.x * z[h][1].y + e2.y * z[h][1].x);
            z[h][0] = make_double2(c2 * x.x - s2 * y.x, c2 * x.y - s2 * y.y);
            z[h][1] = make_double2(s2 * x.x + c2 * y.x, s2 * x.y + c2 * y.y);
          }
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const double2 x = z[0][h], y = make_double2(e1.x * z[1][h].x + e1.y * z[1][h].y,
                                                        e1.x * z[1][h].y - e1.y * z[1][h].x);
            z[0][h] = make_double2(c1 * x.x - s1 * y.x, c1 * x.y - s1 * y.y);
            z[1][h] = make_double2(s1 * x.x + c1 * y.x, s1 * x.y + c1 * y.y);
          }
          if (u == v) {
            z[0][1] = z[1][0] = make_double2(0.0, 0.0);
            z[0][0].y = z[1][1].y = 0.0;
          }
          G[p][a] = z[0][0];
          G[p][b] = z[0][1];
          G[q][a] = z[1][0];
          G[q][b] = z[1][1];
        } else {
          const double2 x = W[u][a], z = W[u][b], e = ph[v];
          const double2 y = make_double2(e.x * z.x - e.y * z.y, e.x * z.y + e.y * z.x);
          W[u][a] = make_double2(cs[v] * x.x - sn[v] * y.x, cs[v] * x.y - sn[v] * y.y);
          W[u][b] = make_double2(sn[v] * x.x + cs[v] * y.x, sn[v] * x.y + cs[v] * y.y);
        }
      }
    }
    __syncthreads();
    if (again == 0) break;
    __syncthreads();
  }
  __syncthreads();
  if (t < M) {   // rank of eigenvalue t: those before it in falling order
    int before = 0;
    for (int i = 0; i < M; ++i) before += G[i][i].x > G[t][t].x || (G[i][i].x == G[t][t].x && i < t);
    order[before] = t;
  }
  __syncthreads();
  const double top = broken ? 0.0 : G[order[0]][order[0]].x;
  for (int i = t; i < S * k; i += 256) {
    const int m = i / k - lo, j = i - (m + lo) * k;
    double2 v = make_double2(0.0, 0.0);
    if (m >= 0 && m < M && j < kk && !broken) {
      const int o = order[j];
      if (G[o][o].x > 1e-24 * fmax(top, 1e-300)) {
        const double2 a = W[m][o], b = W[s - lo][o];
        v = make_double2((a.x * b.x + a.y * b.y) / nrm[m], (a.y * b.x - a.x * b.y) / nrm[m]);
      }
    }
    coef[((size_t)(m + lo) * S + s) * k + j] = v;
  }
}

// ------------------------------------------------------- device Lanczos ----
// Vectors of M FP64 complex values; Q: the Lanczos vectors, one after the other.
__device__ __forceinline__ double2 lz_sum(double2 s, double2* l) {   // over the workgroup
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    s.x += __shfl_xor(s.x, o, 64);
    s.y += __shfl_xor(s.y, o, 64);
  }
  if ((threadIdx.x & 63) == 0) l[threadIdx.x >> 6] = s;
  __syncthreads();
  return make_double2((l[0].x + l[1].x) + (l[2].x + l[3].x), (l[0].y + l[1].y) + (l[2].y + l[3].y));
}
// w = G q, a row per workgroup
__global__ __launch_bounds__(256) void k_lz_matvec(const double2* __restrict__ G, int M,
                                                   const double2* __restrict__ q,
                                                   double2* __restrict__ w) {
  __shared__ double2 l[4];
  const double2* row = G + (size_t)blockIdx.x * M;
  double2 s = make_double2(0.0, 0.0);
  for (int b = threadIdx.x; b < M; b += 256) {
    const double2 g = row[b], x = q[b];
    s.x += g.x * x.x - g.y * x.y;
    s.y += g.x * x.y + g.y * x.x;
  }
  s = lz_sum(s, l);
  if (threadIdx.x == 0) w[blockIdx.x] = s;
}
// c_j = q_j^H w, a Lanczos vector per workgroup; the last one's is alpha
__global__ __launch_bounds__(256) void k_lz_dots(const double2* __restrict__ Q, int M,
                                                 const double2* __restrict__ w,
                                                 double2* __restrict__ c, double* alpha) {
  __shared__ double2 l[4];
  const double2* q = Q + (size_t)blockIdx.x * M;
  double2 s = make_double2(0.0, 0.0);
  for (int i = threadIdx.x; i < M; i += 256) {
    const double2 a = q[i], x = w[i];
    s.x += a.x * x.x + a.y * x.y;
    s.y += a.x * x.y - a.y * x.x;
  }
  s = lz_sum(s, l);
  if (threadIdx.x == 0) {
    c[blockIdx.x] = s;
    if (alpha && blockIdx.x + 1 == gridDim.x) *alpha = s.x;
  }
}
// w -= sum_j c_j q_j: 64 entries a workgroup, four threads an entry
__global__ __launch_bounds__(256) void k_lz_update(const double2* __restrict__ Q, int M, int L,
                                                   const double2* __restrict__ c,
                                                   double2* __restrict__ w) {
  __shared__ double2 sum[4][64];
  const int l = threadIdx.x & 63, g = threadIdx.x >> 6, i = blockIdx.x * 64 + l;
  double2 s = make_double2(0.0, 0.0);
  if (i < M) {
#pragma unroll 8
    for (int j = g; j < L; j += 4) {
      const double2 a = c[j], q = Q[(size_t)j * M + i];
      s.x += a.x * q.x - a.y * q.y;
      s.y += a.x * q.y + a.y * q.x;
    }
  }
  sum[g][l] = s;
  __syncthreads();
  if (g == 0 && i < M) {
    double2 x = w[i];
    x.x -= (sum[0][l].x + sum[1][l].x) + (sum[2][l].x + sum[3][l].x);
    x.y -= (sum[0][l].y + sum[1][l].y) + (sum[2][l].y + sum[3][l].y);
    w[i] = x;
  }
}
// beta = ||w||, the next Lanczos vector w / beta
__global__ __launch_bounds__(256) void k_lz_next(const double2* __restrict__ w, int M, double* beta,
                                                 double2* __restrict__ q) {
  __shared__ double2 l[4];
  double2 s = make_double2(0.0, 0.0);
  for (int i = threadIdx.x; i < M; i += 256) s.x += w[i].x * w[i].x + w[i].y * w[i].y;
  const double b = sqrt(lz_sum(s, l).x);
  if (threadIdx.x == 0) *beta = b;
  for (int i = threadIdx.x; i < M; i += 256)
    q[i] = b > 0.0 ? make_double2(w[i].x / b, w[i].y / b) : make_double2(0.0, 0.0);
}

// ------------------------------------------------------------- host math ----
// Eigen-decomposition of the real symmetric tridiagonal matrix with diagonal d
// and off-diagonal e (n - 1 values) by the implicit QR algorithm with Wilkinson
// shifts (Golub and Van Loan, Matrix Computations, Sec. 8.3): eigenvalues in d,
// eigenvector i in Z[i n .. i n + n).  About 1.5 n^2 rotations of two rows of Z;
// cyclic Jacobi sweeps over the full matrix take six times as many.
static void tridiagonal_eigh(std::vector<double>& d, std::vector<double>& e, int n,
                             std::vector<double>& Z) {
  Z.assign((size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i) Z[(size_t)i * n + i] = 1.0;
  int hi = n - 1, tries = 0;
  while (hi > 0) {
    int lo = hi;
    while (lo > 0 && std::fabs(e[lo - 1]) > 0x1p-53 * (std::fabs(d[lo - 1]) + std::fabs(d[lo]))) --lo;
    if (lo > 0) e[lo - 1] = 0.0;
    if (lo == hi || ++tries > 60 * n) {   // one eigenvalue found (the bound is never met)
      --hi;
      continue;
    }
    const double del = 0.5 * (d[hi - 1] - d[hi]), eh = e[hi - 1];
    const double mu = d[hi] - eh * eh / (del + std::copysign(std::hypot(del, eh), del));
    double x = d[lo] - mu, z = e[lo];
    for (int k = lo; k < hi; ++k) {
      const double r = std::hypot(x, z);
      const double c = r > 0.0 ? x / r : 1.0, s = r > 0.0 ? z / r : 0.0;
      if (k > lo) e[k - 1] = r;
      const double a = d[k], b = e[k], g = d[k + 1];
      d[k] = c * c * a + 2.0 * c * s * b + s * s * g;
      d[k + 1] = s * s * a - 2.0 * c * s * b + c * c * g;
      e[k] = c * s * (g - a) + (c * c - s * s) * b;
      x = e[k];
      if (k + 1 < hi) {
        z = s * e[k + 1];
        e[k + 1] *= c;
      }
      double *p = &Z[(size_t)k * n], *q = p + n;
      for (int i = 0; i < n; ++i) {
        const double u = p[i], v = q[i];
        p[i] = c * u + s * v;
        q[i] = c * v - s * u;
      }
    }
  }
}

// The signs of the tridiagonal eigenvectors (rows of Z) as cyclic
// Jacobi rotations from the identity leave them: the signs of a stored basis
// follow from them, and users compare bases.  The rotation angles shrink
// quadratically, so three sweeps settle the directions; each vector takes the
// sign of its product with the nearest Jacobi vector.
static void jacobi_signs(const std::vector<double>& alpha, const std::vector<double>& beta, int n,
                         std::vector<double>& Z) {
  std::vector<double> A((size_t)n * n, 0.0), V((size_t)n * n, 0.0);   // V: vectors in rows
  for (int i = 0; i < n; ++i) {
    A[(size_t)i * n + i] = alpha[i];
    V[(size_t)i * n + i] = 1.0;
    if (i + 1 < n) A[(size_t)i * n + i + 1] = A[(size_t)(i + 1) * n + i] = beta[i];
  }
  for (int sweep = 0; sweep < 3; ++sweep)
    for (int p = 0; p < n - 1; ++p)
      for (int q = p + 1; q < n; ++q) {
        const double apq = A[(size_t)p * n + q];
        if (apq == 0.0) continue;
        const double app = A[(size_t)p * n + p], aqq = A[(size_t)q * n + q];
        const double theta = (aqq - app) / (2.0 * apq);
        const double t = (theta >= 0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
        const double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
        double *ap = &A[(size_t)p * n], *aq = &A[(size_t)q * n];
        double *vp = &V[(size_t)p * n], *vq = &V[(size_t)q * n];
        for (int r = 0; r < n; ++r) {
          const double x = ap[r], y = aq[r], u = vp[r], v = vq[r];
          ap[r] = c * x - s * y;
          aq[r] = s * x + c * y;
          vp[r] = c * u - s * v;
          vq[r] = s * u + c * v;
        }
        for (int r = 0; r < n; ++r) {   // the columns, by symmetry
          A[(size_t)r * n + p] = ap[r];
          A[(size_t)r * n + q] = aq[r];
        }
        ap[p] = app - t * apq;
        aq[q] = aqq + t * apq;
        ap[q] = aq[p] = 0.0;
      }
  for (int i = 0; i < n; ++i) {
    double best = 0.0;
    for (int j = 0; j < n; ++j) {
      double x = 0.0;
      for (int r = 0; r < n; ++r) x += Z[(size_t)i * n + r] * V[(size_t)j * n + r];
      if (std::fabs(x) > std::fabs(best)) best = x;
    }
    if (best < 0.0)
      for (int r = 0; r < n; ++r) Z[(size_t)i * n + r] = -Z[(size_t)i * n + r];
  }
}

// Whether the Krylov dimension L (alpha, beta: the tridiagonal matrix, beta[L-1]
// to the next vector) holds the k leading Ritz pairs to a residual
// beta_L |s_L,i| <= 1e-12 theta_max; `full` accepts as it is.  evecs, order: the
// tridiagonal eigenvectors (rows) and their order by falling eigenvalue.
static bool ritz_done(const std::vector<double>& alpha, const std::vector<double>& beta, int L, int k,
                      bool full, std::vector<double>& evals, std::vector<double>& evecs,
                      std::vector<int>& order) {
  evals.assign(alpha.begin(), alpha.begin() + L);
  std::vector<double> e(beta.begin(), beta.begin() + L - 1);
  tridiagonal_eigh(evals, e, L, evecs);
  order.resize(L);
  for (int i = 0; i < L; ++i) order[i] = i;
  std::sort(order.begin(), order.end(), [&](int x, int y) { return evals[x] > evals[y]; });
  const double b = beta[L - 1];
  if (full || b == 0.0) return true;
  if (L < k) return false;
  const double tmax = std::fabs(evals[order[0]]);
  for (int i = 0; i < k; ++i)
    if (b * std::fabs(evecs[(size_t)order[i] * L + L - 1]) > 1e-12 * tmax) return false;
  return true;
}

// The Lanczos start: normal random values, the same every time.
static std::vector<cd> lanczos_start(int M) {
  std::mt19937_64 rng(12345);
  std::normal_distribution<double> nd(0.0, 1.0);
  std::vector<cd> q(M);
  double nq = 0.0;
  for (int i = 0; i < M; ++i) { q[i] = cd(nd(rng), nd(rng)); nq += std::norm(q[i]); }
  nq = std::sqrt(nq);
  for (auto& v : q) v /= nq;
  return q;
}

// Complex vector operations on the parts (std::complex products test for NaN and
// are not vectorised): x^H y, x^T y, y += a x.
static cd dotc(const cd* x, const cd* y, int n) {
  const double *a = (const double*)x, *b = (const double*)y;
  double re = 0.0, im = 0.0;
  for (int i = 0; i < n; ++i) {
    re += a[2 * i] * b[2 * i] + a[2 * i + 1] * b[2 * i + 1];
    im += a[2 * i] * b[2 * i + 1] - a[2 * i + 1] * b[2 * i];
  }
  return cd(re, im);
}
static cd dotu(const cd* x, const cd* y, int n) {
  const double *a = (const double*)x, *b = (const double*)y;
  double re = 0.0, im = 0.0;
  for (int i = 0; i < n; ++i) {
    re += a[2 * i] * b[2 * i] - a[2 * i + 1] * b[2 * i + 1];
    im += a[2 * i] * b[2 * i + 1] + a[2 * i + 1] * b[2 * i];
  }
  return cd(re, im);
}
static void axpy(cd s, const cd* x, cd* y, int n) {
  const double sr = s.real(), si = s.imag(), *a = (const double*)x;
  double* b = (double*)y;
  for (int i = 0; i < n; ++i) {
    b[2 * i] += sr * a[2 * i] - si * a[2 * i + 1];
    b[2 * i + 1] += sr * a[2 * i + 1] + si * a[2 * i];
  }
}

// The k leading Ritz vectors W (M x k, row-major) and values theta from L
// Lanczos vectors Q (one after the other).
static void ritz_vectors(const std::vector<cd>& Q, int M, int L, int k,
                         const std::vector<double>& evals, const std::vector<double>& evecs,
                         const std::vector<int>& order, std::vector<double>& theta,
                         std::vector<cd>& W) {
  const int kk = std::min(k, L);
  theta.assign(k, 0.0);
  W.assign((size_t)M * k, cd(0.0));
  std::vector<cd> w(M);
  for (int i = 0; i < kk; ++i) {
    theta[i] = evals[order[i]];
    std::fill(w.begin(), w.end(), cd(0.0));
    for (int j = 0; j < L; ++j) {
      const double s = evecs[(size_t)order[i] * L + j];
      const double* q = (const double*)&Q[(size_t)j * M];
      double* o = (double*)w.data();
      for (int r = 0; r < 2 * M; ++r) o[r] += s * q[r];
    }
    for (int r = 0; r < M; ++r) W[(size_t)r * k + i] = w[r];
  }
}

// Leading k eigenpairs of the Hermitian M x M matrix G (row-major) by Lanczos
// with full reorthogonalisation (twice per step), restarted never: the Krylov
// dimension grows until ritz_done, or L = M.  Returns eigenvalues (descending)
// and eigenvectors (M x k, row-major; signs: of a definite sign).
static void lanczos_top(const std::vector<cd>& G, int M, int k, bool signs,
                        std::vector<double>& theta, std::vector<cd>& W) {
  std::vector<double> alpha, beta;
  std::vector<cd> w(M), Q = lanczos_start(M);
  Q.reserve((size_t)M * std::min(M + 1, 2 * k + 64));
  std::vector<double> evals, evecs;
  std::vector<int> order;
  for (int L = 1; L <= M; ++L) {
    const cd* q = &Q[(size_t)(L - 1) * M];
    for (int a = 0; a < M; ++a) w[a] = dotu(&G[(size_t)a * M], q, M);
    alpha.push_back(dotc(q, w.data(), M).real());
    for (int pass = 0; pass < 2; ++pass)
      for (int j = 0; j < L; ++j) {
        const cd* qj = &Q[(size_t)j * M];
        axpy(-dotc(qj, w.data(), M), qj, w.data(), M);
      }
    const double b = std::sqrt(dotc(w.data(), w.data(), M).real());
    beta.push_back(b);
    const bool full = (L == M);
    if (full || (L >= 2 * k + 10 && (L % 10 == 0)) || b == 0.0) {
      if (ritz_done(alpha, beta, L, k, full, evals, evecs, order)) {
        if (signs) jacobi_signs(alpha, beta, L, evecs);
        ritz_vectors(Q, M, L, k, evals, evecs, order, theta, W);
        return;
      }
    }
    for (int i = 0; i < M; ++i) Q.push_back(w[i] / b);
  }
}

// The same iteration on a device matrix G, six small kernels a step; the host
// looks at the tridiagonal matrix every ten steps.  For 1000 snapshots the host
// iteration took 40 ms (a product with G, 16 MB, in each of 50 steps) after a
// 4 ms copy of G; 1.2 ms here.  pca_build takes it from 128 snapshots on, where 20
// components cross: whole calls on 20,000 elements, on the host and here, 112 snapshots
// 1.44 and 1.66 ms, 128 1.60 and 1.66, 160 2.03 and 1.72, 256 3.81 and 2.17; 5 components
// cross near 170: 128 0.58 and 0.76 ms, 160 0.76 and 0.78, 200 1.27 and 1.14.
static dd_status lanczos_device(const double2* G, int M, int k, std::vector<double>& theta,
                                std::vector<cd>& W, hipStream_t stream) {
  DevBuf bQ, bw;
  int cap = std::min(M, 2 * k + 10 + 40);       // Lanczos vectors that there is room for
  DD_HIP_CHECK(hipMalloc(&bQ.p, sizeof(double2) * (size_t)(cap + 1) * M));
  // w, the dot products, then alpha and beta
  DD_HIP_CHECK(hipMalloc(&bw.p, sizeof(double2) * 2 * (size_t)M + sizeof(double) * 2 * (size_t)M));
  double2 *Q = bQ.as<double2>(), *w = bw.as<double2>(), *c = w + M;
  double *da = (double*)(c + M), *db = da + M;
  const std::vector<cd> q0 = lanczos_start(M);
  DD_HIP_CHECK(hipMemcpyAsync(Q, q0.data(), sizeof(double2) * M, hipMemcpyHostToDevice, stream));
  DD_HIP_CHECK(hipStreamSynchronize(stream));
  std::vector<double> alpha, beta, evals, evecs;
  std::vector<int> order;
  const int nu = (M + 63) / 64;
  for (int L = 1; L <= M; ++L) {
    if (L > cap) {
      DevBuf more;
      const int c2 = std::min(M, 2 * cap);
      DD_HIP_CHECK(hipMalloc(&more.p, sizeof(double2) * (size_t)(c2 + 1) * M));
      DD_HIP_CHECK(hipMemcpyAsync(more.p, Q, sizeof(double2) * (size_t)(cap + 1) * M,
                                  hipMemcpyDeviceToDevice, stream));
      DD_HIP_CHECK(hipStreamSynchronize(stream));
      std::swap(more.p, bQ.p);
      Q = bQ.as<double2>();
      cap = c2;
    }
    k_lz_matvec<<<M, 256, 0, stream>>>(G, M, Q + (size_t)(L - 1) * M, w);
    for (int pass = 0; pass < 2; ++pass) {
      k_lz_dots<<<L, 256, 0, stream>>>(Q, M, w, c, pass == 0 ? da + L - 1 : nullptr);
      k_lz_update<<<nu, 256, 0, stream>>>(Q, M, L, c, w);
    }
    k_lz_next<<<1, 256, 0, stream>>>(w, M, db + L - 1, Q + (size_t)L * M);
    const bool full = (L == M);
    if (!full && !(L >= 2 * k + 10 && L % 10 == 0)) continue;
    DD_HIP_CHECK(hipGetLastError());
    alpha.resize(L);
    beta.resize(L);
    DD_HIP_CHECK(hipMemcpyAsync(alpha.data(), da, sizeof(double) * L, hipMemcpyDeviceToHost, stream));
    DD_HIP_CHECK(hipMemcpyAsync(beta.data(), db, sizeof(double) * L, hipMemcpyDeviceToHost, stream));
    DD_HIP_CHECK(hipStreamSynchronize(stream));
    // an invariant space was met on the way: the vectors past it are zero
    int n = L;
    for (int i = 0; i < L; ++i)
      if (beta[i] == 0.0) { n = i + 1; break; }
    if (!ritz_done(alpha, beta, n, k, full && n == L, evals, evecs, order)) continue;
    std::vector<cd> hQ((size_t)n * M);
    DD_HIP_CHECK(hipMemcpyAsync(hQ.data(), Q, sizeof(cd) * hQ.size(), hipMemcpyDeviceToHost, stream));
    DD_HIP_CHECK(hipStreamSynchronize(stream));
    jacobi_signs(alpha, beta, n, evecs);
    ritz_vectors(hQ, M, n, k, evals, evecs, order, theta, W);
    return DD_OK;
  }
  return DD_OK;
}

// ------------------------------------------------------------------ API ----
// Small Gram of k device vectors (FP64), host side: used for the final Cholesky
// QR pass and for the projection loss.
__global__ __launch_bounds__(256) void k_small_gram(const float2* __restrict__ V, int k, int D,
                                                    const double2* __restrict__ f, int with_f,
                                                    int nslices, double2* __restrict__ part) {
  // part[slice][(k+1) x (k+1)]: Gram of [V; f] restricted to this slice
  const int a = blockIdx.x, slice = blockIdx.y;
  const int per = (D + nslices - 1) / nslices;
  const int e0 = slice * per, e1 = min(D, e0 + per);
  const int K1 = k + 1;
  __shared__ double lds[8];
  for (int b = a; b < K1; ++b) {
    if (!with_f && (a == k || b == k)) continue;
    double sx = 0.0, sy = 0.0;
    for (int e = e0 + threadIdx.x; e < e1; e += 256) {
      double ax, ay, bx, by;
      if (a < k) { const float2 v = V[(size_t)a * D + e]; ax = v.x; ay = v.y; }
      else { const double2 v = f[e]; ax = v.x; ay = v.y; }
      if (b < k) { const float2 v = V[(size_t)b * D + e]; bx = v.x; by = v.y; }
      else { const double2 v = f[e]; bx = v.x; by = v.y; }
      sx += ax * bx + ay * by;
      sy += ax * by - ay * bx;
    }
    sx = block_sum1<double>(sx, lds);
    sy = block_sum1<double>(sy, lds);
    if (threadIdx.x == 0) part[((size_t)slice * K1 + a) * K1 + b] = make_double2(sx, sy);
  }
}

// C = V T (T upper triangular k x k, FP64), in place, one thread per element.
__global__ __launch_bounds__(256) void k_small_combine(float2* __restrict__ V, int k, int D,
                                                       const double2* __restrict__ T) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= D) return;
  float2 x[DD_MAX_KPCA];
  for (int i = 0; i < k; ++i) x[i] = V[(size_t)i * D + e];
  for (int o = 0; o < k; ++o) {
    double sx = 0.0, sy = 0.0;
    for (int i = 0; i <= o; ++i) {
      const double2 c = T[(size_t)i * k + o];
      sx += c.x * x[i].x - c.y * x[i].y;
      sy += c.x * x[i].y + c.y * x[i].x;
    }
    V[(size_t)o * D + e] = make_float2((float)sx, (float)sy);
  }
}

dd_status gram_host(const float2* V, int k, int D, const double2* f, std::vector<cd>& G,
                    hipStream_t stream) {
  const int K1 = k + 1;
  const int nslices = std::max(1, std::min(256, D / 4096));
  DevBuf bpart;
  DD_HIP_CHECK(hipMalloc(&bpart.p, sizeof(double2) * nslices * K1 * K1));
  double2* part = bpart.as<double2>();
  DD_HIP_CHECK(hipMemsetAsync(part, 0, sizeof(double2) * nslices * K1 * K1, stream));
  k_small_gram<<<dim3(f ? K1 : k, nslices), 256, 0, stream>>>(V, k, D, f, f ? 1 : 0, nslices, part);
  std::vector<double2> hp((size_t)nslices * K1 * K1);
  DD_HIP_CHECK(hipMemcpyAsync(hp.data(), part, sizeof(double2) * hp.size(), hipMemcpyDeviceToHost,
                              stream));
  DD_HIP_CHECK(hipStreamSynchronize(stream));
  G.assign((size_t)K1 * K1, cd(0.0));
  for (int s = 0; s < nslices; ++s)
    for (int a = 0; a < K1; ++a)
      for (int b = a; b < K1; ++b) {
        const double2 v = hp[((size_t)s * K1 + a) * K1 + b];
        G[(size_t)a * K1 + b] += cd(v.x, v.y);
      }
  for (int a = 0; a < K1; ++a)
    for (int b = 0; b < a; ++b) G[(size_t)a * K1 + b] = std::conj(G[(size_t)b * K1 + a]);
  return DD_OK;
}

// G_ab = <F_a, F_b> (M x M, FP64) of M device rows of D complex64 values.  Tiles of 64 x 64 from 49 rows on (below, half of
// one would be padding), the elements in as many slices (of 2048 workgroups at
// most) as leave the last round of resident workgroups, three a compute unit,
// fullest.  flag: an int behind G that is 0 where all of it is finite.  The call does not
// wait: the caller keeps bpart until the kernels are done.
static dd_status gram_device(const float2* F, int M, int D, DevBuf& bG, DevBuf& bpart, bool flag,
                             hipStream_t stream) {
  const int tile = M > 48 ? 64 : 32;
  const int nta = (M + tile - 1) / tile, ntiles = nta * (nta + 1) / 2;
  int dev = 0, ncu = 256;
  DD_HIP_CHECK(hipGetDevice(&dev));
  DD_HIP_CHECK(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
  const int most = std::min(std::max(1, std::min(256, 2048 / ntiles)), (D + 4 * PE - 1) / (4 * PE));
  int nslices = 1;
  for (int n = 2; n <= most; ++n) {
    const auto rounds = [&](int x) { return (ntiles * (long long)x + 3 * ncu - 1) / (3 * ncu); };
    if (rounds(n) * nslices < rounds(nslices) * n) nslices = n;   // rounds / slices falls
  }
  const int per = ((D + nslices - 1) / nslices + PE - 1) / PE * PE;
  nslices = (D + per - 1) / per;
  DD_HIP_CHECK(hipMalloc(&bpart.p, sizeof(double2) * (size_t)nslices * ntiles * tile * tile));
  DD_HIP_CHECK(hipMalloc(&bG.p, sizeof(double2) * M * M + sizeof(int)));
  double2 *part = bpart.as<double2>(), *G = bG.as<double2>();
  int* bad = flag ? (int*)(G + (size_t)M * M) : nullptr;
  if (flag) DD_HIP_CHECK(hipMemsetAsync(bad, 0, sizeof(int), stream));
  if (tile == 64) k_pca_gram<2><<<dim3(ntiles, nslices), 256, 0, stream>>>(F, M, D, per, part);
  else k_pca_gram<1><<<dim3(ntiles, nslices), 256, 0, stream>>>(F, M, D, per, part);
  k_pca_gram_reduce<<<dim3(ntiles, tile * tile / 64), 256, 0, stream>>>(part, M, tile, nslices, G,
                                                                        bad);
  DD_HIP_CHECK(hipGetLastError());
  return DD_OK;
}

// The same on the host, and whether all of it is finite.
static dd_status gram_rows(const float2* F, int M, int D, std::vector<cd>& G, bool* finite,
                           hipStream_t stream) {
  DevBuf bG, bpart;
  dd_status rc = gram_device(F, M, D, bG, bpart, false, stream);
  if (rc != DD_OK) return rc;
  G.resize((size_t)M * M);
  static_assert(sizeof(cd) == sizeof(double2), "complex layout");
  DD_HIP_CHECK(hipMemcpyAsync(G.data(), bG.p, sizeof(cd) * G.size(), hipMemcpyDeviceToHost, stream));
  DD_HIP_CHECK(hipStreamSynchronize(stream));
  *finite = true;
  for (const cd& v : G) *finite = *finite && std::isfinite(v.real()) && std::isfinite(v.imag());
  return DD_OK;
}

// Cholesky G = L L^H of the leading k x k block (stride ld); returns false if
// not positive definite.  T = L^{-H} (upper triangular, row-major k x k).
bool chol_inv(const std::vector<cd>& G, int ld, int k, std::vector<cd>& L,
              std::vector<cd>& T) {
  L.assign((size_t)k * k, cd(0.0));
  for (int j = 0; j < k; ++j) {
    double d = G[(size_t)j * ld + j].real();
    for (int l = 0; l < j; ++l) d -= std::norm(L[(size_t)j * k + l]);
    if (!(d > 0.0)) return false;
    const double ljj = std::sqrt(d);
    L[(size_t)j * k + j] = ljj;
    for (int i = j + 1; i < k; ++i) {
      cd s = G[(size_t)i * ld + j];
      for (int l = 0; l < j; ++l) s -= L[(size_t)i * k + l] * std::conj(L[(size_t)j * k + l]);
      L[(size_t)i * k + j] = s / ljj;
    }
  }
  T.assign((size_t)k * k, cd(0.0));
  for (int o = 0; o < k; ++o)
    for (int a = o; a >= 0; --a) {
      cd v = (a == o) ? cd(1.0) : cd(0.0);
      for (int l = a + 1; l <= o; ++l) v -= std::conj(L[(size_t)l * k + a]) * T[(size_t)l * k + o];
      T[(size_t)a * k + o] = v / L[(size_t)a * k + a].real();
    }
  return true;
}

extern "C" dd_status pca_build(const void* Sv, int M, int D, int k, void* Uv, double* sigma,
                               hipStream_t stream) {
  if (!Sv || !Uv || M < 1 || D < 1 || k < 1 || k > M || k > DD_MAX_KPCA) {
    dd_set_error("pca_build: need S, U, 1 <= k <= min(M, %d), D >= 1", DD_MAX_KPCA);
    return DD_EINVAL;
  }
  const float2* S = (const float2*)Sv;
  float2* U = (float2*)Uv;
  // G_ab = <s_a, s_b>; with X = [s_1 .. s_M] (D x M), G = X^H X and the left
  // singular vectors are u_i = X w_i / sigma_i for X^H X w_i = sigma_i^2 w_i.
  DevBuf bG, bpart, bcoef, bT;
  bool finite = true;
  std::vector<double> theta;
  std::vector<cd> W;
  dd_status rc = DD_OK;
  if (M >= 128) {
    rc = gram_device(S, M, D, bG, bpart, true, stream);
    if (rc != DD_OK) return rc;
    int bad = 0;
    DD_HIP_CHECK(hipMemcpyAsync(&bad, bG.as<double2>() + (size_t)M * M, sizeof(int),
                                hipMemcpyDeviceToHost, stream));
    DD_HIP_CHECK(hipStreamSynchronize(stream));
    finite = bad == 0;
    if (finite) rc = lanczos_device(bG.as<double2>(), M, k, theta, W, stream);
  } else {
    std::vector<cd> hG;
    rc = gram_rows(S, M, D, hG, &finite, stream);
    if (rc == DD_OK && finite) lanczos_top(hG, M, k, true, theta, W);
  }
  if (rc != DD_OK) return rc;
  if (!finite) {
    dd_set_error("pca_build: snapshots contain non-finite values");
    return DD_ENONFINITE;
  }
  std::vector<double2> hc((size_t)M * k);
  for (int i = 0; i < k; ++i) {
    const double s = std::sqrt(std::max(theta[i], 0.0));
    if (!(s > 0.0)) {
      dd_set_error("pca_build: snapshot matrix has rank < k");
      return DD_EINVAL;
    }
    if (sigma) sigma[i] = s;
    for (int mrow = 0; mrow < M; ++mrow) {
      const cd c = W[(size_t)mrow * k + i] / s;
      hc[(size_t)mrow * k + i] = make_double2(c.real(), c.imag());
    }
  }
  DD_HIP_CHECK(hipMalloc(&bcoef.p, sizeof(double2) * M * k));
  double2* coef = bcoef.as<double2>();
  DD_HIP_CHECK(hipMemcpyAsync(coef, hc.data(), sizeof(double2) * M * k, hipMemcpyHostToDevice, stream));
  k_field_combine<<<dim3((D + 127) / 128, (k + 31) / 32), 256, 0, stream>>>(
      S, M, D, coef, k, 0, 0, nullptr, U);
  DD_HIP_CHECK(hipGetLastError());
  DD_HIP_CHECK(hipStreamSynchronize(stream));
  // one Cholesky QR pass restores orthonormality lost to FP32 storage
  std::vector<cd> Gu, L, T;
  rc = gram_host(U, k, D, nullptr, Gu, stream);
  if (rc != DD_OK) return rc;
  if (!chol_inv(Gu, k + 1, k, L, T)) {
    dd_set_error("pca_build: basis Gram matrix not positive definite");
    return DD_EINVAL;
  }
  std::vector<double2> hT((size_t)k * k);
  for (size_t i = 0; i < hT.size(); ++i) hT[i] = make_double2(T[i].real(), T[i].imag());
  DD_HIP_CHECK(hipMalloc(&bT.p, sizeof(double2) * k * k));
  double2* dT = bT.as<double2>();
  DD_HIP_CHECK(hipMemcpyAsync(dT, hT.data(), sizeof(double2) * k * k, hipMemcpyHostToDevice, stream));
  k_small_combine<<<(D + 255) / 256, 256, 0, stream>>>(U, k, D, dT);
  DD_HIP_CHECK(hipGetLastError());
  DD_HIP_CHECK(hipStreamSynchronize(stream));
  return DD_OK;
}

// Training targets of the convolutional predictor from one trajectory's
// solution fields: for step s, U_loc = the leading k left singular vectors
// of the (unit-normalised) fields of steps s-window..s+window, and target j
// = u_j (u_j^H f_s).  With the window's Gram matrix G (from the trajectory
// Gram matrix) = W diag(sigma^2) W^H, u_j = sum_m W_mj f_m / sigma_j and
// u_j^H f_s = sum_m conj(W_mj) G_ms / sigma_j, so every target is a combination
// of the trajectory's fields with coefficients from a small host problem.
extern "C" dd_status local_pca_targets(const void* Fv, int S, int D, int window, int k,
                                       void* Tv, hipStream_t stream) {
  if (!Fv || !Tv || S < 1 || D < 1 || k < 1 || window < 0 || k > DD_MAX_KPCA) {
    dd_set_error("local_pca_targets: bad argument");
    return DD_EINVAL;
  }
  const float2* F = (const float2*)Fv;
  const dim3 grid((D + 127) / 128, (S * k + 31) / 32);
  if (std::min((long long)S, 2ll * window + 1) <= PJ_MAX) {
    // the windows' problems fit a workgroup's LDS: nothing leaves the device.
    // 32 fields of 480 x 240, windows of 17: 380 us, on the host's way below 815
    DevBuf bG, bpart, bcoef;
    DD_HIP_CHECK(hipMalloc(&bcoef.p, sizeof(double2) * (size_t)S * S * k));
    dd_status rc = gram_device(F, S, D, bG, bpart, true, stream);
    if (rc != DD_OK) return rc;
    const double2* G = bG.as<double2>();
    double2* coef = bcoef.as<double2>();
    k_window_coefs<<<S, 256, 0, stream>>>(G, S, std::min(window, S), k, coef);
    k_field_combine<<<grid, 256, 0, stream>>>(F, S, D, coef, S * k, k, std::min(window, S),
                                              (const int*)(G + (size_t)S * S), (float2*)Tv);
    DD_HIP_CHECK(hipGetLastError());
    DD_HIP_CHECK(hipStreamSynchronize(stream));
    return DD_OK;
  }
  // trajectory Gram matrix of the normalised fields (normalisation applied here)
  std::vector<cd> G0;
  bool finite = true;
  dd_status rc = gram_rows(F, S, D, G0, &finite, stream);
  if (rc != DD_OK) return rc;
  std::vector<double> nrm(S);
  for (int a = 0; a < S; ++a) nrm[a] = std::sqrt(std::max(G0[(size_t)a * S + a].real(), 1e-300));
  std::vector<double2> hc((size_t)S * S * k, make_double2(0.0, 0.0));
  for (int s = 0; s < S; ++s) {
    const int lo = std::max(0, s - window), hi = std::min(S, s + window + 1), M = hi - lo;
    std::vector<cd> G((size_t)M * M);
    for (int a = 0; a < M; ++a)
      for (int b = 0; b < M; ++b)
        G[(size_t)a * M + b] = G0[(size_t)(lo + a) * S + lo + b] / (nrm[lo + a] * nrm[lo + b]);
    const int kk = std::min(k, M);
    std::vector<double> theta;
    std::vector<cd> W;
    lanczos_top(G, M, kk, false, theta, W);   // phase-free
    for (int j = 0; j < kk; ++j) {
      if (!(theta[j] > 1e-24 * std::max(theta[0], 1e-300))) continue;
      const double sg = std::sqrt(theta[j]);
      cd c = 0.0;  // u_j^H f_s (f_s normalised)
      for (int m = 0; m < M; ++m) c += std::conj(W[(size_t)m * kk + j]) * G[(size_t)m * M + (s - lo)];
      c /= sg;
      for (int m = 0; m < M; ++m) {
        // target_j = sum_m (W_mj / sigma_j) c f_m / ||f_m||  (fields normalised)
        const cd v = W[(size_t)m * kk + j] / sg * c / nrm[lo + m];
        hc[((size_t)(lo + m) * S + s) * k + j] = make_double2(v.real(), v.imag());
      }
    }
  }
  DevBuf bcoef;
  DD_HIP_CHECK(hipMalloc(&bcoef.p, sizeof(double2) * hc.size()));
  double2* coef = bcoef.as<double2>();
  DD_HIP_CHECK(hipMemcpyAsync(coef, hc.data(), sizeof(double2) * hc.size(), hipMemcpyHostToDevice, stream));
  k_field_combine<<<grid, 256, 0, stream>>>(F, S, D, coef, S * k, finite ? k : 0,
                                            std::min(window, S), nullptr, (float2*)Tv);
  DD_HIP_CHECK(hipGetLastError());
  DD_HIP_CHECK(hipStreamSynchronize(stream));
  return DD_OK;
}

extern "C" dd_status proj_loss_batched(const void* Vv, const void* fv, int nb, int k, int D,
                                       double* out, hipStream_t stream) {
  if (!Vv || !fv || !out || nb < 1 || k < 1 || k > DD_MAX_KPCA || D < 1) {
    dd_set_error("proj_loss_batched: bad argument");
    return DD_EINVAL;
  }
  for (int p = 0; p < nb; ++p) {
    const float2* V = (const float2*)Vv + (size_t)p * k * D;
    const double2* f = (const double2*)fv + (size_t)p * D;
    std::vector<cd> G, L, T;
    dd_status rc = gram_host(V, k, D, f, G, stream);
    if (rc != DD_OK) return rc;
    const int K1 = k + 1;
    const double ff = G[(size_t)k * K1 + k].real();
    // l = 1 - c^H G_VV^{-1} c / ||f||^2 with c = V^H f; G_VV^{-1} = T T^H
    if (!(ff > 0.0)) { out[p] = 0.0; continue; }
    if (!chol_inv(G, K1, k, L, T)) {
      dd_set_error("proj_loss_batched: V of problem %d is rank deficient", p);
      return DD_EINVAL;
    }
    double q = 0.0;
    for (int o = 0; o < k; ++o) {
      cd s = 0.0;  // (T^H c)_o = sum_a conj(T[a][o]) c_a
      for (int a = 0; a <= o; ++a) s += std::conj(T[(size_t)a * k + o]) * G[(size_t)a * K1 + k];
      q += std::norm(s);
    }
    // the loss lies in [0, 1] by definition; rounding can step outside by ~1e-16
    out[p] = std::min(1.0, std::max(0.0, 1.0 - q / ff));
  }
  return DD_OK;
}
