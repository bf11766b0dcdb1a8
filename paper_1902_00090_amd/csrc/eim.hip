// Effective-index approximation of the field: the CNN's second input.
//
// The paper feeds its CNN an effective-index simulation of the field next to
// the permittivity (Sec. 3, data-set and CNN paragraphs).  It describes this
// only as a cheap 1D solve of Maxwell's equations.  The separable reading
// used here has three steps.
//
//  1. Every column ix is a 1D slab.  Its fundamental mode phi_ix is the
//     eigenvector of the lowest eigenvalue mu_ix of
//         T = -(second difference in y)/dx^2 - omega^2 eps(ix, .),
//     with zero field outside the column.  phi_ix has unit norm and is
//     positive.
//  2. The amplitude a along x solves the 1D FDFD equation.  It uses the 2D
//     operator's stretched x-differences (periodic wrap) with mu in place of
//     -omega^2 eps:
//         cxm_i (a_i - a_{i-1}) - cxp_i (a_{i+1} - a_i) + mu_i a_i = j_i,
//     where j_i = phi_i^T b[:, i].
//  3. F[iy, ix] = a_ix phi_ix(iy).
//
// The kernels, all in FP64:
//  * k_eim_bound: lower bounds of the lowest eigenvalues, by sections of the
//    Gershgorin interval; four lanes of a column try four points at a time.
//  * k_eim_modes: one thread per column, inverse iteration from just below the
//    eigenvalue.  The shifted matrix is then symmetric positive definite with
//    non-positive off-diagonals, so its LDL^T sweep needs no pivoting and keeps
//    the iterate positive.
//  * k_eim_line: one wave per problem.  The cyclic complex tridiagonal system
//    is solved by Sherman-Morrison over a tridiagonal elimination with partial
//    pivoting.  The matrix is indefinite, so pivoting is needed.
//  * k_eim_assemble: writes F in complex64.
// Measured for 64 problems of 480 x 240: one bisecting thread per column with a
// division in each Sturm step took 4.54 ms and one thread per problem, its rows
// in memory between the steps, 1.04 ms; these kernels take
// 0.17, 0.34 and 0.19 ms.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <utility>
#include <vector>

#include "common.h"
#include "eim.h"
#include "op.h"

#define DD_EIM_MAX_DEVICES 64

namespace {

struct EimDesc {
  int nx, ny;
  double omega, dx;
  const float* eps;    // [ny][nx]
  const double2* cf;   // cxm [0, nx), cxp [nx, 2nx)
  const double2* b;    // [D] right-hand side
  float2* F;           // [D] output
  size_t off2;         // offset in the D-sized scratch arrays
  size_t off1;         // offset in the nx-sized scratch arrays
};

__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 zsub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 zadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double zabs2(double2 a) { return a.x * a.x + a.y * a.y; }
__device__ __forceinline__ double2 zdiv(double2 a, double2 b) {
  const double s = 1.0 / zabs2(b);
  return make_double2((a.x * b.x + a.y * b.y) * s, (a.y * b.x - a.x * b.y) * s);
}

// ------------------------------------------------ column modes (step 1) ----
// Lower bound of the lowest eigenvalue of 16 columns per wave.  T - x I has a
// negative eigenvalue where the sequence of its leading minors changes sign:
// divided by h2^i they obey p_i = t_i p_{i-1} - p_{i-2} with t_i = (d_i - x)/h2,
// one fused multiply-add a step and no division (the pivots are their ratios,
// each a division that waits for the one before).  p is scaled down every four steps
// where it has grown past 2^400: four steps multiply it by less than 2^600 while
// (omega dx)^2 is below 2^20, whatever the FP32 permittivity (|t| < 2^150).  It needs no
// scaling up: where it falls as the mode does, through a cladding, a step's rounding puts
// 2^-53 of it into the solution that grows, which takes over after about 2^-27.  Lane
// 16 s + c tries point s + 1 of five sections of column
// c's interval: 18 rounds leave 2 h2 5^-18 < 2^-40 h2 (the shift below it is off
// by 1e-10 of the diagonal on purpose).  LDS: the columns' permittivities are
// read 18 times.
template <bool LDS>
__global__ __launch_bounds__(64) void k_eim_bound(const EimDesc* __restrict__ desc,
                                                  double* __restrict__ sig) {
  extern __shared__ float eps_l[];
  const EimDesc d = desc[blockIdx.y];
  const int c = threadIdx.x & 15, sct = threadIdx.x >> 4;
  if ((int)blockIdx.x * 16 >= d.nx) return;
  const int ix = min((int)blockIdx.x * 16 + c, d.nx - 1);
  const int nx = d.nx, ny = d.ny;
  const double h2 = 1.0 / (d.dx * d.dx), w2 = d.omega * d.omega;
  const float* eps = d.eps + ix;
  float emin = eps[0], emax = emin;
  for (int i = sct; i < ny; i += 4) {
    const float e = eps[(size_t)i * nx];
    if (LDS) eps_l[i * 16 + c] = e;
    emin = fminf(emin, e);
    emax = fmaxf(emax, e);
  }
  for (int o = 16; o <= 32; o <<= 1) {
    emin = fminf(emin, __shfl_xor(emin, o, 64));
    emax = fmaxf(emax, __shfl_xor(emax, o, 64));
  }
  __syncthreads();
  // Gershgorin: the lowest eigenvalue lies in [min diag - 2 h2, min diag]
  const double dmin = 2.0 * h2 - w2 * (double)emax, dmax = 2.0 * h2 - w2 * (double)emin;
  const double amax = fmax(fabs(dmin), fabs(dmax));
  double lo = dmin - 2.0 * h2, width = 2.0 * h2;
  const double a = -w2 / h2;
  for (int it = 0; it < 18; ++it) {
    const double x = lo + width * (0.2 * (sct + 1));
    const double t0 = 2.0 - x / h2;
    double p1 = 1.0, p2 = 0.0;
    int neg = 0;                    // sign bits of the minors
    int i = 0;
    for (; i + 8 <= ny; i += 8) {
      float e[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) e[q] = LDS ? eps_l[(i + q) * 16 + c] : eps[(size_t)(i + q) * nx];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const double p = fma(fma(a, (double)e[q], t0), p1, -p2);
        neg |= __double2hiint(p);
        p2 = p1;
        p1 = p;
        if (q % 4 == 3) {
          const double f = (fabs(p1) > 0x1p400) ? 0x1p-400 : 1.0;
          p1 *= f;
          p2 *= f;
        }
      }
    }
    for (; i < ny; ++i) {
      const double e = LDS ? eps_l[i * 16 + c] : eps[(size_t)i * nx];
      const double p = fma(fma(a, e, t0), p1, -p2);
      neg |= __double2hiint(p);
      const double f = (fabs(p) > 0x1p400) ? 0x1p-400 : 1.0;
      p2 = p1 * f;
      p1 = p * f;
    }
    // the points without a sign change lie below the eigenvalue
    const unsigned long long below = __ballot(neg >= 0);
    const int k = __popcll((below >> c) & 0x0001000100010001ull);
    lo += width * (0.2 * k);
    width *= 0.2;
  }
  if (sct == 0 && (int)blockIdx.x * 16 + c < nx)
    sig[d.off1 + ix] = lo - 1e-10 * (amax + 2.0 * h2);
}

// Inverse iteration from the shift, one thread per column.  The pivots' inverses
// are formed once (the only divisions); a sweep is then one fused multiply-add a
// row.  Rows are taken sixteen at a time so that their loads are in flight
// together.  Bound by a column's chain of rows, nine times up or down it: 64 problems
// of 480 x 240 take 342 us, 8 of them 295; with eight rows at a time 365, with 24 340,
// with the vector in LDS (one wave a compute unit) 548, with scalar row offsets and
// buffer accesses 484.  The vector is kept in the output array, whose complex64 is as
// large, until the field is assembled: it costs no scratch to allocate and free (a call
// on those 64 problems 962 us, with scratch for it 270 more).  Outputs that share memory
// with a right-hand side, which other columns still read then, are left alone until then
// and phi is scratch.
#define DD_EIM_COLS 64
__global__ __launch_bounds__(DD_EIM_COLS) void k_eim_modes(const EimDesc* __restrict__ desc,
                                                  double* __restrict__ phi,
                                                  double* __restrict__ piv,
                                                  double* __restrict__ mu,
                                                  double2* __restrict__ jp) {
  const EimDesc d = desc[blockIdx.y];
  const int ix = blockIdx.x * DD_EIM_COLS + threadIdx.x;
  if (ix >= d.nx) return;
  const int nx = d.nx, ny = d.ny;
  const double h2 = 1.0 / (d.dx * d.dx), w2 = d.omega * d.omega, e2 = h2 * h2;
  const float* eps = d.eps + ix;
  double* ph = (phi ? phi + d.off2 : (double*)d.F) + ix;
  double* pv = piv + d.off2 + ix;
  const double sigma = mu[d.off1 + ix];
  constexpr int U = 16;
  // rows [i, i + U) up (or down) with valid addresses past the ends
  auto row = [&](int i) { return (size_t)min(max(i, 0), ny - 1) * nx; };
  double ss = 0.0, sum = 0.0;
  // sixteen rows are computed while the next sixteen are in flight
  double v[U], r[U], vn[U], rn[U];
  auto fetch = [&](int i0, int dir, bool first) {
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const size_t at = row(i0 + dir * q);
      vn[q] = first ? (double)eps[at] : ph[at];
      if (!first) rn[q] = pv[at];
    }
  };
  auto take = [&]() {
#pragma unroll
    for (int q = 0; q < U; ++q) {
      v[q] = vn[q];
      r[q] = rn[q];
    }
  };
  for (int it = 0; it < 4; ++it) {
    // L z = v: z_i = v_i + h2 z_{i-1} / p_{i-1}; the first time from ones
    double z = 0.0, rp = 0.0;
    fetch(0, 1, it == 0);
    for (int i0 = 0; i0 < ny; i0 += U) {
      take();
      fetch(i0 + U, 1, it == 0);
#pragma unroll
      for (int q = 0; q < U; ++q) {
        if (i0 + q < ny) {
          if (it == 0) {
            r[q] = 1.0 / (2.0 * h2 - w2 * v[q] - sigma - e2 * rp);
            v[q] = 1.0;
            pv[(size_t)(i0 + q) * nx] = r[q];
          }
          z = fma(h2 * rp, z, v[q]);
          rp = r[q];
          ph[(size_t)(i0 + q) * nx] = z;
        }
      }
    }
    // D L^T x = z: x_i = (z_i + h2 x_{i+1}) / p_i
    double x = 0.0;
    ss = sum = 0.0;
    fetch(ny - 1, -1, false);
    for (int i0 = ny - 1; i0 >= 0; i0 -= U) {
      take();
      fetch(i0 - U, -1, false);
#pragma unroll
      for (int q = 0; q < U; ++q) {
        if (i0 - q >= 0) {
          x = fma(h2 * r[q], x, v[q] * r[q]);
          ph[(size_t)(i0 - q) * nx] = x;
          ss = fma(x, x, ss);
          sum += x;
        }
      }
    }
    // an iteration multiplies the vector by up to 1e10 / h2: scale it if four of
    // them could leave the range at either end
    if (it < 3 && !(ss < 1e120 && ss > 1e-60)) {
      const double f = 1.0 / sqrt(ss);
      for (int i = 0; i < ny; ++i) ph[(size_t)i * nx] *= f;
    }
  }
  // unit norm and sign (positive), Rayleigh quotient and projection of the
  // source column
  const double sc = copysign(1.0 / sqrt(ss), sum);
  double rq = 0.0, prev = 0.0, cur = sc * ph[0];
  double2 jj = make_double2(0.0, 0.0);
  const double2* bc = d.b + ix;
  for (int i0 = 0; i0 < ny; i0 += U) {
    float e[U];
    double2 bv[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      v[q] = ph[row(i0 + q + 1)];
      e[q] = eps[row(i0 + q)];
      bv[q] = bc[row(i0 + q)];
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int i = i0 + q;
      if (i < ny) {
        const double next = (i + 1 < ny) ? sc * v[q] : 0.0;
        rq += cur * ((2.0 * h2 - w2 * (double)e[q]) * cur - h2 * (prev + next));
        jj.x += cur * bv[q].x;
        jj.y += cur * bv[q].y;
        ph[(size_t)i * nx] = cur;
        prev = cur;
        cur = next;
      }
    }
  }
  mu[d.off1 + ix] = rq;
  jp[d.off1 + ix] = jj;
}

// ----------------------------------------- 1D solve along x (step 2) ------
// Row i of the cyclic system: lower -cxm_i (column i-1), diagonal
// cxm_i + cxp_i + mu_i, upper -cxp_i (column i+1); row 0's lower coefficient
// beta sits in column n-1 and row n-1's upper coefficient alpha in column 0.
// With gamma = -diag_0, M = T + u v^T where T is M without the corners and
// with diag_0 - gamma, diag_{n-1} - alpha beta / gamma, u = (gamma, 0.., alpha)
// and v = (1, 0.., beta / gamma).  Then a = y - (v.y / (1 + v.z)) z with
// T y = j and T z = u.
// One wave per problem.  The elimination is a chain of n steps with a division
// each; all lanes do it, the current row in registers, on rows that they have
// laid out 64 at a time in LDS, the even lanes with the first right-hand side, the odd
// ones with the second.  Bound by the instructions of a step, all in one wave: 64
// problems of 480 columns 194 us; with both sides in every lane and the pivoting as
// selects 225.  They then divide the finished rows by their
// pivots, a row each, so that the back substitution's chain is one complex
// multiply-add a step.
struct LineRow {           // a finished row: diagonal, two entries above, right-hand sides
  double2 d, u, w, y, z;
};
__global__ __launch_bounds__(64) void k_eim_line(const EimDesc* __restrict__ desc,
                                                 const double* __restrict__ mu,
                                                 const double2* __restrict__ jp,
                                                 LineRow* __restrict__ rows,
                                                 double2* __restrict__ amp) {
  const EimDesc d = desc[blockIdx.x];
  const int n = d.nx, lane = threadIdx.x;
  const size_t o = d.off1;
  const double2* cxm = d.cf;
  const double2* cxp = d.cf + n;
  LineRow* R = rows + o;
  __shared__ double2 sub_l[64], dg_l[64], up_l[64], j_l[64];
  __shared__ LineRow r_l[64];
  const double2 zero = make_double2(0.0, 0.0);
  auto neg = [](double2 a) { return make_double2(-a.x, -a.y); };
  const double2 beta = neg(cxm[0]), alpha = neg(cxp[n - 1]);
  const double2 diag0 = make_double2(cxm[0].x + cxp[0].x + mu[o], cxm[0].y + cxp[0].y);
  const double2 gamma = neg(diag0);
  const double2 bg = zdiv(beta, gamma);
  // elimination with partial pivoting; the current row's diagonal, upper entry
  // and right-hand side: j in the even lanes, u in the odd ones
  const int odd = lane & 1;
  double2 cd = zero, cu = zero, c = zero;
  for (int i0 = 0; i0 < n; i0 += 64) {
    const int i = i0 + lane;
    __syncthreads();
    if (i < n) {
      double2 t = make_double2(cxm[i].x + cxp[i].x + mu[o + i], cxm[i].y + cxp[i].y);
      if (i == 0) t = zsub(t, gamma);
      if (i == n - 1) t = zsub(t, zmul(alpha, bg));
      sub_l[lane] = neg(cxm[i]);
      dg_l[lane] = t;
      up_l[lane] = (i < n - 1) ? neg(cxp[i]) : zero;
      j_l[lane] = jp[o + i];
    }
    __syncthreads();
    const int m = min(64, n - i0);
    for (int q = 0; q < m; ++q) {
      // row i0 + q joins: it is eliminated by, or takes the place of, the current row
      const double2 sub = sub_l[q], dg = dg_l[q], up = up_l[q];
      const int r = i0 + q;
      double2 j = odd ? zero : j_l[q];
      if (odd && r == 0) j = zadd(j, gamma);
      if (odd && r == n - 1) j = zadd(j, alpha);
      if (r == 0) {
        cd = dg;
        cu = up;
        c = j;
        continue;
      }
      // finished row r - 1, and the current row less f times it; the lanes agree on
      // the pivot, so it is a branch
      LineRow* fin = R + r - 1;
      if (__builtin_amdgcn_readfirstlane(zabs2(cd) >= zabs2(sub))) {
        const double2 f = zdiv(sub, cd);
        if (lane == 0) fin->d = cd, fin->u = cu, fin->w = zero;
        if (lane < 2) (&fin->y)[lane] = c;
        cd = zsub(dg, zmul(f, cu));
        cu = up;
        c = zsub(j, zmul(f, c));
      } else {
        const double2 f = zdiv(cd, sub);
        if (lane == 0) fin->d = sub, fin->u = dg, fin->w = up;
        if (lane < 2) (&fin->y)[lane] = j;
        cd = zsub(cu, zmul(f, dg));
        cu = zsub(zero, zmul(f, up));
        c = zsub(c, zmul(f, j));
      }
    }
  }
  if (lane == 0) R[n - 1].d = cd, R[n - 1].u = zero, R[n - 1].w = zero;
  if (lane < 2) (&R[n - 1].y)[lane] = c;
  __threadfence_block();
  __syncthreads();
  // back substitution of both right-hand sides, y_i and z_i left in the rows
  double2 y1 = zero, y2 = zero;
  for (int i0 = (n - 1) / 64 * 64; i0 >= 0; i0 -= 64) {
    const int m = min(64, n - i0);
    __syncthreads();
    if (lane < m) {
      LineRow a = R[i0 + lane];
      const double2 inv = zdiv(make_double2(1.0, 0.0), a.d);
      a.u = zmul(a.u, inv);
      a.w = zmul(a.w, inv);
      a.y = zmul(a.y, inv);
      a.z = zmul(a.z, inv);
      r_l[lane] = a;
    }
    __syncthreads();
    for (int q = m - 1; q >= 0; --q) {
      const double2 y = zsub(zsub((&r_l[q].y)[odd], zmul(r_l[q].w, y2)), zmul(r_l[q].u, y1));
      if (lane < 2) (&R[i0 + q].y)[lane] = y;
      y2 = y1;
      y1 = y;
    }
  }
  __threadfence_block();
  __syncthreads();
  const double2 vy = zadd(R[0].y, zmul(bg, R[n - 1].y));
  const double2 vz = zadd(make_double2(1.0 + R[0].z.x, R[0].z.y), zmul(bg, R[n - 1].z));
  const double2 f = zdiv(vy, vz);
  for (int i = lane; i < n; i += 64) amp[o + i] = zsub(R[i].y, zmul(f, R[i].z));
}

// ------------------------------------------------------ field (step 3) ----
__global__ __launch_bounds__(256) void k_eim_assemble(const EimDesc* __restrict__ desc,
                                                      const double* phi,
                                                      const double2* __restrict__ amp) {
  const EimDesc d = desc[blockIdx.y];
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= d.nx * d.ny) return;
  const int ix = e % d.nx;
  const double2 a = amp[d.off1 + ix];
  const double v = phi ? phi[d.off2 + e] : ((const double*)d.F)[e];
  d.F[e] = make_float2((float)(a.x * v), (float)(a.y * v));
}

}  // namespace

// Scratch layout of one call: the modes (D doubles; only where they cannot wait in F),
// inverse pivots (D doubles); mu (nx doubles; the shifts until the modes are known); j,
// the finished rows of the line system (five values), amplitude (nx complex each); then
// the descriptor table.  Every word is written by the kernels before it is read, so
// nothing needs clearing between calls.
static size_t even(size_t n) { return (n + 1) & ~(size_t)1; }   // 16-byte alignment for what follows
static size_t eim_used_bytes(size_t s2, size_t s1, int nb, bool apart) {
  return sizeof(double) * ((apart ? 2 * s2 : even(s2)) + even(s1)) + sizeof(double2) * 7 * s1 +
         sizeof(EimDesc) * nb;
}
// The size that a call is charged with where the caller or the library provides the
// scratch: room for the modes, whether this call needs it or not.
static size_t eim_scratch_bytes(size_t s2, size_t s1, int nb) {
  return eim_used_bytes(s2, s1, nb, true);
}

// Whether an output shares memory with a right-hand side or another output: the modes
// then have to wait in scratch.
static bool eim_shared(const std::vector<EimDesc>& hd) {
  std::vector<std::pair<uintptr_t, uintptr_t>> out, in;   // [begin, end)
  for (const auto& d : hd) {
    const size_t D = (size_t)d.nx * d.ny;
    out.push_back({(uintptr_t)d.F, (uintptr_t)(d.F + D)});
    in.push_back({(uintptr_t)d.b, (uintptr_t)(d.b + D)});
  }
  std::sort(out.begin(), out.end());
  std::sort(in.begin(), in.end());
  for (size_t i = 1; i < out.size(); ++i)
    if (out[i].first < out[i - 1].second) return true;
  // the outputs are apart: one pass over both lists (right-hand sides may repeat)
  uintptr_t end = 0;          // of the right-hand sides that begin before this output's end
  size_t q = 0;
  for (const auto& f : out) {
    for (; q < in.size() && in[q].first < f.second; ++q) end = std::max(end, in[q].second);
    if (end > f.first) return true;
  }
  return false;
}

// Validates the arguments and fills the descriptor table; returns the
// scratch bytes the call needs (0 on an invalid argument, message set).
static size_t eim_prepare(const char* who, const fdfd_op* const* ops, int nb,
                          const void* const* b, void* const* F, std::vector<EimDesc>& hd,
                          size_t& s1, int& maxnx, int& maxD) {
  if (!ops || !b || !F || nb < 1) {
    dd_set_error("%s: need nb >= 1 and the ops, b and F arrays", who);
    return 0;
  }
  hd.resize(nb);
  size_t s2 = 0;
  s1 = 0;
  maxnx = 0;
  maxD = 0;
  for (int p = 0; p < nb; ++p) {
    if (!ops[p] || !b[p] || !F[p]) {
      dd_set_error("%s: problem %d has a NULL operator, b or F", who, p);
      return 0;
    }
    const fdfd_op* op = ops[p];
    EimDesc& d = hd[p];
    d.nx = op->nx; d.ny = op->ny; d.omega = op->omega; d.dx = op->dx;
    d.eps = op->eps32; d.cf = op->cf64;
    d.b = (const double2*)b[p]; d.F = (float2*)F[p];
    d.off2 = s2; d.off1 = s1;
    s2 += (size_t)op->D;
    s1 += (size_t)op->nx;
    maxnx = std::max(maxnx, op->nx);
    maxD = std::max(maxD, op->D);
  }
  return eim_scratch_bytes(s2, s1, nb);
}

// Enqueues the four kernels on scratch ws (eim_scratch_bytes long) and waits
// for them.
static hipError_t eim_run(const std::vector<EimDesc>& hd, size_t s1, int maxnx, int maxD,
                          char* ws, hipStream_t stream) {
  const int nb = (int)hd.size();
  size_t s2 = 0;
  for (const auto& d : hd) s2 += (size_t)d.nx * d.ny;
  const bool apart = eim_shared(hd);
  double* phi = apart ? (double*)ws : nullptr;
  double* piv = (double*)ws + (apart ? s2 : 0);
  double* mu = (double*)ws + (apart ? 2 * s2 : even(s2));
  double2* z = (double2*)(mu + even(s1));
  double2 *jp = z, *amp = z + 6 * s1;
  LineRow* rows = (LineRow*)(z + s1);
  static_assert(sizeof(LineRow) == 5 * sizeof(double2), "five values a row");
  int maxny = 0;
  for (const auto& d : hd) maxny = std::max(maxny, d.ny);
  EimDesc* dd = (EimDesc*)(z + 7 * s1);
  hipError_t e = hipMemcpyAsync(dd, hd.data(), sizeof(EimDesc) * nb, hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) {
    // the permittivities of 16 columns fit the 64 KB of LDS up to 1024 rows
    const dim3 gb((maxnx + 15) / 16, nb);
    if (maxny <= 1024) k_eim_bound<true><<<gb, 64, (size_t)maxny * 64, stream>>>(dd, mu);
    else k_eim_bound<false><<<gb, 64, 0, stream>>>(dd, mu);
    k_eim_modes<<<dim3((maxnx + DD_EIM_COLS - 1) / DD_EIM_COLS, nb), DD_EIM_COLS, 0, stream>>>(dd, phi, piv,
                                                                                               mu, jp);
    k_eim_line<<<nb, 64, 0, stream>>>(dd, mu, jp, rows, amp);
    k_eim_assemble<<<dim3((maxD + 255) / 256, nb), 256, 0, stream>>>(dd, phi, amp);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  return e;
}

extern "C" dd_status eim_field(const fdfd_op* const* ops, int nb, const void* const* b,
                               void* const* F, hipStream_t stream) {
  std::vector<EimDesc> hd;
  size_t s1 = 0;
  int maxnx = 0, maxD = 0;
  const size_t bytes = eim_prepare("eim_field", ops, nb, b, F, hd, s1, maxnx, maxD);
  if (bytes == 0) return DD_EINVAL;
  size_t s2 = 0;
  for (const auto& d : hd) s2 += (size_t)d.nx * d.ny;
  char* ws = nullptr;
  DD_HIP_CHECK(hipMalloc((void**)&ws, eim_used_bytes(s2, s1, nb, eim_shared(hd))));
  hipError_t e = eim_run(hd, s1, maxnx, maxD, ws, stream);
  (void)hipFree(ws);
  if (e != hipSuccess) {
    dd_set_error("eim_field: %s", hipGetErrorString(e));
    return DD_EHIP;
  }
  return DD_OK;
}

// eim_field on a workspace the caller owns (ws_bytes >= eim_ws_bytes of the
// batch): used by the predictor, which holds one for its largest batch.
size_t eim_ws_bytes(int nx, int ny, int nb) {
  return eim_scratch_bytes((size_t)nx * ny * nb, (size_t)nx * nb, nb);
}

dd_status eim_field_ws(const fdfd_op* const* ops, int nb, const void* const* b, void* const* F,
                       void* ws, size_t ws_bytes, hipStream_t stream) {
  std::vector<EimDesc> hd;
  size_t s1 = 0;
  int maxnx = 0, maxD = 0;
  const size_t bytes = eim_prepare("eim_field", ops, nb, b, F, hd, s1, maxnx, maxD);
  if (bytes == 0) return DD_EINVAL;
  if (!ws || bytes > ws_bytes) {
    dd_set_error("eim_field: the batch needs %zu bytes of workspace, %zu given", bytes, ws_bytes);
    return DD_EINVAL;
  }
  const hipError_t e = eim_run(hd, s1, maxnx, maxD, (char*)ws, stream);
  if (e != hipSuccess) {
    dd_set_error("eim_field: %s", hipGetErrorString(e));
    return DD_EHIP;
  }
  return DD_OK;
}

// ------------------------------------------- allocation-free variant ----
// The scratch of eim_field_noalloc: a file-scope device array, one copy per
// GPU, held until the process ends.  Host code never uses its name as an
// address: eim_scratch_ptr() resolves the current device's copy once with
// hipGetSymbolAddress and every kernel argument and copy goes through that
// pointer.
static __device__ __align__(256) char eim_scratch[DD_EIM_NOALLOC_BYTES];

static std::mutex g_eim_scratch_mu;
static void* g_eim_scratch_ptr[DD_EIM_MAX_DEVICES];

static dd_status eim_scratch_ptr(char** out) {
  int dev = 0;
  DD_HIP_CHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= DD_EIM_MAX_DEVICES) {
    dd_set_error("eim_field_noalloc: device %d beyond the %d supported", dev, DD_EIM_MAX_DEVICES);
    return DD_EINVAL;
  }
  std::lock_guard<std::mutex> lock(g_eim_scratch_mu);
  if (!g_eim_scratch_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(eim_scratch));
    if (e != hipSuccess || !ptr) {
      dd_set_error("eim_field_noalloc: hipGetSymbolAddress: %s", hipGetErrorString(e));
      return DD_EHIP;
    }
    g_eim_scratch_ptr[dev] = ptr;
  }
  *out = (char*)g_eim_scratch_ptr[dev];
  return DD_OK;
}

extern "C" dd_status eim_field_noalloc(const fdfd_op* const* ops, int nb, const void* const* b,
                                       void* const* F, hipStream_t stream) {
  std::vector<EimDesc> hd;
  size_t s1 = 0;
  int maxnx = 0, maxD = 0;
  const size_t bytes = eim_prepare("eim_field_noalloc", ops, nb, b, F, hd, s1, maxnx, maxD);
  if (bytes == 0) return DD_EINVAL;
  if (bytes > (size_t)DD_EIM_NOALLOC_BYTES) {
    dd_set_error("eim_field_noalloc: the batch needs %zu bytes of scratch, more than the %zu "
                 "the library holds (split the batch, or call eim_field)",
                 bytes, (size_t)DD_EIM_NOALLOC_BYTES);
    return DD_EINVAL;
  }
  char* ws = nullptr;
  dd_status rc = eim_scratch_ptr(&ws);
  if (rc != DD_OK) return rc;
  const hipError_t e = eim_run(hd, s1, maxnx, maxD, ws, stream);
  if (e != hipSuccess) {
    dd_set_error("eim_field_noalloc: %s", hipGetErrorString(e));
    return DD_EHIP;
  }
  return DD_OK;
}
