// One-sweep Arnoldi step: the update of step j, the stencil and
// the dot products of step j + 1 in one pass over the basis.
//
// The Krylov vectors are normalised one step late, q_i = s_i q~_i with FP64
// scales s_i (C columns: s = 1), and z_j = A q~_j is kept unscaled beside the
// basis.  With the update coefficients g the sweep forms
//     q~_{j+1} = zs z_j - sum_v g_v b_v,      b = [C, q~_0 .. q~_j],
// then z_{j+1} = A q~_{j+1} and its raw dots against [C, q~_0 .. q~_{j+1}].
// In complex64 zs and g carry a power of two that keeps ||q~_{j+1}|| at or below one
// (sw_unit): the sums of FP32 products are then of the size of ||A||^2 at most, whatever
// the unit of length, and no result changes by it.
//
// The stencil needs q~_{j+1} on the cells around, so a workgroup walks a strip
// of up to 62 columns (64 lanes with one halo column on either side) down the
// rows and recomputes the halos.  Its eight waves share the basis vectors, not
// the columns: wave w holds the vectors w, w + 8, ... of the whole strip row,
// PER of them, in registers.  Each row the waves exchange their parts of the
// sum through LDS (one barrier; the buffer alternates) and every wave adds the
// eight parts, so that all of them know the new row and apply the stencil to
// the row behind without a second barrier; the wave's dots then use the basis
// values of that row, which are still in its registers.  Every basis value is
// fetched once.  Four register sets rotate: the row behind, the row being
// updated and two rows in flight (about 120 KB per compute unit at 121
// vectors, against the 50 KB that cover the latency of HBM at its rate).
//
// The dots accumulate in FP32 over at most DD_SW_FOLD rows, are then summed
// over the 64 columns and added in FP64: one FP64 partial sum per tile and value,
// added over the tiles in a fixed order by k_post_sweep.
//
// Loads go through buffer descriptors whose range check stands for the bounds:
// vectors past the basis and lanes outside the strip read as zero and move
// nothing.
#pragma once

#include "solver.h"

#define DD_SW_COLS 62                 // owned columns of a strip, at most
#define DD_SW_MAXN 128                // basis vectors
#define DD_SW_TWO 24                  // rows a workgroup from which on there are two per CU
#define DD_SW_FOLD 32                 // rows between the FP64 additions
#define DD_SW_OUT 0x80000000u         // an offset past every descriptor's range

typedef unsigned int sw_u2 __attribute__((ext_vector_type(2)));
typedef unsigned int sw_u4 __attribute__((ext_vector_type(4)));

// A value that no kernel writes while this one runs, at a uniform address:
// a scalar load, which does not queue behind the vector loads in flight.
template <typename X> __device__ __forceinline__ X ld_uni(const X* p) {
  return *(const __attribute__((address_space(4))) X*)p;
}
__device__ __forceinline__ float2 ld_uni(const float2* p) {
  const auto q = (const __attribute__((address_space(4))) float*)p;
  return make_float2(q[0], q[1]);
}
__device__ __forceinline__ double2 ld_uni(const double2* p) {
  const auto q = (const __attribute__((address_space(4))) double*)p;
  return make_double2(q[0], q[1]);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t sw_rsrc(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ double sw_f64(unsigned lo, unsigned hi) {
  return __hiloint2double((int)hi, (int)lo);
}
// A complex and a real value of type T through a descriptor.
template <typename T> __device__ __forceinline__ c2<T> sw_ldc(__amdgpu_buffer_rsrc_t r, unsigned off) {
  if constexpr (sizeof(T) == 4) {
    const sw_u2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
    return make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
  } else {
    const sw_u4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
    return make_double2(sw_f64(v.x, v.y), sw_f64(v.z, v.w));
  }
}
template <typename T> __device__ __forceinline__ T sw_ldr(__amdgpu_buffer_rsrc_t r, unsigned off) {
  if constexpr (sizeof(T) == 4) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
  } else {
    const sw_u2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
    return sw_f64(v.x, v.y);
  }
}
__device__ __forceinline__ float sw_fma(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double sw_fma(double a, double b, double c) { return fma(a, b, c); }

template <typename T> struct OpP;
template <> struct OpP<float> {
  template <typename D> static __device__ __forceinline__ const float2* cf(const D& d) { return d.cf32; }
  template <typename D> static __device__ __forceinline__ const float* eps(const D& d) { return d.eps32; }
};
template <> struct OpP<double> {
  template <typename D> static __device__ __forceinline__ const double2* cf(const D& d) { return d.cf64; }
  template <typename D> static __device__ __forceinline__ const double* eps(const D& d) { return d.eps64; }
};

// Strips of a grid of nx columns, and their common width.
__host__ __device__ inline int sw_strips(int nx) { return (nx + DD_SW_COLS - 1) / DD_SW_COLS; }
__host__ __device__ inline int sw_width(int nx) {
  const int s = sw_strips(nx);
  return (nx + s - 1) / s;
}

// One tile: rows [y0, y0 + rows) of a strip of problem p, with what a workgroup
// needs to know of the problem, so that it addresses the basis after one load.
// The second Gram-Schmidt pass has no stencil: its one strip's rows are runs of
// 64 cells.
struct SweepTile {
  int p, strip, y0, rows;
  int nx, ny, k, pad;
  size_t Dp;
  void *basis, *Z;
  const void *cf, *eps, *pl, *pr;   // of the inner precision
  double omega2;
};

// Workgroup b of the G that walk the tiles takes the tiles sw_first(b) + r G.
// Workgroup b runs on XCD b % 8: each XCD has neighbouring tiles.
__device__ __forceinline__ int sw_first(int b, int G) {
  return (G % 8 == 0) ? (b % 8) * (G / 8) + b / 8 : b;
}
// The record of tile t stands where its workgroup finds it without knowing G
// first: workgroup b's r-th at r G + b.
template <bool PASS2> __device__ __forceinline__ int sw_position(int t, int G) {
  if (PASS2 || G % 8 != 0) return t;
  const int g = t % G;
  return t - g + g % (G / 8) * 8 + g / (G / 8);
}

// complex128 has the range for ||A||^4
template <typename T> constexpr bool sw_has_unit = sizeof(T) == 4;
// The power of two f = 2^-h with f ||A q_j|| in (1/4, 1], from zz = ||A q~_j||^2 and un
// = ||q~_j||^2: the vector that is left of A q_j, times f, is stored.  By the exponents
// alone, so that it does not wait for the square root of un; 1 if a sum is zero or not
// finite.
__device__ __forceinline__ int sw_unit(double zz, double un) {
  const int ez = __double2hiint(zz) >> 20, eu = __double2hiint(un) >> 20;
  const bool ok = (unsigned)(ez - 1) < 0x7feu && (unsigned)(eu - 1) < 0x7feu;
  return ok ? min(max((ez - eu + 2) >> 1, -1000), 1000) : 0;   // zz / un < 2^(ez - eu + 1)
}
__device__ __forceinline__ double sw_pow2(int e) { return __hiloint2double((1023 + e) << 20, 0); }

template <bool PASS2> __device__ __forceinline__ int sw_plan_strips(const ProbDesc& d) {
  return PASS2 ? 1 : sw_strips(d.nx);
}
template <bool PASS2> __device__ __forceinline__ int sw_plan_rows(const ProbDesc& d) {
  return PASS2 ? (d.D + 63) / 64 : d.ny;
}

// Cuts the active problems into the tiles of one cycle's sweeps: strips times
// bands of h rows, the same h for all, chosen so that the tiles fill the fewest
// row steps of G workgroups (a tile takes h + 2 of them: the halo rows are
// recomputed), with at most `most` tiles.  G is one workgroup per compute unit
// (ncu), or two where that leaves each of them DD_SW_TWO rows or more: up to 64
// vectors two are resident, and one computes while the other waits.  Measured
// per step: 64 problems of 480 x 240 729 us with one and 708 with two, one such
// problem alone 28 and 33 us.  Within a problem the strips of a
// band follow each other, so that the workgroups that walk neighbouring strips
// run at the same time on the same XCD and its L2 serves the cache lines that
// the strips share at their edges: 62 columns are 496 bytes, which touch five
// lines of 128.  A problem's tiles, and with them its partial sums, are
// consecutive from tile0[p].
template <typename T, bool PASS2>
__global__ __launch_bounds__(DD_BLOCK) void k_sweep_plan(PlanDev P, int ncu, int most) {
  const SweepPlan& W = PASS2 ? P.sw2 : P.sw;
  __shared__ int cnt[DD_BLOCK];
  __shared__ long long best_l[DD_BLOCK];
  const int t = threadIdx.x;
  // thread t judges the heights t + 1, t + 257, ...
  long long best = 1ll << 62, rows = 0;
  int nymax = 1;
  for (int p = 0; p < P.nb; ++p)
    if (P.stI[p * ST_NI + ST_ACTIVE] != 0) {
      nymax = max(nymax, sw_plan_rows<PASS2>(P.desc[p]));
      rows += (long long)sw_plan_strips<PASS2>(P.desc[p]) * sw_plan_rows<PASS2>(P.desc[p]);
    }
  const int G = (rows >= 2ll * ncu * DD_SW_TWO) ? 2 * ncu : ncu;
  for (int h = t + 1; h <= nymax; h += DD_BLOCK) {
    long long n = 0;
    for (int p = 0; p < P.nb; ++p)
      if (P.stI[p * ST_NI + ST_ACTIVE] != 0)
        n += (long long)sw_plan_strips<PASS2>(P.desc[p]) *
             ((sw_plan_rows<PASS2>(P.desc[p]) + h - 1) / h);
    if (n <= most || h == nymax) {
      const long long steps = (n + G - 1) / G * (h + 2);
      best = min(best, (steps << 31) | (unsigned)h);
    }
  }
  best_l[t] = best;
  __syncthreads();
  for (int o = DD_BLOCK / 2; o >= 1; o >>= 1) {
    if (t < o) best_l[t] = min(best_l[t], best_l[t + o]);
    __syncthreads();
  }
  const int h = (int)(best_l[0] & 0x7fffffff);
  int done = 0;
  for (int b = 0; b < P.nb; b += DD_BLOCK) {
    const int p = b + t;
    int r = 0, strips = 1;
    if (p < P.nb && P.stI[p * ST_NI + ST_ACTIVE] != 0) {
      strips = sw_plan_strips<PASS2>(P.desc[p]);
      r = strips * ((sw_plan_rows<PASS2>(P.desc[p]) + h - 1) / h);
    }
    cnt[t] = r;
    __syncthreads();
    for (int o = 1; o < DD_BLOCK; o <<= 1) {
      const int x = (t >= o) ? cnt[t - o] : 0;
      __syncthreads();
      cnt[t] += x;
      __syncthreads();
    }
    if (p < P.nb) {
      W.tile0[p] = done + cnt[t] - r;
      W.ntile[p] = r;
      if (!PASS2) P.live[p] = r > 0;
    }
    done += cnt[DD_BLOCK - 1];
    __syncthreads();
  }
  for (int i = t; i < done; i += DD_BLOCK) {
    int p = 0, e = P.nb;           // the last problem whose tiles start at or before i
    while (e - p > 1) {
      const int c = (p + e) / 2;
      if (W.tile0[c] <= i) p = c;
      else e = c;
    }
    const ProbDesc& d = P.desc[p];
    const int strips = sw_plan_strips<PASS2>(d), ny = sw_plan_rows<PASS2>(d), q = i - W.tile0[p];
    const int y0 = q / strips * h;
    W.tiles[sw_position<PASS2>(i, G)] = {
        p, q % strips, y0, min(h, ny - y0), d.nx, d.ny, d.k, 0, (size_t)d.Dp, d.basis, d.Z,
        OpP<T>::cf(d), OpP<T>::eps(d), d.pl, d.pr, d.omega2};
  }
  if (t == 0) {
    W.count[0] = done;
    W.count[1] = G;
  }
}

// Adds the lanes' dots to the wave's sums: lanes 2 i and 2 i + 1 hold value i
// (real and imaginary parts alternate).
template <typename T, int PER>
__device__ __forceinline__ void sw_fold(c2<T> (&acc)[PER], double& dsum, int lane) {
  T v[32];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    v[2 * i] = (i < PER) ? acc[i < PER ? i : 0].x : T(0);
    v[2 * i + 1] = (i < PER) ? acc[i < PER ? i : 0].y : T(0);
  }
  butterfly_step<T, 32>(v, lane);
  dsum += (double)(v[0] + __shfl_xor(v[0], 1, 64));
#pragma unroll
  for (int i = 0; i < PER; ++i) acc[i] = cmk<c2<T>>(T(0), T(0));
}

template <typename T, int PER> struct SweepRow {
  c2<T> b[PER];           // the wave's basis values at its lane's column
  c2<T> z;                // z_j (last wave; zero in the others)
  T eps;
  c2<T> pr, pl;           // diagonal preconditioner
};

// The lane's neighbours in the wave (0 past its ends): DPP shifts by one lane.
template <int CTRL> __device__ __forceinline__ float sw_dpp(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xf, 0xf, false));
}
template <int CTRL> __device__ __forceinline__ double sw_dpp(double x) {
  return __hiloint2double(
      __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, false),
      __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, false));
}
template <typename V> __device__ __forceinline__ V from_west(V v) {
  return cmk<V>(sw_dpp<0x138>(v.x), sw_dpp<0x138>(v.y));
}
template <typename V> __device__ __forceinline__ V from_east(V v) {
  return cmk<V>(sw_dpp<0x130>(v.x), sw_dpp<0x130>(v.y));
}

// NW waves of PER vectors each.  PC: the problems carry a diagonal
// preconditioner, z = P_L A P_R q~.
template <typename T, int NW, int PER, bool PC>
__global__ __launch_bounds__(64 * NW, 2) void k_sweep(PlanDev P, int j) {
  // Each level of these scalar loads is a latency that a short step feels: the
  // tile's record is loaded beside the counts, whether there is one or not, and
  // the basis is addressed from it.  Through the count, the tile and the problem's
  // descriptor in turn a step of one 480 x 240 problem took 24.3 us, so 23.5; one
  // of 192 x 96 15.7 and 15.0.
  const auto* tl = (const __attribute__((address_space(4))) SweepTile*)(P.sw.tiles) + blockIdx.x;
  const int count = ld_uni(P.sw.count), G = ld_uni(P.sw.count + 1);
  int nrows = tl->rows;
  asm volatile("" : "+s"(nrows));
  if ((int)blockIdx.x >= G) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  using V = c2<T>;
  constexpr unsigned CB = sizeof(V);                // bytes of a cell's value
  __shared__ V part[2][NW][64];
  const V zero = cmk<V>(T(0), T(0));

  for (int tile = sw_first(blockIdx.x, G); tile < count; tile += G, tl += G) {
    const int p = tl->p, strip = tl->strip, ya = tl->y0;
    nrows = tl->rows;
    const int nx = tl->nx, ny = tl->ny, k = tl->k, n = k + j + 1;
    const size_t Dp = tl->Dp;
    int act = ld_uni(P.stI + p * ST_NI + ST_ACTIVE);
    const V* cS = (const V*)P.coefS + (size_t)p * DD_SW_MAXN + wave;
    V gc[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) gc[i] = ld_uni(cS + NW * i);
    const T zs = (T)ld_uni(P.zs + p);
    const V* B = (const V*)tl->basis + (size_t)(P.kmax - k) * Dp;
    V* qn = (V*)tl->basis + (size_t)(P.kmax + j + 1) * Dp;
    const V* zin = (const V*)tl->Z + (size_t)(j & 1) * Dp;
    V* zout = (V*)tl->Z + (size_t)((j + 1) & 1) * Dp;
    const V* cf = (const V*)tl->cf;
    const T om2 = (T)tl->omega2;
    const __amdgpu_buffer_rsrc_t rB = sw_rsrc(B, (size_t)n * Dp * CB);
    const __amdgpu_buffer_rsrc_t rZ = sw_rsrc(zin, (size_t)Dp * CB);
    const __amdgpu_buffer_rsrc_t rE = sw_rsrc(tl->eps, (size_t)nx * ny * (CB / 2));
    const bool has_pl = PC && tl->pl != nullptr, has_pr = PC && tl->pr != nullptr;
    const __amdgpu_buffer_rsrc_t rL = sw_rsrc(has_pl ? tl->pl : B, has_pl ? (size_t)Dp * CB : 0);
    const __amdgpu_buffer_rsrc_t rR = sw_rsrc(has_pr ? tl->pr : B, has_pr ? (size_t)Dp * CB : 0);
    const unsigned vec = (unsigned)Dp * CB;         // bytes of one vector
    V acc[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) acc[i] = zero;
    V accn = zero;                              // conj(q~_{j+1}) z_{j+1}
    T un2 = T(0), zz2 = T(0);                      // ||q~_{j+1}||^2, ||z_{j+1}||^2
    double dsum = 0.0, dn0 = 0.0, dn1 = 0.0, dn2 = 0.0, dn3 = 0.0;
    auto fold = [&]() {
      sw_fold<T, PER>(acc, dsum, lane);
      if (wave == 0) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
          accn.x += __shfl_xor(accn.x, o, 64);
          accn.y += __shfl_xor(accn.y, o, 64);
          un2 += __shfl_xor(un2, o, 64);
          zz2 += __shfl_xor(zz2, o, 64);
        }
        dn0 += (double)accn.x;
        dn1 += (double)accn.y;
        dn2 += (double)un2;
        dn3 += (double)zz2;
        accn = zero;
        un2 = zz2 = T(0);
      }
    };

    const int sw = sw_width(nx), x0 = strip * sw;
    const int w = min(sw, nx - x0);                          // owned columns (may be 0)
    const bool lane_ok = lane <= w + 1;
    const bool owned = lane >= 1 && lane <= w;
    int c = x0 - 1 + lane;
    c = (c < 0) ? c + nx : ((c >= nx) ? c - nx : c);
    c = lane_ok ? c : 0;
    V cxm = zero, cxp = zero;
    if (owned) {
      cxm = cf[c];
      cxp = cf[nx + c];
    }
    const int N = nrows + 2;
    // rows in flight before they are needed: two, in complex128 (whose sets are
    // twice as large) none
    constexpr int AHEAD = sizeof(T) == 4 ? 2 : 0;
    SweepRow<T, PER> S0, S1, S2, S3;
    // byte offsets of the lane's cell in row 0 of the wave's first vector, of z
    // and of eps; a row adds the same to every lane
    const unsigned ob = lane_ok ? (unsigned)c * CB + (unsigned)wave * vec : DD_SW_OUT;
    const unsigned oz = (lane_ok && wave == NW - 1) ? (unsigned)c * CB : DD_SW_OUT;
    const unsigned oe = lane_ok ? (unsigned)c * (CB / 2) : DD_SW_OUT;
    auto load = [&](SweepRow<T, PER>& s, int t) {
      int y = ya - 1 + t;
      y = (y < 0) ? y + ny : ((y >= ny) ? y - ny : y);
      // rows past the tile are not fetched (a lane outside the strip may wrap
      // into the range there: it is read and not used)
      const unsigned row = (t < N) ? (unsigned)(y * nx) * (CB / 2) : DD_SW_OUT / 2;
      unsigned o = ob + 2 * row;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        s.b[i] = sw_ldc<T>(rB, o);
        o += NW * vec;
        asm("" : "+v"(o));      // one running offset: the multiples would fill the scalar registers
      }
      s.z = sw_ldc<T>(rZ, oz + 2 * row);
      s.eps = sw_ldr<T>(rE, oe + row);
      if (PC) {
        s.pr = sw_ldc<T>(rR, (lane_ok ? (unsigned)c * CB : DD_SW_OUT) + 2 * row);
        s.pl = sw_ldc<T>(rL, (lane_ok ? (unsigned)c * CB : DD_SW_OUT) + 2 * row);
      }
    };
    // the new row's values one and two rows back: q~, P_R q~ and its
    // neighbours to the west and east
    V u1 = zero, r1 = zero, r2 = zero, rw = zero, re = zero;
    auto step = [&](SweepRow<T, PER>& cur, SweepRow<T, PER>& prev, SweepRow<T, PER>& ahead, int t) {
      load(ahead, t + AHEAD);
      __builtin_amdgcn_sched_barrier(0);   // rows are fetched, and so waited for, in order
      const int ys = max(ya, ya + t - 2);
      const V cym = ld_uni(cf + 2 * nx + ys), cyp = ld_uni(cf + 2 * nx + ny + ys);
      V pu = cmk<V>(-zs * cur.z.x, -zs * cur.z.y);
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        pu.x = sw_fma(-gc[i].y, cur.b[i].y, sw_fma(gc[i].x, cur.b[i].x, pu.x));
        pu.y = sw_fma(gc[i].y, cur.b[i].x, sw_fma(gc[i].x, cur.b[i].y, pu.y));
      }
      part[t & 1][wave][lane] = pu;
      __syncthreads();
      V u = zero;
#pragma unroll
      for (int q = 0; q < NW; ++q) u = csub(u, part[t & 1][q][lane]);
      int y = ya - 1 + t;
      y = (y < 0) ? y + ny : ((y >= ny) ? y - ny : y);
      const bool mine = t >= 1 && t <= nrows;
      V r = u;
      if (has_pr) r = cmul(u, cur.pr);
      if (t >= 2) {
        V z = cmul(cxm, csub(r1, rw));
        z = csub(z, cmul(cxp, csub(re, r1)));
        z = cadd(z, cmul(cym, csub(r1, r2)));
        z = csub(z, cmul(cyp, csub(r, r1)));
        const T de = om2 * prev.eps;
        z.x -= de * r1.x;
        z.y -= de * r1.y;
        if (!owned) z = zero;
        if (has_pl) z = cmul(prev.pl, z);
        if (wave == 1 && owned) zout[ys * nx + c] = z;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
          acc[i].x = sw_fma(prev.b[i].y, z.y, sw_fma(prev.b[i].x, z.x, acc[i].x));
          acc[i].y = sw_fma(-prev.b[i].y, z.x, sw_fma(prev.b[i].x, z.y, acc[i].y));
        }
        if (wave == 0) {
          accn.x += u1.x * z.x + u1.y * z.y;
          accn.y += u1.x * z.y - u1.y * z.x;
          zz2 += z.x * z.x + z.y * z.y;
        }
      }
      if (wave == 0 && mine && owned) {
        qn[y * nx + c] = u;
        un2 += u.x * u.x + u.y * u.y;
      }
      rw = from_west(r);
      re = from_east(r);
      r2 = r1;
      r1 = r;
      u1 = u;
    };
    int t = 0;
    if constexpr (AHEAD == 2) {
      load(S0, 0);
      __builtin_amdgcn_sched_barrier(0);
      load(S1, 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("" : "+s"(act) : "s"(gc[0].x), "s"(gc[PER - 1].x), "s"(zs));
    if (act == 0) continue;   // ended within this cycle (the first rows are on their way by now)
    __syncthreads();          // the parts of the tile before have been read
    if constexpr (AHEAD == 2) {
      for (; t + 4 <= N; t += 4) {
        step(S0, S3, S2, t);
        step(S1, S0, S3, t + 1);
        step(S2, S1, S0, t + 2);
        step(S3, S2, S1, t + 3);
        if ((t + 4) % DD_SW_FOLD == 0) fold();
      }
      if (t < N) step(S0, S3, S2, t);
      if (t + 1 < N) step(S1, S0, S3, t + 1);
      if (t + 2 < N) step(S2, S1, S0, t + 2);
    } else {
      for (; t + 2 <= N; t += 2) {
        step(S0, S1, S0, t);
        step(S1, S0, S1, t + 1);
        if ((t + 2) % DD_SW_FOLD == 0) fold();
      }
      if (t < N) step(S0, S1, S0, t);
    }
    fold();
    double* out = (double*)P.partial + tile;
    const size_t ld = P.sw_ld;
    const int idx = lane >> 1, v = wave + NW * (idx >> 1);
    if ((lane & 1) == 0 && idx < 2 * PER && v < n) out[(2 * v + (idx & 1)) * ld] = dsum;
    if (wave == 0 && lane == 0) {
      out[(2 * n) * ld] = dn0;
      out[(2 * n + 1) * ld] = dn1;
      out[(2 * n + 2) * ld] = dn2;
      out[(2 * n + 3) * ld] = dn3;
    }
  }
}

// Whether the step takes the second Gram-Schmidt pass: never, always, or when
// the first pass removes more than half of ||w||^2 (the test of Kahan and
// Parlett, from the sums that the kernel before left).
__device__ __forceinline__ bool sw_second_pass(const PlanDev& P, int p) {
  if (P.reorth_mode != 2) return P.reorth_mode == 1;
  const double* cc = P.ccpart + (size_t)p * 33;     // [0] ||w||^2, then the slices' parts
  const double ww = ld_uni(cc);
  double c = 0.0;
#pragma unroll
  for (int i = 1; i <= 32; ++i) c += ld_uni(cc + i);
  return ww - c < 0.5 * ww;
}

// Second Gram-Schmidt pass of step j: z_j <- zs z_j - sum_v g_v b_v in place and
// the raw dots of the result with the basis, one read of the basis.  The tiles
// are runs of 64 cells; otherwise as k_sweep, without halos and stencil: a run
// is updated and dotted at once, so three register sets rotate.
template <typename T, int NW, int PER>
__global__ __launch_bounds__(64 * NW, 2) void k_pass2(PlanDev P, int j) {
  const auto* tl = (const __attribute__((address_space(4))) SweepTile*)(P.sw2.tiles) + blockIdx.x;
  const int count = ld_uni(P.sw2.count), G = ld_uni(P.sw2.count + 1);
  int N = tl->rows;
  asm volatile("" : "+s"(N));
  if ((int)blockIdx.x >= G) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  using V = c2<T>;
  constexpr unsigned CB = sizeof(V);                // bytes of a cell's value
  __shared__ V part[2][NW][64];
  const V zero = cmk<V>(T(0), T(0));

  for (int tile = blockIdx.x; tile < count; tile += G, tl += G) {
    const int p = tl->p, ya = tl->y0, k = tl->k, n = k + j + 1, cells = tl->nx * tl->ny;
    N = tl->rows;
    int act = ld_uni(P.stI + p * ST_NI + ST_ACTIVE);
    const bool second = sw_second_pass(P, p);
    asm volatile("" : "+s"(act));
    if (act == 0 || !second) continue;
    const size_t Dp = tl->Dp;
    const V* B = (const V*)tl->basis + (size_t)(P.kmax - k) * Dp;
    V* z = (V*)tl->Z + (size_t)(j & 1) * Dp;
    const __amdgpu_buffer_rsrc_t rB = sw_rsrc(B, (size_t)n * Dp * CB);
    const __amdgpu_buffer_rsrc_t rZ = sw_rsrc(z, (size_t)Dp * CB);
    const unsigned vec = (unsigned)Dp * CB;
    const V* cS = (const V*)P.coefS + (size_t)p * DD_SW_MAXN + wave;
    V gc[PER], acc[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      gc[i] = ld_uni(cS + NW * i);
      acc[i] = zero;
    }
    const T zs = (T)ld_uni(P.zs + p);
    double dsum = 0.0;
    struct Run {
      V b[PER], z;
    } S0, S1, S2;
    const unsigned ob = (unsigned)lane * CB + (unsigned)wave * vec;
    const unsigned oz = (wave == NW - 1) ? (unsigned)lane * CB : DD_SW_OUT;
    auto load = [&](Run& s, int t) {
      // a run past the tile is not fetched
      const unsigned row = (t < N) ? (unsigned)(ya + t) * (64 * CB) : DD_SW_OUT;
      unsigned o = ob + row;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        s.b[i] = sw_ldc<T>(rB, o);
        o += NW * vec;
        asm("" : "+v"(o));
      }
      s.z = sw_ldc<T>(rZ, (t < N) ? oz + row : DD_SW_OUT);
    };
    auto step = [&](Run& cur, Run& ahead, int t) {
      load(ahead, t + 2);
      __builtin_amdgcn_sched_barrier(0);
      V pu = cmk<V>(-zs * cur.z.x, -zs * cur.z.y);
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        pu.x = sw_fma(-gc[i].y, cur.b[i].y, sw_fma(gc[i].x, cur.b[i].x, pu.x));
        pu.y = sw_fma(gc[i].y, cur.b[i].x, sw_fma(gc[i].x, cur.b[i].y, pu.y));
      }
      part[t & 1][wave][lane] = pu;
      __syncthreads();
      V u = zero;
#pragma unroll
      for (int q = 0; q < NW; ++q) u = csub(u, part[t & 1][q][lane]);
      // the padding stays zero whatever the coefficients are: no later cycle clears it
      const int e = (ya + t) * 64 + lane;
      if (wave == 1 && e < cells) z[e] = u;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        acc[i].x = sw_fma(cur.b[i].y, u.y, sw_fma(cur.b[i].x, u.x, acc[i].x));
        acc[i].y = sw_fma(-cur.b[i].y, u.x, sw_fma(cur.b[i].x, u.y, acc[i].y));
      }
    };
    __syncthreads();          // the parts of the tile before have been read
    load(S0, 0);
    __builtin_amdgcn_sched_barrier(0);
    load(S1, 1);
    __builtin_amdgcn_sched_barrier(0);
    int t = 0;
    for (; t + 3 <= N; t += 3) {
      step(S0, S2, t);
      step(S1, S0, t + 1);
      step(S2, S1, t + 2);
      if ((t + 3) % (DD_SW_FOLD / 3 * 3) == 0) sw_fold<T, PER>(acc, dsum, lane);
    }
    if (t < N) step(S0, S2, t);
    if (t + 1 < N) step(S1, S0, t + 1);
    sw_fold<T, PER>(acc, dsum, lane);
    const int idx = lane >> 1, v = wave + NW * (idx >> 1);
    if ((lane & 1) == 0 && idx < 2 * PER && v < n)
      ((double*)P.partial)[(size_t)(2 * v + (idx & 1)) * P.sw_ld + tile] = dsum;
  }
}
