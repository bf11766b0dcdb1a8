// Convolutional subspace predictor (Sec. 3 CNN paragraph; Methods): forward,
// backward and Adam on gfx950, bf16 activations with FP32 accumulation on the
// matrix cores.
//
// The paper's architecture figure is not available; the layer list (the
// reading used throughout) is an encoder-decoder of eight 3x3 convolutions,
// zero padding 1, ReLU after all but the last:
//   1->32, 32->64 (stride 2), 64->128 (stride 2), 128->128,
//   x2 nearest upsample + 128->64, x2 nearest upsample + 64->32, 32->32,
//   32->2k (linear).
// The input is (eps - 2.085) / (12.25 - 2.085); output channels (2j, 2j+1)
// are the real and imaginary parts of v_j (complex inputs/outputs as images
// of depth 2, Methods).
//
// Layouts: activations NHWC bf16 with the channel count padded to a multiple
// of 16 (padded channels hold zeros); the normalised input is FP32 [B][H][W];
// the last layer's output is FP32 NHWC with 2k channels.  Master weights,
// gradients and Adam moments are FP32 in [cout][cin][3][3] + [cout] per
// layer; the GEMM copies are bf16, forward Wf[tap][coutp][cinp] and
// backward-data Wb[tap][cinp][coutp].
//
// Convolutions are implicit GEMMs on v_mfma_f32_16x16x32_bf16 with the GEMM
// rows = output channels and columns = pixels: lane l holds A[l%16][8(l/16)+i],
// B[8(l/16)+i][l%16] (i < 8) and receives C[4(l/16)+i][l%16] (i < 4), so one
// lane's results are 4 consecutive channels of one pixel (an 8-byte store).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <random>
#include <vector>

#include "common.h"
#include "op.h"
#include "predfile.h"
#include "resloss.h"

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

#define NL 8
#define CNN_EPS_LO 2.085f
#define CNN_EPS_HI 12.25f

enum { MAP_S1 = 0, MAP_S2 = 1, MAP_UP = 2 };

struct CnnLayer {
  int cin, cout, stride, up, relu;
  int cinp, coutp;           // padded channel counts (32, 64 or 128; layer 1's cin stays 1 or 3)
  int Hin, Win, Hout, Wout;  // per-image grid sizes
  size_t woff, boff;         // offsets of weights / bias in the parameter vector
  int mode;                  // MAP_S1, MAP_S2 or MAP_UP
};

struct dd_cnn {
  int nx, ny, maxB, k;
  int cin0;                  // input planes: 1 (permittivity) or 3 (+ effective-index field)
  int ncu = 1;               // compute units of the device the network was created on
  CnnLayer L[NL];
  size_t nparams = 0;
  float *params = nullptr, *grads = nullptr, *am = nullptr, *av = nullptr;
  int adam_t = 0;
  bf16* wf[NL] = {};
  bf16* wb[NL] = {};
  bf16* wu[NL] = {};         // upsampled layers: effective backward-data weights [16][cinp][coutp]
  float* x0 = nullptr;       // normalised input planes [B][cin0][H][W]
  double* espart = nullptr;  // [maxB][ES_SLICES] partial sums of |F|^2
  // residual-loss scratch (allocated on first use): V = output fields, W = A V,
  // r = b - W c, s = A^H r
  float2 *rl_W = nullptr, *rl_r = nullptr, *rl_s = nullptr;
  void* rl_scratch = nullptr;      // residual-loss descriptors, coefficients, Gram partials
  size_t rl_scratch_bytes = 0;
  bf16* act[NL] = {};        // act[l] = output of layer l (l < NL-1), NHWC bf16
  float* out = nullptr;      // last layer output: complex fields [B][k][D] (FP32 pairs)
  const float* last_fields = nullptr;   // where the last forward pass wrote its fields
  bf16* dz[NL] = {};         // gradient w.r.t. the pre-activation of layer l
  float* wpart = nullptr;    // split partial weight gradients
  size_t wpart_elems = 0;
  float* lpart = nullptr;    // loss partial sums
  float* biaspad = nullptr;  // [NL][256] zero-padded FP32 biases for the GEMM epilogue
  std::vector<void*> allocs;
};

// ------------------------------------------------------------ helpers ----
__device__ __forceinline__ bf16x8 load8(const bf16* p) {
  return __builtin_bit_cast(bf16x8, *(const u32x4*)p);
}
__device__ __forceinline__ bf16x8 zero8() {
  return __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
}
__device__ __forceinline__ float bf2f(bf16 v) { return (float)v; }

// Source pixel (in the layer-input grid) that output pixel (y, x) reads at
// tap (dy, dx); false when it falls in the zero padding.
__device__ __forceinline__ bool fwd_src(int mode, int y, int x, int dy, int dx, int Hin, int Win,
                                        int Hout, int Wout, int& ys, int& xs) {
  if (mode == MAP_S1) {
    ys = y + dy - 1; xs = x + dx - 1;
    return ys >= 0 && ys < Hin && xs >= 0 && xs < Win;
  } else if (mode == MAP_S2) {
    ys = 2 * y + dy - 1; xs = 2 * x + dx - 1;
    return ys >= 0 && ys < Hin && xs >= 0 && xs < Win;
  } else {  // upsampled grid has the output's size
    const int uy = y + dy - 1, ux = x + dx - 1;
    ys = uy >> 1; xs = ux >> 1;
    return uy >= 0 && uy < Hout && ux >= 0 && ux < Wout;
  }
}

// ------------------------------------------ convolutions as MFMA GEMMs ----
// Forward: out[p][r] = act(bias[r] + sum_{tap,c} Wf[tap][r][c] *
//   src[map(p, tap)][c]), p over output pixels, r < M = coutp.
// Backward data: dzprev[q][r] = mask(q, r) * sum_{tap,c} Wb[tap][r][c] *
//   dz[gather(q, tap)][c], q over layer-input pixels, r < M = cinp, mask = the
//   ReLU mask of the previous layer's output (the layer input).
// Operands of v_mfma_f32_16x16x32_bf16: A = 16 rows (result channels) x 32
// source channels of one tap's weights, B = 32 source channels x 16 pixels;
// lane l holds row / pixel l % 16 and channels 8 (l / 16) .. 8 (l / 16) + 7
// (16-byte reads of NHWC data); the accumulator holds rows 4 (l / 16) .. + 3
// of pixel l % 16.  MT = M / 16 row tiles.
struct GemmArgs {
  const bf16* src;       // forward: layer input; backward: dz of this layer
  const bf16* W;         // Wf or Wb
  const float* bias;     // forward only
  const bf16* mask;      // backward: layer input activations (ReLU mask)
  bf16* out;             // bf16 result (NHWC, M channels)
  float* outf;           // final layer: complex fields [B][nreal / 2][Hq Wq] (FP32 pairs)
  int nreal;             // real channels of the final layer (2 k)
  int B, Hq, Wq;         // grid of the result pixels
  int Hs, Ws;            // grid of the source pixels
  int Ksrc;              // channels of the source (multiple of 32)
  int M;                 // result channels (= 16 MT)
  int mode, relu;
};

// Final-layer epilogue: channels r0..r0+3 of pixel e of image b are (Re, Im)
// of fields r0 / 2 and r0 / 2 + 1; they go to the complex field layout
// [B][kf][D] (16 lanes with consecutive pixels write 128 contiguous bytes).
__device__ __forceinline__ void store_fields(float* outf, int kf, int D, int b, int e, int r0,
                                             const float* v) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int j = r0 / 2 + h;
    if (j < kf)
      *(float2*)(outf + (((size_t)b * kf + j) * D + e) * 2) = make_float2(v[2 * h], v[2 * h + 1]);
  }
}

// ---------------------------------------- LDS-tiled forward convolution ----
// Forward pass of the stride-1 layers, plain (MAP_S1) or after a x2 nearest
// upsample (MAP_UP), and (BWD) the backward-data pass of the plain stride-1
// layers: the gradient at a layer-input pixel gathers dz through the kernel
// rotated by 180 degrees (tap t reads weight tap 8 - t of the transposed
// copy), masked by the ReLU of the layer input.  A workgroup of TH waves computes
// a TH x 64 tile of output pixels of one image for 16 MT of the M result
// channels (blockIdx.z: image, then channel group).  For every 32 input channels
// the (TH + 2) x 66 input patch (halo included; zero padding and the upsampling
// are resolved while staging) and the weights of all nine taps are written once
// to LDS and read there by all taps, so each source value is fetched from memory
// once instead of nine times and the tap loop waits on no global load.  Wave w
// owns output row w of the tile (four pixel tiles of 16).  Operand layouts are
// those described at GemmArgs.
//
// Addresses cost the vector units next to nothing.  A thread stages one
// (column, 16-byte quarter) of every patch row: the row's offset is scalar, the
// column's is fixed, and loads and stores go through buffer descriptors whose
// range check is the zero padding and the ragged edge.  A staged pixel is 64
// bytes; quarter q of pixel p sits at q ^ ((p >> 1) & 3), which spreads the 16
// pixels of an operand read over the banks (80-byte rows took half as long
// again: 4.2 against 2.8 clocks a read).  Rows of 72 pixels keep that pattern
// the same for every row and tile, so that taps differ by constants.
#define CT_TW 64
#define CT_PW 72                      // staged row: 66 pixels used, a multiple of 8
#define CT_OUT 0x80000000u            // an offset past every descriptor's range

__device__ __forceinline__ __amdgpu_buffer_rsrc_t cnn_rsrc(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0,
                                           (int)(bytes < 0x7fffffffu ? bytes : 0x7fffffffu),
                                           0x00020000);
}
__device__ __forceinline__ u32x4 buf_load16(__amdgpu_buffer_rsrc_t r, unsigned v, unsigned s) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, v, s, 0);
}
// LDS byte of quarter q of 64-byte item p (a pixel, a weight row)
__device__ __forceinline__ int cnn_place(int p, int q) {
  return p * 64 + ((q ^ ((p >> 1) & 3)) << 4);
}

// LDS item of weight row p (of a tap's multiple of 32): row r of tile i is result
// channel 32 (i / 2) + 8 (r / 4) + 4 (i % 2) + r % 4, so that two tiles leave a lane
// 8 neighbouring channels of its pixel, read from the mask and written 16 bytes
// at a time (480 x 240: layer 2 at batch 64 213 us, with 8 bytes 238; layer 4 137 and
// 151; layer 6 backward at batch 32 138 and 162).
__device__ __forceinline__ int cnn_wrow(int p) {
  return (p & ~31) | ((p & 4) << 2) | ((p & 24) >> 1) | (p & 3);
}

template <int MT, int TH, bool BWD>
__global__ __launch_bounds__(64 * TH) void k_conv_tile(GemmArgs a) {
  constexpr int NT = 64 * TH, PH = TH + 2, RP = NT / 256;   // RP patch rows staged at a time
  __shared__ __attribute__((aligned(16))) unsigned char patch[PH * CT_PW * 64];
  // the chunk's weights, [tap][row], quarters placed as the pixels'
  __shared__ __attribute__((aligned(16))) unsigned char wl[9 * 16 * MT * 64];
  const int t0 = threadIdx.x, lane = t0 & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t0 >> 6);
  const int x0 = blockIdx.x * CT_TW, y0 = blockIdx.y * TH;
  const int nm = a.M / (16 * MT), b = blockIdx.z / nm, m0 = (blockIdx.z - b * nm) * 16 * MT;
  const int Hq = a.Hq, Wq = a.Wq;
  const int sh = (a.mode == MAP_UP) ? 1 : 0;             // source pixel = conv-input pixel >> sh
  f32x4 acc[MT][4];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int pl = lane & 15, kg = lane >> 4;
  // patch rows y0 - 1 .. y0 + TH of the conv-input grid; the descriptor starts at
  // the first source row among them
  const unsigned px2 = 2u * a.Ksrc, row2 = px2 * a.Ws;   // bytes of a source pixel, row
  const int sy0 = max(y0 - 1, 0) >> sh;
  const __amdgpu_buffer_rsrc_t rS =
      cnn_rsrc((const char*)a.src + ((size_t)b * a.Hs + sy0) * row2, (size_t)(a.Hs - sy0) * row2);
  // this thread's column of the patch rows tr, tr + RP, ..
  const int tr = (RP > 1) ? __builtin_amdgcn_readfirstlane(t0 >> 8) : 0, tc = (t0 & 255) >> 2;
  const int ux = x0 + tc - 1;
  const unsigned vcol = (ux >= 0 && ux < Wq) ? (unsigned)(ux >> sh) * px2 + 16u * (t0 & 3) : CT_OUT;
  // columns 64 and 65: eight units a row, threads 0 .. 8 PH - 1
  const int er = t0 >> 3, ex = 64 + ((t0 >> 2) & 1), euy = y0 - 1 + er, eux = x0 + ex - 1;
  const unsigned vedge =
      (er < PH && euy >= 0 && euy < Hq && eux < Wq)
          ? (unsigned)((euy >> sh) - sy0) * row2 + (unsigned)(eux >> sh) * px2 + 16u * (t0 & 3)
          : CT_OUT;
  const int lcol = cnn_place(tc, t0 & 3), ledge = cnn_place(er * CT_PW + ex, t0 & 3);
  // operands: 16 pixels at dx = 0, 1, 2 (rows and pixel tiles are constants away), 16 weight rows
  int lb[3];
#pragma unroll
  for (int dx = 0; dx < 3; ++dx) lb[dx] = cnn_place(wave * CT_PW + pl + dx, kg);
  const int lw = cnn_place(pl, kg), lws = cnn_place(cnn_wrow(t0 >> 2), t0 & 3);
  // thread t0 stages weight item (tap, row, quarter) t0 + NT it
  const unsigned tap2 = (unsigned)a.M * px2;              // bytes of a tap's weights
  const __amdgpu_buffer_rsrc_t rW = cnn_rsrc((const char*)a.W + (size_t)m0 * px2,
                                             (size_t)9 * tap2 - (size_t)m0 * px2);
  constexpr int UT = 16 * MT * 4;                         // items of a tap: 128, 256 or 512
  constexpr int NWI = 9 * UT, NWS = (NWI + NT - 1) / NT;
  const unsigned vwl = (unsigned)((t0 % UT) >> 2) * px2 + 16u * (t0 & 3);
  for (unsigned c2 = 0; c2 < px2; c2 += 64) {
    // all of this thread's loads are issued before the first LDS store
    u32x4 wv[NWS], sv[PH / RP], se;
#pragma unroll
    for (int it = 0; it < NWS; ++it) {
      if constexpr (UT >= NT) {
        const int tap = it / (UT / NT);
        wv[it] = buf_load16(rW, vwl, (unsigned)(BWD ? 8 - tap : tap) * tap2 +
                                         (unsigned)(it % (UT / NT)) * (NT / 4u) * px2 + c2);
      } else {
        const int tap = it * (NT / UT) + t0 / UT;
        wv[it] = buf_load16(rW, tap < 9 ? vwl + (unsigned)(BWD ? 8 - tap : tap) * tap2 : CT_OUT, c2);
      }
    }
#pragma unroll
    for (int r = 0; r < PH / RP; ++r) {
      const int uy = y0 - 1 + r * RP + tr;
      const bool in = uy >= 0 && uy < Hq;
      sv[r] = buf_load16(rS, in ? vcol : CT_OUT, in ? (unsigned)((uy >> sh) - sy0) * row2 + c2 : 0u);
    }
    se = buf_load16(rS, vedge, c2);
    if (c2 > 0) __syncthreads();                          // the chunk before has been read
#pragma unroll
    for (int it = 0; it < NWS; ++it)
      if (t0 + NT * it < NWI) *(u32x4*)(wl + lws + it * NT * 16) = wv[it];
#pragma unroll
    for (int r = 0; r < PH / RP; ++r) *(u32x4*)(patch + lcol + (r * RP + tr) * CT_PW * 64) = sv[r];
    if (er < PH) *(u32x4*)(patch + ledge) = se;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      bf16x8 w[MT], bv[4];
#pragma unroll
      for (int i = 0; i < MT; ++i) w[i] = *(const bf16x8*)(wl + lw + (t * MT + i) * 16 * 64);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        bv[j] = *(const bf16x8*)(patch + lb[t % 3] + ((t / 3) * CT_PW + 16 * j) * 64);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i], bv[j], acc[i][j], 0, 0, 0);
    }
  }
  const int y = y0 + wave;
  if (y >= Hq) return;
  // epilogue operands (bias, or the ReLU mask of the layer input) are all
  // loaded before any result is stored
  const size_t rowp = ((size_t)b * Hq + y) * Wq;          // the row's first pixel
  const unsigned m2 = 2u * a.M, orow = m2 * Wq;
  unsigned vo[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int x = x0 + 16 * j + pl;
    vo[j] = x < Wq ? (unsigned)x * m2 + 2u * m0 + 16u * kg : CT_OUT;
  }
  float bq[MT / 2][8];
  bf16x8 mk[MT / 2][4];
  const __amdgpu_buffer_rsrc_t rM = cnn_rsrc(BWD ? (const char*)a.mask + rowp * m2 : nullptr, BWD ? orow : 0);
#pragma unroll
  for (int i = 0; i < MT / 2; ++i) {
    if (!BWD) {
      const float4* bp = (const float4*)(a.bias + m0 + 32 * i + 8 * kg);
      const float4 lo = bp[0], hi = bp[1];
      bq[i][0] = lo.x, bq[i][1] = lo.y, bq[i][2] = lo.z, bq[i][3] = lo.w;
      bq[i][4] = hi.x, bq[i][5] = hi.y, bq[i][6] = hi.z, bq[i][7] = hi.w;
    }
    if (BWD)
#pragma unroll
      for (int j = 0; j < 4; ++j) mk[i][j] = __builtin_bit_cast(bf16x8, buf_load16(rM, vo[j] + 64 * i, 0));
  }
  const bool fields = !BWD && a.outf;
  const __amdgpu_buffer_rsrc_t rO =
      cnn_rsrc(fields ? nullptr : (const char*)a.out + rowp * m2, fields ? 0 : orow);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int x = x0 + 16 * j + pl;
#pragma unroll
    for (int i = 0; i < MT / 2; ++i) {
      float v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float r = acc[2 * i + (q >> 2)][j][q & 3];
        if (BWD) {
          v[q] = ((float)mk[i][j][q] > 0.f) ? r : 0.f;
        } else {
          v[q] = r + bq[i][q];
          if (a.relu) v[q] = fmaxf(v[q], 0.f);
        }
      }
      if (fields) {
        if (x < Wq)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            store_fields(a.outf, a.nreal / 2, Hq * Wq, b, y * Wq + x, m0 + 32 * i + 8 * kg + 4 * h, v + 4 * h);
      } else {
        bf16x8 h;
#pragma unroll
        for (int q = 0; q < 8; ++q) h[q] = (bf16)v[q];
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, h), rO, vo[j] + 64 * i, 0, 0);
      }
    }
  }
}

// Stride-2 reads from LDS, for two passes of the same form: output pixel
// (y, x) of a 4 x 32 tile sums taps (ty, tx) over a KS x KS window of the
// source at (2 y - 1 + ty, 2 x - 1 + tx), weight tap KS ty + tx:
//  * KS = 3, forward of the stride-2 layers: source = layer input, weights Wf,
//    bias and ReLU epilogue;
//  * KS = 4, backward data of the upsampling layers (BWD): source = dz on the
//    upsampled grid, the 16 effective weights of k_pack_up_weights, ReLU-mask
//    epilogue.
// A workgroup of TH waves computes TH x 32 output pixels for 16 MT of the M
// channels.  It stages the (2 TH + KS - 2) x (62 + KS) source patch of its tile
// and the weights (all nine taps, or eight of the sixteen at a time) in LDS per 32
// source channels and applies the taps from there; wave w owns output row y0 + w
// (two pixel tiles of 16).  Staging and addresses are those of k_conv_tile; even
// and odd source columns are staged apart, so that the 16 pixels of an operand,
// two columns apart in the source, are neighbours in LDS.
#define CS_TW 32
#define CS_PH 40                      // staged half row: 33 pixels used, a multiple of 8
template <int MT, int KS, int TH, bool BWD>
__global__ __launch_bounds__(64 * TH) void k_conv_tile_s2(GemmArgs a) {
  constexpr int NT = 64 * TH, PH = 2 * TH + KS - 2, RP = NT / 256, NR = (PH + RP - 1) / RP;
  constexpr int NTAP = KS * KS, NTW = NTAP > 9 ? NTAP / 2 : NTAP, NE = KS - 2;   // edge columns
  __shared__ __attribute__((aligned(16))) unsigned char patch[PH * 2 * CS_PH * 64];
  __shared__ __attribute__((aligned(16))) unsigned char wl[NTW * 16 * MT * 64];
  const int t0 = threadIdx.x, lane = t0 & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t0 >> 6);
  const int x0 = blockIdx.x * CS_TW, y0 = blockIdx.y * TH;
  const int nm = a.M / (16 * MT), b = blockIdx.z / nm, m0 = (blockIdx.z - b * nm) * 16 * MT;
  const int Hq = a.Hq, Wq = a.Wq, Hs = a.Hs, Ws = a.Ws;
  f32x4 acc[MT][2];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int pl = lane & 15, kg = lane >> 4;
  // patch rows 2 y0 - 1 .. of the source; the descriptor starts at the first one in it
  const unsigned px2 = 2u * a.Ksrc, row2 = px2 * Ws;
  const int sy0 = max(2 * y0 - 1, 0);
  const __amdgpu_buffer_rsrc_t rS =
      cnn_rsrc((const char*)a.src + ((size_t)b * Hs + sy0) * row2, (size_t)(Hs - sy0) * row2);
  // LDS item of source column px (of the patch) in patch row r
  auto item = [](int r, int px) { return (2 * r + (px & 1)) * CS_PH + (px >> 1); };
  const int tr = (RP > 1) ? __builtin_amdgcn_readfirstlane(t0 >> 8) : 0, tc = (t0 & 255) >> 2;
  const int sx = 2 * x0 + tc - 1;
  const unsigned vcol = (sx >= 0 && sx < Ws) ? (unsigned)sx * px2 + 16u * (t0 & 3) : CT_OUT;
  // columns 64 .. 61 + KS: 4 NE units a row
  const int er = t0 / (4 * NE), ex = 64 + (t0 >> 2) % NE, esy = 2 * y0 - 1 + er, esx = 2 * x0 + ex - 1;
  const unsigned vedge = (er < PH && esy >= 0 && esy < Hs && esx < Ws)
                             ? (unsigned)(esy - sy0) * row2 + (unsigned)esx * px2 + 16u * (t0 & 3)
                             : CT_OUT;
  const int lcol = cnn_place(item(0, tc), t0 & 3), ledge = cnn_place(item(er, ex), t0 & 3);
  // operands: 16 pixels from column m or m + 1 of a half row on
  int lb[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) lb[h] = cnn_place(item(2 * wave, 0) + pl + h, kg);
  const int lw = cnn_place(pl, kg), lws = cnn_place(cnn_wrow(t0 >> 2), t0 & 3);
  const unsigned tap2 = (unsigned)a.M * px2;
  const __amdgpu_buffer_rsrc_t rW = cnn_rsrc((const char*)a.W + (size_t)m0 * px2,
                                             (size_t)NTAP * tap2 - (size_t)m0 * px2);
  constexpr int UT = 16 * MT * 4, NWI = NTW * UT, NWS = (NWI + NT - 1) / NT;
  const unsigned vwl = (unsigned)((t0 % UT) >> 2) * px2 + 16u * (t0 & 3);
  u32x4 wv[NWS];
  // weights of taps g0 .. g0 + NTW - 1 of the chunk at byte c2 into registers, then LDS
  auto wfetch = [&](int g0, unsigned c2) {
#pragma unroll
    for (int it = 0; it < NWS; ++it) {
      if constexpr (UT >= NT) {
        wv[it] = buf_load16(rW, vwl, (unsigned)(g0 + it / (UT / NT)) * tap2 +
                                         (unsigned)(it % (UT / NT)) * (NT / 4u) * px2 + c2);
      } else {
        const int tap = it * (NT / UT) + t0 / UT;
        wv[it] = buf_load16(rW, tap < NTW ? vwl + (unsigned)(g0 + tap) * tap2 : CT_OUT, c2);
      }
    }
  };
  auto wstore = [&]() {
#pragma unroll
    for (int it = 0; it < NWS; ++it)
      if (t0 + NT * it < NWI) *(u32x4*)(wl + lws + it * NT * 16) = wv[it];
  };
  for (unsigned c2 = 0; c2 < px2; c2 += 64) {
    wfetch(0, c2);
    u32x4 sv[NR], se;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int py = r * RP + tr, sy = 2 * y0 - 1 + py;
      const bool in = py < PH && sy >= 0 && sy < Hs;
      sv[r] = buf_load16(rS, in ? vcol : CT_OUT, in ? (unsigned)(sy - sy0) * row2 + c2 : 0u);
    }
    se = buf_load16(rS, vedge, c2);
    if (c2 > 0) __syncthreads();                          // the chunk before has been read
    wstore();
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if (r * RP + tr < PH) *(u32x4*)(patch + lcol + (r * RP + tr) * 2 * CS_PH * 64) = sv[r];
    if (er < PH) *(u32x4*)(patch + ledge) = se;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NTAP; ++t) {
      if (t > 0 && t % NTW == 0) {                        // the second half of sixteen taps
        wfetch(t, c2);
        __syncthreads();
        wstore();
        __syncthreads();
      }
      const int ty = t / KS, tx = t % KS;
      bf16x8 w[MT], bv[2];
#pragma unroll
      for (int i = 0; i < MT; ++i)
        w[i] = *(const bf16x8*)(wl + lw + ((t % NTW) * MT + i) * 16 * 64);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        bv[j] = *(const bf16x8*)(patch + lb[tx >> 1] + ((2 * ty + (tx & 1)) * CS_PH + 16 * j) * 64);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i], bv[j], acc[i][j], 0, 0, 0);
    }
  }
  const int y = y0 + wave;
  if (y >= Hq) return;
  const size_t rowp = ((size_t)b * Hq + y) * Wq;
  const unsigned m2 = 2u * a.M, orow = m2 * Wq;
  unsigned vo[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int x = x0 + 16 * j + pl;
    vo[j] = x < Wq ? (unsigned)x * m2 + 2u * m0 + 16u * kg : CT_OUT;
  }
  float bq[MT / 2][8];
  bf16x8 mk[MT / 2][2];
  const __amdgpu_buffer_rsrc_t rM = cnn_rsrc(BWD ? (const char*)a.mask + rowp * m2 : nullptr, BWD ? orow : 0);
#pragma unroll
  for (int i = 0; i < MT / 2; ++i) {
    if (!BWD) {
      const float4* bp = (const float4*)(a.bias + m0 + 32 * i + 8 * kg);
      const float4 lo = bp[0], hi = bp[1];
      bq[i][0] = lo.x, bq[i][1] = lo.y, bq[i][2] = lo.z, bq[i][3] = lo.w;
      bq[i][4] = hi.x, bq[i][5] = hi.y, bq[i][6] = hi.z, bq[i][7] = hi.w;
    }
    if (BWD)
#pragma unroll
      for (int j = 0; j < 2; ++j) mk[i][j] = __builtin_bit_cast(bf16x8, buf_load16(rM, vo[j] + 64 * i, 0));
  }
  const __amdgpu_buffer_rsrc_t rO = cnn_rsrc((const char*)a.out + rowp * m2, orow);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
#pragma unroll
    for (int i = 0; i < MT / 2; ++i) {
      bf16x8 h;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float r = acc[2 * i + (q >> 2)][j][q & 3];
        float v;
        if (BWD) {
          v = ((float)mk[i][j][q] > 0.f) ? r : 0.f;
        } else {
          v = r + bq[i][q];
          if (a.relu) v = fmaxf(v, 0.f);
        }
        h[q] = (bf16)v;
      }
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, h), rO, vo[j] + 64 * i, 0, 0);
    }
  }
}

// Backward data of the stride-2 layers, LDS-tiled: a workgroup computes an
// 8 x 64 tile of layer-input pixels (all M = 16 MT channels, y0 a multiple of
// 8) from the 5 x 33 dz pixels it reads (rows y0/2 .. y0/2 + 4, columns
// x0/2 .. x0/2 + 32), staged in LDS per 32 dz channels with the weights of
// all nine taps (backward-data copy [tap][cinp][coutp]).  Tap (dy, dx)
// reaches input row y only when y + 1 - dy is even (dy = 1 at even y, 0 and 2
// at odd y) and column x only when x + 1 - dx is even (dx = 1 at even x, 0
// and 2 at odd x).  Wave w owns the even row y0 + 2w and the odd row
// y0 + 2w + 1, four pixel tiles of 16 each: even columns x0 + 2i (tiles 0,
// 1) and odd columns x0 + 2i + 1 (tiles 2, 3), so every wave applies each of
// the nine taps to two tiles.  Per dz row a wave reads two B operands per
// tile pair (dz column c for dx = 1 at even x and dx = 2 at odd x, column c + 1
// for dx = 0 at odd x); dz row w serves dy = 1 of the even row and dy = 2 of
// the odd row.  The next chunk's patch and weights are loaded while the
// current chunk's MFMAs run.  Staging and addresses are those of k_conv_tile, and
// the order of the weight rows (cnn_wrow).  The epilogue masks by the ReLU of the layer
// input.  Bound by the traffic of mask, result and dz: at 480 x 240, batch 32,
// layer 2 (590 MB) 135 us, layer 3 97; with 80-byte pixels, tested bounds and
// 8-byte accesses 181 and 128.
#define BS_TH 8
#define BS_TW 64
#define BS_PR 5
#define BS_PC 40                      // staged row: 33 pixels used, a multiple of 8
template <int MT>
__global__ __launch_bounds__(256) void k_bwd_s2_tile(GemmArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char patch[BS_PR * BS_PC * 64];
  __shared__ __attribute__((aligned(16))) unsigned char wl[9 * 16 * MT * 64];
  const int t0 = threadIdx.x, lane = t0 & 63, wave = __builtin_amdgcn_readfirstlane(t0 >> 6);
  const int x0 = blockIdx.x * BS_TW, y0 = blockIdx.y * BS_TH, b = blockIdx.z;
  const int Hq = a.Hq, Wq = a.Wq, py0 = y0 / 2, px0 = x0 / 2;
  const int pl = lane & 15, kg = lane >> 4;
  f32x4 acc[2][4][MT];   // [row: even, odd][tile][row tile]
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < MT; ++i) acc[h][j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int NPI = BS_PR * 33 * 4, NSTG = (NPI + 255) / 256;      // patch items
  constexpr int NWI = 9 * 16 * MT * 4, NWS = (NWI + 255) / 256;      // weight items
  // the descriptor starts at the tile's first dz row and ends with the image
  const unsigned px2 = 2u * a.Ksrc, row2 = px2 * a.Ws;
  const __amdgpu_buffer_rsrc_t rS = cnn_rsrc(
      (const char*)a.src + ((size_t)b * a.Hs + py0) * row2, (size_t)(a.Hs - py0) * row2);
  const __amdgpu_buffer_rsrc_t rW = cnn_rsrc(a.W, (size_t)9 * 16 * MT * px2);
  unsigned vs[NSTG];
  int ls[NSTG];
#pragma unroll
  for (int it = 0; it < NSTG; ++it) {
    const int u = t0 + 256 * it, pix = u >> 2, q = u & 3;
    const int pr = pix / 33, pc = pix - pr * 33;
    vs[it] = (px0 + pc < a.Ws) ? pr * row2 + (px0 + pc) * px2 + 16u * q : CT_OUT;
    ls[it] = cnn_place(pr * BS_PC + pc, q);
  }
  const unsigned vw = (t0 >> 2) * px2 + 16u * (t0 & 3);   // weight item t0; 64 rows on per round
  const int lws = cnn_place(cnn_wrow(t0 >> 2), t0 & 3);
  u32x4 sv[NSTG], wv[NWS];
  auto fetch = [&](int c0) {
#pragma unroll
    for (int it = 0; it < NWS; ++it) wv[it] = buf_load16(rW, vw + it * 64 * px2 + 2 * c0, 0);
#pragma unroll
    for (int it = 0; it < NSTG; ++it) sv[it] = buf_load16(rS, vs[it] + 2 * c0, 0);
  };
  // operands: dz pixels of column pl (rows and tile pairs are constants away), and
  // of the column after; 16 weight rows
  const int pc0 = cnn_place(pl, kg), pc1 = cnn_place(pl + 1, kg), lw = pc0;
  fetch(0);
  for (int c0 = 0; c0 < a.Ksrc; c0 += 32) {
    __syncthreads();   // the previous chunk's readers are done
#pragma unroll
    for (int it = 0; it < NSTG; ++it)
      if (t0 + 256 * it < NPI) *(u32x4*)(patch + ls[it]) = sv[it];
#pragma unroll
    for (int it = 0; it < NWS; ++it)
      if (t0 + 256 * it < NWI) *(u32x4*)(wl + lws + it * 64 * 64) = wv[it];
    __syncthreads();
    if (c0 + 32 < a.Ksrc) fetch(c0 + 32);
    // dz rows w (r = 0) and w + 1 (r = 1) of the patch
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      bf16x8 bc[2], bn[2];   // dz columns c and c + 1 of the two tile pairs
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const unsigned char* pp = patch + ((wave + r) * BS_PC + 16 * jj) * 64;
        bc[jj] = *(const bf16x8*)(pp + pc0);
        bn[jj] = *(const bf16x8*)(pp + pc1);
      }
      // (input row h, dy): r = 0 serves (even, 1) and (odd, 2); r = 1 serves (odd, 0)
#pragma unroll
      for (int s2 = 0; s2 < 2 - r; ++s2) {
        const int h = (r == 0 && s2 == 0) ? 0 : 1;
        const int dy = (r == 1) ? 0 : (s2 == 0 ? 1 : 2);
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
          bf16x8 wcur[MT];
#pragma unroll
          for (int i = 0; i < MT; ++i)
            wcur[i] = *(const bf16x8*)(wl + lw + ((3 * dy + dx) * MT + i) * 16 * 64);
          // dx = 1: even tiles 0, 1 from column c; dx = 2: odd tiles from
          // column c; dx = 0: odd tiles from column c + 1
          const int j0 = (dx == 1) ? 0 : 2;
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) {
            const bf16x8 bv = (dx == 0) ? bn[jj] : bc[jj];
#pragma unroll
            for (int i = 0; i < MT; ++i)
              acc[h][j0 + jj][i] =
                  __builtin_amdgcn_mfma_f32_16x16x32_bf16(wcur[i], bv, acc[h][j0 + jj][i], 0, 0, 0);
          }
        }
      }
    }
  }
  const unsigned m2 = 2u * a.M;
  unsigned vo[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int x = x0 + 2 * (16 * (j & 1) + pl) + (j >> 1);
    vo[j] = x < Wq ? x * m2 + 16u * kg : CT_OUT;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int y = y0 + 2 * wave + h;
    if (y >= Hq) break;
    const size_t rowp = ((size_t)b * Hq + y) * Wq;
    const __amdgpu_buffer_rsrc_t rM = cnn_rsrc((const char*)a.mask + rowp * m2, (size_t)Wq * m2);
    const __amdgpu_buffer_rsrc_t rO = cnn_rsrc((const char*)a.out + rowp * m2, (size_t)Wq * m2);
    bf16x8 mk[4][MT / 2];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < MT / 2; ++i) mk[j][i] = __builtin_bit_cast(bf16x8, buf_load16(rM, vo[j] + 64 * i, 0));
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < MT / 2; ++i) {
        bf16x8 hv;
#pragma unroll
        for (int q = 0; q < 8; ++q)
          hv[q] = (bf16)(((float)mk[j][i][q] > 0.f) ? acc[h][j][2 * i + (q >> 2)][q & 3] : 0.f);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, hv), rO, vo[j] + 64 * i, 0, 0);
      }
  }
}

// ------------------------------------------------------------- layer 1 ----
// Partial sums of |F_b|^2 of the effective-index fields, grid (ES_SLICES, B);
// k_conv1_fwd adds them in slice order.
#define ES_SLICES 64
__global__ __launch_bounds__(256) void k_eim_scale_part(const float2* __restrict__ eim, int D,
                                                        double* __restrict__ part) {
  const float2* f = eim + (size_t)blockIdx.y * D;
  const int per = (D + ES_SLICES - 1) / ES_SLICES, e0 = blockIdx.x * per, e1 = min(D, e0 + per);
  double s = 0.0;
  for (int e = e0 + threadIdx.x; e < e1; e += 256) {
    const float2 v = f[e];
    s += (double)v.x * v.x + (double)v.y * v.y;
  }
  __shared__ double lds[8];
  s = block_sum1<double>(s, lds);
  if (threadIdx.x == 0) part[(size_t)blockIdx.y * ES_SLICES + blockIdx.x] = s;
}

// The network's input and its first layer.  Input planes [B][C][H][W]: plane 0 =
// (eps - 2.085) / (12.25 - 2.085); for C = 3, planes 1 and 2 = real and imaginary
// part of the effective-index field scaled to unit RMS per pixel, by
// sqrt(D) / ||F_b|| (0 for an all-zero field).
//
// C input planes, 32 output channels, FP32 throughout on the matrix cores: per 16
// output pixels the product W[32][9C] . X[9C][16] runs as FP32 16x16x4 MFMAs over
// K = 9C padded to a multiple of 4 (k = 9 c + tap, padded rows zero).  Lane l
// supplies weight row l % 16 / k-slot l / 16 and the input of pixel l % 16 at
// k-slot l / 16; tile i's row r is channel 8 (r / 4) + 4 i + r % 4, so that the two
// tiles leave a lane 8 neighbouring channels of its pixel: one 16-byte store, and
// a wave's stores are contiguous.
//
// A workgroup forms the planes of C1_TH rows of 64 pixels and a ring around them
// in LDS, stores its own pixels' (for the weight gradient) and reads its operands
// there, at addresses that differ by constants.  At 480 x 240 with three planes,
// batch 64, 195 us, of which the writes alone (32 bf16 channels of each pixel, the
// planes) would take 125 and the MFMAs 85; at batch 1, 8.8 us.  With the planes
// formed by kernels before it, and gathered from memory per pixel and tap with the
// bounds tested for each, 234 + 38 us, and 14.8 us in three launches.
#define C1_TH 8
#define C1_PS 80      // floats of a row in LDS: its banks and the next row's differ
template <int C>
__global__ __launch_bounds__(256) void k_conv1_fwd(const float* __restrict__ eps,
                                                   const float2* __restrict__ eim,
                                                   const double* __restrict__ espart,
                                                   const float* __restrict__ w,
                                                   const float* __restrict__ bias, int H, int W,
                                                   float* __restrict__ x0, bf16* __restrict__ out) {
  constexpr int KS = (9 * C + 3) / 4;   // k-steps of 4
  constexpr int PL = (C1_TH + 2) * C1_PS;
  __shared__ float pl[C * PL];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ks = lane >> 4, col = lane & 15;
  const int xa = blockIdx.x * 64, ya = blockIdx.y * C1_TH, b = blockIdx.z;
  const int HW = H * W;
  const float* eb = eps + (size_t)b * HW;
  const float2* fb = eim + (size_t)b * HW;
  float* xb = x0 + (size_t)b * C * HW;
  constexpr int NP = (C1_TH + 2) * 66, NI = (NP + 255) / 256;
  float e[NI];
  float2 f[NI];
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    const int u = threadIdx.x + 256 * it, r = u / 66, y = ya + r - 1, x = xa + u - 66 * r - 1;
    const bool ok = u < NP && (unsigned)y < (unsigned)H && (unsigned)x < (unsigned)W;
    e[it] = ok ? eb[y * W + x] : 0.f;
    if (C == 3) f[it] = ok ? fb[y * W + x] : make_float2(0.f, 0.f);
  }
  float av[2][KS];
  const int ch = 8 * (col >> 2) + (col & 3);
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int k = 4 * s + ks;
#pragma unroll
    for (int i = 0; i < 2; ++i) av[i][s] = (k < 9 * C) ? w[(ch + 4 * i) * 9 * C + k] : 0.f;
  }
  float sc = 0.f;
  if (C == 3) {
    // uniform loads of what the kernel before wrote
    const auto* ep = (const __attribute__((address_space(4))) double*)(espart + (size_t)b * ES_SLICES);
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < ES_SLICES; ++i) s += ep[i];
    sc = (float)((s > 0.0) ? sqrt((double)HW / s) : 0.0);
  }
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    const int u = threadIdx.x + 256 * it, r = u / 66, c = u - 66 * r, y = ya + r - 1, x = xa + c - 1;
    if (u >= NP) break;
    const bool in = (unsigned)y < (unsigned)H && (unsigned)x < (unsigned)W;
    float v[3] = {0.f, 0.f, 0.f};
    if (in) {
      v[0] = (e[it] - CNN_EPS_LO) / (CNN_EPS_HI - CNN_EPS_LO);
      if (C == 3) {
        v[1] = f[it].x * sc;
        v[2] = f[it].y * sc;
      }
    }
#pragma unroll
    for (int q = 0; q < C; ++q) pl[q * PL + r * C1_PS + c] = v[q];
    if (in && r >= 1 && r <= C1_TH && c >= 1 && c <= 64)
#pragma unroll
      for (int q = 0; q < C; ++q) xb[(size_t)q * HW + y * W + x] = v[q];
  }
  // per k-slot: plane and tap, the same for every pixel tile; a padded slot's
  // operand is zeroed after the read
  int koff[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int k = min(4 * s + ks, 9 * C - 1), c = k / 9, t = k - 9 * c;
    koff[s] = c * PL + (t / 3) * C1_PS + t % 3 + col + 2 * wave * C1_PS;
  }
  const bool padded = 4 * (KS - 1) + ks >= 9 * C;
  float bq[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) bq[q] = bias[8 * ks + q];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int y = ya + 2 * wave + r;
    if (y >= H) break;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (xa + 16 * j >= W) break;
      float bv[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) bv[s] = pl[koff[s] + r * C1_PS + 16 * j];
      if (padded) bv[KS - 1] = 0.f;
      f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][s], bv[s], acc[i], 0, 0, 0);
      const int x = xa + 16 * j + col;
      if (x >= W) continue;
      bf16 h[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) h[q] = (bf16)fmaxf(acc[q >> 2][q & 3] + bq[q], 0.f);
      *(u32x4*)(out + ((size_t)b * HW + y * W + x) * 32 + 8 * ks) = __builtin_bit_cast(u32x4, h);
    }
  }
}

// --------------------------------------------------- weight gradients ----
// Waves per SIMD that the weight-gradient kernels' registers are held to: the
// accumulators, 32 for each block of 8 x 8 in flight, 60 others (left to itself
// the compiler takes more and one workgroup less is resident: 224 us for layer 4).
constexpr int wg_waves(int units, int taps, int bpt) {
  return 512 / (4 * units * taps + 32 * bpt + 60) > 1 ? 512 / (4 * units * taps + 32 * bpt + 60) : 1;
}

// Stores an 8 x 8 block (r[i]: pixel i, 8 channels) transposed, channel c's 8 pixels
// at row(c).  Neighbouring threads hold neighbouring channel groups g (of N); groups
// two apart start a multiple of 256 bytes apart whatever the pitch (a multiple of
// 16), so that all of them storing channel q met in the same banks: conflicts took
// 55 to 76% of the LDS's busy cycles, and the LDS was busy 65 to 85% of the time.
// From 8 groups on, group g therefore takes its channels in the order q ^ (g & 6),
// which spreads 16 lanes over all banks (two to a bank with 16 groups) at the
// pitches in use, 9, 11 and 17 times 16 bytes.  At 480 x 240, batch 32, layers 6 to
// 3: 141, 138, 131 and 76 us, before 178, 168, 172 and 103.  Four groups conflict
// two by two; turning one bit there spilled registers in the ring (185 us against
// 144).
template <int N, typename Row>
__device__ __forceinline__ void put_transposed(const bf16x8 (&r)[8], int g, Row row) {
  const int x = N >= 8 ? g & 6 : 0;
  u32x4 w[8];                      // word d of w[i]: channels 2 d and 2 d + 1, d turned by x
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    w[i] = __builtin_bit_cast(u32x4, r[i]);
    if constexpr (N >= 8) {
      const u32x4 v = w[i];
      const bool s = (x & 4) != 0, h = (x & 2) != 0;
      const u32x4 u = u32x4{s ? v[2] : v[0], s ? v[3] : v[1], s ? v[0] : v[2], s ? v[1] : v[3]};
      w[i] = u32x4{h ? u[1] : u[0], h ? u[0] : u[1], h ? u[3] : u[2], h ? u[2] : u[3]};
    }
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    u32x4 t;
#pragma unroll
    for (int d = 0; d < 4; ++d)    // lower or upper halves of two pixels' words
      t[d] = __builtin_amdgcn_perm(w[2 * d + 1][q >> 1], w[2 * d][q >> 1],
                                   (q & 1) ? 0x07060302u : 0x05040100u);
    *(u32x4*)row(q ^ x) = t;
  }
}

// Weight gradients of a 3x3 layer (stride 1, stride 2 or upsampling) as GEMMs
// dW[tap][r][c] = sum_p dz[p][r] in[src(p, tap)][c] over stages of PX = 32 S
// pixels of one output row (the last chunk of a row is ragged).  Work items:
// (pixel slice, channel block of NB = 16 NT input channels, dy), dy fastest,
// or with ND = 3 (slice, channel block) taking all three dy.  Per stage the
// workgroup stages in LDS, transposed to [channel][pixel]:
//  * dz of the stage, all Mr = 16 MT output channels;
//  * per dy, the input row the stage reads, NB channels from channel n0,
//    once for the three dx taps:
//    - stride 1 (MK = MAP_S1): input columns x0 - 8 .. x0 + PX + 7 at columns
//      0 .. PX + 15; dx reads at shifts -1, 0, +1;
//    - upsampling (MAP_UP): the same, the source row expanded x2 while
//      staging;
//    - stride 2 (MAP_S2): output pixel p reads input columns 2p - 1, 2p and
//      2p + 1, so the row is split by parity: odd columns 2j + 1 (j = x0 - 1 ..
//      x0 + PX - 1) at columns j - x0 + 8, even columns 2j (j = x0 ..
//      x0 + PX - 1) at columns PX + 8 + j - x0.  dx = 2 and dx = 1 read the
//      odd and even halves aligned, dx = 0 the odd half shifted by one.  The
//      one odd column left of the chunk (2 x0 - 1) is loaded by a thread of
//      its own rather than as a block of 8.
// A staging block is 8 pixels x 8 channels: loaded with 16-byte reads,
// transposed in registers, stored with 16-byte writes; the next stage's
// blocks are loaded while the current stage's MFMAs run.  Shifted operands
// are built from aligned 16-byte LDS reads by funnel shifts.  Per stage that
// moves PX + 16 (stride 1), PX / 2 + 8 (upsampling) or 2 PX + 1 (stride 2)
// input pixels per dy instead of 3 PX.  A wave owns (row tile, column tile)
// units and applies all three dx to each.  The slice's (dy 0, first channel
// block) item also sums dz over its pixels (the bias gradient) as dz^T times
// a column of ones.  Partials: weights [slice][tap][r][c], bias [slice][r].
// (The network's upsampling layers use k_conv_wgrad_up and its 32-channel
// stride-1 layers k_conv_wgrad_ring; the upsampling map here serves other
// channel counts.)
constexpr int wg_row_blocks(int MT, int NT, int S, int MK, int ND) {
  const int xg = MK == MAP_UP ? 2 * S + 1 : (MK == MAP_S2 ? 8 * S : 4 * S + 2);
  return (4 * S * 2 * MT + ND * xg * 2 * NT + 255) / 256;
}
template <int MT, int NT, int S, int MK, int ND = 1>
__global__ __launch_bounds__(256, wg_waves((MT * NT + 3) / 4, 3 * ND, wg_row_blocks(MT, NT, S, MK, ND)))
void k_conv_wgrad_row(const bf16* __restrict__ dz,
                                                        const bf16* __restrict__ x, int B,
                                                        int Hout, int Wout, int Hin, int Win,
                                                        int Nc, int stages_per, int nwork,
                                                        float* __restrict__ part,
                                                        float* __restrict__ bpart) {
  constexpr bool UP = MK == MAP_UP, S2 = MK == MAP_S2;
  constexpr int Mr = 16 * MT, NB = 16 * NT, PX = 32 * S, LD = PX + 8;
  // staged columns per channel and row pitch (a pitch of an odd number of
  // 16-byte units)
  constexpr int XC = S2 ? 2 * PX + 8 : PX + 16, LDX = S2 ? XC : XC + 8;
  constexpr int ABLK = (PX / 8) * (Mr / 8);
  // source groups of 8 pixels (stride 2: odd groups, then even groups)
  constexpr int XG = UP ? (PX / 16 + 1) : S2 ? 2 * (PX / 8) : (PX / 8 + 2);
  constexpr int XBLK = XG * (NB / 8);
  constexpr int NBLK = ABLK + ND * XBLK, BPT = (NBLK + 255) / 256;
  constexpr int NU = MT * NT, PER_WAVE = (NU + 3) / 4;
  static_assert(!S2 || ND * (NB / 8) <= 256, "stride-2 halo loads: one per thread");
  __shared__ __attribute__((aligned(16))) bf16 As[Mr][LD];
  __shared__ __attribute__((aligned(16))) bf16 Xs[ND][NB][LDX];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // 1D grid, a multiple of 8 long: consecutive work items (the dy and the
  // channel blocks of one pixel slice) go to the same XCD, whose L2 then
  // serves their shared dz and input rows
  const int w = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (w >= nwork) return;
  const int nblk = Nc / NB;
  // ND = 3: one item takes all three dy (first dy0 = 0) and stages dz once
  const int dy0 = (ND == 3) ? 0 : w % 3;
  const int n0 = ((ND == 3) ? w % nblk : (w / 3) % nblk) * NB;
  const int slice = (ND == 3) ? w / nblk : w / (3 * nblk);
  const int nch = (Wout + PX - 1) / PX, nst = B * Hout * nch;
  const int s0 = slice * stages_per, s1 = min(nst, s0 + stages_per);
  bf16x8 reg[BPT][8];
  bf16x8 hreg = zero8();
  unsigned okm[BPT];   // stride 2: bit i, element i of the block is in range
  bool hok = false;
  auto load = [&](int sg) {
    const int b = sg / (Hout * nch), rem = sg - b * Hout * nch, y = rem / nch;
    const int x0 = (rem - y * nch) * PX;
    if constexpr (S2) {
      // Every load is issued unconditionally (reads out of range go to
      // element 0 of their array) and out-of-range values are zeroed when
      // the block is stored to LDS: with conditional loads, or zeroing right
      // after the load, the waves waited for the prefetch before the current
      // stage's MFMAs.  First the odd column 2 x0 - 1 of row rd.
      const bool hv = threadIdx.x < ND * (NB / 8);
      const int rd = hv ? threadIdx.x / (NB / 8) : 0, cg = (threadIdx.x % (NB / 8)) * 8;
      const int ys = 2 * y + dy0 + rd - 1, c = 2 * x0 - 1;
      hok = hv && ys >= 0 && ys < Hin && c >= 0 && c < Win;
      hreg = load8(x + (hok ? (((size_t)b * Hin + ys) * Win + c) * Nc + n0 + cg : 0));
#pragma unroll
      for (int bi = 0; bi < BPT; ++bi) {
        const int blk = threadIdx.x + 256 * bi;
        // element i is input column c0 + 2 i of source row ys (dz: pixel
        // x0 + 8 pg + i), in range for 0 <= column < climit
        const bf16* src = dz;
        long off0 = 0;
        int c0 = 0, cstep = 1, climit = 0, ostep = 0;
        if (blk < ABLK) {
          const int pg = blk / (Mr / 8), cg = (blk % (Mr / 8)) * 8;
          c0 = x0 + pg * 8; climit = Wout; ostep = Mr;
          off0 = (((long)b * Hout + y) * Wout + c0) * Mr + cg;
        } else if (blk < NBLK) {
          const int rd = (blk - ABLK) / XBLK, r = blk - ABLK - rd * XBLK;   // dy row, item
          const int ys = 2 * y + dy0 + rd - 1;
          const int m = r / (NB / 8), cg = (r % (NB / 8)) * 8;
          c0 = 2 * (x0 + 8 * (m % (PX / 8))) + (m < PX / 8 ? 1 : 0);   // odd, then even groups
          cstep = 2;
          climit = (ys >= 0 && ys < Hin) ? Win : 0;
          src = x; ostep = 2 * Nc;
          off0 = (((long)b * Hin + ys) * Win + c0) * Nc + n0 + cg;
        }
        okm[bi] = 0;
        if (blk < NBLK) {   // false only in the last round, for its spare threads
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int c = c0 + cstep * i;
            const bool ok = c >= 0 && c < climit;
            reg[bi][i] = load8(src + (ok ? off0 + (long)i * ostep : 0));
            okm[bi] |= (unsigned)ok << i;
          }
        }
      }
    } else {
#pragma unroll
      for (int bi = 0; bi < BPT; ++bi) {
        const int blk = threadIdx.x + 256 * bi;
#pragma unroll
        for (int i = 0; i < 8; ++i) reg[bi][i] = zero8();
        if (blk < ABLK) {
          const int pg = blk / (Mr / 8), cg = (blk % (Mr / 8)) * 8;
          const bf16* src = dz + (((size_t)b * Hout + y) * Wout + x0) * Mr + cg;
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (x0 + pg * 8 + i < Wout) reg[bi][i] = load8(src + (size_t)(pg * 8 + i) * Mr);
        } else if (blk < NBLK) {
          const int rd = (blk - ABLK) / XBLK, r = blk - ABLK - rd * XBLK;   // dy row, item
          const int uy = y + dy0 + rd - 1;   // row of the stride-1 or upsampled grid
          if (uy >= 0 && uy < Hout) {
            const int ys = UP ? (uy >> 1) : uy;
            const int m = r / (NB / 8), cg = (r % (NB / 8)) * 8;
            const int c0 = UP ? (x0 / 2 - 4 + 8 * m) : (x0 - 8 + 8 * m);   // first source column
            const bf16* src = x + ((size_t)b * Hin + ys) * Win * Nc + n0 + cg;
#pragma unroll
            for (int i = 0; i < 8; ++i)
              if (c0 + i >= 0 && c0 + i < Win) reg[bi][i] = load8(src + (size_t)(c0 + i) * Nc);
          }
        }
      }
    }
  };
  f32x4 acc[PER_WAVE][3 * ND];   // [unit][row (dy - dy0) * 3 + dx]
#pragma unroll
  for (int i = 0; i < PER_WAVE; ++i)
#pragma unroll
    for (int d = 0; d < 3 * ND; ++d) acc[i][d] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int BT = (MT + 3) / 4;
  const bool bias = (dy0 == 0 && n0 == 0);
  f32x4 accb[BT];
#pragma unroll
  for (int i = 0; i < BT; ++i) accb[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 ones;
#pragma unroll
  for (int q = 0; q < 8; ++q) ones[q] = (bf16)1.f;
  const int kq = 8 * (lane >> 4);
  if (s0 < s1) load(s0);
  for (int sg = s0; sg < s1; ++sg) {
    __syncthreads();
#pragma unroll
    for (int bi = 0; bi < BPT; ++bi) {
      if constexpr (S2) {
#pragma unroll
        for (int i = 0; i < 8; ++i) reg[bi][i] = ((okm[bi] >> i) & 1) ? reg[bi][i] : zero8();
      }
      const int blk = threadIdx.x + 256 * bi;
      if (blk < ABLK) {
        const int g = blk % (Mr / 8);
        bf16* dst = &As[g * 8][(blk / (Mr / 8)) * 8];
        put_transposed<Mr / 8>(reg[bi], g, [&](int c) { return dst + c * LD; });
      } else if (blk < NBLK) {
        const int rd = (blk - ABLK) / XBLK, r = blk - ABLK - rd * XBLK;
        const int m = r / (NB / 8), g = r % (NB / 8), cg = g * 8;
        bf16 (*Xr)[LDX] = Xs[rd];
        if constexpr (UP) {   // source pixel i fills columns 16 m + 2 i and 16 m + 2 i + 1
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            bf16x8 lo, hi;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              lo[2 * i] = lo[2 * i + 1] = reg[bi][i][q];
              hi[2 * i] = hi[2 * i + 1] = reg[bi][i + 4][q];
            }
            *(bf16x8*)&Xr[cg + q][16 * m] = lo;
            *(bf16x8*)&Xr[cg + q][16 * m + 8] = hi;
          }
        } else {   // stride 2: odd and even groups both land at column 8 m + 8
          bf16* dst = &Xr[cg][S2 ? 8 * m + 8 : 8 * m];
          put_transposed<NB / 8>(reg[bi], g, [&](int c) { return dst + c * LDX; });
        }
      }
    }
    if (S2 && threadIdx.x < ND * (NB / 8)) {
      const int rd = threadIdx.x / (NB / 8), cg = (threadIdx.x % (NB / 8)) * 8;
#pragma unroll
      for (int q = 0; q < 8; ++q) Xs[rd][cg + q][7] = hok ? hreg[q] : (bf16)0.f;
    }
    __syncthreads();
    if (sg + 1 < s1) load(sg + 1);
#pragma unroll
    for (int kk = 0; kk < S; ++kk) {
#pragma unroll
      for (int i = 0; i < PER_WAVE; ++i) {
        const int u = wave + 4 * i;
        if (u < NU) {
          const int ti = u / NT, tj = u - ti * NT;
          const bf16x8 av = *(const bf16x8*)&As[ti * 16 + (lane & 15)][kk * 32 + kq];
#pragma unroll
          for (int rd = 0; rd < ND; ++rd) {
            // stride 1 / upsampling: the column of dx = 1; stride 2: the
            // odd column of dx = 2
            const bf16* xr = &Xs[rd][tj * 16 + (lane & 15)][kk * 32 + kq + 8];
            const u32x4 a4 = __builtin_bit_cast(u32x4, *(const bf16x8*)(xr - 8));
            const u32x4 b4 = __builtin_bit_cast(u32x4, *(const bf16x8*)xr);
            // stride 1: the next 8 columns; stride 2: the even columns (dx = 1)
            const u32x4 c4 = __builtin_bit_cast(u32x4, *(const bf16x8*)(xr + (S2 ? PX : 8)));
            // columns shifted by one bf16: word j = high half of word j-1, low half of word j
            const unsigned s0w = (a4[3] >> 16) | (b4[0] << 16), s1w = (b4[0] >> 16) | (b4[1] << 16);
            const unsigned s2w = (b4[1] >> 16) | (b4[2] << 16), s3w = (b4[2] >> 16) | (b4[3] << 16);
            const unsigned s4w = (b4[3] >> 16) | (c4[0] << 16);
            const bf16x8 bl = __builtin_bit_cast(bf16x8, u32x4{s0w, s1w, s2w, s3w});   // dx = 0
            const bf16x8 bm = __builtin_bit_cast(bf16x8, S2 ? c4 : b4);                // dx = 1
            const bf16x8 br = __builtin_bit_cast(bf16x8, S2 ? b4 : u32x4{s1w, s2w, s3w, s4w});   // dx = 2
            acc[i][3 * rd] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bl, acc[i][3 * rd], 0, 0, 0);
            acc[i][3 * rd + 1] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bm, acc[i][3 * rd + 1], 0, 0, 0);
            acc[i][3 * rd + 2] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, br, acc[i][3 * rd + 2], 0, 0, 0);
          }
        }
      }
      if (bias) {
#pragma unroll
        for (int i = 0; i < BT; ++i) {
          const int ti = wave + 4 * i;
          if (ti < MT) {
            const bf16x8 av = *(const bf16x8*)&As[ti * 16 + (lane & 15)][kk * 32 + kq];
            accb[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, ones, accb[i], 0, 0, 0);
          }
        }
      }
    }
  }
  if (bias) {
#pragma unroll
    for (int i = 0; i < BT; ++i) {
      const int ti = wave + 4 * i;
      if (ti < MT && (lane & 15) == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) bpart[(size_t)slice * Mr + ti * 16 + 4 * (lane >> 4) + q] = accb[i][q];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < PER_WAVE; ++i) {
    const int u = wave + 4 * i;
    if (u < NU) {
      const int ti = u / NT, tj = u - ti * NT;
      const int c = tj * 16 + (lane & 15);
#pragma unroll
      for (int d = 0; d < 3 * ND; ++d) {   // tap (dy0 + d / 3) * 3 + d % 3 = 3 dy0 + d
        float* out = part + (((size_t)slice * 9 + dy0 * 3 + d) * Mr) * Nc + n0;
#pragma unroll
        for (int q = 0; q < 4; ++q) out[(size_t)(ti * 16 + 4 * (lane >> 4) + q) * Nc + c] = acc[i][d][q];
      }
    }
  }
}

// Weight gradients of a stride-1 layer, all three dy per work item, with the
// input rows kept in a ring: a slice's stages walk down one column chunk
// (stage order image, chunk, row), so stage y needs input rows y - 1, y and
// y + 1 and the next stage only row y + 2, which replaces row y - 1 in the
// ring of three staged rows.  A stage therefore loads its dz row and one
// input row (k_conv_wgrad_row with all three dy loads three input rows).  At
// the first stage of a slice, and where the walk enters a new chunk or image,
// rows y - 1 and y are loaded as well.  Staging blocks, the column shifts of
// the three dx taps and the partials are those of k_conv_wgrad_row (dsplit 1).
template <int MT, int NT, int S>
__global__ __launch_bounds__(256, wg_waves((MT * NT + 3) / 4, 9, (4 * S * 2 * MT + (4 * S + 2) * 2 * NT + 255) / 256))
void k_conv_wgrad_ring(const bf16* __restrict__ dz,
                                                         const bf16* __restrict__ x, int B,
                                                         int H, int W, int Nc, int stages_per,
                                                         int nwork, float* __restrict__ part,
                                                         float* __restrict__ bpart) {
  constexpr int Mr = 16 * MT, NB = 16 * NT, PX = 32 * S, LD = PX + 8;
  constexpr int XC = PX + 16, LDX = XC + 8;          // staged columns x0 - 8 .. x0 + PX + 7
  constexpr int ABLK = (PX / 8) * (Mr / 8);
  constexpr int XBLK = (PX / 8 + 2) * (NB / 8);      // one input row
  constexpr int NBLK = ABLK + XBLK, BPT = (NBLK + 255) / 256;
  constexpr int NU = MT * NT, PER_WAVE = (NU + 3) / 4;
  __shared__ __attribute__((aligned(16))) bf16 As[Mr][LD];
  __shared__ __attribute__((aligned(16))) bf16 Xs[3][NB][LDX];   // ring: row r in slot r mod 3
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int w = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (w >= nwork) return;
  const int nblk = Nc / NB;
  const int n0 = (w % nblk) * NB, slice = w / nblk;
  const int nch = (W + PX - 1) / PX, nst = B * nch * H;
  const int s0 = slice * stages_per, s1 = min(nst, s0 + stages_per);
  auto slot = [](int r) { return (r + 3) % 3; };   // r >= -1
  bf16x8 reg[BPT][8];
  // input row ry (zeros outside the image) of chunk x0 into the X blocks'
  // registers; with dzrow, dz row y of the chunk into the A blocks' too
  auto load = [&](int b, int x0, int y, int ry, bool dzrow) {
#pragma unroll
    for (int bi = 0; bi < BPT; ++bi) {
      const int blk = threadIdx.x + 256 * bi;
#pragma unroll
      for (int i = 0; i < 8; ++i) reg[bi][i] = zero8();
      if (blk < ABLK) {
        if (dzrow) {
          const int pg = blk / (Mr / 8), cg = (blk % (Mr / 8)) * 8;
          const bf16* src = dz + (((size_t)b * H + y) * W + x0) * Mr + cg;
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (x0 + pg * 8 + i < W) reg[bi][i] = load8(src + (size_t)(pg * 8 + i) * Mr);
        }
      } else if (blk < NBLK && ry >= 0 && ry < H) {
        const int r = blk - ABLK, m = r / (NB / 8), cg = (r % (NB / 8)) * 8;
        const int c0 = x0 - 8 + 8 * m;   // first source column
        const bf16* src = x + ((size_t)b * H + ry) * W * Nc + n0 + cg;
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (c0 + i >= 0 && c0 + i < W) reg[bi][i] = load8(src + (size_t)(c0 + i) * Nc);
      }
    }
  };
  auto store = [&](int xslot, bool dzrow) {
#pragma unroll
    for (int bi = 0; bi < BPT; ++bi) {
      const int blk = threadIdx.x + 256 * bi;
      if (blk < ABLK) {
        if (dzrow) {
          const int g = blk % (Mr / 8);
          bf16* dst = &As[g * 8][(blk / (Mr / 8)) * 8];
          put_transposed<Mr / 8>(reg[bi], g, [&](int c) { return dst + c * LD; });
        }
      } else if (blk < NBLK) {
        const int r = blk - ABLK, m = r / (NB / 8), g = r % (NB / 8);
        bf16* dst = &Xs[xslot][g * 8][8 * m];
        put_transposed<NB / 8>(reg[bi], g, [&](int c) { return dst + c * LDX; });
      }
    }
  };
  auto decode = [&](int sg, int& b, int& x0, int& y) {
    b = sg / (nch * H);
    const int rem = sg - b * nch * H, ch = rem / H;
    y = rem - ch * H;
    x0 = ch * PX;
  };
  f32x4 acc[PER_WAVE][9];   // [unit][dy * 3 + dx]
#pragma unroll
  for (int i = 0; i < PER_WAVE; ++i)
#pragma unroll
    for (int d = 0; d < 9; ++d) acc[i][d] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int BT = (MT + 3) / 4;
  const bool bias = (n0 == 0);
  f32x4 accb[BT];
#pragma unroll
  for (int i = 0; i < BT; ++i) accb[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 ones;
#pragma unroll
  for (int q = 0; q < 8; ++q) ones[q] = (bf16)1.f;
  const int kq = 8 * (lane >> 4);
  if (s0 < s1) {
    int b, x0, y;
    decode(s0, b, x0, y);
    load(b, x0, y, y + 1, true);
  }
  for (int sg = s0; sg < s1; ++sg) {
    int b, x0, y;
    decode(sg, b, x0, y);
    __syncthreads();   // the previous stage's readers of As and of row y - 2's slot are done
    store(slot(y + 1), true);
    if (sg == s0 || y == 0) {   // a new walk: rows y - 1 and y as well
      for (int r = y - 1; r <= y; ++r) {
        load(b, x0, y, r, false);
        store(slot(r), false);
      }
    }
    __syncthreads();
    if (sg + 1 < s1) {
      int bn, xn, yn;
      decode(sg + 1, bn, xn, yn);
      load(bn, xn, yn, yn + 1, true);
    }
    const int sl[3] = {slot(y - 1), slot(y), slot(y + 1)};
#pragma unroll
    for (int kk = 0; kk < S; ++kk) {
#pragma unroll
      for (int i = 0; i < PER_WAVE; ++i) {
        const int u = wave + 4 * i;
        if (u < NU) {
          const int ti = u / NT, tj = u - ti * NT;
          const bf16x8 av = *(const bf16x8*)&As[ti * 16 + (lane & 15)][kk * 32 + kq];
#pragma unroll
          for (int dy = 0; dy < 3; ++dy) {
            const bf16* xr = &Xs[sl[dy]][tj * 16 + (lane & 15)][kk * 32 + kq + 8];   // dx = 1
            const u32x4 a4 = __builtin_bit_cast(u32x4, *(const bf16x8*)(xr - 8));
            const u32x4 b4 = __builtin_bit_cast(u32x4, *(const bf16x8*)xr);
            const u32x4 c4 = __builtin_bit_cast(u32x4, *(const bf16x8*)(xr + 8));
            const unsigned s0w = (a4[3] >> 16) | (b4[0] << 16), s1w = (b4[0] >> 16) | (b4[1] << 16);
            const unsigned s2w = (b4[1] >> 16) | (b4[2] << 16), s3w = (b4[2] >> 16) | (b4[3] << 16);
            const unsigned s4w = (b4[3] >> 16) | (c4[0] << 16);
            const bf16x8 bl = __builtin_bit_cast(bf16x8, u32x4{s0w, s1w, s2w, s3w});   // dx = 0
            const bf16x8 bm = __builtin_bit_cast(bf16x8, b4);                          // dx = 1
            const bf16x8 br = __builtin_bit_cast(bf16x8, u32x4{s1w, s2w, s3w, s4w});   // dx = 2
            acc[i][3 * dy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bl, acc[i][3 * dy], 0, 0, 0);
            acc[i][3 * dy + 1] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bm, acc[i][3 * dy + 1], 0, 0, 0);
            acc[i][3 * dy + 2] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, br, acc[i][3 * dy + 2], 0, 0, 0);
          }
        }
      }
      if (bias) {
#pragma unroll
        for (int i = 0; i < BT; ++i) {
          const int ti = wave + 4 * i;
          if (ti < MT) {
            const bf16x8 av = *(const bf16x8*)&As[ti * 16 + (lane & 15)][kk * 32 + kq];
            accb[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, ones, accb[i], 0, 0, 0);
          }
        }
      }
    }
  }
  if (bias) {
#pragma unroll
    for (int i = 0; i < BT; ++i) {
      const int ti = wave + 4 * i;
      if (ti < MT && (lane & 15) == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) bpart[(size_t)slice * Mr + ti * 16 + 4 * (lane >> 4) + q] = accb[i][q];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < PER_WAVE; ++i) {
    const int u = wave + 4 * i;
    if (u < NU) {
      const int ti = u / NT, tj = u - ti * NT;
      const int c = tj * 16 + (lane & 15);
#pragma unroll
      for (int d = 0; d < 9; ++d) {
        float* out = part + (((size_t)slice * 9 + d) * Mr) * Nc + n0;
#pragma unroll
        for (int q = 0; q < 4; ++q) out[(size_t)(ti * 16 + 4 * (lane >> 4) + q) * Nc + c] = acc[i][d][q];
      }
    }
  }
}

// Weight gradients of the upsampling layers at the source resolution.  The
// layer input u is the source x repeated over 2 x 2 blocks, so for output
// pixel (2i + a, 2j + b) tap t reads x at (i + dy, j + dx) with
// d = (parity + t - 1) >> 1: per parity only two row and two column shifts
// occur, d = parity + s - 1 for s = 0, 1.  The sixteen products
//   G[a][b][sy][sx][r][c] = sum_{i,j} dz[2i + a][2j + b][r] x[i + a + sy - 1][j + b + sx - 1][c]
// give every tap as a sum of four, dW[ty][tx] = sum_{a,b} G[a][b][sy(a, ty)][sx(b, tx)]
// with sy(a, t) = ((a + t - 1) >> 1) - a + 1 (k_up_tapmap): 16 products per
// source pixel instead of the 36 of the upsampled grid.  Work items: (pixel
// slice, channel block of NB = 16 NT input channels, output-row parity a),
// a fastest.  A stage is PX = 32 S source pixels of source row i; the
// workgroup stages in LDS, transposed to [channel][pixel]:
//  * dz of output row 2i + a, columns 2j and 2j + 1 (b = 0, 1) in two halves;
//  * source rows i + a - 1 and i + a (sy = 0, 1), columns j0 - 8 ..
//    j0 + PX + 7, read by the column shifts -1, 0, +1 as in k_conv_wgrad_row.
// Loads, staging blocks and funnel shifts are those of k_conv_wgrad_row.
// Partials: [slice][16][r][c] (index ((a 2 + b) 2 + sy) 2 + sx), bias
// [slice][a][r] (every channel-block-0 item sums its dz row).
template <int MT, int NT, int S>
__global__ __launch_bounds__(256, wg_waves((MT * NT + 3) / 4, 8, (8 * S * 2 * MT + (8 * S + 4) * 2 * NT + 255) / 256))
void k_conv_wgrad_up(const bf16* __restrict__ dz,
                                                       const bf16* __restrict__ x, int B,
                                                       int Hout, int Wout, int Hin, int Win,
                                                       int Nc, int stages_per, int nwork,
                                                       float* __restrict__ part,
                                                       float* __restrict__ bpart) {
  constexpr int Mr = 16 * MT, NB = 16 * NT, PX = 32 * S, LD = PX + 8;
  constexpr int XC = PX + 16, LDX = XC + 8;
  constexpr int AHALF = (PX / 8) * (Mr / 8), ABLK = 2 * AHALF;   // dz: b = 0, then b = 1
  constexpr int XBLK = (PX / 8 + 2) * (NB / 8);                  // per source row
  constexpr int NBLK = ABLK + 2 * XBLK, BPT = (NBLK + 255) / 256;
  constexpr int NU = MT * NT, PER_WAVE = (NU + 3) / 4;
  __shared__ __attribute__((aligned(16))) bf16 As[2][Mr][LD];
  __shared__ __attribute__((aligned(16))) bf16 Xs[2][NB][LDX];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int w = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (w >= nwork) return;
  const int nblk = Nc / NB;
  const int a = w & 1, n0 = ((w >> 1) % nblk) * NB, slice = w / (2 * nblk);
  const int nch = (Win + PX - 1) / PX, nst = B * Hin * nch;
  const int s0 = slice * stages_per, s1 = min(nst, s0 + stages_per);
  bf16x8 reg[BPT][8];
  auto load = [&](int sg) {
    const int b = sg / (Hin * nch), rem = sg - b * Hin * nch, i = rem / nch;
    const int j0 = (rem - i * nch) * PX;
#pragma unroll
    for (int bi = 0; bi < BPT; ++bi) {
      const int blk = threadIdx.x + 256 * bi;
#pragma unroll
      for (int e = 0; e < 8; ++e) reg[bi][e] = zero8();
      if (blk < ABLK) {
        const int par = blk / AHALF, r = blk - par * AHALF;
        const int pg = r / (Mr / 8), cg = (r % (Mr / 8)) * 8;
        const int Y = 2 * i + a;
        const bf16* src = dz + ((size_t)b * Hout + Y) * Wout * Mr + cg;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int X = 2 * (j0 + 8 * pg + e) + par;
          if (Y < Hout && X < Wout) reg[bi][e] = load8(src + (size_t)X * Mr);
        }
      } else if (blk < NBLK) {
        const int sy = (blk - ABLK) / XBLK, r = blk - ABLK - sy * XBLK;
        const int ys = i + a + sy - 1;
        if (ys >= 0 && ys < Hin) {
          const int m = r / (NB / 8), cg = (r % (NB / 8)) * 8;
          const int c0 = j0 - 8 + 8 * m;
          const bf16* src = x + ((size_t)b * Hin + ys) * Win * Nc + n0 + cg;
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (c0 + e >= 0 && c0 + e < Win) reg[bi][e] = load8(src + (size_t)(c0 + e) * Nc);
        }
      }
    }
  };
  f32x4 acc[PER_WAVE][8];   // [unit][(b 2 + sy) 2 + sx]
#pragma unroll
  for (int u = 0; u < PER_WAVE; ++u)
#pragma unroll
    for (int d = 0; d < 8; ++d) acc[u][d] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int BT = (MT + 3) / 4;
  const bool bias = (n0 == 0);
  f32x4 accb[BT];
#pragma unroll
  for (int u = 0; u < BT; ++u) accb[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 ones;
#pragma unroll
  for (int q = 0; q < 8; ++q) ones[q] = (bf16)1.f;
  const int kq = 8 * (lane >> 4);
  if (s0 < s1) load(s0);
  for (int sg = s0; sg < s1; ++sg) {
    __syncthreads();
#pragma unroll
    for (int bi = 0; bi < BPT; ++bi) {
      const int blk = threadIdx.x + 256 * bi;
      if (blk < ABLK) {
        const int par = blk / AHALF, r = blk - par * AHALF, g = r % (Mr / 8);
        bf16* dst = &As[par][g * 8][(r / (Mr / 8)) * 8];
        put_transposed<Mr / 8>(reg[bi], g, [&](int c) { return dst + c * LD; });
      } else if (blk < NBLK) {
        const int sy = (blk - ABLK) / XBLK, r = blk - ABLK - sy * XBLK;
        const int m = r / (NB / 8), g = r % (NB / 8);
        bf16* dst = &Xs[sy][g * 8][8 * m];
        put_transposed<NB / 8>(reg[bi], g, [&](int c) { return dst + c * LDX; });
      }
    }
    __syncthreads();
    if (sg + 1 < s1) load(sg + 1);
#pragma unroll
    for (int kk = 0; kk < S; ++kk) {
#pragma unroll
      for (int u = 0; u < PER_WAVE; ++u) {
        const int uu = wave + 4 * u;
        if (uu < NU) {
          const int ti = uu / NT, tj = uu - ti * NT;
          const bf16x8 av0 = *(const bf16x8*)&As[0][ti * 16 + (lane & 15)][kk * 32 + kq];
          const bf16x8 av1 = *(const bf16x8*)&As[1][ti * 16 + (lane & 15)][kk * 32 + kq];
#pragma unroll
          for (int sy = 0; sy < 2; ++sy) {
            const bf16* xr = &Xs[sy][tj * 16 + (lane & 15)][kk * 32 + kq + 8];   // shift 0
            const u32x4 a4 = __builtin_bit_cast(u32x4, *(const bf16x8*)(xr - 8));
            const u32x4 b4 = __builtin_bit_cast(u32x4, *(const bf16x8*)xr);
            const u32x4 c4 = __builtin_bit_cast(u32x4, *(const bf16x8*)(xr + 8));
            const unsigned s0w = (a4[3] >> 16) | (b4[0] << 16), s1w = (b4[0] >> 16) | (b4[1] << 16);
            const unsigned s2w = (b4[1] >> 16) | (b4[2] << 16), s3w = (b4[2] >> 16) | (b4[3] << 16);
            const unsigned s4w = (b4[3] >> 16) | (c4[0] << 16);
            const bf16x8 bl = __builtin_bit_cast(bf16x8, u32x4{s0w, s1w, s2w, s3w});   // -1
            const bf16x8 bm = __builtin_bit_cast(bf16x8, b4);                          // 0
            const bf16x8 br = __builtin_bit_cast(bf16x8, u32x4{s1w, s2w, s3w, s4w});   // +1
            // b = 0: column shifts -1 (sx 0), 0 (sx 1); b = 1: 0 (sx 0), +1 (sx 1)
            acc[u][2 * sy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av0, bl, acc[u][2 * sy], 0, 0, 0);
            acc[u][2 * sy + 1] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(av0, bm, acc[u][2 * sy + 1], 0, 0, 0);
            acc[u][4 + 2 * sy] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(av1, bm, acc[u][4 + 2 * sy], 0, 0, 0);
            acc[u][5 + 2 * sy] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(av1, br, acc[u][5 + 2 * sy], 0, 0, 0);
          }
        }
      }
      if (bias) {
#pragma unroll
        for (int u = 0; u < BT; ++u) {
          const int ti = wave + 4 * u;
          if (ti < MT) {
#pragma unroll
            for (int par = 0; par < 2; ++par) {
              const bf16x8 av = *(const bf16x8*)&As[par][ti * 16 + (lane & 15)][kk * 32 + kq];
              accb[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, ones, accb[u], 0, 0, 0);
            }
          }
        }
      }
    }
  }
  if (bias) {
#pragma unroll
    for (int u = 0; u < BT; ++u) {
      const int ti = wave + 4 * u;
      if (ti < MT && (lane & 15) == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          bpart[((size_t)slice * 2 + a) * Mr + ti * 16 + 4 * (lane >> 4) + q] = accb[u][q];
      }
    }
  }
#pragma unroll
  for (int u = 0; u < PER_WAVE; ++u) {
    const int uu = wave + 4 * u;
    if (uu < NU) {
      const int ti = uu / NT, tj = uu - ti * NT;
      const int c = tj * 16 + (lane & 15);
#pragma unroll
      for (int d = 0; d < 8; ++d) {   // product index (a 2 + b) 2 + sy) 2 + sx = 8 a + d
        float* out = part + (((size_t)slice * 16 + 8 * a + d) * Mr) * Nc + n0;
#pragma unroll
        for (int q = 0; q < 4; ++q) out[(size_t)(ti * 16 + 4 * (lane >> 4) + q) * Nc + c] = acc[u][d][q];
      }
    }
  }
}

// The nine tap gradients of an upsampling layer from the sixteen products
// summed over slices (S [16][Mr][Nc], see k_conv_wgrad_up), in a fixed order.
__global__ void k_up_tapmap(const float* __restrict__ S, int Mr, int Nc, int cout, int cin,
                            float* __restrict__ g) {
  const int id = blockIdx.x * blockDim.x + threadIdx.x;   // (co, ci, tap)
  if (id >= cout * cin * 9) return;
  const int tap = id % 9, ci = (id / 9) % cin, co = id / (9 * cin);
  const int ty = tap / 3, tx = tap % 3;
  float v = 0.f;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int sy = ((a + ty - 1) >> 1) - a + 1, sx = ((b + tx - 1) >> 1) - b + 1;
      v += S[((size_t)(((a * 2 + b) * 2 + sy) * 2 + sx) * Mr + co) * Nc + ci];
    }
  g[id] = v;
}

// Layer-1 weight and bias gradients on FP32 matrix cores: dW[co][j] =
// sum_p dz[p][co] u[p][j], where u[p] is the pixel's 9 C input values
// (plane-major, tap-minor: the [cout][cin][3][3] order of the weights), then 1
// for the bias, then zeros.  Per 4 pixels, 16x16x4 FP32 MFMAs take
// A[r][px] = dz[px][2 r + i] (row r of tile i is channel 2 r + i, so a lane's
// two channels are one 4-byte load) and B[px][jj] = u[px][16 jt + jj].  A
// workgroup owns the contiguous pixel range [p0, p0 + pix_per); per
// iteration it takes 16 pixels, pixel p0 + 16 it + 4 w + px for wave w, and
// C1W_U iterations' loads are issued before their MFMAs.  The four waves are
// summed in LDS; partials [slice][32][32] (column 9 C = bias).
#define C1W_U 4
template <int C>
__global__ __launch_bounds__(256) void k_conv1_wgrad(const float* __restrict__ x0,
                                                     const bf16* __restrict__ dz, int B, int H,
                                                     int W, int pix_per,
                                                     float* __restrict__ part) {
  constexpr int J = 9 * C, NJT = (J + 16) / 16;   // column tiles holding J + 1 columns
  __shared__ float red[4][32 * 32];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, col = lane & 15;
  const int HW = H * W, total = B * HW;
  const int p0 = blockIdx.x * pix_per, p1 = min(total, p0 + pix_per);
  int koff[NJT], kdy[NJT], kdx[NJT];
  bool kone[NJT];
#pragma unroll
  for (int jt = 0; jt < NJT; ++jt) {
    const int j = 16 * jt + col, c = j / 9, t = j - 9 * c;
    kone[jt] = (j == J);
    kdy[jt] = (j < J) ? t / 3 - 1 : -H;   // bias and padding columns read no input
    kdx[jt] = t % 3 - 1;
    koff[jt] = c * HW + kdy[jt] * W + kdx[jt];
  }
  // (b, y, x) of this lane's pixel, advanced by 16 pixels per iteration
  int p = p0 + 4 * wave + g;
  int b = (unsigned)p / (unsigned)HW, x = p - b * HW;
  int y = (unsigned)x / (unsigned)W;
  x -= y * W;
  f32x4 acc[2][NJT];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int jt = 0; jt < NJT; ++jt) acc[i][jt] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int it0 = 0; p0 + 16 * it0 < p1; it0 += C1W_U) {
    uint32_t dv[C1W_U];
    float uv[C1W_U][NJT];
#pragma unroll
    for (int u = 0; u < C1W_U; ++u) {
      const bool pv = p < p1;
      // out-of-range reads go to element 0 / pixel p0 and are zeroed after
      const uint32_t d = *(const uint32_t*)(dz + (size_t)(pv ? p : p0) * 32 + 2 * col);
      dv[u] = pv ? d : 0u;
      const int pb = p + b * (C - 1) * HW;   // element (b, 0, y, x) of the planar input
#pragma unroll
      for (int jt = 0; jt < NJT; ++jt) {
        const bool ok = pv & ((unsigned)(y + kdy[jt]) < (unsigned)H) &
                        ((unsigned)(x + kdx[jt]) < (unsigned)W);
        const float v = x0[ok ? (unsigned)(pb + koff[jt]) : 0u];
        uv[u][jt] = ok ? v : ((pv & kone[jt]) ? 1.f : 0.f);
      }
      p += 16;
      x += 16;
      while (x >= W) {
        x -= W;
        if (++y == H) { y = 0; ++b; }
      }
    }
#pragma unroll
    for (int u = 0; u < C1W_U; ++u) {
      const float a0 = __uint_as_float(dv[u] << 16), a1 = __uint_as_float(dv[u] & 0xffff0000u);
#pragma unroll
      for (int jt = 0; jt < NJT; ++jt) {
        acc[0][jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, uv[u][jt], acc[0][jt], 0, 0, 0);
        acc[1][jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, uv[u][jt], acc[1][jt], 0, 0, 0);
      }
    }
  }
  // lane holds rows 4 g + q (channel 2 (4 g + q) + i) of column 16 jt + col
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float* r = &red[wave][(2 * (4 * g + q) + i) * 32 + col];
#pragma unroll
      for (int jt = 0; jt < NJT; ++jt) r[16 * jt] = acc[i][jt][q];
      if (NJT == 1) r[16] = 0.f;
    }
  __syncthreads();
  float* out = part + (size_t)blockIdx.x * 32 * 32;
  for (int e = threadIdx.x; e < 32 * 32; e += 256)
    out[e] = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
}

// Sum over slices of [slice][nent] partials for 16 consecutive entries per
// workgroup: 16 slice groups (slices g, g + 16, ...) added in group order.
__device__ __forceinline__ float slice_sum16(const float* __restrict__ part, int nslices, int nent,
                                             int ent, float (*red)[16]) {
  const int j = threadIdx.x & 15, grp = threadIdx.x >> 4;
  float s = 0.f;
  if (ent < nent) {
    // slices grp, grp + 16, ... added in order; eight loads in flight at a time
    int sl = grp;
    for (; sl + 112 < nslices; sl += 128) {
      float a[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) a[q] = part[(size_t)(sl + 16 * q) * nent + ent];
#pragma unroll
      for (int q = 0; q < 8; ++q) s += a[q];
    }
    for (; sl < nslices; sl += 16) s += part[(size_t)sl * nent + ent];
  }
  red[grp][j] = s;
  __syncthreads();
  float t = 0.f;
  if (grp == 0)
    for (int g = 0; g < 16; ++g) t += red[g][j];
  return t;
}

// Sum the [slice][32][32] partials of k_conv1_wgrad (16 entries per block).
__global__ __launch_bounds__(256) void k_conv1_rows_reduce(const float* __restrict__ part,
                                                           int nslices, int cout, int C,
                                                           float* __restrict__ gw,
                                                           float* __restrict__ gb) {
  __shared__ float red[16][16];
  const int J = 9 * C;
  const int ent = blockIdx.x * 16 + (threadIdx.x & 15);
  const float s = slice_sum16(part, nslices, 32 * 32, ent, red);
  const int co = ent / 32, j = ent % 32;
  if ((threadIdx.x >> 4) == 0 && co < cout && j <= J) {
    if (j < J) gw[(size_t)co * J + j] = s;
    else gb[co] = s;
  }
}

// Sum the slices (fixed order) into the FP32 gradient in [cout][cin][3][3]
// order.  A workgroup takes 64 consecutive partial entries ([tap][r][c]
// order, coalesced reads) and four slice groups (slices g, g + 4, ...), which
// are then added in group order.
// NE = 9: the tap gradients, written to g ([cout][cin][9]); NE = 16: the
// products of an upsampling layer, written to S ([16][Mr][Nc]) for k_up_tapmap.
template <int NE>
__global__ __launch_bounds__(256) void k_wgrad_reduce(const float* __restrict__ part, int nslices,
                                                      int Mr, int Nc, int cout, int cin,
                                                      float* __restrict__ g) {
  __shared__ float red[4][64];
  const int j = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int ent = blockIdx.x * 64 + j, nent = NE * Mr * Nc;
  float s = 0.f;
  if (ent < nent) {
    // slices grp, grp + 4, ... added in order; eight loads in flight at a time
    int sl = grp;
    for (; sl + 28 < nslices; sl += 32) {
      float a[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) a[q] = part[(size_t)(sl + 4 * q) * nent + ent];
#pragma unroll
      for (int q = 0; q < 8; ++q) s += a[q];
    }
    for (; sl < nslices; sl += 4) s += part[(size_t)sl * nent + ent];
  }
  red[grp][j] = s;
  __syncthreads();
  if (grp == 0 && ent < nent) {
    const float v = ((red[0][j] + red[1][j]) + red[2][j]) + red[3][j];
    if (NE == 16) {
      g[ent] = v;
    } else {
      const int tap = ent / (Mr * Nc), rem = ent - tap * Mr * Nc, co = rem / Nc, ci = rem - co * Nc;
      if (co < cout && ci < cin) g[((size_t)co * cin + ci) * 9 + tap] = v;
    }
  }
}
__global__ __launch_bounds__(256) void k_bgrad_reduce(const float* __restrict__ part, int nslices,
                                                      int Mr, int cout, float* __restrict__ g) {
  __shared__ float red[16][16];
  const int r = blockIdx.x * 16 + (threadIdx.x & 15);
  const float s = slice_sum16(part, nslices, Mr, r, red);
  if ((threadIdx.x >> 4) == 0 && r < cout) g[r] = s;
}

// ------------------------------------------------ input, loss, output ----
// loss partials and dz of the last (linear) layer: out and target are complex
// fields [B][k][D]; dz = 2 (out - t) / count in bf16 with coutp channels.
// One thread per (pixel, group of 8 channels) (coutp is a multiple of 32), so
// that a pixel's dz row is written by consecutive threads 16 B at a time.
__global__ __launch_bounds__(256) void k_mse(const float* __restrict__ out,
                                             const float2* __restrict__ target, int B, int D,
                                             int k, int coutp, float scale,
                                             bf16* __restrict__ dz, float* __restrict__ lpart) {
  const int CG = coutp / 8;
  const long t = (long)blockIdx.x * 256 + threadIdx.x;
  float s = 0.f;
  if (t < (long)B * D * CG) {
    const int p = (int)(t / CG), c0 = (int)(t - (long)p * CG) * 8;
    const int b = p / D, e = p - b * D;
    const float2* o = (const float2*)out + (size_t)b * k * D + e;   // field j at o[j D]
    bf16x8 h;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = c0 / 2 + q;
      float gx = 0.f, gy = 0.f;
      if (j < k) {
        const float2 v = o[(size_t)j * D], tv = target[((size_t)b * k + j) * D + e];
        const float dx = v.x - tv.x, dy = v.y - tv.y;
        s += dx * dx + dy * dy;
        gx = scale * dx; gy = scale * dy;
      }
      h[2 * q] = (bf16)gx;
      h[2 * q + 1] = (bf16)gy;
    }
    *(u32x4*)(dz + (size_t)p * coutp + c0) = __builtin_bit_cast(u32x4, h);
  }
  __shared__ float lds[8];
  s = block_sum1<float>(s, lds);
  if (threadIdx.x == 0) lpart[blockIdx.x] = s;
}

// ------------------------------------------------------- parameters ----
// bf16 GEMM copies of one layer's FP32 weights [cout][cin][3][3].
__global__ void k_pack_weights(const float* __restrict__ w, int cout, int cin, int coutp,
                               int cinp, bf16* __restrict__ wf, bf16* __restrict__ wb) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= 9 * coutp * cinp) return;
  const int tap = idx / (coutp * cinp), rem = idx % (coutp * cinp);
  const int co = rem / cinp, ci = rem % cinp;
  const float v = (co < cout && ci < cin) ? w[((size_t)co * cin + ci) * 9 + tap] : 0.f;
  wf[idx] = (bf16)v;
  if (wb) wb[((size_t)tap * cinp + ci) * coutp + co] = (bf16)v;
}

// Adam (Kingma & Ba) on the FP32 master parameters.
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, size_t n, float lr, float b1, float b2, float c1,
                       float c2, float eps) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Effective backward-data weights of an upsampled layer (k_conv_tile_s2):
// wu[e][ci][co] = sum of w[co][ci][dy][dx] over the taps whose dz offset is
// (oy, ox) = (e / 4 - 1, e % 4 - 1), i.e. sy = oy + dy - 1 and sx = ox + dx - 1
// in {0, 1}; FP32 sums rounded once to bf16.
__global__ void k_pack_up_weights(const float* __restrict__ w, int cout, int cin, int coutp,
                                  int cinp, bf16* __restrict__ wu) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= 16 * cinp * coutp) return;
  const int e = idx / (cinp * coutp), rem = idx % (cinp * coutp);
  const int ci = rem / coutp, co = rem % coutp;
  const int oy = e / 4 - 1, ox = e % 4 - 1;
  float v = 0.f;
  if (co < cout && ci < cin)
    for (int dy = 0; dy < 3; ++dy) {
      const int sy = oy + dy - 1;
      if (sy < 0 || sy > 1) continue;
      for (int dx = 0; dx < 3; ++dx) {
        const int sx = ox + dx - 1;
        if (sx < 0 || sx > 1) continue;
        v += w[((size_t)co * cin + ci) * 9 + dy * 3 + dx];
      }
    }
  wu[idx] = (bf16)v;
}

// bias for layers whose coutp > cout: a zero-padded FP32 copy
__global__ void k_pad_bias(const float* __restrict__ b, int cout, int coutp, float* __restrict__ bp) {
  const int i = threadIdx.x;
  if (i < coutp) bp[i] = (i < cout) ? b[i] : 0.f;
}

// ============================================================ host side ====
// MFMA kernels take 32, 64 or 128 channels (the K loop steps 32 channels)
static int rup32(int c) { return (c + 31) / 32 * 32; }

// pixels per weight-gradient slice: about 256 slices, multiples of 32

template <typename X>
static hipError_t cnn_alloc(dd_cnn* n, X** p, size_t count) {
  hipError_t e = hipMalloc((void**)p, std::max<size_t>(count * sizeof(X), 256));
  if (e == hipSuccess) {
    n->allocs.push_back((void*)*p);
    e = hipMemset(*p, 0, std::max<size_t>(count * sizeof(X), 256));
  }
  return e;
}

extern "C" void dd_cnn_destroy(dd_cnn* net) {
  if (!net) return;
  (void)hipDeviceSynchronize();
  for (void* p : net->allocs) (void)hipFree(p);
  delete net;
}

static dd_status pack_all(dd_cnn* n, hipStream_t st) {
  for (int l = 0; l < NL; ++l) {
    const CnnLayer& L = n->L[l];
    if (l == 0) continue;  // layer 1 reads the FP32 master weights directly
    const int tot = 9 * L.coutp * L.cinp;
    k_pack_weights<<<(tot + 255) / 256, 256, 0, st>>>(n->params + L.woff, L.cout, L.cin, L.coutp,
                                                      L.cinp, n->wf[l], n->wb[l]);
    if (L.up)
      k_pack_up_weights<<<(16 * L.cinp * L.coutp + 255) / 256, 256, 0, st>>>(
          n->params + L.woff, L.cout, L.cin, L.coutp, L.cinp, n->wu[l]);
    k_pad_bias<<<1, 256, 0, st>>>(n->params + L.boff, L.cout, L.coutp, n->biaspad + 256 * l);
  }
  DD_HIP_CHECK(hipGetLastError());
  return DD_OK;
}

extern "C" dd_status dd_cnn_create(int nx, int ny, int max_batch, int k, int in_channels,
                                   unsigned long long seed, dd_cnn** out) {
  if (!out) { dd_set_error("dd_cnn_create: out is NULL"); return DD_EINVAL; }
  *out = nullptr;
  if (nx < 4 || ny < 4 || nx % 4 || ny % 4 || max_batch < 1 || k < 1 || 2 * k > 64 ||
      (in_channels != 1 && in_channels != 3)) {
    dd_set_error("dd_cnn_create: need nx, ny multiples of 4, max_batch >= 1, 1 <= k <= 32 "
                 "and 1 or 3 input channels");
    return DD_EINVAL;
  }
  dd_cnn* n = new dd_cnn();
  n->nx = nx; n->ny = ny; n->maxB = max_batch; n->k = k; n->cin0 = in_channels;
  {
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        ncu > 0)
      n->ncu = ncu;
  }
  const int spec[NL][5] = {{in_channels, 32, 1, 0, 1}, {32, 64, 2, 0, 1}, {64, 128, 2, 0, 1},
                           {128, 128, 1, 0, 1}, {128, 64, 1, 1, 1}, {64, 32, 1, 1, 1},
                           {32, 32, 1, 0, 1}, {32, 2 * k, 1, 0, 0}};
  int H = ny, W = nx;
  size_t off = 0;
  for (int l = 0; l < NL; ++l) {
    CnnLayer& L = n->L[l];
    L.cin = spec[l][0]; L.cout = spec[l][1]; L.stride = spec[l][2]; L.up = spec[l][3];
    L.relu = spec[l][4];
    L.cinp = (l == 0) ? L.cin : rup32(L.cin);
    L.coutp = rup32(L.cout);
    L.Hin = H; L.Win = W;
    if (L.up) { L.Hout = 2 * H; L.Wout = 2 * W; }
    else if (L.stride == 2) { L.Hout = H / 2; L.Wout = W / 2; }
    else { L.Hout = H; L.Wout = W; }
    L.mode = L.up ? MAP_UP : (L.stride == 2 ? MAP_S2 : MAP_S1);
    L.woff = off; off += (size_t)L.cout * L.cin * 9;
    L.boff = off; off += L.cout;
    H = L.Hout; W = L.Wout;
  }
  n->nparams = off;
  // He-uniform initialisation (host mt19937_64), zero biases
  std::vector<float> hp(off, 0.f);
  std::mt19937_64 rng(seed);
  for (int l = 0; l < NL; ++l) {
    const CnnLayer& L = n->L[l];
    const float bound = std::sqrt(6.0f / (L.cin * 9));
    std::uniform_real_distribution<float> ud(-bound, bound);
    for (size_t i = 0; i < (size_t)L.cout * L.cin * 9; ++i) hp[L.woff + i] = ud(rng);
  }
  hipError_t e = hipSuccess;
  auto chk = [&](hipError_t x) { if (x != hipSuccess && e == hipSuccess) e = x; };
  chk(cnn_alloc(n, &n->params, off + 64));
  chk(cnn_alloc(n, &n->grads, off + 64));
  chk(cnn_alloc(n, &n->am, off + 64));
  chk(cnn_alloc(n, &n->av, off + 64));
  const size_t D = (size_t)nx * ny;
  chk(cnn_alloc(n, &n->x0, (size_t)max_batch * D * in_channels));
  chk(cnn_alloc(n, &n->espart, (size_t)max_batch * ES_SLICES));
  size_t wp = 0;
  for (int l = 0; l < NL && e == hipSuccess; ++l) {
    const CnnLayer& L = n->L[l];
    const size_t pix = (size_t)max_batch * L.Hout * L.Wout;
    if (l > 0) {
      chk(cnn_alloc(n, &n->wf[l], (size_t)9 * L.coutp * L.cinp));
      chk(cnn_alloc(n, &n->wb[l], (size_t)9 * L.coutp * L.cinp));
      if (L.up) chk(cnn_alloc(n, &n->wu[l], (size_t)16 * L.coutp * L.cinp));
    }
    if (l < NL - 1) chk(cnn_alloc(n, &n->act[l], pix * L.coutp));
    chk(cnn_alloc(n, &n->dz[l], pix * L.coutp));
    // gradient partials: room for 8 workgroups per CU (256 threads each)
    // over 3 dy and the 64-channel blocks (k_conv_wgrad_row takes fewer
    // slices when its occupancy asks for more than fit); layer 1 uses
    // [slice][32][32] (at most 8 slices per CU)
    if (l > 0) {
      const size_t nblk = (size_t)std::max(1, L.cinp / 64);
      const size_t sl = std::max<size_t>(1, (size_t)8 * n->ncu / (3 * nblk));
      const size_t wl = (size_t)L.coutp * L.cinp;
      wp = std::max(wp, sl * (9 * wl + L.coutp));
      // upsampling (k_conv_wgrad_up, up to 4 workgroups per CU over the two
      // parities): 16 products and two bias rows per slice, then their sums
      if (L.up) wp = std::max(wp, (size_t)2 * n->ncu / nblk * (16 * wl + 2 * L.coutp) + 16 * wl);
    } else {
      wp = std::max(wp, (size_t)8 * n->ncu * 32 * 32);
    }
  }
  n->wpart_elems = wp;
  chk(cnn_alloc(n, &n->wpart, wp));
  chk(cnn_alloc(n, &n->out, (size_t)max_batch * D * 2 * k));
  chk(cnn_alloc(n, &n->lpart, (size_t)max_batch * D * 8 / 256 + 256));   // k_mse: coutp / 8 <= 8
  chk(cnn_alloc(n, &n->biaspad, (size_t)256 * NL));
  if (e == hipSuccess) chk(hipMemcpy(n->params, hp.data(), sizeof(float) * off, hipMemcpyHostToDevice));
  if (e != hipSuccess) {
    dd_set_error("dd_cnn_create: %s", hipGetErrorString(e));
    dd_cnn_destroy(n);
    return e == hipErrorOutOfMemory ? DD_ENOMEM : DD_EHIP;
  }
  dd_status rc = pack_all(n, 0);
  if (rc != DD_OK) { dd_cnn_destroy(n); return rc; }
  DD_HIP_CHECK(hipDeviceSynchronize());
  *out = n;
  return DD_OK;
}

extern "C" int dd_cnn_layer_info(const dd_cnn* n, int l, int* cin, int* cout, int* stride,
                                 int* up, int* relu) {
  if (!n) return -1;
  if (l < 0 || l >= NL) return NL;
  const CnnLayer& L = n->L[l];
  if (cin) *cin = L.cin;
  if (cout) *cout = L.cout;
  if (stride) *stride = L.stride;
  if (up) *up = L.up;
  if (relu) *relu = L.relu;
  return NL;
}

extern "C" size_t dd_cnn_num_params(const dd_cnn* n) { return n ? n->nparams : 0; }

extern "C" dd_status dd_cnn_get_params(const dd_cnn* n, float* host, size_t count) {
  if (!n || !host || count != n->nparams) {
    dd_set_error("dd_cnn_get_params: bad argument (count must be %zu)", n ? n->nparams : (size_t)0);
    return DD_EINVAL;
  }
  DD_HIP_CHECK(hipDeviceSynchronize());
  DD_HIP_CHECK(hipMemcpy(host, n->params, sizeof(float) * count, hipMemcpyDeviceToHost));
  return DD_OK;
}

extern "C" dd_status dd_cnn_set_params(dd_cnn* n, const float* host, size_t count) {
  if (!n || !host || count != n->nparams) {
    dd_set_error("dd_cnn_set_params: bad argument (count must be %zu)", n ? n->nparams : (size_t)0);
    return DD_EINVAL;
  }
  DD_HIP_CHECK(hipDeviceSynchronize());
  DD_HIP_CHECK(hipMemcpy(n->params, host, sizeof(float) * count, hipMemcpyHostToDevice));
  DD_HIP_CHECK(hipMemset(n->am, 0, sizeof(float) * count));
  DD_HIP_CHECK(hipMemset(n->av, 0, sizeof(float) * count));
  n->adam_t = 0;
  dd_status rc = pack_all(n, 0);
  if (rc != DD_OK) return rc;
  DD_HIP_CHECK(hipDeviceSynchronize());
  return DD_OK;
}

// One launch of k_conv_tile: tiles of TH rows, 16 MT channels a workgroup.
template <int MT, int TH>
static void launch_conv_tile(const GemmArgs& a, bool bwd, hipStream_t st) {
  const dim3 grid((a.Wq + CT_TW - 1) / CT_TW, (a.Hq + TH - 1) / TH, a.B * (a.M / (16 * MT)));
  if (bwd) k_conv_tile<MT, TH, true><<<grid, 64 * TH, 0, st>>>(a);
  else k_conv_tile<MT, TH, false><<<grid, 64 * TH, 0, st>>>(a);
}

// The same of k_conv_tile_s2: a 3 x 3 window forward, 4 x 4 backward.
template <int MT, int KS, int TH>
static void launch_conv_s2(const GemmArgs& a, hipStream_t st) {
  const dim3 grid((a.Wq + CS_TW - 1) / CS_TW, (a.Hq + TH - 1) / TH, a.B * (a.M / (16 * MT)));
  k_conv_tile_s2<MT, KS, TH, KS == 4><<<grid, 64 * TH, 0, st>>>(a);
}

static dd_status gemm_dispatch(const GemmArgs& a, bool bwd, int ncu, hipStream_t st) {
  const int MT = a.M / 16;
  if ((MT != 2 && MT != 4 && MT != 8) || a.M % 16 || a.Ksrc % 32) {
    dd_set_error("dd_cnn: no convolution kernel for %d result / %d source channels", a.M, a.Ksrc);
    return DD_EINVAL;
  }
  if (a.mode == MAP_S1 || (!bwd && a.mode == MAP_UP)) {
    // Tall tiles (the halo a smaller share, the weights staged once for twice the
    // rows) with all of up to 64 (128 in tall tiles) channels, where they fill
    // the chip twice; else the most workgroups: 32 channels and 4 rows each.
    // Measured at 480 x 240, batch 64 (and 1): 32 channels 265, 200, 229 us tall
    // against 325, 219, 261 (8.4, 6.3, 7.4 against 9.1, 6.7, 7.9); 64 channels 263 us
    // with all against 274 in halves (13.7 against 9.8); 128 channels 137 us against
    // 157 in quarters (28.2 against 10.0).
    const long long wide = (long long)((a.Wq + CT_TW - 1) / CT_TW) * a.B;
    const long long tall = wide * ((a.Hq + 7) / 8), flat = wide * ((a.Hq + 3) / 4);
    if (MT == 8 && tall >= 2 * ncu) launch_conv_tile<8, 8>(a, bwd, st);
    else if (MT == 4 && flat >= 2 * ncu) launch_conv_tile<4, 4>(a, bwd, st);
    else if (MT == 2 && tall >= 2 * ncu) launch_conv_tile<2, 8>(a, bwd, st);
    else launch_conv_tile<2, 4>(a, bwd, st);
    return DD_OK;
  }
  if ((!bwd && a.mode == MAP_S2 && !a.outf) || (bwd && a.mode == MAP_UP)) {
    // As above: 64 channels and 8 rows, or 32 and 4.  Measured at 480 x 240, batch
    // 64 (and 1): layer 2 213 us against 245 (6.9 against 6.2), layer 3 174 against
    // 192 (9.8 against 7.1); backward at batch 32, layer 6 138 against 156, layer
    // 5 115 against 128.  Four rows of 64 channels (one workgroup a compute unit)
    // are slower than either: with 8-byte stores 305, 227, 223 and 174 us.
    const long long tall = (long long)((a.Wq + CS_TW - 1) / CS_TW) * ((a.Hq + 7) / 8) * a.B * (MT / 4);
    if (tall >= 2 * ncu) {
      if (bwd) launch_conv_s2<4, 4, 8>(a, st);
      else launch_conv_s2<4, 3, 8>(a, st);
    } else {
      if (bwd) launch_conv_s2<2, 4, 4>(a, st);
      else launch_conv_s2<2, 3, 4>(a, st);
    }
    return DD_OK;
  }
  if (bwd && a.mode == MAP_S2) {
    const dim3 grid((a.Wq + BS_TW - 1) / BS_TW, (a.Hq + BS_TH - 1) / BS_TH, a.B);
    // the stride-2 layers have 32- and 64-channel inputs
    switch (MT) {
      case 2: k_bwd_s2_tile<2><<<grid, 256, 0, st>>>(a); return DD_OK;
      case 4: k_bwd_s2_tile<4><<<grid, 256, 0, st>>>(a); return DD_OK;
    }
    dd_set_error("dd_cnn: no stride-2 backward-data kernel for %d channels", a.M);
    return DD_EINVAL;
  }
  dd_set_error("dd_cnn: no convolution kernel for this layer map");
  return DD_EINVAL;
}

// fields: destination of the complex output fields [B][k][D] (n->out if NULL)
static dd_status forward(dd_cnn* n, const float* eps, const void* eim, int B, hipStream_t st,
                         void* fields = nullptr) {
  const int D = n->nx * n->ny;
  {
    const CnnLayer& L = n->L[0];
    const float *w = n->params + L.woff, *bias = n->params + L.boff;
    const float2* F = (const float2*)eim;
    const dim3 grid((n->nx + 63) / 64, (n->ny + C1_TH - 1) / C1_TH, B);
    if (n->cin0 == 3) {
      k_eim_scale_part<<<dim3(ES_SLICES, B), 256, 0, st>>>(F, D, n->espart);
      k_conv1_fwd<3><<<grid, 256, 0, st>>>(eps, F, n->espart, w, bias, n->ny, n->nx, n->x0, n->act[0]);
    } else {
      k_conv1_fwd<1><<<grid, 256, 0, st>>>(eps, F, n->espart, w, bias, n->ny, n->nx, n->x0, n->act[0]);
    }
  }
  for (int l = 1; l < NL; ++l) {
    const CnnLayer& L = n->L[l];
    GemmArgs a{};
    a.src = n->act[l - 1];
    a.W = n->wf[l];
    a.bias = n->biaspad + 256 * l;
    a.B = B; a.Hq = L.Hout; a.Wq = L.Wout;
    a.Hs = L.Hin; a.Ws = L.Win;
    a.Ksrc = L.cinp; a.M = L.coutp; a.mode = L.mode; a.relu = L.relu;
    if (l == NL - 1) {
      a.outf = fields ? (float*)fields : n->out;
      a.nreal = L.cout;
      n->last_fields = a.outf;
    }
    else a.out = n->act[l];
    const dd_status rc = gemm_dispatch(a, false, n->ncu, st);
    if (rc != DD_OK) return rc;
  }
  DD_HIP_CHECK(hipGetLastError());
  return DD_OK;
}

// Work split of the weight-gradient kernel k_conv_wgrad_row
// over nst stages: one round of resident workgroups (cap per CU), within the
// partial buffer (weights, then bias).
struct WgradSplit {
  int slices, stages_per, nwork, grid;
};
// dsplit: work items per (slice, channel block), 3 (one per dy), 2 (one per
// output-row parity, upsampling) or 1.  ne: weight partials per slice (9
// taps, or the 16 products of an upsampling layer, which also keep their
// 16 Mr Nc sums after the partials); nbias: bias partials per slice.
static WgradSplit wgrad_split(const dd_cnn* n, int cap, int Mr, int Nc, int NB, int nst,
                              int dsplit = 3, int ne = 9, int nbias = 1) {
  const int nblk = Nc / NB;
  const size_t per = (size_t)ne * Mr * Nc + (size_t)nbias * Mr;
  const size_t reserve = ne == 9 ? 0 : (size_t)ne * Mr * Nc;
  int slices = std::max(1, cap * n->ncu / (dsplit * nblk));
  slices = (int)std::min<size_t>((size_t)slices, (n->wpart_elems - reserve) / per);
  slices = std::max(1, std::min(slices, nst));
  const int sp = (nst + slices - 1) / slices;
  slices = (nst + sp - 1) / sp;
  const int nwork = slices * dsplit * nblk;
  return {slices, sp, nwork, (nwork + 7) / 8 * 8};
}

// resident workgroups per CU of a kernel (at least 1)
template <typename K>
static int occupancy(K kern) {
  int c = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&c, kern, 256, 0) != hipSuccess || c < 1) c = 1;
  return c;
}

template <int MT, int NT, int S, int MK, int ND = 1>
static int launch_wgrad_row(dd_cnn* n, int l, int B, hipStream_t st) {
  static const int cap = occupancy(k_conv_wgrad_row<MT, NT, S, MK, ND>);
  const CnnLayer& L = n->L[l];
  const int Mr = 16 * MT, Nc = L.cinp;
  const int nst = B * L.Hout * ((L.Wout + 32 * S - 1) / (32 * S));
  const WgradSplit w = wgrad_split(n, cap, Mr, Nc, 16 * NT, nst, ND == 3 ? 1 : 3);
  k_conv_wgrad_row<MT, NT, S, MK, ND><<<w.grid, 256, 0, st>>>(
      n->dz[l], n->act[l - 1], B, L.Hout, L.Wout, L.Hin, L.Win, Nc, w.stages_per, w.nwork,
      n->wpart, n->wpart + (size_t)w.slices * 9 * Mr * Nc);
  return w.slices;
}

template <int MT, int NT, int S>
static int launch_wgrad_ring(dd_cnn* n, int l, int B, hipStream_t st) {
  static const int cap = occupancy(k_conv_wgrad_ring<MT, NT, S>);
  const CnnLayer& L = n->L[l];
  const int Mr = 16 * MT, Nc = L.cinp;
  const int nst = B * L.Hout * ((L.Wout + 32 * S - 1) / (32 * S));
  const WgradSplit w = wgrad_split(n, cap, Mr, Nc, 16 * NT, nst, 1);
  k_conv_wgrad_ring<MT, NT, S><<<w.grid, 256, 0, st>>>(
      n->dz[l], n->act[l - 1], B, L.Hout, L.Wout, Nc, w.stages_per, w.nwork, n->wpart,
      n->wpart + (size_t)w.slices * 9 * Mr * Nc);
  return w.slices;
}

// whether an upsampling layer's weight gradient runs on k_conv_wgrad_up
static bool wgrad_up_kernel(const CnnLayer& L) {
  return (L.coutp == 64 && L.cinp % 32 == 0) || (L.coutp == 32 && L.cinp % 64 == 0);
}

template <int MT, int NT, int S>
static int launch_wgrad_up(dd_cnn* n, int l, int B, hipStream_t st) {
  static const int cap = occupancy(k_conv_wgrad_up<MT, NT, S>);
  const CnnLayer& L = n->L[l];
  const int Mr = 16 * MT, Nc = L.cinp;
  const int nst = B * L.Hin * ((L.Win + 32 * S - 1) / (32 * S));
  const WgradSplit w = wgrad_split(n, cap, Mr, Nc, 16 * NT, nst, 2, 16, 2);
  k_conv_wgrad_up<MT, NT, S><<<w.grid, 256, 0, st>>>(
      n->dz[l], n->act[l - 1], B, L.Hout, L.Wout, L.Hin, L.Win, Nc, w.stages_per, w.nwork,
      n->wpart, n->wpart + (size_t)w.slices * 16 * Mr * Nc);
  return w.slices;
}

// Weight- and bias-gradient partials of layer l >= 1 (row chunks, every
// map).  Returns the number of pixel slices written to n->wpart (weights
// [slice][9][coutp][cinp], then bias [slice][coutp]), 0 (nothing launched)
// for channel counts without an instance.
static int wgrad_partials(dd_cnn* n, int l, int B, hipStream_t st) {
  const CnnLayer& L = n->L[l];
  const int Mr = L.coutp, Nc = L.cinp, NB = std::min(Nc, 64);
  if (Nc % NB) return 0;
  // S (stage width 32 S pixels, 1, 2 or 4): the largest whose 8 x 8 staging
  // blocks (dz, then the input pixels of one dy row) fit one per thread.
  // The kernels with 32 output channels take all three dy per work item
  // (ND = 3: dz staged once for the three input rows).
  auto blocks = [&](int S) {
    const int xg = (L.mode == MAP_S1) ? 4 * S + 2 : (L.mode == MAP_UP) ? 2 * S + 1 : 8 * S;
    return 4 * S * (Mr / 8) + xg * (NB / 8);
  };
  const int S = blocks(4) <= 256 ? 4 : (blocks(2) <= 256 ? 2 : 1);
#define WG_CASES(F, F3)                                                    \
  if (Mr == 32 && NB == 32) return S == 4 ? F3(2, 2, 4) : 0;           \
  if (Mr == 32 && NB == 64) return S == 4 ? F3(2, 4, 4) : F(2, 4, 2);  \
  if (Mr == 64 && NB == 32) return S == 4 ? F(4, 2, 4) : F(4, 2, 2);   \
  if (Mr == 64 && NB == 64) return S == 4 ? F(4, 4, 4) : F(4, 4, 2);   \
  if (Mr == 128 && NB == 32) return S == 2 ? F(8, 2, 2) : 0;           \
  if (Mr == 128 && NB == 64) return S == 2 ? F(8, 4, 2) : F(8, 4, 1);
#define WG_ROW1(a, b, c) launch_wgrad_row<a, b, c, MAP_S1>(n, l, B, st)
#define WG_ROWU(a, b, c) launch_wgrad_row<a, b, c, MAP_UP>(n, l, B, st)
#define WG_ROW2(a, b, c) launch_wgrad_row<a, b, c, MAP_S2>(n, l, B, st)
#define WG_ROW13(a, b, c) launch_wgrad_row<a, b, c, MAP_S1, 3>(n, l, B, st)
#define WG_ROWU3(a, b, c) launch_wgrad_row<a, b, c, MAP_UP, 3>(n, l, B, st)
#define WG_ROW23(a, b, c) launch_wgrad_row<a, b, c, MAP_S2, 3>(n, l, B, st)
  if (L.mode == MAP_S1) {
    // 32 output and 32 input channels (layers 7, 8): input rows in a ring
    if (Mr == 32 && NB == 32) return launch_wgrad_ring<2, 2, 4>(n, l, B, st);
    WG_CASES(WG_ROW1, WG_ROW13)
  }
  else if (L.mode == MAP_UP) {
    // the two upsampling layers (128 -> 64 and 64 -> 32 channels) at the
    // source resolution, sixteen products per pixel
    if (wgrad_up_kernel(L)) {
      return Mr == 64 ? launch_wgrad_up<4, 2, 2>(n, l, B, st) : launch_wgrad_up<2, 4, 2>(n, l, B, st);
    }
    WG_CASES(WG_ROWU, WG_ROWU3)
  }
  else {
    // 64 output and 32 input channels: three dy per item at half the stage
    // width (the 18 accumulators per unit fit; 130 -> 101 us at batch 32)
    if (Mr == 64 && NB == 32) return WG_ROW23(4, 2, 2);
    WG_CASES(WG_ROW2, WG_ROW23)
  }
#undef WG_CASES
#undef WG_ROW1
#undef WG_ROWU
#undef WG_ROW2
#undef WG_ROW13
#undef WG_ROWU3
#undef WG_ROW23
  return 0;
}

// Backward pass from the gradient of the last layer's pre-activation in
// dz[NL-1]; parameter gradients land in n->grads.
static dd_status backward_from_dz(dd_cnn* n, int B, hipStream_t st) {
  for (int l = NL - 1; l >= 1; --l) {
    const CnnLayer& L = n->L[l];
    // weight and bias gradients of layer l
    const int wslices = wgrad_partials(n, l, B, st);
    if (wslices <= 0) {
      dd_set_error("dd_cnn: no weight-gradient kernel for %d x %d channels", L.coutp, L.cinp);
      return DD_EINVAL;
    }
    if (L.mode == MAP_UP && wgrad_up_kernel(L)) {
      // sixteen products per slice, then bias [slice][parity][r]; their sums
      // over slices after both, then mapped onto the nine taps
      const int nent = 16 * L.coutp * L.cinp;
      float* S = n->wpart + (size_t)wslices * (nent + 2 * L.coutp);
      k_wgrad_reduce<16><<<(nent + 63) / 64, 256, 0, st>>>(n->wpart, wslices, L.coutp, L.cinp,
                                                           L.cout, L.cin, S);
      const int nmap = 9 * L.cout * L.cin;
      k_up_tapmap<<<(nmap + 255) / 256, 256, 0, st>>>(S, L.coutp, L.cinp, L.cout, L.cin,
                                                      n->grads + L.woff);
      k_bgrad_reduce<<<(L.coutp + 15) / 16, 256, 0, st>>>(n->wpart + (size_t)wslices * nent,
                                                           2 * wslices, L.coutp, L.cout,
                                                           n->grads + L.boff);
    } else {
      const int nent = 9 * L.coutp * L.cinp;
      k_wgrad_reduce<9><<<(nent + 63) / 64, 256, 0, st>>>(n->wpart, wslices, L.coutp, L.cinp,
                                                          L.cout, L.cin, n->grads + L.woff);
      k_bgrad_reduce<<<(L.coutp + 15) / 16, 256, 0, st>>>(n->wpart + (size_t)wslices * nent,
                                                           wslices, L.coutp, L.cout,
                                                           n->grads + L.boff);
    }
    // data gradient into the previous layer (masked by its ReLU)
    GemmArgs a{};
    a.src = n->dz[l];
    a.W = L.up ? n->wu[l] : n->wb[l];
    a.mask = n->act[l - 1];
    a.out = n->dz[l - 1];
    a.B = B; a.Hq = L.Hin; a.Wq = L.Win;
    a.Hs = L.Hout; a.Ws = L.Wout;
    a.Ksrc = L.coutp; a.M = L.cinp; a.mode = L.mode;
    const dd_status rc = gemm_dispatch(a, true, n->ncu, st);
    if (rc != DD_OK) return rc;
  }
  {
    const CnnLayer& L = n->L[0];
    // about four workgroups per CU (fewer partials to sum), within the
    // partial buffer; each takes a multiple of 16 C1W_U pixels
    const int total = B * n->nx * n->ny;
    const int want = (int)std::min<size_t>((size_t)4 * n->ncu, n->wpart_elems / (32 * 32));
    const int step = 16 * C1W_U;
    const int pp = (total + want - 1) / want, pix_per = (pp + step - 1) / step * step;
    const int slices = (total + pix_per - 1) / pix_per;
    if (n->cin0 == 3)
      k_conv1_wgrad<3><<<slices, 256, 0, st>>>(n->x0, n->dz[0], B, n->ny, n->nx, pix_per,
                                               n->wpart);
    else
      k_conv1_wgrad<1><<<slices, 256, 0, st>>>(n->x0, n->dz[0], B, n->ny, n->nx, pix_per,
                                               n->wpart);
    k_conv1_rows_reduce<<<64, 256, 0, st>>>(n->wpart, slices, L.cout, n->cin0,
                                            n->grads + L.woff, n->grads + L.boff);
  }
  DD_HIP_CHECK(hipGetLastError());
  return DD_OK;
}

// loss + backward; grads land in n->grads.  *loss receives the batch MSE.
static dd_status backward(dd_cnn* n, const void* target, int B, float* loss, hipStream_t st) {
  const int D = n->nx * n->ny;
  const int k = n->k;
  const CnnLayer& LL = n->L[NL - 1];
  const float scale = 2.0f / ((float)B * D * 2 * k);
  const int nlb = (int)(((long)B * D * (LL.coutp / 8) + 255) / 256);
  k_mse<<<nlb, 256, 0, st>>>(n->out, (const float2*)target, B, D, k, LL.coutp, scale,
                             n->dz[NL - 1], n->lpart);
  dd_status rc = backward_from_dz(n, B, st);
  if (rc != DD_OK) return rc;
  DD_HIP_CHECK(hipGetLastError());
  if (loss) {
    std::vector<float> lp(nlb);
    DD_HIP_CHECK(hipMemcpyAsync(lp.data(), n->lpart, sizeof(float) * nlb, hipMemcpyDeviceToHost, st));
    DD_HIP_CHECK(hipStreamSynchronize(st));
    double s = 0.0;
    for (float v : lp) s += v;
    *loss = (float)(s / ((double)B * D * 2 * k));
  }
  return DD_OK;
}

static dd_status check_batch(const dd_cnn* n, const void* eps, const void* eim, int B,
                             const char* who) {
  if (!n || !eps || B < 1 || B > n->maxB) {
    dd_set_error("%s: need a network, eps and 1 <= B <= max_batch (%d)", who, n ? n->maxB : 0);
    return DD_EINVAL;
  }
  if ((n->cin0 == 3) != (eim != nullptr)) {
    dd_set_error("%s: this network takes %s", who,
                 n->cin0 == 3 ? "the effective-index field (eim must not be NULL)"
                              : "the permittivity only (eim must be NULL)");
    return DD_EINVAL;
  }
  return DD_OK;
}

static dd_status predict(dd_cnn* n, const float* eps, const void* eim, int B, void* U,
                         hipStream_t st, const char* who) {
  dd_status rc = check_batch(n, eps, eim, B, who);
  if (rc != DD_OK) return rc;
  if (!U) { dd_set_error("%s: U is NULL", who); return DD_EINVAL; }
  rc = forward(n, eps, eim, B, st, U);
  if (rc != DD_OK) return rc;
  DD_HIP_CHECK(hipGetLastError());
  DD_HIP_CHECK(hipStreamSynchronize(st));
  return DD_OK;
}

extern "C" dd_status dd_cnn_predict(dd_cnn* n, const float* eps, int B, void* U,
                                    hipStream_t st) {
  return predict(n, eps, nullptr, B, U, st, "dd_cnn_predict");
}

extern "C" dd_status dd_cnn_predict_eim(dd_cnn* n, const float* eps, const void* eim, int B,
                                        void* U, hipStream_t st) {
  if (!eim) { dd_set_error("dd_cnn_predict_eim: eim is NULL"); return DD_EINVAL; }
  return predict(n, eps, eim, B, U, st, "dd_cnn_predict_eim");
}

extern "C" dd_status dd_cnn_dims(const dd_cnn* n, int* nx, int* ny, int* k, int* in_channels,
                                 int* max_batch) {
  if (!n) { dd_set_error("dd_cnn_dims: NULL network"); return DD_EINVAL; }
  if (nx) *nx = n->nx;
  if (ny) *ny = n->ny;
  if (k) *k = n->k;
  if (in_channels) *in_channels = n->cin0;
  if (max_batch) *max_batch = n->maxB;
  return DD_OK;
}

extern "C" dd_status dd_cnn_save(const dd_cnn* n, const char* path) {
  if (!n || !path) { dd_set_error("dd_cnn_save: NULL argument"); return DD_EINVAL; }
  const size_t np = n->nparams;
  std::vector<float> buf(3 * np);
  DD_HIP_CHECK(hipDeviceSynchronize());
  DD_HIP_CHECK(hipMemcpy(buf.data(), n->params, sizeof(float) * np, hipMemcpyDeviceToHost));
  DD_HIP_CHECK(hipMemcpy(buf.data() + np, n->am, sizeof(float) * np, hipMemcpyDeviceToHost));
  DD_HIP_CHECK(hipMemcpy(buf.data() + 2 * np, n->av, sizeof(float) * np, hipMemcpyDeviceToHost));
  PredFileHeader h{};
  std::memcpy(h.magic, DD_PRED_MAGIC, 8);
  h.kind = DD_PRED_CNN;
  h.nx = n->nx; h.ny = n->ny; h.k = n->k; h.in_channels = n->cin0;
  h.count = (int64_t)np;
  h.adam_t = n->adam_t;
  FILE* f = std::fopen(path, "wb");
  if (!f) { dd_set_error("dd_cnn_save: cannot open '%s' for writing", path); return DD_EINVAL; }
  const bool ok = std::fwrite(&h, sizeof(h), 1, f) == 1 &&
                  std::fwrite(buf.data(), sizeof(float), buf.size(), f) == buf.size();
  if (std::fclose(f) != 0 || !ok) {
    dd_set_error("dd_cnn_save: writing '%s' failed", path);
    return DD_EINVAL;
  }
  return DD_OK;
}

extern "C" dd_status dd_cnn_load(const char* path, int max_batch, dd_cnn** out) {
  if (!out) { dd_set_error("dd_cnn_load: out is NULL"); return DD_EINVAL; }
  *out = nullptr;
  PredFileHeader h{};
  char msg[512];
  FILE* f = pred_open(path, h, msg, sizeof(msg));
  if (!f) { dd_set_error("dd_cnn_load: %s", msg); return DD_EINVAL; }
  if (h.kind != DD_PRED_CNN) {
    std::fclose(f);
    dd_set_error("dd_cnn_load: '%s' holds a PCA basis, not a network", path);
    return DD_EINVAL;
  }
  std::vector<float> buf(3 * (size_t)h.count);
  const bool ok = std::fread(buf.data(), sizeof(float), buf.size(), f) == buf.size();
  std::fclose(f);
  if (!ok) { dd_set_error("dd_cnn_load: reading '%s' failed", path); return DD_EINVAL; }
  dd_cnn* n = nullptr;
  dd_status rc = dd_cnn_create(h.nx, h.ny, max_batch, h.k, h.in_channels, 0, &n);
  if (rc != DD_OK) return rc;
  if ((int64_t)n->nparams != h.count) {
    dd_cnn_destroy(n);
    dd_set_error("dd_cnn_load: '%s' holds %lld parameters, the network has %zu", path,
                 (long long)h.count, n->nparams);
    return DD_EINVAL;
  }
  const size_t np = n->nparams;
  hipError_t e = hipMemcpy(n->params, buf.data(), sizeof(float) * np, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(n->am, buf.data() + np, sizeof(float) * np, hipMemcpyHostToDevice);
  if (e == hipSuccess)
    e = hipMemcpy(n->av, buf.data() + 2 * np, sizeof(float) * np, hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    dd_cnn_destroy(n);
    dd_set_error("dd_cnn_load: %s", hipGetErrorString(e));
    return DD_EHIP;
  }
  n->adam_t = (int)h.adam_t;
  rc = pack_all(n, 0);
  if (rc == DD_OK && hipDeviceSynchronize() != hipSuccess) rc = DD_EHIP;
  if (rc != DD_OK) { dd_cnn_destroy(n); return rc; }
  *out = n;
  return DD_OK;
}

extern "C" dd_status dd_cnn_grad(dd_cnn* n, const float* eps, const void* eim, const void* target,
                                 int B, float* loss, float* host_grad, size_t count,
                                 hipStream_t st) {
  dd_status rc = check_batch(n, eps, eim, B, "dd_cnn_grad");
  if (rc != DD_OK) return rc;
  if (!target || (host_grad && count != n->nparams)) {
    dd_set_error("dd_cnn_grad: bad target or gradient size");
    return DD_EINVAL;
  }
  rc = forward(n, eps, eim, B, st);
  if (rc != DD_OK) return rc;
  rc = backward(n, target, B, loss, st);
  if (rc != DD_OK) return rc;
  if (host_grad) {
    DD_HIP_CHECK(hipMemcpyAsync(host_grad, n->grads, sizeof(float) * count, hipMemcpyDeviceToHost, st));
  }
  DD_HIP_CHECK(hipStreamSynchronize(st));
  return DD_OK;
}

extern "C" dd_status dd_cnn_train_step(dd_cnn* n, const float* eps, const void* eim,
                                       const void* target, int B, float lr, float b1, float b2,
                                       float* loss, hipStream_t st) {
  dd_status rc = check_batch(n, eps, eim, B, "dd_cnn_train_step");
  if (rc != DD_OK) return rc;
  if (!target || !(lr > 0.f) || !(b1 >= 0.f && b1 < 1.f) || !(b2 >= 0.f && b2 < 1.f)) {
    dd_set_error("dd_cnn_train_step: bad target or Adam parameters");
    return DD_EINVAL;
  }
  rc = forward(n, eps, eim, B, st);
  if (rc != DD_OK) return rc;
  rc = backward(n, target, B, loss, st);
  if (rc != DD_OK) return rc;
  n->adam_t += 1;
  const float c1 = 1.f - std::pow(b1, (float)n->adam_t);
  const float c2 = 1.f - std::pow(b2, (float)n->adam_t);
  k_adam<<<(unsigned)((n->nparams + 255) / 256), 256, 0, st>>>(n->params, n->grads, n->am, n->av,
                                                                n->nparams, lr, b1, b2, c1, c2, 1e-8f);
  rc = pack_all(n, st);
  if (rc != DD_OK) return rc;
  DD_HIP_CHECK(hipStreamSynchronize(st));
  return DD_OK;
}

// Residual-loss step (Sec. 3, eq:res_loss): forward, the loss of every image's
// predicted fields against its own operator and right-hand side, the
// gradient through A^H into the last layer, backward.  *loss = batch mean.
static dd_status res_step(dd_cnn* n, const float* eps, const void* eim,
                          const fdfd_op* const* ops, const void* const* b, int B, float* loss,
                          hipStream_t st, const char* who) {
  dd_status rc = check_batch(n, eps, eim, B, who);
  if (rc != DD_OK) return rc;
  if (!ops || !b) { dd_set_error("%s: need ops and b", who); return DD_EINVAL; }
  for (int p = 0; p < B; ++p)
    if (!ops[p] || !b[p] || ops[p]->nx != n->nx || ops[p]->ny != n->ny) {
      dd_set_error("%s: problem %d needs an operator of %d x %d and b", who, p, n->nx, n->ny);
      return DD_EINVAL;
    }
  const size_t D = (size_t)n->nx * n->ny;
  if (!n->rl_W) {
    hipError_t e = hipSuccess;
    auto chk = [&](hipError_t x) { if (x != hipSuccess && e == hipSuccess) e = x; };
    chk(cnn_alloc(n, &n->rl_W, (size_t)n->maxB * n->k * D));
    chk(cnn_alloc(n, &n->rl_r, (size_t)n->maxB * D));
    chk(cnn_alloc(n, &n->rl_s, (size_t)n->maxB * D));
    n->rl_scratch_bytes = res_loss_scratch_bytes(n->maxB, n->k);
    chk(cnn_alloc(n, (float2**)&n->rl_scratch, (n->rl_scratch_bytes + 7) / 8));
    if (e != hipSuccess) {
      dd_set_error("%s: %s", who, hipGetErrorString(e));
      return e == hipErrorOutOfMemory ? DD_ENOMEM : DD_EHIP;
    }
  }
  rc = forward(n, eps, eim, B, st);   // fields V in n->out
  if (rc != DD_OK) return rc;
  DD_HIP_CHECK(hipGetLastError());
  std::vector<const void*> Vp(B);
  for (int p = 0; p < B; ++p) Vp[p] = (const float2*)n->out + (size_t)p * n->k * D;
  std::vector<double> lv(B);
  rc = res_loss_core(ops, b, Vp.data(), B, n->k, n->rl_W, n->rl_r, n->rl_s, lv.data(),
                     n->dz[NL - 1], n->L[NL - 1].coutp, 1.0 / B, st, nullptr, n->rl_scratch,
                     n->rl_scratch_bytes);
  if (rc != DD_OK) return rc;
  rc = backward_from_dz(n, B, st);
  if (rc != DD_OK) return rc;
  if (loss) {
    double s = 0.0;
    for (double v : lv) s += v;
    *loss = (float)(s / B);
  }
  return DD_OK;
}

extern "C" dd_status dd_cnn_grad_res(dd_cnn* n, const float* eps, const void* eim,
                                     const fdfd_op* const* ops, const void* const* b, int B,
                                     float* loss, float* host_grad, size_t count,
                                     hipStream_t st) {
  if (n && host_grad && count != n->nparams) {
    dd_set_error("dd_cnn_grad_res: gradient size must be %zu", n->nparams);
    return DD_EINVAL;
  }
  dd_status rc = res_step(n, eps, eim, ops, b, B, loss, st, "dd_cnn_grad_res");
  if (rc != DD_OK) return rc;
  if (host_grad) {
    DD_HIP_CHECK(hipMemcpyAsync(host_grad, n->grads, sizeof(float) * count, hipMemcpyDeviceToHost, st));
  }
  DD_HIP_CHECK(hipStreamSynchronize(st));
  return DD_OK;
}

extern "C" dd_status dd_cnn_train_step_res(dd_cnn* n, const float* eps, const void* eim,
                                           const fdfd_op* const* ops, const void* const* b, int B,
                                           float lr, float b1, float b2, float* loss,
                                           hipStream_t st) {
  if (!(lr > 0.f) || !(b1 >= 0.f && b1 < 1.f) || !(b2 >= 0.f && b2 < 1.f)) {
    dd_set_error("dd_cnn_train_step_res: bad Adam parameters");
    return DD_EINVAL;
  }
  dd_status rc = res_step(n, eps, eim, ops, b, B, loss, st, "dd_cnn_train_step_res");
  if (rc != DD_OK) return rc;
  n->adam_t += 1;
  const float c1 = 1.f - std::pow(b1, (float)n->adam_t);
  const float c2 = 1.f - std::pow(b2, (float)n->adam_t);
  k_adam<<<(unsigned)((n->nparams + 255) / 256), 256, 0, st>>>(n->params, n->grads, n->am, n->av,
                                                                n->nparams, lr, b1, b2, c1, c2, 1e-8f);
  rc = pack_all(n, st);
  if (rc != DD_OK) return rc;
  DD_HIP_CHECK(hipStreamSynchronize(st));
  return DD_OK;
}

extern "C" dd_status dd_cnn_debug_activation(const dd_cnn* n, int layer, int B, float* host,
                                             size_t count) {
  if (!n || !host || layer < -1 || layer >= NL || B < 1 || B > n->maxB) {
    dd_set_error("dd_cnn_debug_activation: bad argument");
    return DD_EINVAL;
  }
  DD_HIP_CHECK(hipDeviceSynchronize());
  const size_t D = (size_t)n->nx * n->ny;
  if (layer == -1) {
    const size_t cnt = B * D * n->cin0;
    if (count != cnt) { dd_set_error("dd_cnn_debug_activation: count must be %zu", cnt); return DD_EINVAL; }
    DD_HIP_CHECK(hipMemcpy(host, n->x0, sizeof(float) * count, hipMemcpyDeviceToHost));
    return DD_OK;
  }
  const CnnLayer& L = n->L[layer];
  const size_t pix = (size_t)B * L.Hout * L.Wout;
  if (layer == NL - 1) {   // n->out holds complex fields [B][k][D]: back to [pixel][2k]
    if (count != pix * L.cout) { dd_set_error("dd_cnn_debug_activation: count must be %zu", pix * L.cout); return DD_EINVAL; }
    std::vector<float> f(count);
    if (!n->last_fields) { dd_set_error("dd_cnn_debug_activation: no forward pass yet"); return DD_EINVAL; }
    DD_HIP_CHECK(hipMemcpy(f.data(), n->last_fields, sizeof(float) * count, hipMemcpyDeviceToHost));
    const int kf = n->k;
    for (size_t p = 0; p < pix; ++p) {
      const size_t b = p / D, e = p % D;
      for (int j = 0; j < kf; ++j)
        for (int c = 0; c < 2; ++c) host[p * 2 * kf + 2 * j + c] = f[((b * kf + j) * D + e) * 2 + c];
    }
    return DD_OK;
  }
  if (count != pix * L.cout) { dd_set_error("dd_cnn_debug_activation: count must be %zu", pix * L.cout); return DD_EINVAL; }
  std::vector<bf16> tmp(pix * L.coutp);
  DD_HIP_CHECK(hipMemcpy(tmp.data(), n->act[layer], sizeof(bf16) * tmp.size(), hipMemcpyDeviceToHost));
  for (size_t p = 0; p < pix; ++p)
    for (int c = 0; c < L.cout; ++c) host[p * L.cout + c] = (float)tmp[p * L.coutp + c];
  return DD_OK;
}
