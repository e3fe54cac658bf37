// Learned angular reconstruction: a small 3x3 convolutional network whose
// inference and training run on BF16 MFMA (v_mfma_f32_16x16x32_bf16, FP32
// accumulate).  It stands in for 4x angular supersampling (Sec. 4) and is
// applied to every view v of a frame.  Angular supersampling plus the angular
// filter averages sub-views within about one view interval; a surface at
// disparity d = D/Z - 1 moves k*d pixels across per view step, so away from
// occlusions that average is a horizontal blur of width proportional to |d|.
// The input at a pixel is (R, G, B, d) of views v-2 .. v+2 (zero beyond the
// rig) and the disparity blur of view v (9 Gaussian taps over +-1 view step,
// the angular filter's profile): 24 channels; layers 24 -> 32 -> 32 -> 32 -> 3
// with ReLU, 3x3 kernels dilated horizontally by 1, 3, 9, 1; output = blurred
// RGB + network.
//
// Layouts: the compact input is [view][H][W][4] BF16 and layer 1 gathers the
// neighbour views from it directly, and the blur from its own [view][H][W][4]
// buffer; hidden activations are [view][H][W][32]
// BF16; the output [view][H][W][4] (RGB, 0).  Parameters: FP32 master vector,
// per layer W [tap][cout][cin] then b [cout] (unpadded); BF16 copies padded
// to 32 input channels (layer 1) and 16 output channels (layer 4).
//
// MFMA 16x16x32 lane layout used throughout: lane l feeds row (l % 16) of A
// and column (l % 16) of B with 8 K-values each (group l / 16); the 4 results
// of lane l are D[4*(l/16) + e][l % 16].  A and B take their K-values in the
// same order, so the K ordering inside a group does not matter.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/lfdpr.h"
#include "lfdpr_internal.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace lfdpr {
namespace net {

constexpr int kHidden = 32;
enum Mode { MODE_RELU = 0, MODE_OUT = 1, MODE_BWD = 2 };

__device__ __forceinline__ uint16_t to_bf16(float v) {
  uint32_t u = __float_as_uint(v);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// Two values rounded to BF16 (nearest, ties to even) by one v_cvt_pk_bf16_f32,
// lo in bits 0-15.  For every non-NaN binary32 input it gives the same bits as
// to_bf16 (checked exhaustively on gfx950).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

union Frag {
  uint4 u;
  bf16x8 v;
};

// ---------------------------------------------------------------- 3x3 convolution
constexpr int kNeigh = 2;   // views v-2 .. v+2
constexpr int kViewCh = 4 * (2 * kNeigh + 1);  // 20 channels of the five views
constexpr int kCin0 = kViewCh + 4;             // + blurred (R, G, B, 0) of view v
constexpr int kK = 32;      // padded input channels of every layer (one MFMA K step per tap)
// Horizontal dilation per layer: one view step shifts content by several
// pixels across, so the stack sees +-14 px horizontally and +-4 px vertically.
constexpr int kDilation[4] = {1, 3, 9, 1};

// Loads the 8 K-values of lane group g for input pixel (n, yy, xx), zero
// outside the image.  GATHER: from the compact [n][H][W][4] input, channels
// 8g..8g+7 = views n+2g-2, n+2g-1; the slot after view n+2 (channels 20..23)
// takes the blur XB of view n.  Pixel indices fit in 32 bits: a network holds
// at most 2^26 pixels.
template <bool GATHER>
__device__ __forceinline__ uint4 load_a(const uint16_t* __restrict__ X, const uint16_t* __restrict__ XB, int n, int yy,
                                        int xx, int H, int W, int g, int V) {
  if (yy < 0 || yy >= H || xx < 0 || xx >= W) return uint4{0u, 0u, 0u, 0u};
  if (!GATHER) return *reinterpret_cast<const uint4*>(X + (size_t)((n * H + yy) * W + xx) * kK + 8 * g);
  const int v = n % V, f0 = n - v;
  uint2 lo = {0u, 0u}, hi = {0u, 0u};
  const int o0 = 2 * g - kNeigh, o1 = 2 * g + 1 - kNeigh;
  if (o0 <= kNeigh && v + o0 >= 0 && v + o0 < V)
    lo = *reinterpret_cast<const uint2*>(X + (size_t)(((f0 + v + o0) * H + yy) * W + xx) * 4);
  if (o1 <= kNeigh) {
    if (v + o1 >= 0 && v + o1 < V)
      hi = *reinterpret_cast<const uint2*>(X + (size_t)(((f0 + v + o1) * H + yy) * W + xx) * 4);
  } else if (o1 == kNeigh + 1) {
    hi = *reinterpret_cast<const uint2*>(XB + (size_t)((n * H + yy) * W + xx) * 4);
  }
  return uint4{lo.x, lo.y, hi.x, hi.y};
}

// One block = kTY waves, persistent over output tiles of kTY rows x kTX pixels of
// one image (wave w computes row w: four 16-pixel M tiles); NT = COUT/16
// output-channel tiles.  All nine taps' [COUT][32] weights stay in LDS; each
// tile's input, rows y0-1 .. y0+kTY and columns x0-DIL .. x0+kTX-1+DIL with
// zero padding, is staged in LDS once and read by all nine taps.  LDS rows of
// 32 channels are four 16-byte groups stored at slot g ^ ((px >> 1) & 3): LDS
// serves 16-byte reads eight lanes (128 bytes) at a time, and any 8
// consecutive pixels then fall into 8 distinct bank groups (no conflicts on
// gfx950 by the SQ_LDS_BANK_CONFLICT counter).  aux: GATHER, the blur buffer;
// MODE_OUT, the residual (stride AUX_C); MODE_BWD, the activation whose ReLU
// masks the gradient.
//
// Memory bounds the hidden layers (48 x 512 x 512 pixels: 1.6 GB read and written,
// 326 us at the rate of a copy), so what counts is whole lines and waves in
// flight: 16-byte stores that cover 16 whole pixels, and tiles of eight rows,
// two workgroups of eight waves per compute unit, which the dilation as a
// constant makes room for (at most 128 registers).  Measured there with four
// rows, three workgroups of four waves and 8-byte stores of half a pixel: layers
// 1 to 4 370, 360, 362 and 245 us; eight rows 360, 344, 342 and 221; and with the
// wide stores 305, 326, 323 and 220.
constexpr int kTX = 64, kTY = 8, kConvThreads = 64 * kTY;
constexpr int kConvGrid = 512;  // two workgroups (16 waves) per compute unit
constexpr int kPlanes = 2 * kNeigh + 2;  // layer 1's sources: five views and the blur

__device__ __forceinline__ int swz(int row, int g) { return row * 4 + (g ^ ((row >> 1) & 3)); }

template <int NT, int DIL>
constexpr size_t conv_lds_bytes() {
  return (size_t)9 * NT * 16 * 4 * 16 + (size_t)(kTY + 2) * (kTX + 2 * DIL) * 4 * 16;
}

template <int NT, int MODE, bool GATHER, int DIL>
__global__ void __launch_bounds__(kConvThreads, 4) k_conv3x3(const uint16_t* __restrict__ X, const uint16_t* __restrict__ Wt,
                                                  const float* __restrict__ bias, int N, int H, int W, int V,
                                                  uint16_t* __restrict__ Y, int YS, const uint16_t* __restrict__ aux,
                                                  int AUX_C) {
  constexpr int COUT = NT * 16;
  extern __shared__ uint4 smem[];
  uint4* wlds = smem;                  // [9 * COUT rows][4 groups]
  uint4* tl = smem + 9 * COUT * 4;     // [(kTY + 2) rows][TW pixels][4 groups]
  constexpr int TW = kTX + 2 * DIL;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int g = lane >> 4, r16 = lane & 15, c0 = 4 * NT * g;
  struct alignas(8 * NT) Chans {  // 4 NT channels of a pixel
    uint32_t w[2 * NT];
  };
  for (int k = threadIdx.x; k < 9 * COUT * 4; k += blockDim.x) {
    const int c = (k >> 2) % COUT;  // kept in row t * 16 + 4 g + e for channel 4 NT g + 4 t + e
    const int row = (k >> 2) - c + (c / 4 % NT) * 16 + c / (4 * NT) * 4 + c % 4;
    wlds[swz(row, k & 3)] = reinterpret_cast<const uint4*>(Wt)[k];
  }
  // Loads whose results the epilogue uses are unconditional (clamped indices):
  // a load issued under a branch leaves the compiler unsure that a later wait
  // covered it, and it would then wait for all memory traffic in the epilogue.
  // The MFMA computes D = W x A (rows: output channels, columns: pixels), so
  // lane (g, r16) ends with rows t*16 + 4g .. +3 of pixel r16 of each M tile: the
  // weights' rows are ordered so that these are the 4 NT channels from 4 NT g on,
  // and a wave stores 16 whole pixels at once.
  float bco[NT][4];  // their biases (3 in the output layer)
  const int nbias = MODE == MODE_BWD ? 0 : (MODE == MODE_OUT ? 3 : YS);
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = 4 * NT * g + 4 * t + e;
      if (MODE == MODE_BWD) {
        bco[t][e] = 0.0f;
      } else {
        const float bv = bias[c < nbias ? c : 0];
        bco[t][e] = c < nbias ? bv : 0.0f;
      }
    }
  const int tiles_x = (W + kTX - 1) / kTX, tiles_y = (H + kTY - 1) / kTY;
  const int ntile = N * tiles_x * tiles_y;
  constexpr int nstage = (kTY + 2) * TW * 4;
  // Tile order.  Image-major ([n][row band][column]), except for the gathering
  // first layer: position-major with the view fastest, so the five output views
  // that read one input view's tile follow each other.  Workgroups are handed to
  // the 8 XCDs round robin and each XCD has its own L2, so the blocks of XCD c
  // (blockIdx % 8 == c) take the c-th eighth of that order, in order: tiles that
  // share halo rows and columns (or input views) then run at about the same time
  // on the XCD that caches them.  Any other grid takes tiles blockIdx + k*grid.
  const bool by_xcd = gridDim.x % 8 == 0 && ntile >= (int)gridDim.x;
  const int xc = blockIdx.x % 8;
  const int t_end = by_xcd ? (int)((int64_t)ntile * (xc + 1) / 8) : ntile;
  const int t_first = by_xcd ? (int)((int64_t)ntile * xc / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
  const int t_step = by_xcd ? (int)(gridDim.x / 8) : (int)gridDim.x;
  auto decode = [&](int tile, int& n, int& y0, int& x0) {
    int pos;
    if (GATHER) {
      n = tile % N;
      pos = tile / N;
    } else {
      n = tile / (tiles_x * tiles_y);
      pos = tile % (tiles_x * tiles_y);
    }
    y0 = (pos / tiles_x) * kTY;
    x0 = (pos % tiles_x) * kTX;
  };
  // Staging items of this thread, the same for every tile.  Layers 2-4: item j
  // is 16-byte group threadIdx % 4 of LDS pixel q = threadIdx / 4 + kConvThreads / 4 j, at
  // tile row q / TW and column q % TW (rows from kTY + 2 on lie past the staged
  // tile).  Layer 1 (GATHER) stages plane by plane -- views v-2 .. v+2 of the
  // compact input, then the blur, 8 bytes per pixel -- in pairs of pixels from
  // an even column xs = x0 - DIL - (DIL & 1), so each wave load reads 128
  // consecutive pixels of one plane (16 bytes a lane where the pair is inside
  // the image and 16-byte aligned, else two 8-byte loads): item j' = threadIdx
  // + kConvThreads j is plane j' / ((kTY + 2) NP), then row and pair (NP pairs a row);
  // plane p fills half p % 2 of group p / 2, pixels outside the tile's columns
  // are dropped, and group 3 (channels 24-31) stays zero.
  constexpr int NP = kTX / 2 + DIL + (DIL & 1);  // pixel pairs per staged row (layer 1)
  constexpr int kSlots = ((GATHER ? (kTY + 2) * NP * kPlanes : nstage) + kConvThreads - 1) / kConvThreads;  // items of a thread
  int geo[kSlots];
#pragma unroll
  for (int j = 0; j < kSlots; ++j) {
    if (GATHER) {
      const int i = (int)threadIdx.x + kConvThreads * j, m = (kTY + 2) * NP;
      const int pl = i / m, rem = i % m;
      geo[j] = (pl << 24) | ((rem / NP) << 16) | (rem % NP);
    } else {
      const int q = (int)(threadIdx.x >> 2) + kConvThreads / 4 * j;
      geo[j] = ((q / TW) << 16) | (q % TW);
    }
  }
  const int sg = threadIdx.x & 3;
  if (GATHER) {  // the zero group: the whole tile once, before any staging
    for (int k = threadIdx.x; k < nstage; k += blockDim.x) tl[k] = uint4{0u, 0u, 0u, 0u};
    __syncthreads();
  }
  // the next tile's input is fetched into registers while this one computes
  uint4 pre[kSlots];
  auto fetch = [&](int tile) {
    int n, y0, x0;
    decode(tile, n, y0, x0);
    if constexpr (GATHER) {
      const int vv = n % V, f0 = n - vv;
      const int xs = x0 - DIL - (DIL & 1);
#pragma unroll
      for (int j = 0; j < kSlots; ++j) {
        const int pl = geo[j] >> 24, r = (geo[j] >> 16) & 0xFF, q = geo[j] & 0xFFFF;
        const int yy = y0 - 1 + r, xx = xs + 2 * q;
        uint4 val = {0u, 0u, 0u, 0u};
        const int vo = vv + pl - kNeigh;
        const bool plane_ok = pl < kPlanes - 1 ? (vo >= 0 && vo < V) : pl == kPlanes - 1;
        if (plane_ok && yy >= 0 && yy < H) {
          const uint16_t* src = pl < kPlanes - 1 ? X : aux;
          const int img = pl < kPlanes - 1 ? f0 + vo : n;
          const bool ok0 = xx >= 0 && xx < W, ok1 = xx + 1 >= 0 && xx + 1 < W;
          const int p0 = (img * H + yy) * W + xx;  // dereferenced only where in the image
          const uint16_t* a0 = src + (size_t)p0 * 4;
          if (ok0 && ok1 && ((uintptr_t)a0 & 15) == 0) {
            val = *reinterpret_cast<const uint4*>(a0);
          } else {
            if (ok0) {
              const uint2 a = *reinterpret_cast<const uint2*>(src + (size_t)p0 * 4);
              val.x = a.x;
              val.y = a.y;
            }
            if (ok1) {
              const uint2 b = *reinterpret_cast<const uint2*>(src + (size_t)(p0 + 1) * 4);
              val.z = b.x;
              val.w = b.y;
            }
          }
        }
        pre[j] = val;
      }
    } else {
#pragma unroll
      for (int j = 0; j < kSlots; ++j) {
        const int r = geo[j] >> 16, c = geo[j] & 0xFFFF;
        pre[j] = r < kTY + 2 ? load_a<false>(X, nullptr, n, y0 - 1 + r, x0 - DIL + c, H, W, sg, V) : uint4{0u, 0u, 0u, 0u};
      }
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
      if constexpr (GATHER) {
        const int pl = geo[j] >> 24, r = (geo[j] >> 16) & 0xFF, q = geo[j] & 0xFFFF;
        const int c0 = 2 * q - (DIL & 1);  // tile column of the pair's first pixel
        if (pl < kPlanes) {
          if (c0 >= 0) reinterpret_cast<uint2*>(&tl[swz(r * TW + c0, pl >> 1)])[pl & 1] = uint2{pre[j].x, pre[j].y};
          if (c0 + 1 < TW)
            reinterpret_cast<uint2*>(&tl[swz(r * TW + c0 + 1, pl >> 1)])[pl & 1] = uint2{pre[j].z, pre[j].w};
        }
      } else {
        const int k = threadIdx.x + j * kConvThreads;
        if (k < nstage) tl[swz(k >> 2, k & 3)] = pre[j];
      }
    }
  };
  // Software pipeline per tile: MFMAs on the staged tile; then the next tile
  // (already in registers) goes to LDS, the one after it is requested, and only
  // then do this tile's results leave.  Vector-memory waits count stores as well
  // as loads, so each wait (before staging) covers requests that have had a
  // whole tile of MFMAs to complete, never the stores just issued.
  if (t_first < t_end) {
    fetch(t_first);
    stage();
    __syncthreads();  // weights and the first tile in LDS
    if (t_first + t_step < t_end) fetch(t_first + t_step);
  }
  for (int tile = t_first; tile < t_end; tile += t_step) {
    int n, y0, x0;
    decode(tile, n, y0, x0);
    const int y = y0 + wv;
    // the epilogue's side input (residual or ReLU mask), clamped into the image
    // and used only where in range: the residual is requested before the MFMAs;
    // the mask (two 32-channel tiles) after them, which keeps the backward
    // instantiation within 128 registers (four waves per SIMD)
    Chans side[4];
    auto load_side = [&]() {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int x = min(x0 + m * 16 + r16, W - 1), yc = min(y, H - 1);
        side[m] = *reinterpret_cast<const Chans*>(aux + (((size_t)n * H + yc) * W + x) * AUX_C + (c0 < YS ? c0 : 0));
      }
    };
#pragma unroll
    for (int m = 0; m < 4; ++m) side[m] = Chans{};
    if (MODE == MODE_OUT) load_side();
    f32x4 acc[4][NT];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // all nine taps unrolled: in a rolled loop the compiler moves the
    // accumulators between AGPRs on every iteration (about 40 moves per 8 MFMAs)
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int dy = tap / 3 - 1, dx = tap % 3 - 1;
      Frag b[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) b[t].u = wlds[swz(tap * COUT + t * 16 + r16, g)];
      const int rowbase = (wv + 1 + dy) * TW + DIL + dx * DIL + r16;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        Frag a;
        a.u = tl[swz(rowbase + m * 16, g)];
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[t].v, a.v, acc[m][t], 0, 0, 0);
      }
    }
    if (MODE == MODE_BWD) load_side();
    const int next = tile + t_step;
    __syncthreads();  // every wave has finished reading this tile
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0) on every path: all requests so far have landed
    if (next < t_end) stage();
    __syncthreads();
    if (next + t_step < t_end) fetch(next + t_step);
    // epilogue: 4 NT consecutive channels of pixel x0 + 16m + r16 (row y0 + wv) leave as one store
    if (y < H) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int x = x0 + m * 16 + r16;
        if (x >= W || c0 >= YS) continue;
        Chans o;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const uint32_t side0 = side[m].w[2 * t], side1 = side[m].w[2 * t + 1];
          const float sv[4] = {from_bf16((uint16_t)(side0 & 0xFFFFu)), from_bf16((uint16_t)(side0 >> 16)),
                               from_bf16((uint16_t)(side1 & 0xFFFFu)), from_bf16((uint16_t)(side1 >> 16))};
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float u = acc[m][t][e];
            if (MODE == MODE_RELU) {
              u = fmaxf(u + bco[t][e], 0.0f);
            } else if (MODE == MODE_OUT) {
              u = c0 + 4 * t + e < 3 ? (u + bco[t][e]) + sv[e] : 0.0f;
            } else {
              u = sv[e] > 0.0f ? u : 0.0f;
            }
            v[e] = u;
          }
          o.w[2 * t] = pack_bf16x2(v[0], v[1]);
          o.w[2 * t + 1] = pack_bf16x2(v[2], v[3]);
        }
        *reinterpret_cast<Chans*>(Y + (((size_t)n * H + y) * W + x) * YS + c0) = o;
      }
    }
  }
}

// ---------------------------------------------------------------- weight gradient
// dW[tap][co][ci] = sum_p dZ[p][co] * A[p + off(tap)][ci], db[co] = sum_p dZ[p][co].
//
// The contraction runs over pixels, so both operands need eight pixels of one
// channel in a lane while memory holds 32 channels of one pixel: the tile is
// staged as it lies (dZ of kGY x kGX pixels, A with the taps' halo, loaded once
// for all nine taps) and read through the transposing LDS loads, four pixels x
// 16 channels per 16 lanes.  Wave w of three takes the taps of row w - 1: per 16
// pixels one dZ operand and, for each tap, the shifted A operand and one
// v_mfma_f32_32x32x16_bf16 over all 32 x 32 channels; no sums cross waves.  The
// next tile is fetched into registers meanwhile.  48 x 128 x 128 pixels: 60-72 us a
// layer, and 9 for its biases, when each tap's shifted pixels were staged channel
// by channel through two-byte LDS writes; 30-39 now.  (Four waves with a row of the
// tile each and all nine taps: 60, most of it adding up the waves' sums.)
//
// Workgroups take tiles grid, 2 grid, .. apart and write their sums to their own
// row of a partials buffer laid out as the parameter vector, which
// k_sum_partials adds in row order: gradients come out the same on every run.
// The accumulators of kGRun tiles (128 products) join a second set of sums, so
// that a workgroup of hundreds of tiles rounds as one of a few does (64 views of
// 1024 x 1024, a smooth error: root mean square error 4.8e-8 of the largest
// gradient in one chain, 1.0e-8 so, in the same time).
constexpr int kGX = 64, kGY = 4, kGThreads = 192;
constexpr int kGRun = 8;
constexpr int kGradBlocks = 512;  // rows of the partials buffer: two workgroups per CU
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Eight pixels (p0 .. p0+3 and p0+4 .. p0+7 of this lane's half, in tile order)
// of channel lane % 32 from rows of 32 channels; `at` is this lane's address in
// the first read: pixel (lane >> 2) & 3 of its half, channels 16 ((lane >> 4) & 1)
// + 4 (lane & 3).
__device__ __forceinline__ bf16x8 read_pixels(const uint16_t* at) {
  typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
  union {
    i16x4 q[2];
    bf16x8 v;
  } f;
  f.q[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)at);
  f.q[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(at + 4 * kK));
  return f.v;
}

template <bool GATHER, int DIL>
__global__ void __launch_bounds__(kGThreads, 2) k_conv_wgrad(const uint16_t* __restrict__ dZ, int CO,
                                                     const uint16_t* __restrict__ A, const uint16_t* __restrict__ AB,
                                                     int CI, int N, int H, int W, int V, float* __restrict__ part,
                                                     int part_row) {
  constexpr int TW = kGX + 2 * DIL, kAPix = (kGY + 2) * TW, kZPix = kGY * kGX;
  constexpr int kAItems = (kAPix * 4 + kGThreads - 1) / kGThreads, kZItems = (kZPix * 4 + kGThreads - 1) / kGThreads;
  static_assert(kGThreads % 4 == 0, "a thread stages one 16-byte group of its pixels");
  __shared__ __attribute__((aligned(16))) uint16_t at[kAPix * kK], zt[kZPix * kK];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int tiles_x = (W + kGX - 1) / kGX, tiles_y = (H + kGY - 1) / kGY, ntile = N * tiles_x * tiles_y;
  const int sg = threadIdx.x & 3;
  uint4 pa[kAItems], pz[kZItems];
  auto fetch = [&](int tile) {
    const int n = tile / (tiles_x * tiles_y), pos = tile % (tiles_x * tiles_y);
    const int y0 = pos / tiles_x * kGY, x0 = pos % tiles_x * kGX;
#pragma unroll
    for (int j = 0; j < kZItems; ++j) {
      const int q = (int)(threadIdx.x >> 2) + kGThreads / 4 * j, y = y0 + q / kGX, x = x0 + q % kGX;
      pz[j] = q < kZPix && y < H && x < W ? *reinterpret_cast<const uint4*>(dZ + (size_t)((n * H + y) * W + x) * kK + 8 * sg)
                                          : uint4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int j = 0; j < kAItems; ++j) {
      const int q = (int)(threadIdx.x >> 2) + kGThreads / 4 * j;
      pa[j] = q < kAPix ? load_a<GATHER>(A, AB, n, y0 - 1 + q / TW, x0 - DIL + q % TW, H, W, sg, V) : uint4{0u, 0u, 0u, 0u};
    }
  };
  float bsum = 0.f;  // wave 0: dZ of channel lane % 32, this half's pixels
  const int px = 8 * (lane >> 5) + ((lane >> 2) & 3), ch = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  fetch(blockIdx.x);
  f32x16 sum[3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int e = 0; e < 16; ++e) sum[k][e] = 0.f;
  for (int tile = blockIdx.x; tile < ntile;) {
    f32x16 acc[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[k][e] = 0.f;
    for (int run = 0; run < kGRun && tile < ntile; ++run, tile += gridDim.x) {
      __syncthreads();  // the previous tile's reads are done
#pragma unroll
      for (int j = 0; j < kZItems; ++j)
        if ((int)threadIdx.x + kGThreads * j < kZPix * 4) reinterpret_cast<uint4*>(zt)[threadIdx.x + kGThreads * j] = pz[j];
#pragma unroll
      for (int j = 0; j < kAItems; ++j)
        if ((int)threadIdx.x + kGThreads * j < kAPix * 4) reinterpret_cast<uint4*>(at)[threadIdx.x + kGThreads * j] = pa[j];
      __syncthreads();
      if (tile + (int)gridDim.x < ntile) fetch(tile + gridDim.x);
      float btile = 0.f;  // the tile's terms first: a workgroup may take hundreds of tiles
#pragma unroll
      for (int row = 0; row < kGY; ++row)
#pragma unroll
        for (int k = 0; k < kGX / 16; ++k) {
          const bf16x8 fz = read_pixels(zt + (row * kGX + 16 * k + px) * kK + ch);
          if (wv == 0)
#pragma unroll
            for (int e = 0; e < 8; ++e) btile += (float)fz[e];
#pragma unroll
          for (int t = 0; t < 3; ++t) {
            const bf16x8 fa = read_pixels(at + ((row + wv) * TW + 16 * k + t * DIL + px) * kK + ch);
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fz, fa, acc[t], 0, 0, 0);
          }
        }
      bsum += btile;
    }
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) sum[t][e] += acc[t][e];
  }
  // lane holds D[8 (e / 4) + 4 (lane / 32) + e % 4][lane % 32]
  float* const out = part + (size_t)blockIdx.x * part_row;
  const int ci = lane & 31;
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int co = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
      if (co < CO && ci < CI) out[((3 * wv + t) * CO + co) * CI + ci] = sum[t][e];
    }
  bsum += __shfl_xor(bsum, 32, 64);
  if (wv == 0 && lane < CO && lane < 32) out[9 * CO * CI + lane] = bsum;
}

// out[i] = sum over the nblk rows of part[b][i] in a fixed order: in a block of
// 256, lane (phase f = t / 32, column j = t % 32) adds rows f, f + 8, .. in
// ascending order, then the 8 phase sums of each column are added in phase
// order.  The last workgroup adds the loss's nloss partial sums (lane t those of
// t, t + 256, .., then the lanes' by halves) and writes it to *loss0 and, if
// given, *loss1.  Grid: ceil(n / 32) + 1 blocks.
__global__ void __launch_bounds__(256) k_sum_partials(const float* __restrict__ part, int nblk, int n,
                                                       float* __restrict__ out, const float* __restrict__ loss_part,
                                                       int nloss, float* __restrict__ loss0, float* __restrict__ loss1) {
  __shared__ float red[8][32];
  const int j = threadIdx.x & 31, f = threadIdx.x >> 5;
  const bool last = blockIdx.x == gridDim.x - 1;
  const int i = blockIdx.x * 32 + j;
  float sum = 0.0f;
  if (last) {
    for (int b = threadIdx.x; b < nloss; b += 256) sum += loss_part[b];
  } else if (i < n) {
#pragma unroll 16
    for (int b = f; b < nblk; b += 8) sum += part[(size_t)b * n + i];
  }
  red[f][j] = sum;
  __syncthreads();
  if (last) {
    float* const r = red[0];
    for (int k = 128; k > 0; k >>= 1) {
      if ((int)threadIdx.x < k) r[threadIdx.x] += r[threadIdx.x + k];
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      *loss0 = r[0];
      if (loss1) *loss1 = r[0];
    }
  } else if (f == 0 && i < n) {
    float total = 0.0f;
    for (int k = 0; k < 8; ++k) total += red[k][j];
    out[i] = total;
  }
}

// loss = mean((y - t)^2) over the 3 colour channels of npx pixels (inputs
// [p][4]), as one partial sum per workgroup; dZ = bf16(2 (y - t) / n) into a
// [p][32] buffer (other channels 0).  Four lanes per pixel, one 16-byte store
// each, so that a wave writes 1 KiB in a row.  16 pixels' squares are summed
// before they join a lane's sum (up to 512 pixels a lane: 64 views of
// 1024 x 1024 -5.4e-6 of the loss in one chain).
constexpr int kMseBlocks = 2048;
__global__ void __launch_bounds__(256) k_mse(const uint16_t* __restrict__ Yb, const uint16_t* __restrict__ T, int npx,
                                              uint16_t* __restrict__ dZ, float* __restrict__ loss_part) {
  const int64_t n = (int64_t)npx * 3;
  float sq = 0.0f, run = 0.0f;
  int k = 0;
  const int g = threadIdx.x & 3;
  for (int64_t p = (int64_t)blockIdx.x * 64 + (threadIdx.x >> 2); p < npx; p += (int64_t)gridDim.x * 64) {
    uint4 o{0u, 0u, 0u, 0u};
    if (g == 0) {
      const uint2 yv = *reinterpret_cast<const uint2*>(Yb + p * 4);
      const uint2 tv = *reinterpret_cast<const uint2*>(T + p * 4);
      const float d0 = from_bf16((uint16_t)(yv.x & 0xFFFFu)) - from_bf16((uint16_t)(tv.x & 0xFFFFu));
      const float d1 = from_bf16((uint16_t)(yv.x >> 16)) - from_bf16((uint16_t)(tv.x >> 16));
      const float d2 = from_bf16((uint16_t)(yv.y & 0xFFFFu)) - from_bf16((uint16_t)(tv.y & 0xFFFFu));
      run += (d0 * d0 + d1 * d1) + d2 * d2;
      if ((++k & 15) == 0) {
        sq += run;
        run = 0.0f;
      }
      o.x = (uint32_t)to_bf16((2.0f * d0) / (float)n) | ((uint32_t)to_bf16((2.0f * d1) / (float)n) << 16);
      o.y = (uint32_t)to_bf16((2.0f * d2) / (float)n);
    }
    reinterpret_cast<uint4*>(dZ + p * kK)[g] = o;
  }
  __shared__ float red[256];
  red[threadIdx.x] = sq + run;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss_part[blockIdx.x] = red[0] / (float)n;
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                       int64_t n, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// BF16 weights for the forward pass ([tap][cof][32], zero-padded from the
// master [tap][co][ci]) and the flipped, transposed copy for the input
// gradient ([8 - tap][ci][32], zero beyond co).
__global__ void k_pack_w(const float* __restrict__ master, int CO, int CI, int COF, uint16_t* __restrict__ wf,
                         uint16_t* __restrict__ wb) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (int64_t)9 * COF * kK) {
    const int tap = (int)(i / (COF * kK)), rem = (int)(i % (COF * kK));
    const int co = rem / kK, ci = rem % kK;
    wf[i] = (co < CO && ci < CI) ? to_bf16(master[((int64_t)tap * CO + co) * CI + ci]) : (uint16_t)0;
  }
  if (wb && i < (int64_t)9 * CI * kK) {
    const int tapb = (int)(i / (CI * kK)), rem = (int)(i % (CI * kK));
    const int ci = rem / kK, co = rem % kK;
    wb[i] = co < CO ? to_bf16(master[((int64_t)(8 - tapb) * CO + co) * CI + ci]) : (uint16_t)0;
  }
}

// views (V, H, W) RGBA8 + depth -> x[v][p][4] = (R/255, G/255, B/255, D/Z - 1), d = -1 when empty
__global__ void k_pack_input(const uint32_t* __restrict__ views, const float* __restrict__ depth, int64_t n, float D,
                             uint16_t* __restrict__ x) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t c = views[i];
  const float z = depth ? depth[i] : INFINITY;
  const float d = z < INFINITY ? D / z - 1.0f : -1.0f;
  uint2 o;
  o.x = (uint32_t)to_bf16((float)(c & 255u) / 255.0f) | ((uint32_t)to_bf16((float)((c >> 8) & 255u) / 255.0f) << 16);
  o.y = (uint32_t)to_bf16((float)((c >> 16) & 255u) / 255.0f) | ((uint32_t)(depth ? to_bf16(d) : 0u) << 16);
  reinterpret_cast<uint2*>(x)[i] = o;
}

// Disparity blur of each view (the binary32 steps are fixed, so the result is
// reproducible bit for bit): per pixel, s = k*d (0 where d <= -1, empty); for
// tap t = -1, -3/4, .., 1: u = min(max(x + t*s, -1), W), x0 = floor(u),
// f = u - x0, c = (1 - f)*C[x0] + f*C[x0 + 1] (indices clamped to the row),
// acc += w_t*c; XB = (bf16(acc_R), bf16(acc_G), bf16(acc_B), 0).
struct BlurTaps {
  float w[9];
};

// One output pixel of the blur with the packed disparity word `dw` (d in bits
// 16-31); pair(i, a, b) sets a, b to the colours of pixels i and i + 1 of the
// row, i = -1 .. W, indices clamped to the row.
struct Colour {
  float r, g, b;
};
__device__ __forceinline__ Colour unpack_colour(uint2 c) {
  return {from_bf16((uint16_t)(c.x & 0xFFFFu)), from_bf16((uint16_t)(c.x >> 16)), from_bf16((uint16_t)(c.y & 0xFFFFu))};
}
template <typename Pair>
__device__ __forceinline__ uint2 blur_pixel(Pair pair, uint32_t dw, int x, int W, float k, const BlurTaps& bw) {
  const float d = from_bf16((uint16_t)(dw >> 16));
  const float s = d > -1.0f ? k * d : 0.0f;
  float acc[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    const float ts = (j < 4 ? 4 - j : j - 4) * 0.25f * s;
    float u = j < 4 ? (float)x - ts : (float)x + ts;
    u = __builtin_amdgcn_fmed3f(u, -1.0f, (float)W);  // a NaN gives -1, as max and min do
    const float fl = floorf(u);
    const float f = u - fl;
    Colour a, b;
    pair((int)fl, a, b);
    const float g = 1.0f - f;
    acc[0] = acc[0] + bw.w[j] * (g * a.r + f * b.r);
    acc[1] = acc[1] + bw.w[j] * (g * a.g + f * b.g);
    acc[2] = acc[2] + bw.w[j] * (g * a.b + f * b.b);
  }
  uint2 o;
  o.x = pack_bf16x2(acc[0], acc[1]);
  o.y = pack_bf16x2(acc[2], 0.0f);
  return o;
}

// Rows of up to kBlurRowMax pixels: a block stages whole rows in LDS with
// coalesced loads, and every tap is gathered from there.  Vector instructions
// bound it (24 a tap, about the same time as the taps' LDS reads), so colours are
// unpacked once, when staged, and a staged row carries one copy of its first and
// two of its last pixel: the clamped indices of a tap are then two neighbouring
// pixels.  Rows are taken in groups of about kBlurGroup pixels, so that few
// threads of the last pass over a group are idle, as long as kBlurGroups groups
// are left.  48 x 512 x 512 pixels: 90 us
// with packed, unpadded rows, 75 now (groups of 512 pixels 78, of 2048 80).
constexpr int kBlurRowMax = 4096;
constexpr int kBlurGroup = 1024, kBlurGroups = 1536;

inline int blur_rows(int64_t nrows, int W) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(nrows / kBlurGroups, std::min(64, kBlurGroup / W)));
}

__global__ void __launch_bounds__(256) k_disparity_blur_rows(const uint16_t* __restrict__ X, int64_t nrows, int W, int R,
                                                              int4 st, float k, BlurTaps bw, uint16_t* __restrict__ XB) {
  extern __shared__ Colour lrow[];  // R rows of W + 3 pixels: pixel i at i + 1
  const int P = W + 3;  // st: 256 pixels are st.x rows and st.y pixels of W, st.z rows and st.w of P
  const int64_t ngroups = (nrows + R - 1) / R;
  for (int64_t gr = blockIdx.x; gr < ngroups; gr += gridDim.x) {
    const int64_t r0 = gr * R;
    const int nr = (int)min((int64_t)R, nrows - r0);
    const uint2* src = reinterpret_cast<const uint2*>(X) + r0 * W;
    uint2* dst = reinterpret_cast<uint2*>(XB) + r0 * W;
    __syncthreads();  // the previous group's gathers are finished
    for (int i = threadIdx.x, r = i / P, c = i % P; r < nr; i += blockDim.x) {
      lrow[i] = unpack_colour(src[r * W + min(max(c - 1, 0), W - 1)]);
      r += st.z;
      c += st.w;
      if (c >= P) { c -= P; ++r; }
    }
    __syncthreads();
    for (int i = threadIdx.x, r = i / W, x = i % W; r < nr; i += blockDim.x) {
      const Colour* row = lrow + r * P + 1;
      dst[i] = blur_pixel(
          [&](int a, Colour& ca, Colour& cb) {
            ca = row[a];
            cb = row[a + 1];
          },
          src[i].y, x, W, k, bw);
      r += st.x;
      x += st.y;
      if (x >= W) { x -= W; ++r; }
    }
  }
}

// Wider rows: one thread per pixel, taps gathered from global memory.
__global__ void __launch_bounds__(256) k_disparity_blur(const uint16_t* __restrict__ X, int64_t npx, int W, float k,
                                                         BlurTaps bw, uint16_t* __restrict__ XB) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npx) return;
  const int x = (int)(p % W);
  const uint2* row = reinterpret_cast<const uint2*>(X) + (p - x);
  reinterpret_cast<uint2*>(XB)[p] = blur_pixel(
      [&](int a, Colour& ca, Colour& cb) {
        ca = unpack_colour(row[min(max(a, 0), W - 1)]);
        cb = unpack_colour(row[min(max(a + 1, 0), W - 1)]);
      },
      row[x].y, x, W, k, bw);
}

// y[v][p][4] -> RGBA8, clamp(floor(255 y + 0.5)), alpha 255
__global__ void k_unpack_output(const uint16_t* __restrict__ y, int64_t n, uint32_t* __restrict__ views) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t o = 0xFF000000u;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    float f = floorf(from_bf16(y[i * 4 + c]) * 255.0f + 0.5f);
    f = f < 0.0f ? 0.0f : (f > 255.0f ? 255.0f : f);
    o |= (uint32_t)f << (8 * c);
  }
  views[i] = o;
}

}  // namespace net
}  // namespace lfdpr

using namespace lfdpr;
using namespace lfdpr::net;

struct lfdpr_net {
  lfdpr_ctx* ctx = nullptr;
  bool counted = false;  // registered as a child of ctx
  hipStream_t stream = nullptr;
  int device = 0;
  int V = 0;
  int64_t maxpx = 0;  // views * H * W
  int ci[4], co[4], cof[4];
  int64_t off_w[4], off_b[4], nparams = 0;
  float* master = nullptr;
  float* grad = nullptr;
  float* adam_m = nullptr;
  float* adam_v = nullptr;
  int64_t step = 0;
  uint16_t* wf[4] = {nullptr, nullptr, nullptr, nullptr};
  uint16_t* wb[4] = {nullptr, nullptr, nullptr, nullptr};
  uint16_t* act[4] = {nullptr, nullptr, nullptr, nullptr};  // act[1..3]
  uint16_t* dz[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  uint16_t* xb = nullptr;  // disparity blur of the last forward input, [view][H][W][4]
  float kscale = 0.0f;     // pixels per view step per unit d
  BlurTaps taps{};
  const uint16_t* last_x = nullptr;
  const uint16_t* last_y = nullptr;
  int last_n = 0, last_h = 0, last_w = 0;
  float* d_loss = nullptr;
  float* part = nullptr;   // per-block partial gradients (kGradBlocks rows of nparams), then kMseBlocks of the loss
  std::string err;
};

namespace {

int nfail(lfdpr_net* n, int code, const std::string& m) {
  if (n) n->err = m;
  return code;
}

#define NHIP(call)                                                                                    \
  do {                                                                                                \
    hipError_t e_ = (call);                                                                           \
    if (e_ != hipSuccess) return nfail(net, LFDPR_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

template <int NT, int MODE, bool GATHER, int DIL>
void launch_conv(const uint16_t* X, const uint16_t* Wt, const float* b, int N, int H, int W, int V,
                 uint16_t* Y, int YS, const uint16_t* aux, int AUXC, hipStream_t s) {
  const int64_t tiles = (int64_t)N * ((H + kTY - 1) / kTY) * ((W + kTX - 1) / kTX);
  const int grid = (int)std::min<int64_t>(tiles, kConvGrid);  // persistent
  k_conv3x3<NT, MODE, GATHER, DIL><<<grid, kConvThreads, conv_lds_bytes<NT, DIL>(), s>>>(X, Wt, b, N, H, W, V, Y, YS, aux, AUXC);
}

void pack_weights(lfdpr_net* net) {
  for (int k = 0; k < 4; ++k) {
    const int64_t n = 9ll * kK * (net->cof[k] > net->ci[k] ? net->cof[k] : net->ci[k]);
    k_pack_w<<<(unsigned)((n + 255) / 256), 256, 0, net->stream>>>(net->master + net->off_w[k], net->co[k], net->ci[k],
                                                                   net->cof[k], net->wf[k], net->wb[k]);
  }
}

}  // namespace

extern "C" {

int lfdpr_net_create(lfdpr_ctx* ctx, int32_t V, int32_t max_h, int32_t max_w, lfdpr_net** out) {
  if (!ctx || !out) return LFDPR_EINVAL;
  *out = nullptr;
  if (V < 1 || V > 4096 || max_h < 1 || max_w < 1 || (int64_t)V * max_h * max_w > (1ll << 26)) return LFDPR_EINVAL;
  lfdpr_net* net = new lfdpr_net();
  net->ctx = ctx;
  net->stream = ctx_stream_of(ctx);
  net->device = ctx_device_of(ctx);
  net->V = V;
  net->maxpx = (int64_t)V * max_h * max_w;
  const int ci[4] = {kCin0, kHidden, kHidden, kHidden}, co[4] = {kHidden, kHidden, kHidden, 3};
  int64_t off = 0;
  for (int k = 0; k < 4; ++k) {
    net->ci[k] = ci[k];
    net->co[k] = co[k];
    net->cof[k] = k == 3 ? 16 : kHidden;
    net->off_w[k] = off;
    off += 9ll * co[k] * ci[k];
    net->off_b[k] = off;
    off += co[k];
  }
  net->nparams = off;
  bool ok = hipSetDevice(net->device) == hipSuccess;
  auto al = [&](auto*& p, size_t n) { if (ok) ok = hipMalloc((void**)&p, n * sizeof(*p)) == hipSuccess; };
  al(net->master, off);
  al(net->grad, off);
  al(net->adam_m, off);
  al(net->adam_v, off);
  al(net->d_loss, 1);
  al(net->part, (size_t)kGradBlocks * off + kMseBlocks);
  for (int k = 0; k < 4; ++k) {
    al(net->wf[k], 9ll * net->cof[k] * kK);
    if (k > 0) al(net->wb[k], 9ll * ci[k] * kK);
    if (k > 0) al(net->act[k], (size_t)net->maxpx * kHidden);
  }
  for (int k = 1; k <= 4; ++k) al(net->dz[k], (size_t)net->maxpx * kK);
  al(net->xb, (size_t)net->maxpx * 4);
  {  // the angular filter's Gaussian profile (sigma = half a view step), normalised in binary32
    long long wi[9], tot = 0;
    for (int j = 0; j < 9; ++j) {
      const double t = (j - 4) / 4.0;
      wi[j] = std::llround(65535.0 * std::exp(-t * t / 0.5));
      tot += wi[j];
    }
    for (int j = 0; j < 9; ++j) net->taps.w[j] = (float)wi[j] / (float)tot;
  }
  if (!ok) {
    lfdpr_net_destroy(net);
    return LFDPR_ENOMEM;
  }
  // the widest dilation's staged tile takes 71 KB, above the 64 KB a launch has by default
  constexpr int wide = (int)conv_lds_bytes<2, kDilation[2]>();
  if (hipFuncSetAttribute((const void*)k_conv3x3<2, MODE_RELU, false, kDilation[2]>,
                          hipFuncAttributeMaxDynamicSharedMemorySize, wide) != hipSuccess ||
      hipFuncSetAttribute((const void*)k_conv3x3<2, MODE_BWD, false, kDilation[2]>,
                          hipFuncAttributeMaxDynamicSharedMemorySize, wide) != hipSuccess) {
    lfdpr_net_destroy(net);
    return LFDPR_EDEVICE;
  }
  if (hipMemset(net->master, 0, off * 4) != hipSuccess) {
    lfdpr_net_destroy(net);
    return LFDPR_EDEVICE;
  }
  *out = net;
  ctx_children_add(ctx, 1);
  net->counted = true;
  int rc = lfdpr_net_set_params(net, nullptr, 0);
  if (rc) {
    lfdpr_net_destroy(net);
    *out = nullptr;
  }
  return rc;
}

int lfdpr_net_destroy(lfdpr_net* net) {
  if (!net) return LFDPR_OK;
  (void)hipSetDevice(net->device);
  (void)hipStreamSynchronize(net->stream);
  if (net->counted) ctx_children_add(net->ctx, -1);
  (void)hipFree(net->master);
  (void)hipFree(net->grad);
  (void)hipFree(net->adam_m);
  (void)hipFree(net->adam_v);
  (void)hipFree(net->d_loss);
  (void)hipFree(net->part);
  for (int k = 0; k < 4; ++k) { (void)hipFree(net->wf[k]); (void)hipFree(net->wb[k]); (void)hipFree(net->act[k]); }
  for (int k = 0; k < 5; ++k) (void)hipFree(net->dz[k]);
  (void)hipFree(net->xb);
  delete net;
  return LFDPR_OK;
}

const char* lfdpr_net_last_error(lfdpr_net* net) { return net ? net->err.c_str() : "null network"; }

int lfdpr_net_param_count(lfdpr_net* net, int64_t* n) {
  if (!net || !n) return LFDPR_EINVAL;
  *n = net->nparams;
  return LFDPR_OK;
}

int lfdpr_net_set_params(lfdpr_net* net, const float* host, int64_t n) {
  if (!net) return LFDPR_EINVAL;
  if (host && n != net->nparams) return nfail(net, LFDPR_EINVAL, "parameter count mismatch");
  for (int64_t k = 0; host && k < n; ++k)
    if (!std::isfinite(host[k])) return nfail(net, LFDPR_EINVAL, "non-finite parameter");
  NHIP(hipSetDevice(net->device));
  NHIP(hipStreamSynchronize(net->stream));
  if (host) NHIP(hipMemcpy(net->master, host, n * 4, hipMemcpyHostToDevice));
  NHIP(hipMemset(net->adam_m, 0, net->nparams * 4));
  NHIP(hipMemset(net->adam_v, 0, net->nparams * 4));
  net->step = 0;
  pack_weights(net);
  NHIP(hipGetLastError());
  NHIP(hipStreamSynchronize(net->stream));
  return LFDPR_OK;
}

int lfdpr_net_get_params(lfdpr_net* net, float* host, int64_t n) {
  if (!net || !host || n != net->nparams) return LFDPR_EINVAL;
  NHIP(hipSetDevice(net->device));
  NHIP(hipStreamSynchronize(net->stream));
  NHIP(hipMemcpy(host, net->master, n * 4, hipMemcpyDeviceToHost));
  return LFDPR_OK;
}

int lfdpr_net_set_disparity_scale(lfdpr_net* net, float k) {
  if (!net) return LFDPR_EINVAL;
  if (!(k >= 0.0f) || !(k < 1.0e6f)) return nfail(net, LFDPR_EINVAL, "disparity scale out of range");
  net->kscale = k;
  return LFDPR_OK;
}

int lfdpr_net_set_rig(lfdpr_net* net, const lfdpr_view_params* v) {
  if (!net || !v) return LFDPR_EINVAL;
  if (v->V != net->V || v->W < 1 || !(v->aspect > 0.0f) || !(v->fovy_deg > 0.0f && v->fovy_deg < 180.0f) ||
      !(v->cone_deg >= 0.0f && v->cone_deg < 180.0f))
    return nfail(net, LFDPR_EINVAL, "rig does not match the network or is out of range");
  // a view step moves the eye by 2 D tan(cone/2) / V, which shifts a surface at
  // depth Z by fx * 2 D tan(cone/2) / V * (1/Z - 1/D) pixels = k * d, d = D/Z - 1
  const double fx = (v->W / 2.0) / ((double)v->aspect * std::tan((double)v->fovy_deg * M_PI / 360.0));
  const double k = fx * 2.0 * std::tan((double)v->cone_deg * M_PI / 360.0) / v->V;
  return lfdpr_net_set_disparity_scale(net, (float)k);
}

int lfdpr_net_pack_input(lfdpr_net* net, const uint32_t* views, const float* depth, int32_t n_views, int32_t H,
                         int32_t W, float D, void* x) {
  if (!net || !views || !x || n_views < 1 || H < 1 || W < 1 || !(D > 0.0f)) return LFDPR_EINVAL;
  NHIP(hipSetDevice(net->device));
  const int64_t n = (int64_t)n_views * H * W;
  k_pack_input<<<(unsigned)((n + 255) / 256), 256, 0, net->stream>>>(views, depth, n, D, (uint16_t*)x);
  NHIP(hipGetLastError());
  return LFDPR_OK;
}

int lfdpr_net_forward(lfdpr_net* net, const void* x, int32_t n_views, int32_t H, int32_t W, void* y) {
  if (!net || !x || !y) return LFDPR_EINVAL;
  if (n_views < 1 || n_views % net->V || H < 1 || W < 1 || (int64_t)n_views * H * W > net->maxpx)
    return nfail(net, LFDPR_EINVAL, "views must be whole frames of V views and fit the network's maximum");
  NHIP(hipSetDevice(net->device));
  const uint16_t* in = (const uint16_t*)x;
  hipStream_t s = net->stream;
  const int N = n_views, V = net->V;
  const int64_t npx = (int64_t)N * H * W;
  if (W <= kBlurRowMax) {
    const int rows = blur_rows((int64_t)N * H, W);
    const int64_t groups = ((int64_t)N * H + rows - 1) / rows;
    k_disparity_blur_rows<<<(unsigned)(groups < 4096 ? groups : 4096), 256, (size_t)rows * (W + 3) * sizeof(Colour), s>>>(
        in, (int64_t)N * H, W, rows, int4{256 / W, 256 % W, 256 / (W + 3), 256 % (W + 3)}, net->kscale, net->taps, net->xb);
  } else {
    k_disparity_blur<<<(unsigned)((npx + 255) / 256), 256, 0, s>>>(in, npx, W, net->kscale, net->taps, net->xb);
  }
  launch_conv<2, MODE_RELU, true, kDilation[0]>(in, net->wf[0], net->master + net->off_b[0], N, H, W, V, net->act[1], kHidden, net->xb, 4, s);
  launch_conv<2, MODE_RELU, false, kDilation[1]>(net->act[1], net->wf[1], net->master + net->off_b[1], N, H, W, V, net->act[2], kHidden, nullptr, 0, s);
  launch_conv<2, MODE_RELU, false, kDilation[2]>(net->act[2], net->wf[2], net->master + net->off_b[2], N, H, W, V, net->act[3], kHidden, nullptr, 0, s);
  launch_conv<1, MODE_OUT, false, kDilation[3]>(net->act[3], net->wf[3], net->master + net->off_b[3], N, H, W, V, (uint16_t*)y, 4, net->xb, 4, s);
  NHIP(hipGetLastError());
  net->last_x = in;
  net->last_y = (const uint16_t*)y;
  net->last_n = N;
  net->last_h = H;
  net->last_w = W;
  return LFDPR_OK;
}

int lfdpr_net_backward(lfdpr_net* net, const void* target, float* loss) {
  if (!net || !target) return LFDPR_EINVAL;
  if (!net->last_x) return nfail(net, LFDPR_ESTATE, "lfdpr_net_forward first");
  NHIP(hipSetDevice(net->device));
  hipStream_t s = net->stream;
  const int N = net->last_n, H = net->last_h, W = net->last_w, V = net->V;
  const int npx = N * H * W;
  float* const loss_part = net->part + (size_t)kGradBlocks * net->nparams;
  const int mse_blocks = (int)std::min<int64_t>(((int64_t)npx + 63) / 64, kMseBlocks);
  k_mse<<<mse_blocks, 256, 0, s>>>(net->last_y, (const uint16_t*)target, npx, net->dz[4], loss_part);
  const int64_t tiles = (int64_t)N * ((H + kGY - 1) / kGY) * ((W + kGX - 1) / kGX);
  const int rows = (int)std::min<int64_t>(tiles, kGradBlocks);
  auto layer = [&](auto index) {
    constexpr int k = decltype(index)::value;
    k_conv_wgrad<k == 0, kDilation[k]><<<rows, kGThreads, 0, s>>>(
        net->dz[k + 1], net->co[k], k == 0 ? net->last_x : net->act[k], k == 0 ? net->xb : nullptr, net->ci[k], N, H, W, V,
        net->part + net->off_w[k], (int)net->nparams);  // the layer's weights, then its biases
    if constexpr (k > 0)  // input gradient through the flipped, transposed weights, masked by the ReLU
      launch_conv<2, MODE_BWD, false, kDilation[k]>(net->dz[k + 1], net->wb[k], nullptr, N, H, W, V, net->dz[k], kHidden,
                                                    net->act[k], kHidden, s);
  };
  layer(std::integral_constant<int, 3>());
  layer(std::integral_constant<int, 2>());
  layer(std::integral_constant<int, 1>());
  layer(std::integral_constant<int, 0>());
  k_sum_partials<<<(unsigned)((net->nparams + 31) / 32) + 1, 256, 0, s>>>(net->part, rows, (int)net->nparams, net->grad,
                                                                          loss_part, mse_blocks, net->d_loss, loss);
  NHIP(hipGetLastError());
  return LFDPR_OK;
}

int lfdpr_net_adam_step(lfdpr_net* net, float lr, float b1, float b2, float eps) {
  if (!net || !(lr >= 0.0f) || !(b1 >= 0.0f && b1 < 1.0f) || !(b2 >= 0.0f && b2 < 1.0f) || !(eps > 0.0f))
    return nfail(net, LFDPR_EINVAL, "Adam hyper-parameters out of range");
  NHIP(hipSetDevice(net->device));
  net->step += 1;
  const float c1 = (float)(1.0 - std::pow((double)b1, (double)net->step));
  const float c2 = (float)(1.0 - std::pow((double)b2, (double)net->step));
  k_adam<<<(unsigned)((net->nparams + 255) / 256), 256, 0, net->stream>>>(net->master, net->grad, net->adam_m,
                                                                          net->adam_v, net->nparams, lr, b1, b2, eps,
                                                                          c1, c2);
  pack_weights(net);
  NHIP(hipGetLastError());
  return LFDPR_OK;
}

int lfdpr_net_unpack_output(lfdpr_net* net, const void* y, int32_t n_views, int32_t H, int32_t W, uint32_t* views) {
  if (!net || !y || !views || n_views < 1 || H < 1 || W < 1) return LFDPR_EINVAL;
  NHIP(hipSetDevice(net->device));
  const int64_t n = (int64_t)n_views * H * W;
  k_unpack_output<<<(unsigned)((n + 255) / 256), 256, 0, net->stream>>>((const uint16_t*)y, n, views);
  NHIP(hipGetLastError());
  return LFDPR_OK;
}

int lfdpr_net_copy_state(lfdpr_net* net, int32_t which, void* dst, int64_t n_bytes) {
  if (!net || !dst) return LFDPR_EINVAL;
  const int64_t npx = (int64_t)net->last_n * net->last_h * net->last_w;
  const void* src = nullptr;
  int64_t bytes = 0;
  if (which >= 1 && which <= 3) { src = net->act[which]; bytes = npx * kHidden * 2; }
  else if (which == 4) { src = net->xb; bytes = npx * 4 * 2; }
  else if (which >= 11 && which <= 14) { src = net->dz[which - 10]; bytes = npx * kK * 2; }
  else if (which == 20) { src = net->grad; bytes = net->nparams * 4; }
  else return nfail(net, LFDPR_EINVAL, "unknown state");
  if (n_bytes < bytes) return nfail(net, LFDPR_EINVAL, "destination too small");
  NHIP(hipSetDevice(net->device));
  NHIP(hipStreamSynchronize(net->stream));
  NHIP(hipMemcpy(dst, src, (size_t)bytes, hipMemcpyDeviceToDevice));
  return LFDPR_OK;
}

int lfdpr_net_save(lfdpr_net* net, const char* path) {
  if (!net || !path) return LFDPR_EINVAL;
  std::vector<float> buf(3 * net->nparams);
  NHIP(hipSetDevice(net->device));
  NHIP(hipStreamSynchronize(net->stream));
  NHIP(hipMemcpy(buf.data(), net->master, net->nparams * 4, hipMemcpyDeviceToHost));
  NHIP(hipMemcpy(buf.data() + net->nparams, net->adam_m, net->nparams * 4, hipMemcpyDeviceToHost));
  NHIP(hipMemcpy(buf.data() + 2 * net->nparams, net->adam_v, net->nparams * 4, hipMemcpyDeviceToHost));
  FILE* f = std::fopen(path, "wb");
  if (!f) return nfail(net, LFDPR_EINVAL, "cannot open file for writing");
  const char magic[8] = {'L', 'F', 'D', 'P', 'R', 'N', 'E', '1'};
  int64_t hdr[3] = {net->V, net->nparams, net->step};
  bool ok = std::fwrite(magic, 1, 8, f) == 8 && std::fwrite(hdr, 8, 3, f) == 3 &&
            std::fwrite(buf.data(), 4, buf.size(), f) == buf.size();
  ok = (std::fclose(f) == 0) && ok;
  return ok ? LFDPR_OK : nfail(net, LFDPR_EINVAL, "write failed");
}

int lfdpr_net_load(lfdpr_net* net, const char* path) {
  if (!net || !path) return LFDPR_EINVAL;
  FILE* f = std::fopen(path, "rb");
  if (!f) return nfail(net, LFDPR_EINVAL, "cannot open file");
  char magic[8];
  int64_t hdr[3];
  std::vector<float> buf(3 * net->nparams);
  bool ok = std::fread(magic, 1, 8, f) == 8 && std::memcmp(magic, "LFDPRNE1", 8) == 0 && std::fread(hdr, 8, 3, f) == 3 &&
            hdr[0] == net->V && hdr[1] == net->nparams && hdr[2] >= 0 &&
            std::fread(buf.data(), 4, buf.size(), f) == buf.size();
  std::fclose(f);
  if (!ok) return nfail(net, LFDPR_EINVAL, "not a checkpoint of this network");
  int rc = lfdpr_net_set_params(net, buf.data(), net->nparams);
  if (rc) return rc;
  NHIP(hipMemcpy(net->adam_m, buf.data() + net->nparams, net->nparams * 4, hipMemcpyHostToDevice));
  NHIP(hipMemcpy(net->adam_v, buf.data() + 2 * net->nparams, net->nparams * 4, hipMemcpyHostToDevice));
  net->step = hdr[2];
  return LFDPR_OK;
}

}  // extern "C"
