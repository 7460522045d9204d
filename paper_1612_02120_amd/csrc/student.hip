// Student network: conv5x5 1->8 ReLU, conv3x3 8->8 ReLU, conv1x1 8->1 sigmoid
// (receptive radius 6). A thinner net that runs everywhere as the fast pass;
// tiles where it disagrees with the plain net on sampled windows fall back to
// the plain net (multi-pass: extra effort only where errors are likely,
// arXiv 1612.02120, Sections 1 and 3).
//
// Parameters (801) in the cnn_create layout: W1[8][1][5][5], b1[8],
// W2[8][8][3][3], b2[8], Wh[8], bh. The library keeps FP32 master weights,
// Adam moments, and "working" weights used by the kernels: W1 / 255 (the input
// is the raw uint8 value) and, in BF16 mode, W1 / 255 and W2 rounded to bf16.
// In BF16 mode conv2's input (h1) and the backward operands dh1, dh2 are also
// rounded to bf16; every product of two bf16 values is exact in FP32 and sums
// accumulate in FP32. The head runs in FP32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/emcnn.h"
#include "common.h"
#include "device_util.h"
#include "runtime.h"

namespace emcnn {

// n < 2^31 workgroups as a grid: a launch holds at most 2^32 threads along x, so in
// rows of at most 2^20, the last of which may have some to spare (grid_block() >= n).
static dim3 grid_rows(int64_t n) {
  const int64_t x = std::min<int64_t>(n, 1 << 20);
  return dim3((unsigned)x, (unsigned)((n + x - 1) / x));
}
__device__ __forceinline__ unsigned grid_block() { return blockIdx.y * gridDim.x + blockIdx.x; }

constexpr int S_C = 8;  // student channels
constexpr int S_NP = 801;
constexpr int OFF_W1 = 0, OFF_B1 = 200, OFF_W2 = 208, OFF_B2 = 784, OFF_WH = 792, OFF_BH = 800;
// Working weights again, in the orders the training kernels read them: eight
// consecutive floats (one scalar load) per tap and channel.
//   OFF_W1T [tap][co], OFF_W2T [tap][ci][co], OFF_W2U [tap][co][ci]
constexpr int OFF_W1T = 808, OFF_W2T = OFF_W1T + 200, OFF_W2U = OFF_W2T + 576, S_NWW = OFF_W2U + 576;

__device__ __forceinline__ float s_relu(float v) { return v > 0.0f ? v : 0.0f; }
__device__ __forceinline__ float s_bf16(float v) { return (float)(__bf16)v; }
__device__ __forceinline__ float s_sigmoid(float t) {
  if (t >= 0.0f) return 1.0f / (1.0f + expf(-t));
  float e = expf(t);
  return e / (1.0f + e);
}

// ------------------------------------------------------------------ fused inference

// out(z, y, x) = student probability at student-output position (y + crop, x + crop)
// of slice z; student output (y, x) is centred on input (y + 3, x + 3).
template <int TY, int TX>
__global__ __launch_bounds__((TY * TX)) void student_fused(const uint8_t* __restrict__ in, int64_t in_rs, int64_t in_zs,
                                                           float* __restrict__ out, int64_t out_rs, int64_t out_zs,
                                                           int Ho, int Wo, int crop, const float* __restrict__ ww,
                                                           int bf16) {
  constexpr int IR = TY + 6, IC = TX + 6, HR = TY + 2, HC = TX + 2;
  __shared__ float xin[IR * IC];
  __shared__ float h1[S_C][HR * HC];
  const int tid = threadIdx.x;
  const int y0 = blockIdx.y * TY, x0 = blockIdx.x * TX, z = blockIdx.z;
  const uint8_t* src = in + (int64_t)z * in_zs;
  // input rows needed: student coords y0+crop .. +TY+5 (clamped to the last valid input row)
  const int hin_lim = Ho + 2 * crop + 6, win_lim = Wo + 2 * crop + 6;  // input dims implied by the output
  for (int t = tid; t < IR * IC; t += TY * TX) {
    int r = t / IC, c = t % IC;
    int y = min(y0 + crop + r, hin_lim - 1), x = min(x0 + crop + c, win_lim - 1);
    xin[t] = (float)src[(int64_t)y * in_rs + x];
  }
  __syncthreads();
  for (int t = tid; t < HR * HC; t += TY * TX) {
    const int r = t / HC, c = t % HC;
    float a[S_C];
#pragma unroll
    for (int co = 0; co < S_C; ++co) a[co] = ww[OFF_B1 + co];
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const float xv = xin[(r + i) * IC + c + j];
#pragma unroll
        for (int co = 0; co < S_C; ++co) a[co] = fmaf(ww[OFF_W1 + co * 25 + i * 5 + j], xv, a[co]);
      }
#pragma unroll
    for (int co = 0; co < S_C; ++co) {
      float v = s_relu(a[co]);
      h1[co][t] = bf16 ? s_bf16(v) : v;
    }
  }
  __syncthreads();
  const int ty = tid / TX, tx = tid % TX;
  float a2[S_C];
#pragma unroll
  for (int co = 0; co < S_C; ++co) a2[co] = ww[OFF_B2 + co];
#pragma unroll
  for (int ci = 0; ci < S_C; ++ci)
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const float hv = h1[ci][(ty + i) * HC + tx + j];
#pragma unroll
        for (int co = 0; co < S_C; ++co) a2[co] = fmaf(ww[OFF_W2 + (co * 8 + ci) * 9 + i * 3 + j], hv, a2[co]);
      }
  float zl = ww[OFF_BH];
#pragma unroll
  for (int co = 0; co < S_C; ++co) zl = fmaf(ww[OFF_WH + co], s_relu(a2[co]), zl);
  const int y = y0 + ty, x = x0 + tx;
  if (y < Ho && x < Wo) out[(int64_t)z * out_zs + (int64_t)y * out_rs + x] = s_sigmoid(zl);
}

// BF16 mode on MFMA. Both convs run as D = W X on 16x16x32 bf16 MFMAs: the
// working weights and h1 are bf16 values and uint8 inputs are exact in bf16,
// so every product is exact and sums are FP32 (in the MFMA's order).
//
// The 8 channels would leave half of an MFMA's 16 rows empty:
//   conv1: two MFMAs on one accumulator, the channels in the weights' rows 0..7 for
//          the first 16 pixels and in rows 8..15 for the next 16. K slot t is tap t,
//          as h1 is rounded to bf16 after this sum: in another order of the slots, a few
//          h1 pixels in a million round the other way.
//   conv2: a column is the pixel pair 2n, 2n + 1, rows 0..7 the channels of pixel 2n,
//          rows 8..15 those of pixel 2n + 1, whose weights are the same ones one tap
//          to the right. A pair's window, 3 x 4 taps x 8 channels, is the K of three
//          MFMAs; lane group g of MFMA i reads h1 pixel (i, g), 16 bytes.
// conv1's operand is two pixels a dword, each row kept twice in LDS, from an even
// and from an odd pixel, so that any two neighbours are one; the two dwords that hold
// a row's end and the next one's start in some lane groups are put together from two.
// A wave computes a strip of 62 output columns (64 of h1, two MFMA columns of 32)
// from the top down, with rings of its own (6 input rows in LDS, each in two places so
// that five consecutive ones always lie in order; three h1 rows as conv2's operands in
// registers, where LDS turns each row once): no barrier, no halo rows but the strip's
// first six, and the loads of the row after next in flight. One sigmoid and one store
// per lane and row. On 8 x 2048^2: 312 us with tiles of 16 x 64 outputs shared by
// four waves and half of each MFMA empty, 157 now, of which the vector instructions
// (95 per row of 62 outputs, 16 of them the sigmoid) fill 77 % and LDS about as much.

// Outputs (y0 .. y0 + n - 1, x) of slice z, one lane each (see where it is called).
__device__ __forceinline__ void student_pixels(const uint8_t* in, int64_t in_rs, int64_t in_zs, float* out, int64_t out_rs,
                                               int64_t out_zs, int Ho, int Wo, int crop, const float* ww, int z, int y0,
                                               int n, int x, bool mine) {
  if (!mine || x >= Wo) return;
  for (int y = y0; y < y0 + n; ++y) {
    const uint8_t* src = in + (int64_t)z * in_zs + (int64_t)(y + crop) * in_rs + x + crop;
    float a[S_C];
#pragma unroll
    for (int co = 0; co < S_C; ++co) a[co] = ww[OFF_B2 + co];
#pragma clang loop unroll(disable)
    for (int e = 0; e < S_C * 9; ++e) {
      const int ci = e / 9, i = e % 9 / 3, j = e % 3;
      float s = 0.f;
#pragma clang loop unroll(disable)
      for (int k = 0; k < 25; ++k) s = fmaf(ww[OFF_W1 + ci * 25 + k], (float)src[(i + k / 5) * in_rs + j + k % 5], s);
      const float h = s_bf16(s_relu(s + ww[OFF_B1 + ci]));
#pragma unroll
      for (int co = 0; co < S_C; ++co) a[co] = fmaf(ww[OFF_W2 + (co * 8 + ci) * 9 + i * 3 + j], h, a[co]);
    }
    float zl = ww[OFF_BH];
#pragma unroll
    for (int co = 0; co < S_C; ++co) zl = fmaf(ww[OFF_WH + co], s_relu(a[co]), zl);
    out[(int64_t)z * out_zs + (int64_t)y * out_rs + x] = s_sigmoid(zl);
  }
}

constexpr int SW = 62;            // output columns of a strip
constexpr int SXP = 42 * 4;       // bytes per input row: 70 pixels of bf16, padded
constexpr int SXC = 528 * 4;      // from the copy that starts at pixel 0 to the one that starts at pixel 1
constexpr int SX = 2 * SXC;       // both copies of 12 rows
constexpr int SHO = 40 * 16;      // in an h1 row, from its even pixels to its odd ones: lanes that read every other pixel read on end
constexpr int SHP = SHO + 33 * 16;  // bytes per h1 row: 64 pixels of 8 channels, and what the last pair over-reads
constexpr int SLDS = SX + 2 * SHP;
static_assert(SXC >= 12 * SXP && SX % 16 == 0 && SHO >= 33 * 16, "rows do not overlap");
__global__ __launch_bounds__(256, 4) void student_strip(const uint8_t* in, int64_t in_rs, int64_t in_zs, float* out,
                                                     int64_t out_rs, int64_t out_zs, int Ho, int Wo, int crop,
                                                     const float* ww, int rows, int nsy, int nsx, int nstrips) {
  __shared__ __attribute__((aligned(16))) unsigned char lds_all[4 * SLDS];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned at = grid_block() * 4 + wave;
  if (at >= (unsigned)nstrips) return;
  const int strip = (int)at;
  unsigned char* const xr = lds_all + wave * SLDS;
  unsigned char* const hr = xr + SX;
  const int g = lane >> 4, n16 = lane & 15;
  const int sx = strip % nsx, sy = (strip / nsx) % nsy, z = strip / (nsx * nsy);
  const int x0 = sx * SW, y0 = sy * rows;
  const int nout = min(rows, Ho - y0);
  // the strip's input: 71 columns from x0 + crop, clamped to the last valid row and column
  const int ylim = Ho + 2 * crop + 5, xlim = Wo + 2 * crop + 5;
  const gbyte* srow = gin(in) + (int64_t)z * in_zs + (int64_t)min(y0 + crop, ylim) * in_rs;  // the next row to load
  int below = ylim - (y0 + crop);                                                            // rows below it
  const unsigned ca = min(x0 + crop + 2 * lane, xlim), cb = min(x0 + crop + 2 * lane + 1, xlim),
                 cc = min(x0 + crop + 2 * lane + 2, xlim);  // this lane's pixels
  unsigned pa[2], pb[2], pc[2];  // rows r and r + 1 ahead of their use
  auto load = [&](int i) __attribute__((always_inline)) {
    pa[i] = srow[ca];
    pb[i] = srow[cb];
    pc[i] = srow[cc];
    srow += below > 0 ? in_rs : 0;
    --below;
  };
  load(0);
  load(1);
  // weight fragments: lane (g, m) holds row m's K slots 8g..8g+7 (every load is
  // unconditional, from a clamped index, and the padding is selected afterwards,
  // so that all of them are in flight together)
  const int ch = n16 & 7, dx = n16 >> 3;
  bf16x8 w1f[2], w2f[3];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const __bf16 v = (__bf16)ldf(ww, OFF_W1 + ch * 25 + min(8 * g + e, 24));
#pragma unroll
    for (int b = 0; b < 2; ++b) w1f[b][e] = b == dx && 8 * g + e < 25 ? v : (__bf16)0.f;
  }
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int j = g - dx;
      const float v = ldf(ww, OFF_W2 + (ch * 8 + e) * 9 + i * 3 + min(max(j, 0), 2));
      w2f[i][e] = (__bf16)(j >= 0 && j < 3 ? v : 0.f);
    }
  // accumulator row 4g + k is channel 4 (g & 1) + k of pixel 2n + (g >> 1)
  f4 b1, b2, wh;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int co = 4 * (g & 1) + k;
    b1[k] = ldf(ww, OFF_B1 + co);
    b2[k] = ldf(ww, OFF_B2 + co);
    wh[k] = ldf(ww, OFF_WH + co);
  }
  const float bh = ldf(ww, OFF_BH);
  // A pair's window holds a pixel that one of the two has zero weights for: were its
  // h1 infinite, the product would be NaN. Weights that bound h1 well below the
  // largest bf16 (any but a diverged student's) rule that out; with others the strip
  // is computed pixel by pixel.
  float top = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) top += 255.f * (fabsf((float)w1f[0][e]) + fabsf((float)w1f[1][e]));
#pragma unroll
  for (int k = 0; k < 4; ++k) top += fabsf(b1[k]);
  if (__any(!(top < 1e36f))) {
    student_pixels(in, in_rs, in_zs, out, out_rs, out_zs, Ho, Wo, crop, ww, z, y0, nout, x0 + lane, lane < SW);
    return;
  }
  // per-lane bases: pixel pairs from taps 8g + 2k (xa) and 8g + 2k + 1 (xb) of pixel n16, h1 writes and reads
  auto tap_at = [&](int tap) __attribute__((always_inline)) {
    tap = tap > 24 ? tap - 8 : tap;  // zero weights there: the address of the lane group before
    const int i = tap / 5, px = n16 + tap % 5;
    return xr + (px & 1) * SXC + i * SXP + (px >> 1) * 4;
  };
  const unsigned char *xa[4], *xb[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) xa[k] = tap_at(8 * g + 2 * k);
#pragma unroll
  for (int k = 0; k < 2; ++k) xb[k] = tap_at(8 * g + 5 + 2 * k);
  unsigned char* const hw = hr + (n16 & 1) * SHO + (8 * (g >> 1) + (n16 >> 1)) * 16 + (g & 1) * 8;
  const unsigned char* const hrd = hr + (g & 1) * SHO + (n16 + (g >> 1)) * 16;
  // the lane's output column after the exchange below: MFMA column g & 1, pixel 2n + (g >> 1)
  const int xo = 32 * (g & 1) + 2 * n16 + (g >> 1);
  const unsigned xo4 = xo * 4;
  const bool col_ok = xo < SW && x0 + xo < Wo;
  gbyte* orow = gout(out) + ((int64_t)z * out_zs + (int64_t)y0 * out_rs + x0) * 4;  // the next output row

  // LDS between lanes of one wave needs no wait (its accesses stay in order), only
  // that the compiler keeps that order
  auto in_order = []() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  u4v h[3][2];  // conv2's operands of the last three h1 rows
  // input row r = p (mod 6) to LDS
  auto take_row = [&](int p) __attribute__((always_inline)) {
    // uint8 -> bf16 is exact: the float of an integer below 256 has a zero low half
    auto pair = [](unsigned lo, unsigned hi) __attribute__((always_inline)) {
      return __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, (float)hi), __builtin_bit_cast(unsigned, (float)lo),
                                   0x07060302u);
    };
    if (lane < 35) {
      const unsigned even = pair(pa[p & 1], pb[p & 1]), odd = pair(pb[p & 1], pc[p & 1]);
      unsigned char* const x = xr + p * SXP + lane * 4;
      st<uint32_t>(x, even);
      st<uint32_t>(x + 6 * SXP, even);
      st<uint32_t>(x + SXC, odd);
      st<uint32_t>(x + SXC + 6 * SXP, odd);
    }
    load(p & 1);
    in_order();
  };
  // input rows r - 4 .. r as conv1 reads them
  unsigned x[2][2][6];
  auto conv1_in = [&](int p) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int k = 0; k < 6; ++k)
          x[c][b][k] = ld<uint32_t>((k < 4 ? xa[k & 3] : xb[k & 1]) + (p + 2) % 6 * SXP + c * 64 + b * 32);
  };
  // conv1: h1 row r - 4, and its operands back for conv2
  auto h1_row = [&](int p) __attribute__((always_inline)) {
    typedef float f2v __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
    auto pack = [](float lo, float hi) __attribute__((always_inline)) {
      return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2v){lo, hi}, bf16x2v));
    };
    f4 d[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      d[c] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        u4v xv;
#pragma unroll
        for (int k = 0; k < 4; ++k) xv[k] = k < 2 ? x[c][b][k] : __builtin_amdgcn_perm(x[c][b][k + 2], x[c][b][k], 0x05040100u);
        d[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1f[b], __builtin_bit_cast(bf16x8, xv), d[c], 0, 0, 0);
      }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
      st<u2v>(hw + (p & 1) * SHP + c * 256, u2v{pack(s_relu(d[c][0] + b1[0]), s_relu(d[c][1] + b1[1])),
                                                pack(s_relu(d[c][2] + b1[2]), s_relu(d[c][3] + b1[3]))});
    in_order();
#pragma unroll
    for (int c = 0; c < 2; ++c) h[p % 3][c] = ld<u4v>(hrd + (p & 1) * SHP + c * 256);
  };
  // conv2 and head: output row r - 6 from h1 rows r - 6 .. r - 4
  auto out_row = [&](int p) __attribute__((always_inline)) {
    float part[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 3; ++i)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2f[i], __builtin_bit_cast(bf16x8, h[(p + 1 + i) % 3][c]), acc, 0, 0, 0);
      part[c] = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) part[c] = fmaf(wh[k], s_relu(acc[k] + b2[k]), part[c]);
    }
    // channels 0..3 (even lane groups) and 4..7 (odd ones) of each pixel: even
    // groups take MFMA column 0, odd ones column 1
    const bool odd = g & 1;
    const float give = odd ? part[0] : part[1], keep = odd ? part[1] : part[0];
    const int got = __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, give), 16 << 10 | 31);  // of lane ^ 16
    const float zl = keep + __builtin_bit_cast(float, got) + bh;
    const float e = expf(-fabsf(zl));
    // (z >= 0 ? 1 : e) / d, d in [1, 2]: the reciprocal and the quotient each corrected
    // once by their residual, which needs no scaling here
    const float num = zl >= 0.0f ? 1.0f : e, d = 1.0f + e;
    float rc = __builtin_amdgcn_rcpf(d);
    rc = fmaf(fmaf(-d, rc, 1.0f), rc, rc);
    const float q = num * rc;
    const float prob = fmaf(fmaf(-d, q, num), rc, q);
    if (col_ok) st<float>(orow + xo4, prob);
    orow += out_rs * 4;
  };
#pragma unroll
  for (int r = 0; r < 7; ++r) {
    take_row(r % 6);
    if (r >= 4) {
      conv1_in(r % 6);
      h1_row(r % 6);
    }
  }
  // an output row a step behind, so that its MFMAs and its sigmoid run while conv1's
  // operands come from LDS
  for (int left = nout; left > 0; left -= 6) {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const int p = (q + 1) % 6;
      take_row(p);
      conv1_in(p);
      out_row(q);
      if (q + 1 >= left) return;
      h1_row(p);
    }
  }
}

// ------------------------------------------------------------------ training kernels

// Forward, loss and the activation gradients of one FY x FX tile of h1
// positions of one patch: h1, h2, dz, dh2 and dh1 in one kernel. Writes, per
// position and FP32 (bf16-valued in BF16 mode where noted):
//   h1[b][y][x][c]  over (P-4)^2 positions, post-ReLU (bf16-valued)
//   h2              over (P-6)^2 positions, post-ReLU
//   dz              (sigmoid(z) - t) / N
//   dh2             dz wh [h2 > 0] (bf16-valued)
//   dh1             sum over co, i, j of W2[co][ci][i][j] dh2[co][y-i][x-j],
//                   masked by h1 > 0 (bf16-valued)
// and one FP64 partial of sum(softplus(z) - t z) per block (fixed-order tree).
// dh1 of a tile needs dh2 two rows and columns before it, which the block
// recomputes (18 x 34 of h2, 20 x 36 of h1 for 16 x 32): 1.3x the multiply-adds
// of the layers run one after another, but one launch instead of three, and no
// layer waits for another's maps. The kernel is bound by the FP32 vector rate;
// a thread computes up to three positions at once, so that the eight weights of
// a tap and channel (two broadcast LDS reads) serve 24 FMAs. 32 us at 16 x 128^2 (10 us of them FMAs
// at the vector rate, 4 us stores; 16 x 16 and 8 x 32 tiles 33 and 35 us, 512
// threads 37 us). Every value is the same
// chain of FMAs in the same order as when each layer was a kernel of its own.
constexpr int FY = 16, FX = 32, FT = 256;  // tile, threads
__global__ __launch_bounds__(FT) void st_forward(const uint8_t* __restrict__ patches, int P, int tiles_y, int tiles_x,
                                                  const float* __restrict__ ww, const float* __restrict__ teacher,
                                                  float* __restrict__ h1, float* __restrict__ h2,
                                                  float* __restrict__ dz, float* __restrict__ dh2,
                                                  float* __restrict__ dh1, double* __restrict__ loss_part,
                                                  double invN, int bf16, int nblocks) {
  constexpr int XR = FY + 8, XC = FX + 8;  // input tile, from (y0 - 2, x0 - 2)
  constexpr int HR = FY + 4, HC = FX + 4;  // h1, from (y0 - 2, x0 - 2)
  constexpr int DR = FY + 2, DC = FX + 2;  // h2 and dh2, from (y0 - 2, x0 - 2)
  constexpr int N1 = (HR * HC + FT - 1) / FT, N2 = (DR * DC + FT - 1) / FT, N3 = FY * FX / FT;
  __shared__ float xin[XR * XC];
  __shared__ float s1[S_C][HR * HC];
  __shared__ float sd[S_C][DR * DC];
  __shared__ double red[FT];
  __shared__ __attribute__((aligned(16))) float wl[S_NWW - OFF_W1T];  // W1T, W2T, W2U
  const int tid = threadIdx.x;
  const int P1 = P - 4, P2 = P - 6;
  const int tiles = tiles_y * tiles_x;
  const unsigned block = grid_block();
  if (block >= (unsigned)nblocks) return;
  const int64_t b = block / (unsigned)tiles;
  const int rt = (int)(block % (unsigned)tiles);
  const int y0 = (rt / tiles_x) * FY, x0 = (rt % tiles_x) * FX;
  const uint8_t* src = patches + b * P * P;
  // every load of the block's inputs in flight before the first is used: input
  // tile, weights, and the targets of this thread's h2 positions
  constexpr int NX = (XR * XC + FT - 1) / FT, NW = ((S_NWW - OFF_W1T) / 4 + FT - 1) / FT;
  static_assert((S_NWW - OFF_W1T) % 4 == 0 && OFF_W1T % 4 == 0, "weights copied in 16-byte chunks");
  unsigned char xb[NX];
  f4 wb[NW];
  float tv[N2];
#pragma unroll
  for (int k = 0; k < NX; ++k) {
    const int t = min(tid + k * FT, XR * XC - 1);
    const int y = min(max(y0 - 2 + t / XC, 0), P - 1), x = min(max(x0 - 2 + t % XC, 0), P - 1);
    xb[k] = src[(int64_t)y * P + x];
  }
#pragma unroll
  for (int k = 0; k < NW; ++k)
    wb[k] = reinterpret_cast<const f4*>(ww + OFF_W1T)[min(tid + k * FT, (S_NWW - OFF_W1T) / 4 - 1)];
#pragma unroll
  for (int k = 0; k < N2; ++k) {
    const int t = min(tid + k * FT, DR * DC - 1);
    const int y = min(max(y0 - 2 + t / DC, 0), P2 - 1), x = min(max(x0 - 2 + t % DC, 0), P2 - 1);
    tv[k] = teacher[(b * P2 + y) * P2 + x];
  }
#pragma unroll
  for (int k = 0; k < NX; ++k)
    if (tid + k * FT < XR * XC) xin[tid + k * FT] = (float)xb[k];
#pragma unroll
  for (int k = 0; k < NW; ++k)
    if (tid + k * FT < (S_NWW - OFF_W1T) / 4) reinterpret_cast<f4*>(wl)[tid + k * FT] = wb[k];
  __syncthreads();
  {
    float a[N1][S_C];
    int xp[N1];
#pragma unroll
    for (int k = 0; k < N1; ++k) {
      const int t = min(tid + k * FT, HR * HC - 1);
      xp[k] = (t / HC) * XC + t % HC;
#pragma unroll
      for (int co = 0; co < S_C; ++co) a[k][co] = ww[OFF_B1 + co];
    }
    // rows rolled: unrolled, the 200 weights overflow the scalar registers
#pragma unroll 1
    for (int i = 0; i < 5; ++i)
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const f4* wv = reinterpret_cast<const f4*>(wl + (i * 5 + j) * 8);
        const f4 wa = wv[0], wb = wv[1];
#pragma unroll
        for (int k = 0; k < N1; ++k) {
          const float xv = xin[xp[k] + i * XC + j];
#pragma unroll
          for (int co = 0; co < S_C; ++co) a[k][co] = fmaf(co < 4 ? wa[co & 3] : wb[co & 3], xv, a[k][co]);
        }
      }
#pragma unroll
    for (int k = 0; k < N1; ++k) {
      const int t = tid + k * FT;
      if (t >= HR * HC) break;
      const int r = t / HC, c = t % HC, y = y0 - 2 + r, x = x0 - 2 + c;
      f4 v[2];
#pragma unroll
      for (int co = 0; co < S_C; ++co) {
        const float q = s_relu(a[k][co]);
        v[co >> 2][co & 3] = bf16 ? s_bf16(q) : q;
        s1[co][t] = v[co >> 2][co & 3];
      }
      if (r >= 2 && c >= 2 && r < 2 + FY && c < 2 + FX && y < P1 && x < P1) {  // this tile's own positions
        f4* o = reinterpret_cast<f4*>(h1 + ((b * P1 + y) * P1 + x) * S_C);
        o[0] = v[0];
        o[1] = v[1];
      }
    }
  }
  __syncthreads();
  double term = 0.0;
  {
    float a[N2][S_C];
    int hp[N2];
#pragma unroll
    for (int k = 0; k < N2; ++k) {
      const int t = min(tid + k * FT, DR * DC - 1);
      hp[k] = (t / DC) * HC + t % DC;
#pragma unroll
      for (int co = 0; co < S_C; ++co) a[k][co] = ww[OFF_B2 + co];
    }
#pragma unroll 1
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int ci = 0; ci < S_C; ++ci) {
          const f4* wv = reinterpret_cast<const f4*>(wl + OFF_W2T - OFF_W1T + ((i * 3 + j) * 8 + ci) * 8);
          const f4 wa = wv[0], wb = wv[1];
#pragma unroll
          for (int k = 0; k < N2; ++k) {
            const float hv = s1[ci][hp[k] + i * HC + j];
#pragma unroll
            for (int co = 0; co < S_C; ++co) a[k][co] = fmaf(co < 4 ? wa[co & 3] : wb[co & 3], hv, a[k][co]);
          }
        }
#pragma unroll
    for (int k = 0; k < N2; ++k) {
      const int t = tid + k * FT;
      if (t >= DR * DC) break;
      const int r = t / DC, c = t % DC, y = y0 - 2 + r, x = x0 - 2 + c;
      float d[S_C];
#pragma unroll
      for (int co = 0; co < S_C; ++co) d[co] = 0.f;
      if (y >= 0 && x >= 0 && y < P2 && x < P2) {
        float zl = ww[OFF_BH];
#pragma unroll
        for (int co = 0; co < S_C; ++co) {
          a[k][co] = s_relu(a[k][co]);
          zl = fmaf(ww[OFF_WH + co], a[k][co], zl);
        }
        const int64_t p = (b * P2 + y) * P2 + x;
        const float g = (s_sigmoid(zl) - tv[k]) * (float)invN;
#pragma unroll
        for (int co = 0; co < S_C; ++co) {
          const float q = a[k][co] > 0.0f ? g * ww[OFF_WH + co] : 0.0f;
          d[co] = bf16 ? s_bf16(q) : q;
        }
        if (r >= 2 && c >= 2) {  // this tile's own positions
          dz[p] = g;
          f4* o2 = reinterpret_cast<f4*>(h2 + p * S_C);
          o2[0] = f4{a[k][0], a[k][1], a[k][2], a[k][3]};
          o2[1] = f4{a[k][4], a[k][5], a[k][6], a[k][7]};
          f4* od = reinterpret_cast<f4*>(dh2 + p * S_C);
          od[0] = f4{d[0], d[1], d[2], d[3]};
          od[1] = f4{d[4], d[5], d[6], d[7]};
          const double zd = (double)zl;
          term += fmax(zd, 0.0) + log1p(exp(-fabs(zd))) - (double)tv[k] * zd;
        }
      }
#pragma unroll
      for (int co = 0; co < S_C; ++co) sd[co][t] = d[co];
    }
  }
  red[tid] = term;
  __syncthreads();
  {
    float a[N3][S_C];
#pragma unroll
    for (int k = 0; k < N3; ++k)
#pragma unroll
      for (int ci = 0; ci < S_C; ++ci) a[k][ci] = 0.f;
#pragma unroll 1
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int k = 0; k < N3; ++k) {
          const int r = (tid + k * FT) / FX, c = tid % FX;
          const int yy = y0 + r - i, xx = x0 + c - j;
          if (yy < 0 || xx < 0 || yy >= P2 || xx >= P2) continue;
          const int dp = (r + 2 - i) * DC + c + 2 - j;
#pragma unroll
          for (int co = 0; co < S_C; ++co) {
            const f4* wv = reinterpret_cast<const f4*>(wl + OFF_W2U - OFF_W1T + ((i * 3 + j) * 8 + co) * 8);
            const f4 wa = wv[0], wb = wv[1];
            const float dv = sd[co][dp];
#pragma unroll
            for (int ci = 0; ci < S_C; ++ci) a[k][ci] = fmaf(ci < 4 ? wa[ci & 3] : wb[ci & 3], dv, a[k][ci]);
          }
        }
#pragma unroll
    for (int k = 0; k < N3; ++k) {
      const int r = (tid + k * FT) / FX, c = tid % FX, y = y0 + r, x = x0 + c;
      if (y < P1 && x < P1) {
        f4 v[2];
#pragma unroll
        for (int ci = 0; ci < S_C; ++ci) {
          const float q = s1[ci][(r + 2) * HC + c + 2] > 0.0f ? a[k][ci] : 0.0f;
          v[ci >> 2][ci & 3] = bf16 ? s_bf16(q) : q;
        }
        f4* o = reinterpret_cast<f4*>(dh1 + ((b * P1 + y) * P1 + x) * S_C);
        o[0] = v[0];
        o[1] = v[1];
      }
    }
  }
  for (int s = FT / 2; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  if (tid == 0) loss_part[block] = red[0];
}

// Partial weight gradients over a chunk of 2048 positions, in FP32: element
// (co, ci, i, j) sums dY[p][co] X[p + (i, j)][ci] over the chunk's positions in
// ascending order (one FMA chain per element, so the result does not depend on
// how the work is laid out), the bias elements sum dY.
//   layer 0: dY = dh1 (P-4)^2 x 8, X = uint8 patch / 255 (5x5, 1 channel)
//   layer 1: dY = dh2 (P-6)^2 x 8, X = h1 (3x3, 8 channels)
//   layer 2: dY = dz  (P-6)^2 x 1, X = h2 (1x1, 8 channels)
// One launch for all layers: the first blocks take layer 1's chunks together
// with layer 2's (the same positions), the rest layer 0's.
//
// A chain of 2048 dependent FMAs per element bounds a chunk from below, so what
// counts is how few other instructions each position costs. Rows of a chunk are
// laid out one after another at the input's row pitch, channel planes apart: a
// position's K taps of a filter row are then consecutive columns, and dY is zero
// in the K - 1 columns past a row's outputs (an FMA with 0 leaves a finite chain
// as it is). A thread holds three taps of one filter row of one (co, ci): per
// eight columns two 16-byte LDS reads of dY, two of X, and 24 FMAs whose X slides
// through registers; the biases read an X of ones. Four producer waves stage the
// next 256 columns meanwhile. Loading dY and X from global memory for every
// element and position instead (two loads per FMA) left the texture addresser as
// the bound: 0.26 - 0.40 ms per layer at 16 x 128^2, against 25 us for all three.
constexpr int WQ = 256;          // columns staged at a time
constexpr int WPITCH = WQ + 4;   // plane pitch in floats: 8 planes' 16-byte reads fall in distinct banks
constexpr int kChunk = 2048;     // positions per chunk
struct WgradArgs {
  const float *dh1, *h1, *dh2, *h2, *dz;
  const uint8_t* patches;
  float* part[3];
  int64_t n1, n2;
  int P, nc1;  // nc1: chunks of layers 1 and 2
};

// A stage. Entry e of a dY plane is column q0 + e; entry e of an X plane is the
// last of the three taps there, the two columns before it being carried along:
//   layer 1: x[8 i + ci] = h1 at (row i, column q0 + e + 2), x[24 + c] = h2,
//            d[co] = dh2, d[8] = dz
//   layer 0: x[i], x[5 + i] = patch / 255 at (row i, columns q0 + e + 2, + 4)
//            for taps 0..2 and 2..4, d[co] = dh1
struct WgBuf {
  float x[32][WPITCH];
  float d[9][WPITCH];
};

// Layout of a chunk in columns: output rows of Ho positions at a pitch of Hi.
struct WgChunk {
  unsigned row0;  // first output row, over all patches (batch P^2 <= 2^31: 32 bits)
  int x0;         // first position's column
  int nq;         // columns of the chunk
  __device__ WgChunk(int64_t p0, int64_t p1, int Ho, int Hi) {
    row0 = (unsigned)p0 / (unsigned)Ho;
    x0 = (int)((unsigned)p0 % (unsigned)Ho);
    const unsigned last = (unsigned)(p1 - 1), row1 = last / (unsigned)Ho;
    nq = (int)(row1 - row0) * Hi + (int)(last % (unsigned)Ho) - x0 + 1;
  }
};

__global__ __launch_bounds__(512) void st_wgrad(WgradArgs a) {
  __shared__ __attribute__((aligned(16))) WgBuf buf[2];
  __shared__ __attribute__((aligned(16))) float ones[WPITCH];
  __shared__ int odd[2][4];  // per stage and producer wave: it staged an h1 that is not finite
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int P = a.P, P1 = P - 4, P2 = P - 6;
  const bool l1 = (int)blockIdx.x < a.nc1;  // uniform: layers 1 and 2, or layer 0
  const int chunk = l1 ? blockIdx.x : blockIdx.x - a.nc1;
  const int Ho = l1 ? P2 : P1, Hi = l1 ? P1 : P;
  const int64_t p0 = (int64_t)chunk * kChunk, p1 = min(l1 ? a.n2 : a.n1, p0 + kChunk);
  const WgChunk w(p0, p1, Ho, Hi);
  const int nst = (w.nq + WQ - 1) / WQ;
  const unsigned rows = (unsigned)(l1 ? a.n2 : a.n1) / (unsigned)Ho;  // output rows over all patches
  // output row and input column of chunk column q (past the chunk's end: read, never used)
  auto at = [&](int q, unsigned& row, int& col) __attribute__((always_inline)) {
    const unsigned v = (unsigned)(q + w.x0);
    row = min(w.row0 + v / (unsigned)Hi, rows - 1);
    col = (int)(v % (unsigned)Hi);
  };
  // X at (row, col): filter rows i are P1 (P) pixels apart
  auto x1_at = [&](unsigned row, int col) __attribute__((always_inline)) {
    const int64_t b = row / (unsigned)P2, y = row % (unsigned)P2;
    return gin(a.h1) + ((b * P1 + y) * P1 + col) * (S_C * 4);
  };
  auto x0_at = [&](unsigned row, int col) __attribute__((always_inline)) {
    const int64_t b = row / (unsigned)P1, y = row % (unsigned)P1;
    return gin(a.patches) + (b * P + y) * P + col;
  };

  if (wave >= 4) {
    // ---------------- producer waves: one column per thread; the next stage's
    // loads are in flight while this stage is computed
    const int pt = tid - 256;
    ones[pt] = 1.0f;
    if (pt < WPITCH - 256) ones[256 + pt] = 1.0f;
    f4 v[3][2], dv[2], hv[2];
    float zv = 0.f;
    unsigned char b5[2][5];
    bool live = false;
    auto load = [&](int k) __attribute__((always_inline)) {
      const int q = k * WQ + pt;
      unsigned row, rx;
      int col, cx;
      at(q, row, col);
      at(q + 2, rx, cx);
      live = col < Ho && q < w.nq;
      const int64_t p = (int64_t)row * Ho + min(col, Ho - 1);
      if (l1) {
        const gbyte* s = x1_at(rx, cx);
        const gbyte* dsrc = gin(a.dh2) + p * (S_C * 4);
        const gbyte* hsrc = gin(a.h2) + p * (S_C * 4);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int h = 0; h < 2; ++h) v[i][h] = ld<f4>(s + (int64_t)i * P1 * (S_C * 4) + h * 16);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          dv[h] = ld<f4>(dsrc + h * 16);
          hv[h] = ld<f4>(hsrc + h * 16);
        }
        zv = ld<float>(gin(a.dz) + p * 4);
      } else {
        unsigned r4;
        int c4;
        at(q + 4, r4, c4);
        const gbyte* s2 = x0_at(rx, cx);
        const gbyte* s4 = x0_at(r4, c4);
        const gbyte* dsrc = gin(a.dh1) + p * (S_C * 4);
#pragma unroll
        for (int i = 0; i < 5; ++i) {
          b5[0][i] = ld<unsigned char>(s2 + (int64_t)i * P);
          b5[1][i] = ld<unsigned char>(s4 + (int64_t)i * P);
        }
        dv[0] = ld<f4>(dsrc);
        dv[1] = ld<f4>(dsrc + 16);
      }
    };
    load(0);
    for (int k = 0; k < nst; ++k) {
      WgBuf& o = buf[k & 1];
      if (l1) {
        bool fin = true;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int c = 0; c < S_C; ++c) {
            const float xv = v[i][c >> 2][c & 3];
            o.x[8 * i + c][pt] = xv;
            fin = fin && isfinite(xv);
          }
#pragma unroll
        for (int c = 0; c < S_C; ++c) o.x[24 + c][pt] = live ? hv[c >> 2][c & 3] : 0.f;
        o.d[8][pt] = live ? zv : 0.f;
        const uint64_t bad = __ballot(!fin);
        if (lane == 0) odd[k & 1][wave - 4] = bad != 0;
      } else {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
          o.x[i][pt] = (float)b5[0][i] * (1.0f / 255.0f);
          o.x[5 + i][pt] = (float)b5[1][i] * (1.0f / 255.0f);
        }
        if (lane == 0) odd[k & 1][wave - 4] = 0;
      }
#pragma unroll
      for (int c = 0; c < S_C; ++c) o.d[c][pt] = live ? dv[c >> 2][c & 3] : 0.f;
      if (k + 1 < nst) load(k + 1);
      __syncthreads();  // stage k ready; the compute waves are done with stage k - 1
    }
    return;
  }

  // ---------------- compute waves: the planes of this lane's elements, and X at
  // the two columns before the first entry
  //   layer 1: waves 0..2: filter row i = wave, lane (co, ci); wave 3: lanes
  //            0..7 layer 2's weights, 8 its bias, 16..23 layer 1's biases, all
  //            in the chain of the last tap
  //   layer 0: waves 0, 1: taps 0..2 and 2..4 of filter row i = lane / 8 for
  //            channel co = lane % 8; lanes 40..47 of wave 1 the biases
  const int lo = lane & 7, hi8 = lane >> 3;
  const bool one = l1 ? wave == 3 && lane >= 8 : wave == 1 && lane >= 40;  // X of ones
  const int xpl = l1 ? (wave < 3 ? 8 * wave + lo : 24 + lo) : (wave & 1) * 5 + min(hi8, 4);
  const int dpl = l1 ? (wave < 3 ? hi8 : lane < 16 ? 8 : lo) : lo;
  float c0 = 1.f, c1 = 1.f;
  {
    const int q = l1 ? 0 : 2 * (wave & 1);
    unsigned row;
    int cc;
    if (l1 && wave < 3) {
      at(q, row, cc);
      c0 = ld<float>(x1_at(row, cc) + (int64_t)wave * P1 * (S_C * 4) + lo * 4);
      at(q + 1, row, cc);
      c1 = ld<float>(x1_at(row, cc) + (int64_t)wave * P1 * (S_C * 4) + lo * 4);
    } else if (!l1) {
      at(q, row, cc);
      c0 = (float)ld<unsigned char>(x0_at(row, cc) + (int64_t)min(hi8, 4) * P) * (1.0f / 255.0f);
      at(q + 1, row, cc);
      c1 = (float)ld<unsigned char>(x0_at(row, cc) + (int64_t)min(hi8, 4) * P) * (1.0f / 255.0f);
    }
  }
  float acc[3] = {0.f, 0.f, 0.f};
  for (int k = 0; k < nst; ++k) {
    __syncthreads();
    if (!l1 && wave > 1) continue;
    const WgBuf& o = buf[k & 1];
    const float* pd = o.d[dpl];
    const float* px = one ? ones : o.x[xpl];
    const int n = min(WQ, w.nq - k * WQ);
    const int* od = odd[k & 1];
    // (c0 and c1 are of the stage before, or of the chunk's start)
    if (od[0] | od[1] | od[2] | od[3] || __any(!isfinite(c0) || !isfinite(c1))) {
      // an h1 of this stage is not finite (0 times it is NaN): only positions, one by one
      for (int q = 0; q < n; ++q) {
        const float x = px[q], d = pd[q];
        if ((k * WQ + q + w.x0) % Hi < Ho) {
          acc[0] = fmaf(d, c0, acc[0]);
          acc[1] = fmaf(d, c1, acc[1]);
          acc[2] = fmaf(d, x, acc[2]);
        }
        c0 = c1;
        c1 = x;
      }
      if (n < WQ) break;
      continue;
    }
#pragma unroll 1
    for (int q = 0; q < n; q += 32) {  // entries past n: dY is zero
      f4 d[8], x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        d[e] = *reinterpret_cast<const f4*>(pd + q + 4 * e);
        x[e] = *reinterpret_cast<const f4*>(px + q + 4 * e);
      }
#pragma unroll
      for (int e = 0; e < 32; ++e) {
        const float xv = x[e >> 2][e & 3], dv = d[e >> 2][e & 3];
        acc[0] = fmaf(dv, c0, acc[0]);
        acc[1] = fmaf(dv, c1, acc[1]);
        acc[2] = fmaf(dv, xv, acc[2]);
        c0 = c1;
        c1 = xv;
      }
    }
  }
  if (l1) {
    float* q1 = a.part[1] + (int64_t)chunk * (S_C * 72 + S_C);
    float* q2 = a.part[2] + (int64_t)chunk * 9;
    if (wave < 3) {
#pragma unroll
      for (int j = 0; j < 3; ++j) q1[(hi8 * 8 + lo) * 9 + wave * 3 + j] = acc[j];
    } else if (lane < 9) {
      q2[lane] = acc[2];
    } else if (lane >= 16 && lane < 24) {
      q1[S_C * 72 + lo] = acc[2];
    }
  } else {
    float* q0 = a.part[0] + (int64_t)chunk * 208;
    if (lane < 40) {
      if (wave == 0) {
#pragma unroll
        for (int j = 0; j < 3; ++j) q0[lo * 25 + hi8 * 5 + j] = acc[j];
      } else if (wave == 1) {
#pragma unroll
        for (int j = 1; j < 3; ++j) q0[lo * 25 + hi8 * 5 + 2 + j] = acc[j];
      }
    } else if (wave == 1 && lane < 48) {
      q0[200 + lo] = acc[2];
    }
  }
}

struct ReduceArgs {
  const float* part[3];
  int nchunk[3];
  const double* loss_part;
  int nloss;
  double invN;
  float* master;
  float* m;
  float* v;
  float* ww;
  float* grad_out;
  double* loss_out;
  double* gnorm_out;
  int do_update;
  int bf16;
  float lr, b1, b2, eps;
  float c1, c2;  // 1 - b1^t, 1 - b2^t
};

__device__ __forceinline__ void refresh_working(float* ww, float w, int e, int bf16) {
  if (e < OFF_B1) w = w * (1.0f / 255.0f);  // the kernels read raw uint8 input
  if (bf16 && (e < OFF_B1 || (e >= OFF_W2 && e < OFF_B2))) w = s_bf16(w);
  ww[e] = w;
  if (e < OFF_B1) {
    ww[OFF_W1T + (e % 25) * 8 + e / 25] = w;
  } else if (e >= OFF_W2 && e < OFF_B2) {
    const int r = e - OFF_W2, co = r / 72, ci = (r / 9) % 8, tap = r % 9;
    ww[OFF_W2T + (tap * 8 + ci) * 8 + co] = w;
    ww[OFF_W2U + (tap * 8 + co) * 8 + ci] = w;
  }
}

// FP64 sum over the block's 1024 threads in a fixed order: butterflies inside
// each wave, then over the 16 waves' sums. Every thread receives it.
__device__ __forceinline__ double block_sum(double v, double* lds16) {
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s);
  if ((threadIdx.x & 63) == 0) lds16[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int k = 0; k < 16; ++k) t += lds16[k];
  return t;
}

// One block of 1024 threads: fixed-order reduction of the chunk partials into
// the gradient, FP64 sums of the loss and of g^2, and the Adam update. One block
// on one CU: its time is latency, so every load is issued ahead of the sums.
__global__ __launch_bounds__(1024) void st_reduce_adam(ReduceArgs a) {
  __shared__ double red[2][16];
  const int e = threadIdx.x;
  const int ec = min(e, S_NP - 1);
  const float w0 = a.master[ec], m0 = a.m[ec], v0 = a.v[ec];
  double l = 0.0;
  for (int i = e; i < a.nloss; i += 1024) l += a.loss_part[i];
  float g = 0.f;
  if (e < S_NP) {
    int layer, local, ne;
    if (e < OFF_W2) {
      layer = 0;
      local = e;
      ne = OFF_W2;
    } else if (e < OFF_WH) {
      layer = 1;
      local = e - OFF_W2;
      ne = OFF_WH - OFF_W2;
    } else {
      layer = 2;
      local = e - OFF_WH;
      ne = S_NP - OFF_WH;
    }
    // chunk after chunk, 64 loads in flight
    const float* src = a.part[layer] + local;
    const int nch = a.nchunk[layer];
    for (int c = 0; c < nch; c += 64) {
      float v[64];
#pragma unroll
      for (int k = 0; k < 64; ++k) v[k] = src[(int64_t)min(c + k, nch - 1) * ne];
#pragma unroll
      for (int k = 0; k < 64; ++k) g = c + k < nch ? g + v[k] : g;
    }
    if (a.grad_out) a.grad_out[e] = g;
  }
  if (e < S_NP && a.do_update) {
    const float m = fmaf(g, 1.0f - a.b1, a.b1 * m0);
    const float v = fmaf(a.b2, v0, (1.0f - a.b2) * g * g);
    a.m[e] = m;
    a.v[e] = v;
    const float mh = m / a.c1, vh = v / a.c2;
    const float w = w0 - a.lr * mh / (sqrtf(vh) + a.eps);
    a.master[e] = w;
    refresh_working(a.ww, w, e, a.bf16);
  }
  const double g2 = block_sum((double)g * (double)g, red[0]);
  const double ls = block_sum(l, red[1]);
  if (e == 0) {
    if (a.loss_out) *a.loss_out = ls * a.invN;
    if (a.gnorm_out) *a.gnorm_out = sqrt(g2);
  }
}

__global__ void st_refresh(float* ww, const float* master, int bf16) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < S_NP) refresh_working(ww, master[e], e, bf16);
}

// ------------------------------------------------------------------ fallback decisions

// One block per fallback tile: counts sampled voxels whose 0.5-threshold
// decision differs between the student map (already in `prob`) and the
// teacher's sample windows; flags the tile when flips > tau * count.
__global__ __launch_bounds__(256) void st_flag_tiles(const float* __restrict__ prob, int64_t rs, int64_t zs,
                                                      const float* __restrict__ samples, const int32_t* __restrict__ win,
                                                      int n_samples, float tau, int32_t* __restrict__ flags) {
  __shared__ int cnt[256], tot[256];
  const int t = blockIdx.x;
  int c = 0, n = 0;
  for (int s = 0; s < n_samples; ++s) {
    const int32_t* w = win + ((int64_t)t * n_samples + s) * 5;  // z, y, x, h, w
    const int wh = w[3], wwid = w[4];
    const float* sp = samples + ((int64_t)t * n_samples + s) * 256;
    for (int q = threadIdx.x; q < wh * wwid; q += blockDim.x) {
      const int yy = q / wwid, xx = q % wwid;
      const float st = prob[(int64_t)w[0] * zs + (int64_t)(w[1] + yy) * rs + w[2] + xx];
      const float te = sp[yy * 16 + xx];
      c += ((st >= 0.5f) != (te >= 0.5f)) ? 1 : 0;
      n += 1;
    }
  }
  cnt[threadIdx.x] = c;
  tot[threadIdx.x] = n;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      cnt[threadIdx.x] += cnt[threadIdx.x + s];
      tot[threadIdx.x] += tot[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) flags[t] = ((float)cnt[0] > tau * (float)tot[0]) ? 1 : 0;
}

__global__ __launch_bounds__(256) void st_count_flags(const int32_t* __restrict__ flags, int n, int32_t* stats) {
  __shared__ int red[256];
  int c = 0;
  for (int i = threadIdx.x; i < n; i += 256) c += flags[i];
  red[threadIdx.x] = c;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    stats[0] = red[0];
    stats[1] = n;
  }
}

// ------------------------------------------------------------------ training batches

// One training batch gathered from device volumes and their teacher maps:
// block (., b) copies patch b (P x P bytes) and its centred targets
// ((P-6) x (P-6) floats). Sources are passed by value (at most 64).
struct GatherSrc {
  const uint8_t* vol;  // first byte of the patch
  const float* map;    // first target value
  int64_t vol_rs;      // bytes per volume row
  int64_t map_rs;      // floats per map row
};
struct GatherArgs {
  GatherSrc src[64];
  int batch, P;
};

__global__ __launch_bounds__(256) void st_gather(GatherArgs a, uint8_t* __restrict__ patches,
                                                  float* __restrict__ targets) {
  const int b = blockIdx.y;
  const GatherSrc g = a.src[b];
  const int P = a.P, Pt = a.P - 6;
  const gbyte* vs = gin(g.vol);
  const gbyte* ms = gin(g.map);
  gbyte* po = gout(patches) + (int64_t)b * P * P;
  gbyte* to = gout(targets) + (int64_t)b * Pt * Pt * 4;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < P * P; i += gridDim.x * 256) {
    const int r = i / P, c = i % P;
    st<uint8_t>(po + i, ld<uint8_t>(vs + (int64_t)r * g.vol_rs + c));
  }
  for (int i = blockIdx.x * 256 + threadIdx.x; i < Pt * Pt; i += gridDim.x * 256) {
    const int r = i / Pt, c = i % Pt;
    st<float>(to + (int64_t)i * 4, ld<float>(ms + ((int64_t)r * g.map_rs + c) * 4));
  }
}

// ------------------------------------------------------------------ host object

struct Student {
  int prec = 1;
  int device = 0;
  float* master = nullptr;  // [801] device
  float* m = nullptr;
  float* v = nullptr;
  float* ww = nullptr;
  int64_t step = 0;
  // training workspace
  void* ws = nullptr;
  size_t ws_bytes = 0;
  // fallback workspace
  void* fb = nullptr;
  size_t fb_bytes = 0;
  // sample-window table: pinned host memory, uploaded asynchronously; rewritten
  // only after the event recorded behind the previous upload has completed
  int32_t* win_host = nullptr;
  size_t win_host_n = 0;
  hipEvent_t win_done = nullptr;
  bool win_pending = false;
};

static int student_ws(Student* s, size_t need) {
  if (need <= s->ws_bytes) return CNN_OK;
  hipDeviceSynchronize();
  if (s->ws) hipFree(s->ws);
  s->ws = nullptr;
  s->ws_bytes = 0;
  if (hipMalloc(&s->ws, need) != hipSuccess) return fail(CNN_ENOMEM, "student workspace");
  s->ws_bytes = need;
  return CNN_OK;
}

static int grad_impl(Student* s, const uint8_t* patches, const float* teacher, int B, int P, float* grad_out,
                     double* loss_out, double* gnorm_out, const cnn_adam* hp, hipStream_t st) {
  const int P1 = P - 4, P2 = P - 6;
  const int64_t n1 = (int64_t)B * P1 * P1, n2 = (int64_t)B * P2 * P2;
  const int nc0 = (int)((n1 + kChunk - 1) / kChunk), nc1 = (int)((n2 + kChunk - 1) / kChunk), nc2 = nc1;
  const int tiles_y = (P1 + FY - 1) / FY, tiles_x = (P1 + FX - 1) / FX;
  const int nloss = B * tiles_y * tiles_x;  // one loss partial per forward block
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t sz_h1 = al(n1 * S_C * 4), sz_h2 = al(n2 * S_C * 4), sz_dz = al(n2 * 4);
  const size_t sz_p0 = al((size_t)nc0 * 208 * 4), sz_p1 = al((size_t)nc1 * 584 * 4), sz_p2 = al((size_t)nc2 * 9 * 4);
  const size_t sz_l = al((size_t)nloss * 8);
  const size_t need = sz_h1 * 2 + sz_h2 * 2 + sz_dz + sz_p0 + sz_p1 + sz_p2 + sz_l + 256;
  int rc = student_ws(s, need);
  if (rc) return rc;
  unsigned char* w = reinterpret_cast<unsigned char*>(s->ws);
  float* h1 = reinterpret_cast<float*>(w);
  w += sz_h1;
  float* dh1 = reinterpret_cast<float*>(w);
  w += sz_h1;
  float* h2 = reinterpret_cast<float*>(w);
  w += sz_h2;
  float* dh2 = reinterpret_cast<float*>(w);
  w += sz_h2;
  float* dz = reinterpret_cast<float*>(w);
  w += sz_dz;
  float* p0 = reinterpret_cast<float*>(w);
  w += sz_p0;
  float* p1 = reinterpret_cast<float*>(w);
  w += sz_p1;
  float* p2 = reinterpret_cast<float*>(w);
  w += sz_p2;
  double* lp = reinterpret_cast<double*>(w);
  const int bf = s->prec == CNN_PREC_BF16;
  const double invN = 1.0 / (double)n2;
  hipLaunchKernelGGL(st_forward, grid_rows(nloss), dim3(FT), 0, st, patches, P, tiles_y, tiles_x, s->ww, teacher, h1, h2,
                     dz, dh2, dh1, lp, invN, bf, nloss);
  WgradArgs wa;
  wa.dh1 = dh1;
  wa.h1 = h1;
  wa.dh2 = dh2;
  wa.h2 = h2;
  wa.dz = dz;
  wa.patches = patches;
  wa.part[0] = p0;
  wa.part[1] = p1;
  wa.part[2] = p2;
  wa.n1 = n1;
  wa.n2 = n2;
  wa.P = P;
  wa.nc1 = nc1;
  hipLaunchKernelGGL(st_wgrad, dim3(nc1 + nc0), dim3(512), 0, st, wa);
  ReduceArgs a;
  std::memset(&a, 0, sizeof(a));
  a.part[0] = p0;
  a.part[1] = p1;
  a.part[2] = p2;
  a.nchunk[0] = nc0;
  a.nchunk[1] = nc1;
  a.nchunk[2] = nc2;
  a.loss_part = lp;
  a.nloss = nloss;
  a.invN = invN;
  a.master = s->master;
  a.m = s->m;
  a.v = s->v;
  a.ww = s->ww;
  a.grad_out = grad_out;
  a.loss_out = loss_out;
  a.gnorm_out = gnorm_out;
  a.bf16 = bf;
  if (hp) {
    s->step += 1;
    a.do_update = 1;
    a.lr = hp->lr;
    a.b1 = hp->beta1;
    a.b2 = hp->beta2;
    a.eps = hp->eps;
    a.c1 = (float)(1.0 - std::pow((double)hp->beta1, (double)s->step));
    a.c2 = (float)(1.0 - std::pow((double)hp->beta2, (double)s->step));
  }
  hipLaunchKernelGGL(st_reduce_adam, dim3(1), dim3(1024), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "student kernels");
  return CNN_OK;
}

}  // namespace emcnn

using namespace emcnn;

extern "C" int student_create(const double* w_init, int64_t n, int32_t precision, cnn_student** out) {
  clear_error();
  if (!w_init || !out) return fail(CNN_EINVAL, "student_create: null argument");
  if (n != S_NP) return fail(CNN_EINVAL, "student_create: expected 801 parameters");
  if (precision != CNN_PREC_FP32 && precision != CNN_PREC_BF16)
    return fail(CNN_EUNSUPPORTED, "student_create: precision must be FP32 or BF16");
  *out = nullptr;
  Student* s = new Student();
  s->prec = precision;
  hipGetDevice(&s->device);
  std::vector<float> w(S_NP);
  for (int i = 0; i < S_NP; ++i) w[i] = (float)w_init[i];
  hipError_t e;
  // master, m, v, then the working weights at a multiple of 32 bytes
  constexpr size_t ww_at = (3 * S_NP + 7) / 8 * 8;
  if ((e = hipMalloc(&s->master, (ww_at + S_NWW) * sizeof(float))) != hipSuccess) {
    delete s;
    return fail(CNN_ENOMEM, "student_create: hipMalloc");
  }
  s->m = s->master + S_NP;
  s->v = s->m + S_NP;
  s->ww = s->master + ww_at;
  e = hipMemcpy(s->master, w.data(), S_NP * sizeof(float), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemset(s->m, 0, 2 * S_NP * sizeof(float));
  if (e == hipSuccess) {
    hipLaunchKernelGGL(st_refresh, dim3(4), dim3(256), 0, 0, s->ww, s->master, s->prec == CNN_PREC_BF16 ? 1 : 0);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    hipFree(s->master);
    delete s;
    return hip_fail(e, "student_create");
  }
  *out = reinterpret_cast<cnn_student*>(s);
  return CNN_OK;
}

extern "C" int student_destroy(cnn_student* h) {
  clear_error();
  if (!h) return CNN_OK;
  Student* s = reinterpret_cast<Student*>(h);
  hipDeviceSynchronize();
  if (s->master) hipFree(s->master);
  if (s->ws) hipFree(s->ws);
  if (s->fb) hipFree(s->fb);
  if (s->win_host) hipHostFree(s->win_host);
  if (s->win_done) hipEventDestroy(s->win_done);
  delete s;
  return CNN_OK;
}

extern "C" int student_get_state(cnn_student* h, double* w_out, double* m_out, double* v_out, int64_t* step_out) {
  clear_error();
  if (!h) return fail(CNN_EINVAL, "student_get_state: null student");
  Student* s = reinterpret_cast<Student*>(h);
  std::vector<float> buf(3 * S_NP);
  hipError_t e = hipDeviceSynchronize();
  if (e != hipSuccess) return hip_fail(e, "student_get_state");
  if ((e = hipMemcpy(buf.data(), s->master, 3 * S_NP * sizeof(float), hipMemcpyDeviceToHost)) != hipSuccess)
    return hip_fail(e, "student_get_state: copy");
  for (int i = 0; i < S_NP; ++i) {
    if (w_out) w_out[i] = buf[i];
    if (m_out) m_out[i] = buf[S_NP + i];
    if (v_out) v_out[i] = buf[2 * S_NP + i];
  }
  if (step_out) *step_out = s->step;
  return CNN_OK;
}

extern "C" int student_set_state(cnn_student* h, const double* w, const double* m, const double* v, int64_t step) {
  clear_error();
  if (!h || !w || !m || !v || step < 0) return fail(CNN_EINVAL, "student_set_state: bad argument");
  Student* s = reinterpret_cast<Student*>(h);
  std::vector<float> buf(3 * S_NP);
  for (int i = 0; i < S_NP; ++i) {
    buf[i] = (float)w[i];
    buf[S_NP + i] = (float)m[i];
    buf[2 * S_NP + i] = (float)v[i];
  }
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(s->master, buf.data(), 3 * S_NP * sizeof(float), hipMemcpyHostToDevice);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(st_refresh, dim3(4), dim3(256), 0, 0, s->ww, s->master, s->prec == CNN_PREC_BF16 ? 1 : 0);
    e = hipGetLastError();
  }
  if (e == hipSuccess) s->step = step;
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) return hip_fail(e, "student_set_state");
  return CNN_OK;
}

static int check_batch(int32_t batch, int32_t patch) {
  if (batch < 1 || patch < 7 || patch > 4096 || (int64_t)batch * patch * patch > (1ll << 31))
    return fail(CNN_EINVAL, "student: batch >= 1 and 7 <= patch <= 4096 required");
  return CNN_OK;
}

extern "C" int student_grad(cnn_student* h, const uint8_t* patches, const float* teacher, int32_t batch, int32_t patch,
                            float* grad_out, double* loss_out, void* stream) {
  clear_error();
  if (!h || !patches || !teacher || !grad_out) return fail(CNN_EINVAL, "student_grad: null argument");
  int rc = check_batch(batch, patch);
  if (rc) return rc;
  return grad_impl(reinterpret_cast<Student*>(h), patches, teacher, batch, patch, grad_out, loss_out, nullptr, nullptr,
                   reinterpret_cast<hipStream_t>(stream));
}

extern "C" int student_train_step(cnn_student* h, const uint8_t* patches, const float* teacher, int32_t batch,
                                  int32_t patch, const cnn_adam* hp, double* loss_out, double* gnorm_out,
                                  void* stream) {
  clear_error();
  if (!h || !patches || !teacher || !hp) return fail(CNN_EINVAL, "student_train_step: null argument");
  if (!(hp->lr > 0) || !(hp->beta1 >= 0 && hp->beta1 < 1) || !(hp->beta2 >= 0 && hp->beta2 < 1) || !(hp->eps > 0))
    return fail(CNN_EINVAL, "student_train_step: bad Adam hyper-parameters");
  int rc = check_batch(batch, patch);
  if (rc) return rc;
  return grad_impl(reinterpret_cast<Student*>(h), patches, teacher, batch, patch, nullptr, loss_out, gnorm_out, hp,
                   reinterpret_cast<hipStream_t>(stream));
}

static int student_launch(Student* s, const uint8_t* vol, int64_t Z, int64_t H, int64_t W, float* out, int64_t out_rs,
                          int64_t out_zs, int Ho, int Wo, int crop, hipStream_t st) {
  hipError_t e;
  if (s->prec == CNN_PREC_BF16) {
    // strips as tall as still give every SIMD eight (a strip computes six input and
    // two h1 rows beyond its own; with four 180 us, with sixteen 164)
    const int64_t nsx = (Wo + SW - 1) / SW;
    int rows = 128;
    while (rows > 8 && Z * nsx * ((Ho + rows - 1) / rows) < 8192) rows /= 2;
    const int64_t nsy = (Ho + rows - 1) / rows, n = Z * nsx * nsy;
    if (n > 2147483647ll - 4) return fail(CNN_EUNSUPPORTED, "student: volume too large");
    hipLaunchKernelGGL(student_strip, grid_rows((n + 3) / 4), dim3(256), 0, st, vol, W, H * W, out, out_rs, out_zs,
                       Ho, Wo, crop, s->ww, rows, (int)nsy, (int)nsx, (int)n);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "student_strip");
    return CNN_OK;
  }
  constexpr int TY = 16, TX = 16;
  dim3 grid((Wo + TX - 1) / TX, (Ho + TY - 1) / TY, (unsigned)Z);
  hipLaunchKernelGGL((student_fused<TY, TX>), grid, dim3(TY * TX), 0, st, vol, W, H * W, out, out_rs, out_zs, Ho, Wo,
                     crop, s->ww, 0);
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "student_fused");
  return CNN_OK;
}

extern "C" int student_infer(cnn_student* h, const uint8_t* vol, const int64_t dims[3], float* prob, void* stream) {
  clear_error();
  if (!h || !vol || !dims || !prob) return fail(CNN_EINVAL, "student_infer: null argument");
  const int64_t Z = dims[0], H = dims[1], W = dims[2];
  if (Z < 1 || Z > 65535 || H < 7 || W < 7 || H >= (1 << 30) || W >= (1 << 30))
    return fail(CNN_EINVAL, "student_infer: bad dims");
  Student* s = reinterpret_cast<Student*>(h);
  return student_launch(s, vol, Z, H, W, prob, W - 6, (H - 6) * (W - 6), (int)(H - 6), (int)(W - 6), 0,
                        reinterpret_cast<hipStream_t>(stream));
}

static uint64_t mix64(uint64_t x) {
  // splitmix64 finaliser
  x += 0x9e3779b97f4a7c15ull;
  x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
  x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
  return x ^ (x >> 31);
}

extern "C" int student_infer_with_fallback(cnn_student* h, cnn_net* th, const uint8_t* vol, const int64_t dims[3],
                                           float* prob, float tau, int32_t tile, int32_t n_samples, uint64_t seed,
                                           int32_t* stats, int32_t* flags_out, void* stream) {
  clear_error();
  if (!h || !th || !vol || !dims || !prob) return fail(CNN_EINVAL, "student_infer_with_fallback: null argument");
  Student* s = reinterpret_cast<Student*>(h);
  Net* net = reinterpret_cast<Net*>(th);
  const int64_t Z = dims[0], H = dims[1], W = dims[2];
  const int R = net->R;
  if (R < 6 || (R - 6) % 2 || net->out_stride != 1 || net->in_channels != 1)
    return fail(CNN_EUNSUPPORTED, "fallback: teacher radius must be even and >= 6, output at full resolution");
  if (Z < 1 || Z > 65535 || H < R + 1 || W < R + 1 || H >= (1 << 30) || W >= (1 << 30))
    return fail(CNN_EINVAL, "fallback: bad dims");
  if (tile < 16 || n_samples < 1 || n_samples > 64 || tau != tau)
    return fail(CNN_EINVAL, "fallback: tile >= 16, 1 <= n_samples <= 64, tau not NaN required");
  int rc = check_device(net);
  if (rc) return rc;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int Ho = (int)(H - R), Wo = (int)(W - R);
  const int crop = (R - 6) / 2;
  const int ty = (Ho + tile - 1) / tile, tx = (Wo + tile - 1) / tile;
  const int64_t ntile = Z * ty * tx;
  if (ntile > (1 << 24)) return fail(CNN_EINVAL, "fallback: too many tiles");
  // workspace: teacher samples, window table, flags (this and the teacher's are grown
  // before anything is enqueued, so that a call that fails for memory writes nothing)
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t nwin = (size_t)ntile * n_samples * 5;
  const size_t sz_samp = al((size_t)ntile * n_samples * 256 * 4), sz_win = al(nwin * 4), sz_flag = al((size_t)ntile * 4);
  const size_t need = sz_samp + sz_win + sz_flag;
  hipError_t e;
  if (need > s->fb_bytes) {
    if ((e = hipDeviceSynchronize()) != hipSuccess) return hip_fail(e, "fallback: workspace grow");
    if (s->fb) hipFree(s->fb);
    s->fb = nullptr;
    s->fb_bytes = 0;
    if (hipMalloc(&s->fb, need) != hipSuccess) return fail(CNN_ENOMEM, "fallback workspace");
    s->fb_bytes = need;
  }
  // the pinned window table is rewritten only after the previous call's upload has run
  if (s->win_pending) {
    if ((e = hipEventSynchronize(s->win_done)) != hipSuccess) return hip_fail(e, "fallback: previous window upload");
    s->win_pending = false;
  }
  if (s->win_host_n < nwin) {
    if (s->win_host) hipHostFree(s->win_host);
    s->win_host = nullptr;
    s->win_host_n = 0;
    if (hipHostMalloc((void**)&s->win_host, nwin * 4) != hipSuccess) return fail(CNN_ENOMEM, "fallback: pinned window table");
    s->win_host_n = nwin;
  }
  if (!s->win_done && (e = hipEventCreateWithFlags(&s->win_done, hipEventDisableTiming)) != hipSuccess)
    return hip_fail(e, "fallback: hipEventCreate");
  float* samples = reinterpret_cast<float*>(s->fb);
  int32_t* win_dev = reinterpret_cast<int32_t*>(reinterpret_cast<unsigned char*>(s->fb) + sz_samp);
  int32_t* flags = reinterpret_cast<int32_t*>(reinterpret_cast<unsigned char*>(s->fb) + sz_samp + sz_win);
  // 1) seeded sample windows per tile (positions do not depend on the data)
  std::vector<Region> sample_regs, rerun_regs;
  for (int64_t z = 0; z < Z; ++z)
    for (int a = 0; a < ty; ++a)
      for (int b = 0; b < tx; ++b) {
        const int64_t t = (z * ty + a) * tx + b;
        const int y0 = a * tile, x0 = b * tile;
        const int th_ = std::min(tile, Ho - y0), tw_ = std::min(tile, Wo - x0);
        const int wh = std::min(16, th_), wwid = std::min(16, tw_);
        for (int k = 0; k < n_samples; ++k) {
          const uint64_t r = mix64(seed ^ mix64((uint64_t)t * 64 + k));
          const int oy = (int)(r % (uint64_t)(th_ - wh + 1));
          const int ox = (int)((r >> 32) % (uint64_t)(tw_ - wwid + 1));
          int32_t* w = s->win_host + ((size_t)t * n_samples + k) * 5;
          w[0] = (int32_t)z;
          w[1] = y0 + oy;
          w[2] = x0 + ox;
          w[3] = wh;
          w[4] = wwid;
          Region g;
          g.in = vol + z * H * W + (int64_t)(y0 + oy) * W + (x0 + ox);
          g.in_rs = W;
          g.in_zs = H * W;
          g.z = 1;
          g.h = wh + R;
          g.w = wwid + R;
          g.out = samples + ((size_t)t * n_samples + k) * 256;
          g.out_rs = 16;
          g.out_zs = 256;
          g.gate = nullptr;
          sample_regs.push_back(g);
        }
        Region q;
        q.in = vol + z * H * W + (int64_t)y0 * W + x0;
        q.in_rs = W;
        q.in_zs = H * W;
        q.z = 1;
        q.h = th_ + R;
        q.w = tw_ + R;
        q.out = prob + z * (int64_t)Ho * Wo + (int64_t)y0 * Wo + x0;
        q.out_rs = Wo;
        q.out_zs = (int64_t)Ho * Wo;
        q.gate = flags + t;
        rerun_regs.push_back(q);
      }
  const size_t nj1 = count_region_jobs(net, sample_regs), nj2 = count_region_jobs(net, rerun_regs);
  rc = arena_reserve(net, nj1 + nj2);
  if (rc) return rc;
  std::vector<Launch> l1, l2;
  size_t used1 = 0, used2 = 0, ws1 = 0, ws2 = 0;
  // both passes are planned before either is submitted: size the shared
  // workspace for the larger one first, so that planning the second cannot
  // reallocate the workspace the first one's jobs point into
  rc = plan_regions(net, sample_regs, 0, l1, used1, ws1, true);
  if (rc) return rc;
  rc = plan_regions(net, rerun_regs, 0, l2, used2, ws2, true);
  if (rc) return rc;
  rc = ensure_ws(net, std::max(ws1, ws2));
  if (rc) return rc;
  // 2) student everywhere, in the teacher's output frame (it runs while the teacher's passes are planned)
  rc = student_launch(s, vol, Z, H, W, prob, Wo, (int64_t)Ho * Wo, Ho, Wo, crop, st);
  if (rc) return rc;
  const void* ws_before = net->ws;
  rc = plan_regions(net, sample_regs, 0, l1, used1, ws1);
  if (rc) return rc;
  rc = plan_regions(net, rerun_regs, used1, l2, used2, ws2);
  if (rc) return rc;
  if (net->ws != ws_before) return fail(CNN_EHIP, "fallback: internal: workspace moved during planning");
  if ((e = hipMemcpyAsync(win_dev, s->win_host, nwin * 4, hipMemcpyHostToDevice, st)) != hipSuccess)
    return hip_fail(e, "fallback: window upload");
  if ((e = hipEventRecord(s->win_done, st)) != hipSuccess) return hip_fail(e, "fallback: hipEventRecord");
  s->win_pending = true;
  // 3) teacher on the sample windows, then the per-tile decisions on the device
  rc = submit(net, l1, 0, used1 + used2, st, false);
  if (rc) return rc;
  hipLaunchKernelGGL(st_flag_tiles, dim3((unsigned)ntile), dim3(256), 0, st, prob, (int64_t)Wo, (int64_t)Ho * Wo,
                     samples, win_dev, n_samples, tau, flags);
  if (stats) hipLaunchKernelGGL(st_count_flags, dim3(1), dim3(256), 0, st, flags, (int)ntile, stats);
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "fallback: flag kernels");
  if (flags_out && (e = hipMemcpyAsync(flags_out, flags, (size_t)ntile * 4, hipMemcpyDeviceToDevice, st)) != hipSuccess)
    return hip_fail(e, "fallback: flag copy");
  // 4) teacher re-run of flagged tiles (unflagged tiles are skipped by the gate);
  // the job table of both passes went up with the first submission
  for (const Launch& la : l2) {
    rc = launch_planned(net, la, st);
    if (rc) return rc;
  }
  if ((e = hipEventRecord(net->arena[net->cur].done, st)) != hipSuccess) return hip_fail(e, "fallback: hipEventRecord");
  return CNN_OK;
}

extern "C" int student_gather(const cnn_patch_src* src, int32_t batch, int32_t patch, int32_t teacher_R,
                              uint8_t* patches_out, float* teacher_out, void* stream) {
  clear_error();
  if (!src || !patches_out || !teacher_out) return fail(CNN_EINVAL, "student_gather: null argument");
  if (batch < 1 || batch > 64 || patch < 7 || patch > 4096)
    return fail(CNN_EINVAL, "student_gather: 1 <= batch <= 64 and 7 <= patch <= 4096 required");
  if (teacher_R < 6 || (teacher_R - 6) % 2) return fail(CNN_EINVAL, "student_gather: teacher radius even and >= 6");
  const int m = (teacher_R - 6) / 2;  // centring offset between the two output frames
  GatherArgs a;
  std::memset(&a, 0, sizeof(a));
  a.batch = batch;
  a.P = patch;
  for (int b = 0; b < batch; ++b) {
    const cnn_patch_src& q = src[b];
    if (!q.volume || !q.teacher) return fail(CNN_EINVAL, "student_gather: source " + std::to_string(b) + " is null");
    if (q.H < teacher_R + 1 || q.W < teacher_R + 1 || q.Z < 1 || q.z < 0 || q.z >= q.Z || q.y < m || q.x < m ||
        (int64_t)q.y + patch + m > q.H || (int64_t)q.x + patch + m > q.W)
      return fail(CNN_EINVAL, "student_gather: source " + std::to_string(b) +
                                  " is outside its volume (origin must lie in [m, side - patch - m], m = (R-6)/2)");
    const int64_t Hm = q.H - teacher_R, Wm = q.W - teacher_R;
    a.src[b].vol = q.volume + ((int64_t)q.z * q.H + q.y) * q.W + q.x;
    a.src[b].map = q.teacher + ((int64_t)q.z * Hm + (q.y - m)) * Wm + (q.x - m);
    a.src[b].vol_rs = q.W;
    a.src[b].map_rs = Wm;
  }
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int gx = std::max(1, std::min(64, (patch * patch + 1023) / 1024));
  hipLaunchKernelGGL(st_gather, dim3(gx, batch), dim3(256), 0, st, a, patches_out, teacher_out);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "student_gather");
  return CNN_OK;
}
