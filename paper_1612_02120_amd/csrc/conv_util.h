// Device code shared by the conv kernels: operand types and fragments, max
// filters, the 1x1 head epilogue, persistent work distribution, tile walks.
#pragma once

#include "common.h"
#include "device_util.h"

namespace emcnn {

template <int P>
struct PT;
template <>
struct PT<F32> {
  static constexpr int CHB = 4, U = 1, BYTES = 4, CB = 16;
};
template <>
struct PT<BF16> {
  static constexpr int CHB = 8, U = 1, BYTES = 2, CB = 24;
};
template <>
struct PT<FP8> {
  static constexpr int CHB = 16, U = 2, BYTES = 1, CB = 48;
};

// Pixel stride of an LDS operand tile, in dwords: the smallest w' >= w with
// w' = 8 (mod 16). gfx950 serves a 16-byte LDS read per half-wave (32 lanes,
// 512 B) from 128 dword banks (measured with SQ_LDS_BANK_CONFLICT). An A
// fragment read has 16 consecutive pixels x 2 chunk groups (+16 B) per half
// wave; with the stride = 8 (mod 16) the 16 pixel starts are exactly the
// multiples of 8 dwords mod 128, the second chunk group fills the gaps, and the
// 128 dwords hit 128 distinct banks.
__host__ __device__ constexpr int pad_words(int w) {
  return (w % 16 == 8) ? w : w + ((24 - (w % 16)) % 16);
}

// CBO: channels staged per LDS pass (0: the precision's default block).
// NMEM > 1: the operand tiles of NMEM phases stacked row-wise (conv_phase over
// phase groups), NMEM times the m-blocks.
template <int P, int CIN, int COUT, int KS, int TY, int TX, int MW, bool HEAD = false, int CBO = 0, int NMEM = 1>
struct Cfg {
  using T = PT<P>;
  static constexpr int CB = CBO ? CBO : (T::CB < CIN) ? T::CB : CIN;
  static_assert(CIN % CB == 0, "channel block must divide CIN");
  static constexpr int NCB = CIN / CB;
  static constexpr int NCHB = CB / T::CHB;  // 16-byte chunks per pixel per block
  static_assert(NCHB * T::CHB == CB, "block must be whole chunks");
  static constexpr int NCHK = KS * KS * NCHB;  // chunks of K per block
  static constexpr int SLOTS = 4 * T::U;       // chunks consumed per group-step
  static constexpr int NGS = (NCHK + SLOTS - 1) / SLOTS;
  static constexpr int NB = COUT / 16;
  static_assert(NB * 16 == COUT, "COUT must be a multiple of 16");
  static constexpr int LR = TY + KS - 1, LC = TX + KS - 1;
  static constexpr int PSB = pad_words(CB * T::BYTES / 4) * 4;
  static constexpr int LDS_IN = NMEM * LR * LC * PSB;
  static constexpr int LDS_TILE = LDS_IN;
  static constexpr int MBLK = NMEM * TY * TX / 16;
  static_assert(TX % 16 == 0, "TX must be a multiple of 16");
  static_assert(MBLK % MW == 0, "m-blocks must split evenly over waves");
  static constexpr int WAVES = MBLK / MW;
  static constexpr int THREADS = WAVES * 64;
};

// ---------------------------------------------------------------- helpers

__device__ __forceinline__ float relu(float v) { return v > 0.0f ? v : 0.0f; }  // +0 for v <= 0

__device__ __forceinline__ float sigmoid_f(float t) {
  if (t >= 0.0f) return 1.0f / (1.0f + expf(-t));
  float e = expf(t);
  return e / (1.0f + e);
}

__device__ __forceinline__ unsigned char to_e4m3(float v) {
  // v >= 0 here (post-ReLU); saturate at the largest finite e4m3fn value.
  v = fminf(v, 448.0f);
  int packed = __builtin_amdgcn_cvt_pk_fp8_f32(v, 0.0f, 0, false);
  return (unsigned char)(packed & 0xff);
}

// Two floats to bf16 (round to nearest even), lo in the low half: one packed
// conversion (converted one at a time, the compiler adds a shift and an or)
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2v){lo, hi}, bf16x2v));
}

__device__ __forceinline__ uint32_t pack_e4m3x2(float lo, float hi) {
  // non-negative inputs; saturate at the largest finite e4m3fn value
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(fminf(lo, 448.0f), fminf(hi, 448.0f), 0, false) & 0xffffu;
}

// Signed bf16 activations (nets without ReLU) are stored as order-preserving
// keys: key = b ^ (b < 0 ? 0xffff : 0x8000) per 16-bit half, so that unsigned
// order is float order and a max filter is one packed unsigned max per dword
// (chunk_max<BF16>). bf16_key / bf16_unkey convert two halves at a time.
typedef short s16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_key(uint32_t x) {
  const uint32_t neg = __builtin_bit_cast(uint32_t, __builtin_bit_cast(s16x2, x) >> (short)15);  // 0xffff if < 0
  return x ^ (neg | 0x80008000u);
}
__device__ __forceinline__ uint32_t bf16_unkey(uint32_t k) {
  const uint32_t pos = __builtin_bit_cast(uint32_t, __builtin_bit_cast(s16x2, k) >> (short)15);  // 0xffff if b >= 0
  return k ^ (~pos | 0x80008000u);
}

// Pixel index, inside a slice, of map pixel (y, x) when the map is stored
// fragment-major modulo D = 2^lg (lg = 0: row-major, row stride rs): fragment
// (y mod D, x mod D) is a row-major block of zs / D^2 pixels holding rows y / D
// and columns x / D.
__device__ __forceinline__ int64_t frag_pix(int y, int x, int lg, int64_t rs, int64_t zs) {
  const int m = (1 << lg) - 1;
  return (int64_t)(((y & m) << lg) + (x & m)) * (zs >> (2 * lg)) + (int64_t)(y >> lg) * rs + (x >> lg);
}

// Operand addressing of one phase tile of a spaced conv (taps d apart, 2x2 max
// filter pd = d / 2 apart before it) whose input map is stored fragment-major
// modulo d. Operand pixel (r, c) of phase (py, px) is the filter at input
// (py + d (y0 + r), px + d (x0 + c)): row y0 + r, column x0 + c of fragment
// (py, px). Its partners at +pd lie at the same row and column of fragments
// (py + pd) mod d and (px + pd) mod d, one row / column further where that
// wraps, so each is a fixed offset from the first element for the whole tile.
// Rows and columns are clamped to the last valid filter origin; clamped ones
// only feed outputs that are not stored.
struct FragTile {
  const gbyte* base;  // fragment (py, px), row 0, column 0
  int64_t rowb;       // bytes per fragment row
  int64_t o01, o10, o11;  // byte offsets of the partners at (0, +pd), (+pd, 0), (+pd, +pd)
  int rmax, cmax;     // last valid filter row / column (fragment coordinates)
  __device__ __forceinline__ const gbyte* at(int r, int c, int elb) const {
    return base + (int64_t)min(r, rmax) * rowb + (int64_t)min(c, cmax) * elb;
  }
};

__device__ __forceinline__ FragTile frag_tile(const gbyte* slice, int elb, const LayerJob& J, int py, int px) {
  // pd = 0: no max filter before this conv (its partners are the pixel itself)
  const int d = max(J.geom & 0xff, 1), pd = (J.geom >> 8) & 0xff;
  const int lg = __builtin_ctz(d);
  const int64_t plane = (J.in_zs >> (2 * lg)) * elb;  // bytes per fragment
  FragTile f;
  f.rowb = J.in_rs * elb;
  f.base = slice + (int64_t)(py * d + px) * plane;
  const int fy = (py + pd) & (d - 1), cy = (py + pd) >> lg;
  const int fx = (px + pd) & (d - 1), cx = (px + pd) >> lg;
  f.o01 = (int64_t)(fx - px) * plane + (int64_t)cx * elb;
  f.o10 = (int64_t)(fy - py) * d * plane + (int64_t)cy * f.rowb;
  f.o11 = f.o01 + f.o10;
  f.rmax = (J.hin - 1 - pd - py) >> lg;  // y + pd <= hin - 1
  f.cmax = (J.win - 1 - pd - px) >> lg;
  return f;
}

// Store element idx of an activation array (LDS or global) in the layer's format.
template <int P, class B>
__device__ __forceinline__ void store_act(B* base, int64_t idx, float v, float inv) {
  if constexpr (P == F32) st<float>(base + idx * 4, v);
  else if constexpr (P == BF16) st<__bf16>(base + idx * 2, (__bf16)v);
  else st<unsigned char>(base + idx, to_e4m3(v * inv));
}

// Elementwise max of two 16-byte chunks of non-negative activations. For
// non-negative bf16 and e4m3fn values the bit patterns are ordered like the
// values, so an unsigned integer max is the float max.
template <int P>
__device__ __forceinline__ i4v chunk_max(i4v a, i4v b);
template <>
__device__ __forceinline__ i4v chunk_max<F32>(i4v a, i4v b) {
  f4 x = __builtin_bit_cast(f4, a), y = __builtin_bit_cast(f4, b);
  f4 r;
  r[0] = fmaxf(x[0], y[0]);
  r[1] = fmaxf(x[1], y[1]);
  r[2] = fmaxf(x[2], y[2]);
  r[3] = fmaxf(x[3], y[3]);
  return __builtin_bit_cast(i4v, r);
}
template <>
__device__ __forceinline__ i4v chunk_max<BF16>(i4v a, i4v b) {
  u16x8 x = __builtin_bit_cast(u16x8, a), y = __builtin_bit_cast(u16x8, b);
  return __builtin_bit_cast(i4v, __builtin_elementwise_max(x, y));
}
// e4m3fn codes of non-negative values are 0x00..0x7e (bit 7 clear), so a
// per-byte a - b + 128 never borrows across bytes and its bit 7 is (a >= b).
__device__ __forceinline__ uint32_t max_u7x4(uint32_t a, uint32_t b) {
  const uint32_t hm = ((a | 0x80808080u) - b) & 0x80808080u;  // 0x80 per byte where a >= b
  const uint32_t m = hm | (hm - (hm >> 7));                   // 0xff per byte where a >= b
  return (a & m) | (b & ~m);
}
// The 2x2 max filter of a 3x3 neighbourhood of FP8 chunks (q row-major) into
// its four outputs (o[2d + e] = max over rows d, d+1 and columns e, e+1), per
// byte. A packed u16 max orders each half by its high byte first, so on the
// raw words it gives the odd bytes' max; the even bytes take a packed u16 max
// of the words masked to them. 9 masks, 20 packed maxes and 4 bit-field
// inserts per dword, against 10 SWAR maxes of 7 operations each.
typedef unsigned short u16x2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pkmax_u16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t,
                            __builtin_elementwise_max(__builtin_bit_cast(u16x2v, a), __builtin_bit_cast(u16x2v, b)));
}
__device__ __forceinline__ void max_filter_fp8(const i4v (&q)[9], i4v (&o)[4]) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    uint32_t hi[9], lo[9];
#pragma unroll
    for (int j = 0; j < 9; ++j) {
      hi[j] = (uint32_t)q[j][w];
      lo[j] = hi[j] & 0x00ff00ffu;
    }
    uint32_t hh[3][2], hl[3][2];  // horizontal maxes of each row
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        hh[r][e] = pkmax_u16(hi[3 * r + e], hi[3 * r + e + 1]);
        hl[r][e] = pkmax_u16(lo[3 * r + e], lo[3 * r + e + 1]);
      }
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t mh = pkmax_u16(hh[d][e], hh[d + 1][e]), ml = pkmax_u16(hl[d][e], hl[d + 1][e]);
        o[2 * d + e][w] = (int)((mh & 0xff00ff00u) | ml);
      }
  }
}

template <>
__device__ __forceinline__ i4v chunk_max<FP8>(i4v a, i4v b) {
  i4v r;
  r[0] = (int)max_u7x4((uint32_t)a[0], (uint32_t)b[0]);
  r[1] = (int)max_u7x4((uint32_t)a[1], (uint32_t)b[1]);
  r[2] = (int)max_u7x4((uint32_t)a[2], (uint32_t)b[2]);
  r[3] = (int)max_u7x4((uint32_t)a[3], (uint32_t)b[3]);
  return r;
}

template <int P>
struct Frag;
template <>
struct Frag<F32> {
  f4 v;
};
template <>
struct Frag<BF16> {
  bf16x8 v;
};
template <>
struct Frag<FP8> {
  i8v v;
};

template <int P>
__device__ __forceinline__ void mma(f4& acc, const Frag<P>& a, const Frag<P>& b);
template <>
__device__ __forceinline__ void mma<F32>(f4& acc, const Frag<F32>& a, const Frag<F32>& b) {
  // one 16-byte chunk = 4 channels = 4 MFMA k-steps of 4 (one channel per lane group)
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[0], b.v[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[1], b.v[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[2], b.v[2], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[3], b.v[3], acc, 0, 0, 0);
}
template <>
__device__ __forceinline__ void mma<BF16>(f4& acc, const Frag<BF16>& a, const Frag<BF16>& b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, acc, 0, 0, 0);
}
template <>
__device__ __forceinline__ void mma<FP8>(f4& acc, const Frag<FP8>& a, const Frag<FP8>& b) {
  // format 0 = e4m3 for both operands; unit block scales (E8M0 127 = 2^0)
  acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a.v, b.v, acc, 0, 0, 0, 127, 0, 127);
}

// Load an MFMA operand fragment (16 bytes per lane, FP8: two 16-byte chunks)
// from LDS or global memory.
template <int P, class B>
__device__ __forceinline__ void load_frag(Frag<P>& f, const B* p0, const B* p1) {
  if constexpr (P == F32) {
    f.v = ld<f4>(p0);
  } else if constexpr (P == BF16) {
    f.v = ld<bf16x8>(p0);
  } else {
    const i4v lo = ld<i4v>(p0), hi = ld<i4v>(p1);
    f.v = i8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  }
}

// Lane exchange inside groups of 4 lanes (DPP quad permutation).
template <int CTRL>
__device__ __forceinline__ int quad_perm(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
constexpr int kQuadXor1 = 0xB1;  // lanes [1, 0, 3, 2]
constexpr int kQuadXor2 = 0x4E;  // lanes [2, 3, 0, 1]
constexpr int kRowMirror = 0x140;      // lane i <- lane 15 - i of its 16-lane row
constexpr int kRowHalfMirror = 0x141;  // lane i <- lane 7 - i of its 8-lane half row

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, quad_perm<CTRL>(__builtin_bit_cast(int, v)));
}

// Sums of four per-lane values v[0..3] over the 16 lanes of each row, with
// DPP exchanges only (no LDS): two pairing steps that each keep half of the
// values (across the row mirror, then the half-row mirror), then a quad
// reduction. On return every lane n16 of a row holds the row sum of
// v[n16 >> 2].
__device__ __forceinline__ float row_sum4_transposed(const float v[4], int n16) {
  const bool lo = n16 < 8, q0 = ((n16 >> 2) & 1) == 0;
  const float a = (lo ? v[0] : v[2]) + dpp_f<kRowMirror>(lo ? v[2] : v[0]);
  const float b = (lo ? v[1] : v[3]) + dpp_f<kRowMirror>(lo ? v[3] : v[1]);
  float r = (q0 ? a : b) + dpp_f<kRowHalfMirror>(q0 ? b : a);
  r += dpp_f<kQuadXor1>(r);
  r += dpp_f<kQuadXor2>(r);
  return r;
}


// 1x1 head + sigmoid straight from MFMA accumulators, for NU m-blocks of 16
// pixels. val(u, nb, k) is lane (g, n16)'s accumulator for pixel 4g + k of
// m-block u and channel nb * 16 + n16; pos(u, y, x) gives m-block u's output
// row and first column. The channel sums go through row_sum4_transposed, after
// which the four lanes of a quad hold four different m-blocks, so one sigmoid
// and one store per lane serve four m-blocks.
template <int NU, int NB, class Val, class Pos>
__device__ __forceinline__ void head_epilogue(Val val, Pos pos, const float (&bias)[NB], const float (&osc)[NB],
                                              const float (&hw)[NB], float head_b, int g, int n16, gbyte* out,
                                              int64_t zoff, int64_t rs, int hout, int wout) {
  const int jq = n16 & 3;
#pragma unroll
  for (int grp = 0; grp < (NU + 3) / 4; ++grp) {
    float mine = 0.f;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int u = grp * 4 + jj;
      if (u < NU) {
        float part[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float pv = 0.f;
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) pv = fmaf(relu(fmaf(val(u, nb, k), osc[nb], bias[nb])), hw[nb], pv);
          part[k] = pv;
        }
        const float r = row_sum4_transposed(part, n16);
        mine = jq == jj ? r : mine;
      }
    }
    const int u = grp * 4 + jq;
    int y, xb;
    pos(u, y, xb);
    const int x = xb + 4 * g + (n16 >> 2);
    if (u < NU && y < hout && x < wout) st<float>(out + (zoff + (int64_t)y * rs + x) * 4, sigmoid_f(mine + head_b));
  }
}

// Persistent work distribution: workgroup b serves XCD b % 8 (hardware
// round-robin) and walks the matching eighth of the item range.
struct ItemRange {
  int64_t begin, end, step;
};

__device__ __forceinline__ ItemRange item_range(int64_t total) {
  const int64_t G = gridDim.x;
  const int64_t b = blockIdx.x;
  if ((G & 7) != 0) return {b, total, G};
  const int64_t per = (total + 7) >> 3;
  const int64_t begin = (b & 7) * per;
  int64_t end = begin + per;
  if (end > total) end = total;
  return {begin + (b >> 3), end, G >> 3};
}

__device__ __forceinline__ const EMCNN_GLOBAL LayerJob* gtab(const LayerJob* t) {
  return (const EMCNN_GLOBAL LayerJob*)t;
}

__device__ __forceinline__ int find_job(const LayerJob* table, int n, int64_t item) {
  const EMCNN_GLOBAL LayerJob* t = gtab(table);
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (t[mid].item0 <= item) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Job of a work item: advance the cursor through the table (items ascend).
__device__ __forceinline__ LayerJob job_at(const JobSet& js, int& cur, int64_t item) {
  if (!js.table) return js.single;
  const EMCNN_GLOBAL LayerJob* t = gtab(js.table);
  while (cur + 1 < js.njobs && t[cur + 1].item0 <= item) ++cur;
  static_assert(sizeof(LayerJob) % 16 == 0, "job copied in 16-byte chunks");
  LayerJob J;
  const gbyte* src = reinterpret_cast<const gbyte*>(t + cur);
#pragma unroll
  for (int k = 0; k < (int)sizeof(LayerJob) / 16; ++k) reinterpret_cast<i4v*>(&J)[k] = ld<i4v>(src + 16 * k);
  return J;
}

__device__ __forceinline__ bool gated_off(const LayerJob& J) {
  return J.gate && *(const EMCNN_GLOBAL int32_t*)J.gate == 0;
}

// The workgroup's item at or after `item` (of its sequence item, item + step, ...
// < end) whose job is not gated off, with its job; false: none. A launch may find
// most of its jobs closed (the tiles that a fallback leaves to the student), so after a
// closed one the wave's lanes look at the gates of the next 64 jobs at a time and the
// walk goes on at the first open one: one by one, each step is three dependent
// loads, and the three launches over 512 closed 128 x 128 tiles took 145 us, 29
// this way. For the FP32 kernels, a fallback's usual teacher: in the BF16 and FP8
// ones the longer walk cost 0.5-0.8 % of every other call (bf16 net B on 5 x 1237 x
// 1511 1440 -> 1452 us). Every lane must be active.
__device__ __forceinline__ bool open_item(const JobSet& js, int& cur, int64_t& item, int64_t end, int64_t step, LayerJob& J) {
  while (item < end) {
    J = job_at(js, cur, item);
    if (!gated_off(J)) return true;
    if (!js.table) return false;
    const EMCNN_GLOBAL LayerJob* t = gtab(js.table);
    const int lane = threadIdx.x & 63;
    uint64_t open = 0;
    int n = cur + 1;
    for (; n < js.njobs; n += 64) {
      const int32_t* gate = t[min(n + lane, js.njobs - 1)].gate;
      open = __ballot(n + lane < js.njobs && !(gate && *(const EMCNN_GLOBAL int32_t*)gate == 0));
      if (open) break;
    }
    if (!open) return false;
    cur = n + __builtin_ctzll(open);
    item += (t[cur].item0 - item + step - 1) / step * step;
  }
  return false;
}

// Output fields of a job that a conv_ws epilogue needs after the tile walk
// has moved on to the next item.
struct EpiJob {
  void* out;
  int64_t out_rs, out_zs;
  int32_t hout, wout;
};

// Walk of the work items of one workgroup (see item_range), skipping items
// of gated-off jobs. Every wave of the workgroup walks the same sequence.
struct TileWalk {
  int64_t item, end, step;
  int cur;
  LayerJob J;
  __device__ void init(const JobSet& js, const ItemRange& rg) {
    item = rg.begin - rg.step;
    end = rg.end;
    step = rg.step;
    cur = 0;
    if (js.table && rg.begin < rg.end) cur = find_job(js.table, js.njobs, rg.begin);
  }
  __device__ bool next(const JobSet& js) {
    for (item += step; item < end; item += step) {
      J = job_at(js, cur, item);
      if (gated_off(J)) continue;
      return true;
    }
    return false;
  }
  // The same, by open_item.
  __device__ bool next_open(const JobSet& js) {
    item += step;
    return open_item(js, cur, item, end, step, J);
  }
  // tile origin and slice of the current item
  template <int TY, int TX>
  __device__ void coords(int& zz, int& y0, int& x0) const {
    const int64_t local = item - J.item0;
    const int bx = (int)(local % J.tiles_x);
    const int64_t t2 = local / J.tiles_x;
    y0 = (int)(t2 % J.tiles_y) * TY;
    x0 = bx * TX;
    zz = (int)(t2 / J.tiles_y);
  }
  // items over groups of four phases (head_taps4's order: tile column, then
  // group, then tile row, then slice); the group's first phase (gy, gx), gy,
  // gx < d / 2; (y0, x0) in sub-lattice coordinates
  template <int TY, int TX>
  __device__ void group_coords(int& zz, int& gy, int& gx, int& y0, int& x0) const {
    const int h = (J.geom & 0xff) >> 1;
    const int tpy = J.tiles_y / (h * h);
    const int64_t local = item - J.item0;
    const int bx = (int)(local % J.tiles_x);
    const int64_t t2 = local / J.tiles_x;
    const int grp = (int)(t2 % (h * h));
    const int64_t t3 = t2 / (h * h);
    y0 = (int)(t3 % tpy) * TY;
    x0 = bx * TX;
    zz = (int)(t3 / tpy);
    gy = grp / h;
    gx = grp % h;
  }
  // phase-tiled items of a spaced conv (the order of conv_phase: tile column,
  // then phase, then tile row, then slice); (y0, x0) in sub-lattice coordinates
  template <int TY, int TX>
  __device__ void phase_coords(int& zz, int& py, int& px, int& y0, int& x0) const {
    const int d = max(J.geom & 0xff, 1);
    const int tpy = J.tiles_y / (d * d);
    const int64_t local = item - J.item0;
    const int bx = (int)(local % J.tiles_x);
    const int64_t t2 = local / J.tiles_x;
    const int ph = (int)(t2 % (d * d));
    const int64_t t3 = t2 / (d * d);
    y0 = (int)(t3 % tpy) * TY;
    x0 = bx * TX;
    zz = (int)(t3 / tpy);
    py = ph / d;
    px = ph % d;
  }
};

// A contiguous block of BYTES bytes (packed weights) held in producer
// registers between its global loads and its LDS writes.
template <int BYTES, int NPT>
struct WStage {
  static constexpr int N = BYTES / 16;
  static_assert(N * 16 == BYTES, "whole 16-byte chunks");
  static constexpr int NIT = (N + NPT - 1) / NPT;
  i4v v[NIT];
  __device__ __forceinline__ void load(const gbyte* src, int ptid) {
#pragma unroll
    for (int k = 0; k < NIT; ++k) {
      const int t = ptid + k * NPT;
      if (t < N) v[k] = ld<i4v>(src + (int64_t)t * 16);
    }
  }
  __device__ __forceinline__ void store(unsigned char* dst, int ptid) const {
#pragma unroll
    for (int k = 0; k < NIT; ++k) {
      const int t = ptid + k * NPT;
      if (t < N) reinterpret_cast<i4v*>(dst)[t] = v[k];
    }
  }
};

}  // namespace emcnn
