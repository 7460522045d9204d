// FP32 convolutions on the 16-bit matrix cores, for gfx950.
//
// The FP32 MFMA (16x16x4) runs at 1/16 of the rate of the 16-bit ones (16x16x32),
// and the FP32 body convs are bound by it (conv_mfma: 84 % of its peak). Here
// every FP32 operand is a sum of 16-bit values, and a product is the products of
// the parts that matter, accumulated in FP32, as Ootomo and Yokota (2022,
// "Recovering single precision accuracy from Tensor Cores ...") do with f16 and
// Henry, Tang and Heinecke (2019, "Leveraging the bfloat16 artificial
// intelligence datatype for higher-precision computations") with bf16:
//
// * Triples, x = x0 + x1 + x2 with x0 = bf16(x), x1 = bf16(x - x0), x2 the rest:
//   bf16 has FP32's exponents and 3 x 8 bits hold all 24, so a triple is x itself.
//   Six products (the three others are below 2^-24 of the whole). Nothing depends
//   on the range of the values.
// * Pairs, x = hi + lo with hi = f16(x), lo = f16(x - hi), and three products, hi
//   hi + hi lo + lo hi (lo lo is below 2^-22 of the product): half the work.
//   hi + lo holds x to within one unit of the 24th bit, and a K = 32 MFMA rounds
//   its FP32 accumulator an eighth as often as K = 4 steps do; the measured error
//   against 64 bits is no larger than the FP32 MFMA's (rms on a K = 1200 / 512 /
//   432 contraction: 3.9 / 2.6 / 2.3e-7 against 4.5 / 4.0 / 2.6e-7 of the
//   result's rms).
//
// f16 has a 5-bit exponent, so both sides of a pair's products are scaled by powers
// of two that the host derives (exactly, see split_scales in runtime.hip): each
// input channel by a bound on its activations, which uint8 input and known weights
// give by interval arithmetic, and each output channel's weights by their largest
// magnitude. Values down to 2^-11 of a channel's bound keep all their bits; below,
// the error is 2^-40 of the bound (f16 subnormals, which the MFMA does not flush).
// Convs whose bounds or weights leave an ordinary value fewer bits than FP32's own
// rounding keep the FP32 kernels (split_scales), and nets on real-valued maps, which
// have no bound, take triples.
//
// The kernel is warp-specialised as conv_ws: NCW consumer waves run the
// implicit GEMM with both operands in LDS, NPW producer waves fill it. A stage
// is (tile, CB channels). Its operand tile (max filter applied on the FP32
// values, then scaled and split) is double-buffered; the packed weights of a
// stage (78 KB for 5x5, 16 channels) do not fit beside it, so they stream
// through a double buffer of slices of SS group-steps, with one workgroup
// barrier per slice. While the consumers run slice w the producers store slice
// w + 1 and the w-th part of the next stage's operand tile, and issue the loads
// of the parts after those: the loads and registers are spread evenly over the
// stage. LDS reads per MFMA are 2/3 of the BF16 kernel's with pairs (two fragments
// of each operand feed three MFMAs) and half with triples (three feed six). What
// bounds it (counters on net B, FastMemb and MaskExtend at 8 to 32 slices of 1024^2):
// the matrix cores are busy for 69-75 % of the cycles (MaskExtend's first layer 63 %), at
// the 1.6-1.8 GHz that their power leaves; LDS is active for a third, vector
// instructions issue in 10-28 %.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "common.h"
#include "conv_util.h"
#include "device_util.h"

namespace emcnn {

typedef _Float16 h4v __attribute__((ext_vector_type(4)));
typedef _Float16 h8v __attribute__((ext_vector_type(8)));
typedef __bf16 b4v __attribute__((ext_vector_type(4)));

// Kinds of layer: a plain conv (bias, ReLU, NHWC output), the same with the
// 1x1 sigmoid head fused, a spaced max-out conv per phase, and over groups of
// four phases whose max filters share fragments.
enum SplitKind : int { SK_RELU = 0, SK_HEAD = 1, SK_PHASE = 2, SK_GROUP = 3 };

// NP: 16-bit values per operand, 2 (f16 pairs) or 3 (bf16 triples).
template <int CIN, int COUT, int KS, int KIND, int TY, int TX, int NCW, int NPW, int CB_, int SS_, int NP>
struct CfgSplit {
  static_assert(NP == 2 || NP == 3, "pairs or triples");
  static constexpr int KSZ = KS, CB = CB_, SS = SS_;
  static constexpr int NMEM = KIND == SK_GROUP ? 4 : 1;
  static_assert(CIN % 4 == 0 && CB % 8 == 0, "whole 16-byte chunks, stored and of f16");
  // channels past CIN of the last block are zeros (12 input maps: 16 channels, a
  // quarter of the products padding)
  static constexpr int NCB = (CIN + CB - 1) / CB;
  static constexpr int CINP = NCB * CB;
  static constexpr int NCIN = CIN;
  static constexpr int NCHB = CB / 8;  // 16-byte chunks per pixel in each half
  static constexpr int NCHK = KS * KS * NCHB;
  static constexpr int NGS = (NCHK + 3) / 4;         // group-steps of a stage
  static constexpr int NSL = (NGS + SS - 1) / SS;    // weight slices of a stage
  static constexpr int NB = COUT / 16;
  static_assert(NB * 16 == COUT, "COUT must be a multiple of 16");
  static constexpr int LR = TY + KS - 1, LC = TX + KS - 1;
  // the parts' chunks in separate planes of a buffer: 32 B (16 channels) or
  // 16 B per pixel in each. A half-wave reads 16 pixels x 2 lane groups: 512
  // contiguous bytes (32 B), or two 256-byte runs 16 B apart whose common
  // addresses broadcast (16 B), free of bank conflicts without padding.
  static constexpr int PSB = 16 * NCHB;
  static constexpr int PLANE = NMEM * LR * LC * PSB;
  static constexpr int BUF = NP * PLANE;
  static constexpr int STEPB = NB * NP * 1024;  // packed weights of one group-step
  static constexpr int SLB = SS * STEPB;
  static constexpr int WOFF = 2 * BUF;
  static constexpr int LDS = WOFF + 2 * SLB;
  static_assert(LDS <= 160 * 1024, "LDS budget of a gfx950 workgroup");
  static constexpr int MBLK = NMEM * TY * TX / 16;
  static_assert(TX % 16 == 0 && MBLK % NCW == 0, "m-blocks must split evenly over consumer waves");
  static constexpr int MW = MBLK / NCW;
  static_assert(MW % (TX / 16) == 0, "each consumer wave owns whole tile rows");
  static constexpr int WROWS = MW / (TX / 16);
  static_assert(NMEM == 1 || (TX == 16 && TY % WROWS == 0), "a consumer wave's rows lie in one member's tile");
  static constexpr int THREADS = (NCW + NPW) * 64;
  static_assert(THREADS <= 1024, "workgroup size limit");
  static constexpr size_t PACKB = (size_t)NCB * NSL * SLB;  // fragments; pairs: then iscale[CINP], oscale[COUT]
};

// Four scaled FP32 values to f16 hi and lo halves (8 bytes each).
__device__ __forceinline__ void split4(f4 v, f4 sc, u2v& hi, u2v& lo) {
  const f4 x = v * sc;
  const h4v h = __builtin_convertvector(x, h4v);
  const h4v l = __builtin_convertvector(x - __builtin_convertvector(h, f4), h4v);
  hi = __builtin_bit_cast(u2v, h);
  lo = __builtin_bit_cast(u2v, l);
}

// Four FP32 values to the three bf16 values whose sum each is.
__device__ __forceinline__ void split4(f4 x, u2v (&part)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const b4v b = __builtin_convertvector(x, b4v);
    part[k] = __builtin_bit_cast(u2v, b);
    if (k < 2) x = x - __builtin_convertvector(b, f4);
  }
}

// The producers' walk over the operand tile of one stage: item t = 4 channels
// (16 stored bytes) of a 2x2 block of operand pixels (plain, POOL), of one
// operand position of all four members (group) or of one operand pixel. NL
// 16-byte loads per item; the max filter runs on the FP32 values.
template <class C, int KIND, bool POOL, int NPT, int NP>
struct SplitStage {
  static constexpr int NC4 = C::CB / 4;
  static constexpr bool BLK = KIND <= SK_HEAD && POOL;
  static_assert(!BLK || (C::LR % 2 == 0 && C::LC % 2 == 0), "2x2 staging blocks need even tile sides");
  static constexpr int NST = (BLK ? (C::LR / 2) * (C::LC / 2) : C::LR * C::LC) * NC4;
  static constexpr int NIT = (NST + NPT - 1) / NPT;
  static constexpr int NL = KIND == SK_GROUP ? 9 : !POOL ? 1 : KIND == SK_PHASE ? 4 : 9;
  static constexpr int IPB = (NIT + C::NSL - 1) / C::NSL;  // items per thread and slice window
  static_assert(NPT % NC4 == 0, "a thread keeps its channel chunk");
  f4 q[IPB][NL];

  // Addressing of the tile being loaded.
  const gbyte* base;  // first channel of the stage in the slice (spaced: in fragment (py, px))
  int64_t rowb, o01, o10;
  int y0, x0, rA, rB, cA, cB;  // tile origin; last valid rows / columns (group: of the two fragment parities)
  int elb;

  __device__ __forceinline__ void load_item(int k, int n, int ptid) {
    const int t = ptid + k * NPT;
    if (t >= NST) return;
    const int cg = t % NC4, it = t / NC4;
    const gbyte* b = base + cg * 16;
    if constexpr (C::CINP != C::NCIN) {
      static_assert(C::NCB == 1 || C::CINP == C::NCIN, "padding in a single channel block");
      if (cg * 4 >= C::NCIN) {
#pragma unroll
        for (int i = 0; i < NL; ++i) q[n][i] = f4{0.f, 0.f, 0.f, 0.f};
        return;
      }
    }
    if constexpr (KIND == SK_GROUP) {
      const int R = y0 + it / C::LC, Cc = x0 + it % C::LC;
      const int64_t a0 = (int64_t)min(R, rA) * rowb, b0 = (int64_t)min(R, rB) * rowb;
      const int64_t a1 = (int64_t)min(R + 1, rA) * rowb;
      const int64_t c0 = (int64_t)min(Cc, cA) * elb, d0 = (int64_t)min(Cc, cB) * elb;
      const int64_t c1 = (int64_t)min(Cc + 1, cA) * elb;
      q[n][0] = ld<f4>(b + a0 + c0);              // F00[R][C]
      q[n][1] = ld<f4>(b + o01 + a0 + d0);        // F01[R][C]
      q[n][2] = ld<f4>(b + o10 + b0 + c0);        // F10[R][C]
      q[n][3] = ld<f4>(b + o10 + o01 + b0 + d0);  // F11[R][C]
      q[n][4] = ld<f4>(b + a0 + c1);              // F00[R][C+1]
      q[n][5] = ld<f4>(b + o10 + b0 + c1);        // F10[R][C+1]
      q[n][6] = ld<f4>(b + a1 + c0);              // F00[R+1][C]
      q[n][7] = ld<f4>(b + o01 + a1 + d0);        // F01[R+1][C]
      q[n][8] = ld<f4>(b + a1 + c1);              // F00[R+1][C+1]
    } else if constexpr (KIND == SK_PHASE && POOL) {
      const gbyte* p = b + (int64_t)min(y0 + it / C::LC, rA) * rowb + (int64_t)min(x0 + it % C::LC, cA) * elb;
      q[n][0] = ld<f4>(p);
      q[n][1] = ld<f4>(p + o01);
      q[n][2] = ld<f4>(p + o10);
      q[n][3] = ld<f4>(p + o01 + o10);
    } else if constexpr (BLK) {
      // the stored 3x3 neighbourhood of a 2x2 operand block (see stage_tile
      // for the clamping: rA, cA are the last valid operand row and column)
      const int r = 2 * (it / (C::LC / 2)), c = 2 * (it % (C::LC / 2));
      const int ya = min(y0 + r, rA), yb = min(y0 + r + 1, rA) + 1;
      const int xa = min(x0 + c, cA), xb = min(x0 + c + 1, cA) + 1;
      const gbyte* pr[3] = {b + (int64_t)ya * rowb, b + (int64_t)(ya + 1) * rowb, b + (int64_t)yb * rowb};
      const int64_t pc[3] = {(int64_t)xa * elb, (int64_t)(xa + 1) * elb, (int64_t)xb * elb};
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) q[n][i * 3 + j] = ld<f4>(pr[i] + pc[j]);
    } else {
      q[n][0] = ld<f4>(b + (int64_t)min(y0 + it / C::LC, rA) * rowb + (int64_t)min(x0 + it % C::LC, cA) * elb);
    }
  }

  static __device__ __forceinline__ f4 mx(f4 a, f4 b) {
    return f4{fmaxf(a[0], b[0]), fmaxf(a[1], b[1]), fmaxf(a[2], b[2]), fmaxf(a[3], b[3])};
  }
  static __device__ __forceinline__ void put(unsigned char* lds, int pix, int cg, f4 v, f4 sc) {
    u2v part[NP];
    if constexpr (NP == 2) split4(v, sc, part[0], part[1]);
    else split4(v, part);
#pragma unroll
    for (int k = 0; k < NP; ++k) st<u2v>(lds + k * C::PLANE + pix * C::PSB + cg * 8, part[k]);
  }
  __device__ __forceinline__ void store_item(int k, int n, unsigned char* lds, f4 sc, int ptid) const {
    const int t = ptid + k * NPT;
    if (t >= NST) return;
    const int cg = t % NC4, it = t / NC4;
    const f4* v = q[n];
    if constexpr (KIND == SK_GROUP) {
      const f4 m13 = mx(v[1], v[3]), m23 = mx(v[2], v[3]), m35 = mx(v[3], v[5]);
      put(lds, it, cg, mx(mx(v[0], v[2]), m13), sc);
      put(lds, C::LR * C::LC + it, cg, mx(mx(v[1], v[4]), m35), sc);
      put(lds, 2 * C::LR * C::LC + it, cg, mx(m23, mx(v[6], v[7])), sc);
      put(lds, 3 * C::LR * C::LC + it, cg, mx(m35, mx(v[7], v[8])), sc);
    } else if constexpr (KIND == SK_PHASE && POOL) {
      put(lds, it, cg, mx(mx(v[0], v[1]), mx(v[2], v[3])), sc);
    } else if constexpr (BLK) {
      const int r = 2 * (it / (C::LC / 2)), c = 2 * (it % (C::LC / 2));
      f4 hm[3][2];
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int e = 0; e < 2; ++e) hm[i][e] = mx(v[3 * i + e], v[3 * i + e + 1]);
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int e = 0; e < 2; ++e) put(lds, (r + d) * C::LC + c + e, cg, mx(hm[d][e], hm[d + 1][e]), sc);
    } else {
      put(lds, it, cg, v[0], sc);
    }
  }
  // the part of the tile that slice window w carries
  __device__ __forceinline__ void load(int w, int ptid) {
#pragma unroll
    for (int n = 0; n < IPB; ++n)
      if (w * IPB + n < NIT) load_item(w * IPB + n, n, ptid);
  }
  __device__ __forceinline__ void store(int w, unsigned char* lds, f4 sc, int ptid) const {
#pragma unroll
    for (int n = 0; n < IPB; ++n)
      if (w * IPB + n < NIT) store_item(w * IPB + n, n, lds, sc, ptid);
  }
};

template <int CIN, int COUT, int KS, bool POOL, int KIND, int TY, int TX, int NCW, int NPW, int CB, int SS, int NP>
__global__ __launch_bounds__((CfgSplit<CIN, COUT, KS, KIND, TY, TX, NCW, NPW, CB, SS, NP>::THREADS)) void conv_split(
    JobSet js, ConvParams prm) {
  using C = CfgSplit<CIN, COUT, KS, KIND, TY, TX, NCW, NPW, CB, SS, NP>;
  constexpr bool SPACED = KIND >= SK_PHASE;
  constexpr int MCOLS = TX / 16;
  constexpr int ELB = CIN * 4;  // bytes per stored input pixel (NHWC)
  __shared__ __attribute__((aligned(16))) unsigned char lds[C::LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform role
  const gbyte* wglob = gin(prm.wpack);

  const ItemRange rg = item_range(js.total_items);
  TileWalk w;
  w.init(js, rg);
  if (!w.next_open(js)) return;  // no work for this workgroup (uniform)

  // origin of the walk's tile: slice, first phase (spaced), tile origin
  auto origin = [&](int& zz, int& py, int& px, int& y0, int& x0) __attribute__((always_inline)) {
    py = px = 0;
    if constexpr (KIND == SK_GROUP) w.group_coords<TY, TX>(zz, py, px, y0, x0);
    else if constexpr (KIND == SK_PHASE) w.phase_coords<TY, TX>(zz, py, px, y0, x0);
    else w.coords<TY, TX>(zz, y0, x0);
  };

  if (wave >= NCW) {
    // ---------------- producer waves
    const int ptid = tid - NCW * 64;
    constexpr int NPT = NPW * 64;
    SplitStage<C, KIND, POOL, NPT, NP> a;
    WStage<C::SLB, NPT> ws;
    a.elb = ELB;
    const gbyte* isc = wglob + C::PACKB + (ptid % (C::CB / 4)) * 16;  // this thread's channel scales
    f4 sc = {};
    int cb = 0;
    const gbyte* tile0 = nullptr;  // channel 0 of the tile's slice (spaced: of its fragment)
    auto new_tile = [&]() __attribute__((always_inline)) {
      const LayerJob& J = w.J;
      int zz, py, px;
      origin(zz, py, px, a.y0, a.x0);
      const gbyte* slice = gin(J.in) + (int64_t)zz * J.in_zs * ELB;
      a.rowb = J.in_rs * ELB;
      if constexpr (KIND == SK_GROUP) {
        const int d = J.geom & 0xff, h = d >> 1, lg = __builtin_ctz(d);
        const int64_t plane = (J.in_zs >> (2 * lg)) * ELB;  // bytes per fragment
        tile0 = slice + (int64_t)(py * d + px) * plane;
        a.o01 = h * plane;
        a.o10 = (int64_t)h * d * plane;
        a.rA = (J.hin - 1 - py) >> lg;
        a.rB = (J.hin - 1 - py - h) >> lg;
        a.cA = (J.win - 1 - px) >> lg;
        a.cB = (J.win - 1 - px - h) >> lg;
      } else if constexpr (KIND == SK_PHASE) {
        const FragTile f = frag_tile(slice, ELB, J, py, px);
        tile0 = f.base;
        a.o01 = f.o01;
        a.o10 = f.o10;
        a.rA = f.rmax;
        a.cA = f.cmax;
      } else {
        tile0 = slice;
        a.rA = J.hin - 1 - (POOL ? 1 : 0);
        a.cA = J.win - 1 - (POOL ? 1 : 0);
      }
    };
    auto new_stage = [&]() __attribute__((always_inline)) {
      a.base = tile0 + cb * (C::CB * 4);
      if constexpr (NP == 2) sc = ld<f4>(isc + cb * (C::CB * 4));
    };
    // the next stage of the walk; false past the last
    auto advance = [&]() __attribute__((always_inline)) -> bool {
      if (++cb == C::NCB) {
        cb = 0;
        if (!w.next_open(js)) return false;
        new_tile();
      }
      new_stage();
      return true;
    };
    // weight slices in the order the consumers use them, cyclic over a tile
    int wq = 0;
    auto load_w = [&]() __attribute__((always_inline)) {
      ws.load(wglob + (size_t)wq * C::SLB, ptid);
      wq = wq + 1 == C::NCB * C::NSL ? 0 : wq + 1;
    };
    // stage 0 and slice 0
    new_tile();
    new_stage();
    load_w();
    ws.store(lds + C::WOFF, ptid);
#pragma unroll 1
    for (int p = 0; p < C::NSL; ++p) {
#pragma unroll
      for (int n = 0; n < a.IPB; ++n)
        if (p * a.IPB + n < a.NIT) a.load_item(p * a.IPB + n, n, ptid);
#pragma unroll
      for (int n = 0; n < a.IPB; ++n)
        if (p * a.IPB + n < a.NIT) a.store_item(p * a.IPB + n, n, lds, sc, ptid);
    }
    bool more = advance();  // does the stage after the consumers' stage exist
    if (more) a.load(0, ptid);
    load_w();
    __syncthreads();  // stage 0, slice 0 ready
    int sel = 1, wsel = 1;
    for (;;) {
      bool more2 = false;
#pragma unroll
      for (int p = 0; p < C::NSL; ++p) {
        // the consumers run slice p of their stage
        ws.store(lds + C::WOFF + wsel * C::SLB, ptid);  // slice p + 1 (past the end: a slice nobody reads)
        wsel ^= 1;
        load_w();
        if (more) {
          a.store(p, lds + sel * C::BUF, sc, ptid);
          if (p + 1 < C::NSL) {
            a.load(p + 1, ptid);
          } else {
            more2 = advance();
            if (more2) a.load(0, ptid);
          }
        }
        __syncthreads();  // slice p + 1 ready, slice p done
      }
      if (!more) return;
      more = more2;
      sel ^= 1;
    }
  }

  // ---------------- consumer waves: tile rows wave*WROWS .. +WROWS-1 (group:
  // of one member, whose operand rows are stacked after the earlier members')
  const int g = lane >> 4, n16 = lane & 15;
  const int wrow0 = KIND == SK_GROUP ? (wave * C::WROWS) % TY : wave * C::WROWS;
  const int wmem = KIND == SK_GROUP ? (wave * C::WROWS) / TY : 0;
  const int lrow0 = wmem * C::LR + wrow0;
  // Weights as the MFMA's A operand and pixels as B: lane (g, n16) accumulates
  // four channels of pixel n16, stored as 16 bytes. With the fused head the
  // other way round: channel n16 of pixels 4g .. 4g + 3 (head_epilogue).
  constexpr bool TRANS = KIND != SK_HEAD;
  static_assert(NP == 2 || TRANS, "triples: max-out convs");
  f4 acc[C::MW][C::NB];
  int cb = 0, sel = 0, wsel = 0;

  // one group-step: three (pairs) or six (triples) products per (m-block, n-block), small terms first
  using Frag16 = std::conditional_t<NP == 2, h8v, bf16x8>;
  // the products: part of the pixels, part of the weights (triples: weights part by part)
  constexpr int XP[6] = {NP == 2 ? 1 : 0, NP == 2 ? 0 : 1, 0, 2, 1, 0};
  constexpr int WP[6] = {NP == 2 ? 0 : 2, 1, NP == 2 ? 0 : 1, 0, 0, 0};
  auto step = [&](const unsigned char* abase, const unsigned char* wl, int s) __attribute__((always_inline)) {
    // LDS offset of this lane group's chunk: slot 4 s + g, chunk-major inside a tap
    int o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const KSlot k = k_slot(4 * s + e, KS, C::NCHB, false);
      o[e] = (k.i * C::LC + k.j) * C::PSB + k.cg * 16;
    }
    const int off = g < 2 ? (g == 0 ? o[0] : o[1]) : (g == 2 ? o[2] : o[3]);
    const unsigned char* ap = abase + off;
    auto mm = [&](f4& c, const Frag16& x, const Frag16& wv) __attribute__((always_inline)) {
      if constexpr (NP == 3) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv, x, c, 0, 0, 0);
      else if constexpr (TRANS) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(wv, x, c, 0, 0, 0);
      else c = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, wv, c, 0, 0, 0);
    };
    auto a_at = [&](int u, int k) __attribute__((always_inline)) {
      return ap + ((u / MCOLS) * C::LC + (u % MCOLS) * 16) * C::PSB + k * C::PLANE;
    };
    auto w_at = [&](int nb, int k) __attribute__((always_inline)) { return wl + (nb * NP + k) * 1024; };
    // the operand with fewer fragments stays in registers, the other streams
    if constexpr (NP == 2 && C::NB <= C::MW) {
      Frag16 wv[C::NB][NP];
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb)
#pragma unroll
        for (int k = 0; k < NP; ++k) wv[nb][k] = ld<Frag16>(w_at(nb, k));
#pragma unroll
      for (int u = 0; u < C::MW; ++u) {
        Frag16 x[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) x[k] = ld<Frag16>(a_at(u, k));
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
          for (int nb = 0; nb < C::NB; ++nb) mm(acc[u][nb], x[XP[t]], wv[nb][WP[t]]);
      }
    } else {
      Frag16 x[C::MW][NP];
#pragma unroll
      for (int u = 0; u < C::MW; ++u)
#pragma unroll
        for (int k = 0; k < NP; ++k) x[u][k] = ld<Frag16>(a_at(u, k));
      if constexpr (NP == 2) {
        // the next n-block's weights are loaded ahead of this one's MFMAs, and no
        // earlier (the scheduler would hoist them until the registers spill)
        Frag16 wv[2][NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) wv[0][k] = ld<Frag16>(w_at(0, k));
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb) {
          if (nb + 1 < C::NB) {
#pragma unroll
            for (int k = 0; k < NP; ++k) wv[(nb + 1) & 1][k] = ld<Frag16>(w_at(nb + 1, k));
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int u = 0; u < C::MW; ++u) mm(acc[u][nb], x[u][XP[t]], wv[nb & 1][WP[t]]);
        }
      } else {
        // The small products are summed in accumulators of their own, which a sum takes
        // with the large one: six roundings of a whole sum per step would cost what the
        // operands gain (MaskExtend's rms error against 64 bits 1.26 of that with pairs,
        // 0.6 this way, for 8 % of the time). A part of the weights makes way for the next
        // n-block's where its last product is issued.
        Frag16 wv[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) wv[k] = ld<Frag16>(w_at(0, k));
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb) {
          f4 low[C::MW];
#pragma unroll
          for (int t = 0; t < 6; ++t) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < C::MW; ++u) {
              if (t == 0) low[u] = f4{0.f, 0.f, 0.f, 0.f};
              if (t == 5) acc[u][nb] += low[u];
              mm(t < 5 ? low[u] : acc[u][nb], x[u][XP[t]], wv[WP[t]]);
            }
            if (nb + 1 < C::NB && (t == 5 || WP[t + 1] != WP[t])) wv[WP[t]] = ld<Frag16>(w_at(nb + 1, WP[t]));
          }
        }
      }
    }
  };

  const gbyte* osc_p = wglob + C::PACKB + C::CINP * 4;
  auto epilogue = [&]() __attribute__((always_inline)) {
    int zz, py, px, y0, x0;
    origin(zz, py, px, y0, x0);
    const LayerJob& J = w.J;
    if constexpr (KIND == SK_HEAD) {
      float bias[C::NB], osc[C::NB], hw[C::NB];
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb) {
        bias[nb] = ldf(prm.bias, nb * 16 + n16);
        osc[nb] = ld<float>(osc_p + (nb * 16 + n16) * 4);
        hw[nb] = ldf(prm.head_w, nb * 16 + n16);
      }
      head_epilogue<C::MW, C::NB>(
          [&](int u, int nb, int k) __attribute__((always_inline)) { return acc[u][nb][k]; },
          [&](int u, int& y, int& xb) __attribute__((always_inline)) {
            y = y0 + wrow0 + u / MCOLS;
            xb = x0 + (u % MCOLS) * 16;
          },
          bias, osc, hw, prm.head_b, g, n16, gout(J.out), (int64_t)zz * J.out_zs, J.out_rs, J.hout, J.wout);
    } else {
      // biases and scales of this lane's channels, all at once where the
      // accumulators leave the registers for it (4 n-blocks: FastMemb's convs 7 %
      // faster than with a load at each use), else where they are used
      constexpr bool PRE = C::NB <= 4;
      f4 bsv[PRE ? C::NB : 1], scv[PRE ? C::NB : 1];
      auto chan4 = [&](int nb) __attribute__((always_inline)) { return split_chan(nb, 4 * g, C::NB, SPACED) * 4; };
      if constexpr (PRE) {
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb) {
          bsv[nb] = ld<f4>(gin(prm.bias) + chan4(nb));
          if constexpr (NP == 2) scv[nb] = ld<f4>(osc_p + chan4(nb));
        }
      }
      // this lane's four channels of n-block nb: acc * sc + bs (triples are not scaled)
      auto value = [&](f4 v, int nb) __attribute__((always_inline)) {
        const f4 bs = PRE ? bsv[PRE ? nb : 0] : ld<f4>(gin(prm.bias) + chan4(nb));
        if constexpr (NP == 3) return v + bs;
        const f4 sc = PRE ? scv[PRE ? nb : 0] : ld<f4>(osc_p + chan4(nb));
        f4 t;
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = fmaf(v[k], sc[k], bs[k]);
        return t;
      };
      if constexpr (SPACED) {
        const int d = max(J.geom & 0xff, 1), lgo = (J.geom >> 16) & 0xf;
        if constexpr (KIND == SK_GROUP) {
          const int h = d >> 1;
          py += (wmem >> 1) * h;  // member (a, b) = (wmem / 2, wmem % 2): phase (gy + a h, gx + b h)
          px += (wmem & 1) * h;
        }
        gbyte* o[C::MW];
        bool ok[C::MW];
#pragma unroll
        for (int u = 0; u < C::MW; ++u) {
          const int y = py + d * (y0 + wrow0 + u / MCOLS), x = px + d * (x0 + (u % MCOLS) * 16 + n16);
          ok[u] = y < J.hout && x < J.wout;
          o[u] = gout(J.out) + ((int64_t)zz * J.out_zs + frag_pix(y, x, lgo, J.out_rs, J.out_zs)) * (COUT * 2);
        }
        // a pair of n-blocks at a time (all biases and scales at once would spill)
#pragma unroll
        for (int nb = 0; nb < C::NB; nb += 2) {
          const int at = split_chan(nb, 4 * g, C::NB, true) * 2;
#pragma unroll
          for (int u = 0; u < C::MW; ++u) {
            const f4 p = value(acc[u][nb], nb);
            if (nb + 1 < C::NB) {
              const f4 q = value(acc[u][nb + 1 < C::NB ? nb + 1 : nb], nb + 1 < C::NB ? nb + 1 : nb);
              if (ok[u])
                st<f4>(o[u] + at, f4{fmaxf(p[0], p[1]), fmaxf(p[2], p[3]), fmaxf(q[0], q[1]), fmaxf(q[2], q[3])});
            } else if (ok[u]) {
              st<f2>(o[u] + at, f2{fmaxf(p[0], p[1]), fmaxf(p[2], p[3])});
            }
          }
          if constexpr (!PRE) __builtin_amdgcn_sched_barrier(0);
        }
      } else {
#pragma unroll
        for (int u = 0; u < C::MW; ++u) {
          const int y = y0 + wrow0 + u / MCOLS, x = x0 + (u % MCOLS) * 16 + n16;
          if (y < J.hout && x < J.wout) {
            gbyte* o = gout(J.out) + ((int64_t)zz * J.out_zs + (int64_t)y * J.out_rs + x) * (COUT * 4) + g * 16;
#pragma unroll
            for (int nb = 0; nb < C::NB; ++nb) {
              f4 t = value(acc[u][nb], nb);
#pragma unroll
              for (int k = 0; k < 4; ++k) t[k] = relu(t[k]);
              st<f4>(o + nb * 64, t);
            }
          }
        }
      }
    }
  };

  __syncthreads();  // stage 0, slice 0 ready
  for (;;) {
    if (cb == 0) {
#pragma unroll
      for (int u = 0; u < C::MW; ++u)
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb) acc[u][nb] = f4{0.f, 0.f, 0.f, 0.f};
    }
    const unsigned char* abase = lds + sel * C::BUF + (lrow0 * C::LC + n16) * C::PSB;
#pragma unroll
    for (int p = 0; p < C::NSL; ++p) {
      const unsigned char* wl = lds + C::WOFF + wsel * C::SLB + lane * 16;
#pragma unroll
      for (int e = 0; e < SS; ++e)
        if (p * SS + e < C::NGS) step(abase, wl + e * C::STEPB, p * SS + e);
      wsel ^= 1;
      if (p + 1 == C::NSL && cb == C::NCB - 1) epilogue();
      __syncthreads();  // slice done; the next one is ready
    }
    sel ^= 1;
    if (++cb == C::NCB) {
      cb = 0;
      if (!w.next_open(js)) return;
    }
  }
}

// ---------------------------------------------------------------- registry

#define EMCNN_SPLITN(NAME, CIN, COUT, KS, POOL, KIND, TY, TX, NCW, NPW, CB, SS, NP, LONE, RATE)           \
  VariantInfo{F32, CIN, COUT, KS, KIND >= SK_PHASE ? 1 : POOL, KIND == SK_HEAD, TY, TX,                    \
              CfgSplit<CIN, COUT, KS, KIND, TY, TX, NCW, NPW, CB, SS, NP>::MW,                             \
              CfgSplit<CIN, COUT, KS, KIND, TY, TX, NCW, NPW, CB, SS, NP>::THREADS, CB, 8, 1,              \
              CfgSplit<CIN, COUT, KS, KIND, TY, TX, NCW, NPW, CB, SS, NP>::NSL * SS, 0, 0,                 \
              KIND >= SK_PHASE ? 1 : 0, CfgSplit<CIN, COUT, KS, KIND, TY, TX, NCW, NPW, CB, SS, NP>::LDS,  \
              reinterpret_cast<const void*>(&conv_split<CIN, COUT, KS, POOL, KIND, TY, TX, NCW, NPW, CB, SS, NP>), \
              NAME, 0, KIND == SK_GROUP, KIND >= SK_PHASE ? 2 : 1, TileCost{LONE, RATE}, NP}
#define EMCNN_SPLIT(CIN, COUT, KS, POOL, HEAD, TY, TX, NCW, NPW, CB, SS, LONE, RATE)                       \
  EMCNN_SPLITN("conv_split<" #CIN "," #COUT "," #KS "," #POOL "," #HEAD "," #TY "," #TX "," #NCW "," #NPW "," #CB \
               "," #SS ">",                                                                                 \
               CIN, COUT, KS, POOL, (HEAD ? SK_HEAD : SK_RELU), TY, TX, NCW, NPW, CB, SS, 2, LONE, RATE)
#define EMCNN_SPLIT_PHASE(CIN, COUT, KS, POOL, TY, TX, NCW, NPW, CB, SS, LONE, RATE)                        \
  EMCNN_SPLITN("conv_phase<F32S," #CIN "," #COUT "," #KS "," #POOL "," #TY "," #TX "," #NCW "," #NPW "," #CB "," #SS \
               ">",                                                                                         \
               CIN, COUT, KS, POOL, SK_PHASE, TY, TX, NCW, NPW, CB, SS, 2, LONE, RATE)
#define EMCNN_SPLIT_GROUP(CIN, COUT, KS, TY, NCW, NPW, CB, SS, LONE, RATE)                                  \
  EMCNN_SPLITN("conv_phase_group<F32S," #CIN "," #COUT "," #KS "," #TY "," #NCW "," #NPW "," #CB "," #SS ">", \
               CIN, COUT, KS, true, SK_GROUP, TY, 16, NCW, NPW, CB, SS, 2, LONE, RATE)
// the same over bf16 triples
#define EMCNN_SPLIT3_PHASE(CIN, COUT, KS, POOL, TY, TX, NCW, NPW, CB, SS, LONE, RATE)                       \
  EMCNN_SPLITN("conv_phase<F32S,3xbf16," #CIN "," #COUT "," #KS "," #POOL "," #TY "," #TX "," #NCW "," #NPW "," #CB \
               "," #SS ">",                                                                                 \
               CIN, COUT, KS, POOL, SK_PHASE, TY, TX, NCW, NPW, CB, SS, 3, LONE, RATE)
#define EMCNN_SPLIT3_GROUP(CIN, COUT, KS, TY, NCW, NPW, CB, SS, LONE, RATE)                                 \
  EMCNN_SPLITN("conv_phase_group<F32S,3xbf16," #CIN "," #COUT "," #KS "," #TY "," #NCW "," #NPW "," #CB "," #SS ">", \
               CIN, COUT, KS, true, SK_GROUP, TY, 16, NCW, NPW, CB, SS, 3, LONE, RATE)

// First entry per signature: the default; last two arguments its TileCost. All shapes of a signature contract in
// the same order (16-channel stages), so their outputs are bitwise the same.
// Against the FP32 kernels, on 32 x 1024^2 (net B) and 8 x 1024^2 (FastMemb):
// conv2 28.2 -> 8.6 ms (1.33 PFLOP/s of f16 products, 98 % of them useful),
// conv3 11.2 -> 3.5 ms, FastMemb's body convs 4.4 -> 1.28 ms each.
static const VariantInfo kSplit[] = {
    // net B conv2: 24 x 32 tiles, 6 m-blocks per consumer wave (8.6 ms on
    // 32 x 1024^2; 16 x 32 8.8, 8 x 32 9.9, 8 x 16 12.9)
    EMCNN_SPLIT(48, 48, 5, true, false, 24, 32, 8, 4, 16, 2, 45, 50),
    EMCNN_SPLIT(48, 48, 5, true, false, 16, 32, 8, 4, 16, 3, 31, 34.3),
    EMCNN_SPLIT(48, 48, 5, true, false, 8, 32, 8, 4, 16, 4, 20, 19.5),
    EMCNN_SPLIT(48, 48, 5, true, false, 8, 16, 8, 4, 16, 4, 14, 12.7),
    // net B conv3 and head (3.5 ms; 16 x 32 3.6, 8 x 32 4.1, 8 x 16 5.6; the
    // whole stage's weights as one slice of 5 steps spills at 16 x 32, 7.0 ms)
    EMCNN_SPLIT(48, 48, 3, true, true, 16, 48, 8, 4, 16, 3, 19, 20),
    EMCNN_SPLIT(48, 48, 3, true, true, 16, 32, 8, 4, 16, 3, 14.5, 13.9),
    EMCNN_SPLIT(48, 48, 3, true, true, 8, 32, 8, 4, 16, 5, 9.8, 8.1),
    EMCNN_SPLIT(48, 48, 3, true, true, 8, 16, 8, 4, 16, 5, 6.5, 5.5),
    // net A conv2 and head (0.30 ms on 8 x 1024^2; 8 x 16 0.50)
    EMCNN_SPLIT(16, 16, 5, false, true, 16, 32, 8, 4, 16, 7, 6.5, 4.7),
    EMCNN_SPLIT(16, 16, 5, false, true, 8, 16, 8, 4, 16, 13, 3, 1.95),
    // FastMemb and FastMemb_ss body convs: over phase groups (1.28 ms; 12-row
    // members 1.27-1.29, 4-row ones 1.56), per phase 1.32 (8 x 32 1.53)
    EMCNN_SPLIT_GROUP(32, 64, 4, 8, 8, 4, 16, 2, 20, 20), EMCNN_SPLIT_GROUP(32, 64, 4, 12, 8, 4, 16, 1, 28, 29.8),
    EMCNN_SPLIT_GROUP(32, 64, 4, 4, 8, 4, 16, 2, 13, 12.3),
    EMCNN_SPLIT_PHASE(32, 64, 4, true, 16, 32, 8, 4, 16, 2, 21.5, 20.6),
    EMCNN_SPLIT_PHASE(32, 64, 4, true, 8, 32, 8, 4, 16, 2, 13, 12),
    // MaskExtend, on bf16 triples. ms on 2 x 512 x 600 and 4 x 800^2 maps (f16 pairs, for
    // whose scales real-valued maps have no bound; the FP32 kernels):
    //   12 -> 64, no max filter   0.10 and 0.41 (0.07 and 0.30; 0.14 and 0.62)
    //   32 -> 80                  0.23 and 0.91 (0.18 and 0.58; 0.53 and 2.30), 4-row members 0.23 and 0.96
    //   40 -> 96                  0.29 and 1.38 (0.21 and 0.81; 0.66 and 3.16), 4-row members 0.29 and 1.38
    //   48 -> 112                 0.44 and 1.71 (0.30 and 1.02; 0.94 and 3.74), 6-row members 10 % slower
    //   56 -> 128                 0.42 and 2.07 (0.24 and 1.32; 0.89 and 4.63), 6-row members 27 % slower
    // In 8-channel stages: 16-channel ones leave room for one weight slice per barrier
    // (32 -> 80 2 % slower, 48 -> 112 4 %). Taller members spill: 3 x 4 registers of
    // weights and of each m-block's pixels beside the accumulators.
    EMCNN_SPLIT3_PHASE(12, 64, 4, false, 24, 16, 8, 4, 16, 1, 15, 15.4),
    EMCNN_SPLIT3_PHASE(12, 64, 4, false, 8, 32, 8, 4, 16, 1, 10.5, 10.9),
    EMCNN_SPLIT3_GROUP(32, 80, 4, 6, 8, 4, 8, 2, 34, 35.3), EMCNN_SPLIT3_GROUP(32, 80, 4, 4, 8, 4, 8, 2, 24, 24.9),
    EMCNN_SPLIT3_GROUP(40, 96, 4, 6, 8, 4, 8, 1, 50, 51.5), EMCNN_SPLIT3_GROUP(40, 96, 4, 4, 8, 4, 8, 2, 33.5, 34.7),
    EMCNN_SPLIT3_GROUP(48, 112, 4, 4, 8, 4, 8, 2, 0, 0), EMCNN_SPLIT3_GROUP(56, 128, 4, 4, 8, 4, 8, 2, 0, 0),
};

int split_variant_count() { return (int)(sizeof(kSplit) / sizeof(kSplit[0])); }
const VariantInfo* split_variant(int i) { return &kSplit[i]; }

}  // namespace emcnn
