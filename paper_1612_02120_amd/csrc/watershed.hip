// 3-D watershed of a membrane probability map (Section 2.1: the stage after
// membrane classification turns the map into an over-segmentation with a 3-D
// watershed). Watershed by steepest descent with seeded minima:
//   order   u < v iff p[u] < p[v], or p[u] == p[v] and index(u) < index(v)
//   seeds   S = { v : p[v] < t }, its 6-connected components labelled
//           1 + the least index in each
//   descent next(v) = v on S, else the least of v and its 6-neighbours
//   label   of v: the seed component's label where the descent from v ends
//           in S, else 1 + the index of the local minimum it ends at.
// The result is unique (a total order, no flooding order to choose), so the
// kernels reproduce it exactly whatever the scheduling. One forest a[] holds
// both parts: a non-seed points along its descent, a seed into its
// component's tree. Roots are fixed points: component minima and non-seed
// local minima.
//   ws_tile   a workgroup per tile of 4 x 8 x 128 voxels, its forest in LDS. A seed
//             points to the first seed of its run along x in the tile, any other
//             voxel to next(v); runs adjacent along y or z in the tile are united
//             by a lock-free union-find (the structure of ECL-CC): find both
//             roots, hook the larger root under the smaller with a
//             compare-and-swap that only succeeds while it is still a root, and
//             retry from the new roots when another thread hooked it first. Then
//             every voxel follows its parents as far as the tile goes, and a[]
//             takes where it got: its tile component's least voxel, a local
//             minimum, or the voxel of another tile that its descent goes on at.
//   ws_border the same union-find on a[] for seeds that touch across the faces of
//             tiles. Of touching pairs that are linked anyway through their
//             neighbours' pair (one column left, one row up) one is united.
//   ws_label  every voxel follows its parents to its root r, and takes r + 1.
// A seed's parent index only decreases, so every component ends rooted at its
// least index. Path halving points a node at its grandparent, an ancestor in the
// same tree, so concurrent finds stay valid; it never writes a root.
//
// A wave works on rows, four consecutive columns to a lane, as one 16-byte access
// where rows and pointers allow it. On a 32 x 1012^2 membrane map
// with seeds below 0.05 (44 % of the voxels): ws_tile 173 us (reading, links and
// writing 93, unions 43, walks 40), ws_border 57, ws_label 109. With the whole forest
// in memory, links, unions, the flattening of runs and walks to the root were passes
// of 90, 220-234, 55 and 227 us; a step of a walk costs a trip to the L2 or the memory
// there, and every union is one of 1.4 M compare-and-swaps, on one address where a
// volume is one component (2 M voxels: 350 us per call, in tiles 69).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "../../include/emcnn.h"
#include "device_util.h"
#include "runtime.h"

namespace emcnn {

struct Vol3 {
  int Z, H, W;
  int64_t N;
};

// Parents while other threads may be changing them, read through the caches: an
// older value is an ancestor all the same, and a root that has been hooked since
// shows in the compare-and-swap, whose answer the walk goes on from. (Past the
// caches, the root of a large component is one address that every find of every
// CU waits for: unions over a whole forest in memory took 268 us there, 217-234 here.)
__device__ __forceinline__ int32_t wa(const int32_t* a, int64_t v) {
  return __hip_atomic_load(a + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

typedef int32_t i4 __attribute__((ext_vector_type(4)));

// Four values at v .. v + 3 of a row that holds n of them (the others read as 0).
// VEC: rows and pointers are 16-byte aligned, so all four are there or none.
template <bool VEC>
__device__ __forceinline__ f4 row4(const float* p, int v, int n) {
  if constexpr (VEC) {
    return n > 0 ? ld<f4>(gin(p) + (int64_t)v * 4) : f4{0.f, 0.f, 0.f, 0.f};
  } else {
    f4 r;
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = k < n ? ld<float>(gin(p) + ((int64_t)v + k) * 4) : 0.f;
    return r;
  }
}

// Bits k < n with q[k] < t.
__device__ __forceinline__ unsigned below4(f4 q, int n, float t) {
  unsigned m = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) m |= (k < n && q[k] < t) ? 1u << k : 0u;
  return m;
}

// Columns per step of a wave.
constexpr int WC = 256;

// body(row) for the rows of this wave: groups of four rows, one per wave of a
// workgroup, dealt out so that consecutive groups run on the same XCD (workgroup
// b on XCD b % 8) and its L2 serves the rows that neighbours share.
template <class Body>
__device__ __forceinline__ void wave_rows(unsigned nrow, Body body) {
  const unsigned per = ((nrow + 3) / 4 + 7) / 8;  // groups per XCD (nrow < 2^31)
  for (unsigned k = blockIdx.x >> 3; k < per; k += gridDim.x >> 3) {
    const unsigned row = ((blockIdx.x & 7) * per + k) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (row < nrow) body((int)row);
  }
}

// Bits of m whose left neighbour's bit is clear, in rows of 32 lanes: the first
// columns of m's runs.
__device__ __forceinline__ unsigned half_starts(unsigned m, int l32) {
  const unsigned left = (unsigned)__shfl_up((int)(m >> 3), 1);
  return m & ~((m << 1) | (l32 ? left : 0u));
}

// ---- tiles
// LDS answers a step of a walk in a tenth of the time of the caches, and a tile of 4 x
// 8 x 128 leaves to ws_border a quarter of the contacts along z, an eighth along y and
// the ends along x. us on 32 x 1012^2 (tile, border, label) and on 2^20 voxels in all:
// 4 x 8 rows 173, 59, 109 and 35; 4 x 16 197, 50, 103 and 45; 2 x 8 175, 89, 134 and
// 32; 2 x 16 172, 77, 127 and 35; 4 x 4 179, 79, 122 and 34.
constexpr int TX = 128;

// parents in LDS, as ws_find and ws_unite below
__device__ __forceinline__ int lp(const int* par, int l) {
  return __hip_atomic_load(par + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ int tile_find(int* par, int r) {
  int up = lp(par, r);
  while (up != r) {
    const int gp = lp(par, up);
    if (gp == up) return up;
    __hip_atomic_store(par + r, gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    r = gp;
    up = lp(par, r);
  }
  return r;
}
__device__ __forceinline__ void tile_unite(int* par, int u, int v) {
  int ru = tile_find(par, u), rv = tile_find(par, v);
  while (ru != rv) {
    const int hi = ru > rv ? ru : rv, lo = ru < rv ? ru : rv;
    int old = hi;
    if (__hip_atomic_compare_exchange_strong(par + hi, &old, lo, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP))
      return;
    ru = tile_find(par, old);
    rv = lo;
  }
}

template <bool VEC, int TZ, int TY>
__global__ __launch_bounds__(512) void ws_tile(const float* __restrict__ p, Vol3 g, float t, int32_t* __restrict__ a,
                                               unsigned ntz, unsigned ntx, unsigned ntiles) {
  constexpr int STEPS = TZ * TY / 16;  // of 16 rows, two per wave
  static_assert(TZ * TY == 16 * STEPS && STEPS <= 4, "whole steps; four fill the masks below");
  __shared__ __attribute__((aligned(16))) int par[TX * TY * TZ];  // >= 0: a voxel of the tile; else ~ one outside it
  // consecutive tiles (along z, then x, then y: the largest shared faces first) on the
  // same XCD (workgroup b on XCD b % 8), whose L2 serves the rows that neighbours share
  const unsigned tile = blockIdx.y * gridDim.x + (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (tile >= ntiles) return;
  const int z0 = (int)(tile % ntz) * TZ, x0 = (int)(tile / ntz % ntx) * TX, y0 = (int)(tile / (ntz * ntx)) * TY;
  const int HW = g.H * g.W, lane = threadIdx.x & 63, l32 = lane & 31;
  const int base = (z0 * g.H + y0) * g.W + x0;
  const int x = x0 + 4 * l32;
  // step s of wave w: two rows of the tile, lanes 0..31 and lanes 32..63
  const int row0 = (int)(threadIdx.x >> 6) * 2 * STEPS + (lane >> 5);
  unsigned touch = 0, first = 0;  // per step: columns to unite along y, along z; first columns of runs
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int r = row0 + 2 * s, lz = r / TY, ly = r % TY, z = z0 + lz, y = y0 + ly;
    const int n = z < g.Z && y < g.H ? min(max(g.W - x, 0), 4) : 0;
    const int v = n ? base + lz * HW + ly * g.W + 4 * l32 : 0, l = r * TX + 4 * l32;
    const f4 q = row4<VEC>(p, v, n);
    const f4 zm = row4<VEC>(p, v - HW, z > 0 ? n : 0), zp = row4<VEC>(p, v + HW, z < g.Z - 1 ? n : 0);
    const f4 ym = row4<VEC>(p, v - g.W, y > 0 ? n : 0), yp = row4<VEC>(p, v + g.W, y < g.H - 1 ? n : 0);
    float left = __shfl_up(q[3], 1), right = __shfl_down(q[0], 1);
    if (l32 == 0 && n && x > 0) left = ld<float>(gin(p) + ((int64_t)v - 1) * 4);
    if (l32 == 31 && n && x + 4 < g.W) right = ld<float>(gin(p) + ((int64_t)v + 4) * 4);
    const unsigned m = below4(q, n, t);
    // the last column before this lane's that is no seed (columns past the row count as none)
    const int last = m == 15u ? -1 : 4 * l32 + 31 - __builtin_clz(~m & 15u);
    const uint64_t brk = __ballot(m != 15u);
    const unsigned before = (unsigned)(brk >> (lane & 32)) & ((1u << l32) - 1);
    const int from = __shfl(last, (lane & 32) + (before ? 31 - __builtin_clz(before) : 0));
    int lb = before ? from : -1;
    i4 up;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (m >> k & 1) {
        up[k] = r * TX + lb + 1;  // the run's first seed
        continue;
      }
      lb = 4 * l32 + k;
      const int self = l + k;
      int best = self;
      float pb = q[k];
      // candidates in ascending index order: an equal one wins only over v itself, from
      // before v; one of another tile is held as ~ its index
      auto cand = [&](bool there, bool lower, float pu, bool inside, int lu, int u) __attribute__((always_inline)) {
        const bool take = there && (pu < pb || (lower && pu == pb && best == self));
        pb = take ? pu : pb;
        best = take ? (inside ? lu : ~u) : best;
      };
      cand(z > 0, true, zm[k], lz > 0, self - TY * TX, v + k - HW);
      cand(y > 0, true, ym[k], ly > 0, self - TX, v + k - g.W);
      cand(x + k > 0, true, k > 0 ? q[k > 0 ? k - 1 : 0] : left, k > 0 || l32 > 0, self - 1, v + k - 1);
      cand(x + k < g.W - 1, false, k < 3 ? q[k < 3 ? k + 1 : 3] : right, k < 3 || l32 < 31, self + 1, v + k + 1);
      cand(y < g.H - 1, false, yp[k], ly < TY - 1, self + TX, v + k + g.W);
      cand(z < g.Z - 1, false, zp[k], lz < TZ - 1, self + TY * TX, v + k + HW);
      up[k] = best;
    }
    *reinterpret_cast<i4*>(par + l) = up;
    // first columns where the run of this row touches one of the next row / slice of the tile
    const unsigned my = ly < TY - 1 && y < g.H - 1 ? m & below4(yp, n, t) : 0u;
    const unsigned mz = lz < TZ - 1 && z < g.Z - 1 ? m & below4(zp, n, t) : 0u;
    touch |= (half_starts(my, l32) | half_starts(mz, l32) << 4) << 8 * s;
    first |= half_starts(m, l32) << 4 * s;
  }
  __syncthreads();
  for (unsigned b = touch; b; b &= b - 1) {
    const int i = __builtin_ctz(b), l = (row0 + 2 * (i >> 3)) * TX + 4 * l32 + (i & 3);
    tile_unite(par, l, l + (i & 4 ? TY * TX : TX));
  }
  __syncthreads();
  for (unsigned b = first; b; b &= b - 1) {
    const int i = __builtin_ctz(b), l = (row0 + 2 * (i >> 2)) * TX + 4 * l32 + (i & 3);
    const int r = tile_find(par, l);
    __hip_atomic_store(par + l, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int r = row0 + 2 * s, lz = r / TY, ly = r % TY;
    const int n = z0 + lz < g.Z && y0 + ly < g.H ? min(max(g.W - x, 0), 4) : 0;
    if (n == 0) continue;
    const int l = r * TX + 4 * l32;
    i4 c = {l, l + 1, l + 2, l + 3}, up = *reinterpret_cast<const i4*>(par + l);
#pragma unroll
    for (int k = 1; k < 4; ++k) up[k] = k < n ? up[k] : c[k];
    // the four walks step together
    auto open = [&](int k) __attribute__((always_inline)) { return up[k] >= 0 && up[k] != c[k]; };
    while (open(0) || open(1) || open(2) || open(3)) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool o = open(k);
        c[k] = o ? up[k] : c[k];
        up[k] = o ? par[c[k]] : up[k];
      }
    }
    i4 out;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      out[k] = up[k] < 0 ? ~up[k] : base + c[k] / (TY * TX) * HW + c[k] / TX % TY * g.W + c[k] % TX;
    const int64_t v = base + lz * HW + ly * g.W + 4 * l32;
    if constexpr (VEC) {
      st<i4>(gout(a) + v * 4, out);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < n) st<int32_t>(gout(a) + (v + k) * 4, out[k]);
    }
  }
}

// ---- across tiles
// Root of r with path halving (any node may be passed; roots are fixed points).
__device__ __forceinline__ int32_t ws_find(int32_t* a, int32_t r) {
  int32_t par = wa(a, r);
  while (par != r) {
    if (par < 0) return ~par;  // ws_label has written the root here
    const int32_t gp = wa(a, par);
    if (gp == par) return par;
    if (gp < 0) return ~gp;
    // r is not a root: an ancestor is a valid parent
    __hip_atomic_store(a + r, gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    r = gp;
    par = wa(a, r);
  }
  return r;
}

// The larger root may have been hooked since the caches saw it: a fresh look at it
// costs a load, where a compare-and-swap that fails is one more on an address that
// many threads may be at (465 -> 388 us on a map whose seeds are many small runs,
// 333 -> 324 on one with fewer and longer ones, both 32 x 1012^2).
__device__ __forceinline__ void ws_unite(int32_t* a, int32_t u, int32_t v) {
  int32_t ru = ws_find(a, u), rv = ws_find(a, v);
  while (ru != rv) {
    const int32_t hi = ru > rv ? ru : rv, lo = ru < rv ? ru : rv;
    int32_t old = __hip_atomic_load(a + hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == hi) {
      old = atomicCAS(a + hi, hi, lo);
      if (old == hi) return;  // hooked while hi was still a root
    }
    // hi had been hooked (under old < hi): continue from there
    ru = ws_find(a, old);
    rv = lo;
  }
}

// Bits of m whose left neighbour's bit is clear: the first columns of m's runs.
// prev: the bit left of the wave's step (updated to its last one).
__device__ __forceinline__ unsigned run_starts(unsigned m, int lane, unsigned& prev) {
  unsigned left = (unsigned)__shfl_up((int)(m >> 3), 1);
  if (lane == 0) left = prev;
  prev = (unsigned)__shfl((int)(m >> 3), 63);
  return m & ~((m << 1) | left);
}

// Finds are chains of dependent loads, and the columns that start one are sparse
// (a few per wave and step), so a wave queues them in LDS and works them off 64 at
// a time.
constexpr int WQCAP = 64 + 2 * WC;
struct WaveQueue {
  int* q;
  int n = 0;  // uniform
  int lane;
  // queue e of the lanes with `there` (at most 64 at a time)
  __device__ __forceinline__ void push(bool there, int e) {
    const uint64_t b = __ballot(there);
    if (there) q[n + __builtin_popcountll(b & ((1ull << lane) - 1))] = e;
    n += __builtin_popcountll(b);
  }
  // work(e) on the last 64 entries while there are that many (all: on every entry)
  template <class Work>
  __device__ __forceinline__ void drain(bool all, Work work) {
    while (n >= 64 || (all && n > 0)) {
      const int k = min(n, 64);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int e = lane < k ? q[n - k + lane] : 0;
      if (lane < k) work(e);
      n -= k;
      __builtin_amdgcn_wave_barrier();
    }
  }
};

// Contacts across the faces of tiles. A pair of touching voxels needs no union
// where a neighbouring pair is united and the links between the two pairs are made
// without this pair's: across y, the pair one column left; across z, the pair one
// column left or one row up; across x, the pair one row up in the same tiles (the
// links along y inside a tile, whose runs start at its edge, need none across x).
template <bool VEC, int TZ, int TY>
__global__ __launch_bounds__(256) void ws_border(const float* __restrict__ p, Vol3 g, float t, int32_t* a) {
  __shared__ int queue[4][WQCAP];
  const int HW = g.H * g.W, lane = threadIdx.x & 63;
  WaveQueue wq{queue[threadIdx.x >> 6], 0, lane};
  // entry v: unite v with the voxel below it; ~v: with the one in the next slice
  auto work = [&](int e) __attribute__((always_inline)) {
    const int v = e < 0 ? ~e : e;
    ws_unite(a, v, e < 0 ? v + HW : v + g.W);
  };
  wave_rows((unsigned)(g.Z * g.H), [&](int row) __attribute__((always_inline)) {
    const int z = row / g.H, y = row - z * g.H, base = row * g.W;
    const bool fy = y % TY == TY - 1 && y < g.H - 1, fz = z % TZ == TZ - 1 && z < g.Z - 1;
    const bool up = fz && y > 0;
    if (fy || fz) {
      unsigned prevy = 0, prevz = 0;
      for (int x0 = 0; x0 < g.W; x0 += WC) {
        const int x = x0 + 4 * lane, v = base + x, n = min(max(g.W - x, 0), 4);
        const f4 q = row4<VEC>(p, v, n), qy = row4<VEC>(p, v + g.W, fy ? n : 0), qz = row4<VEC>(p, v + HW, fz ? n : 0);
        const f4 qu = row4<VEC>(p, v - g.W, up ? n : 0), qzu = row4<VEC>(p, v + HW - g.W, up ? n : 0);
        const unsigned m = below4(q, n, t);
        const unsigned my = m & below4(qy, fy ? n : 0, t), mz = m & below4(qz, fz ? n : 0, t);
        const unsigned sy = run_starts(my, lane, prevy);
        const unsigned sz = run_starts(mz, lane, prevz) & ~(below4(qu, up ? n : 0, t) & below4(qzu, up ? n : 0, t));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          wq.push(sy >> k & 1, v + k);
          wq.push(sz >> k & 1, ~(v + k));
        }
        wq.drain(false, work);
      }
    }
    for (int x0 = TX; x0 < g.W; x0 += 64 * TX) {
      const int64_t x = x0 + (int64_t)lane * TX;
      if (x >= g.W) continue;
      auto both = [&](int64_t v) __attribute__((always_inline)) {
        return ld<float>(gin(p) + v * 4) < t && ld<float>(gin(p) + (v - 1) * 4) < t;
      };
      const int64_t v = base + x;
      if (both(v) && !(y % TY != 0 && both(v - g.W))) ws_unite(a, (int32_t)v, (int32_t)v - 1);
    }
  });
  wq.drain(true, work);
}

// Parents followed before a walk goes on with writes. Walks are short here (a
// tile's component, the components it was hooked under; the tiles of a descent), and
// writes from every voxel cost more than they save; a component whose tree is deep
// all the same gets its paths halved, and its root's complement, which ends a walk,
// where the walk was after these steps.
constexpr int kPlainSteps = 16;

template <bool VEC>
__global__ __launch_bounds__(256) void ws_label(Vol3 g, int32_t* a, int32_t* out) {
  const gbyte* ab = gin(a);
  const int64_t v = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (v >= g.N) return;
  i4 r, par;
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = (int32_t)(VEC ? v + k : min(v + k, g.N - 1));
  if constexpr (VEC) {
    par = ld<i4>(ab + v * 4);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) par[k] = wa(a, r[k]);
  }
  // the four walks step together, so that their loads overlap
  auto open = [&](int k) __attribute__((always_inline)) { return par[k] >= 0 && par[k] != r[k]; };
  for (int i = 0; i < kPlainSteps && (open(0) || open(1) || open(2) || open(3)); ++i) {
    i4 nx;
#pragma unroll
    for (int k = 0; k < 4; ++k) nx[k] = open(k) ? wa(a, par[k]) : par[k];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      r[k] = open(k) ? par[k] : r[k];
      par[k] = nx[k];
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (open(k)) {
      const int32_t root = ws_find(a, par[k]);
      // (r is no root, and its complement is only ever read as the end of a walk)
      __hip_atomic_store(a + r[k], ~root, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      par[k] = ~root;
    }
    r[k] = (par[k] < 0 ? ~par[k] : r[k]) + 1;
  }
  if constexpr (VEC) {
    st<i4>(gout(out) + v * 4, r);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (v + k < g.N) st<int32_t>(gout(out) + (v + k) * 4, r[k]);
  }
}

// Voxels up to which tiles of 2 x 8 rows are taken: a step of a wave less, twice the
// workgroups (us with 2 x 8 against 4 x 8 rows: 25.6 against 30.7 on 2^19 voxels, 32 against
// 35 on 2^20, 48-50 against 46 on 1.2 M, 62 against 60 on 2^22). Single slices take them
// too, though they leave three quarters of a tile empty: 100 us on 1100^2, 342 on 4096^2
// (134 and 860 with rows as waves and all links in memory).
constexpr int64_t kSmall = 1 << 20;

template <bool VEC, int TZ, int TY>
static hipError_t ws_run(const float* p, const Vol3& g, float t, int32_t* labels, int32_t* work, hipStream_t st) {
  const int64_t ntz = (g.Z + TZ - 1) / TZ, ntx = (g.W + TX - 1) / TX, nty = (g.H + TY - 1) / TY, nt = ntz * ntx * nty;
  const int64_t groups = ((int64_t)g.Z * g.H + 3) / 4;  // of four rows
  // grids in multiples of 8, one share per XCD; ws_border runs persistent waves, which keep their queues filled.
  // Thin volumes have more tiles than a row of the grid may hold threads for (2^32): then in several rows
  const int64_t gx = std::min<int64_t>((nt + 7) / 8 * 8, 1 << 20);
  hipLaunchKernelGGL((ws_tile<VEC, TZ, TY>), dim3((unsigned)gx, (unsigned)((nt + gx - 1) / gx)), dim3(512), 0, st, p, g, t,
                     work, (unsigned)ntz, (unsigned)ntx, (unsigned)nt);
  hipLaunchKernelGGL((ws_border<VEC, TZ, TY>), dim3((unsigned)std::min<int64_t>((groups + 7) / 8 * 8, 2048)), dim3(256), 0,
                     st, p, g, t, work);
  hipLaunchKernelGGL(ws_label<VEC>, dim3((unsigned)((g.N + 1023) / 1024)), dim3(256), 0, st, g, work, labels);
  return hipGetLastError();
}

}  // namespace emcnn

using namespace emcnn;

extern "C" int watershed_3d(const float* prob, const int64_t dims[3], float seed_threshold, int32_t* labels_out,
                            int32_t* work, void* stream) {
  clear_error();
  if (!prob || !dims || !labels_out || !work) return fail(CNN_EINVAL, "watershed_3d: null argument");
  int64_t Z = dims[0], H = dims[1], W = dims[2];
  if (Z < 1 || H < 1 || W < 1 || Z > (1 << 30) || H > (1 << 30) || W > (1 << 30) || Z * H * W >= 2147483647ll)
    return fail(CNN_EINVAL, "watershed_3d: dims must be >= 1 with Z H W < 2^31 - 1");
  if (seed_threshold != seed_threshold) return fail(CNN_EINVAL, "watershed_3d: NaN threshold");
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  // Sides of one voxel come first: neither a voxel's index nor its neighbours change, and a
  // tile's 128 columns lie along a side that has some (us on 1.2 M voxels in all: 1 x N x 1
  // 1650 -> 327, N x 1 x 1 2610 -> 327).
  for (int k = 0; k < 2 && W == 1; ++k) {
    W = H;
    H = Z;
    Z = 1;
  }
  if (H == 1) {
    H = Z;
    Z = 1;
  }
  Vol3 g{(int)Z, (int)H, (int)W, Z * H * W};
  // 16-byte accesses where every row starts at one
  const bool vec = W % 4 == 0 && ((uintptr_t)prob | (uintptr_t)work | (uintptr_t)labels_out) % 16 == 0;
  const bool small = g.N <= kSmall;
  const auto run = vec ? (small ? ws_run<true, 2, 8> : ws_run<true, 4, 8>)
                       : (small ? ws_run<false, 2, 8> : ws_run<false, 4, 8>);
  const hipError_t e = run(prob, g, seed_threshold, labels_out, work, st);
  if (e != hipSuccess) return hip_fail(e, "watershed_3d");
  return CNN_OK;
}
