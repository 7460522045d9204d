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
//   ws_init   one pass: a seed points to the first seed of its run along x
//             (the run's least index), any other voxel to next(v). The x-links
//             of the seed graph are then made.
//   ws_union  one pass over the seeds: runs adjacent along y or z are united
//             by a lock-free union-find (the structure of ECL-CC): find both
//             roots, hook the larger root under the smaller with a
//             compare-and-swap that only succeeds while it is still a root,
//             and retry from the new roots when another thread hooked it
//             first. Two runs that touch are united once, at the first column
//             where they do (the pair one column left, when both are seeds,
//             joins the same two runs). A seed's parent index only
//             decreases, so every component ends rooted at its least index.
//   ws_flat   every run's first seed finds its component's root r, halving the
//             path as it goes, and takes ~r, which ends a walk.
//   ws_label  every voxel follows its parents to a run's ~r (a seed in two
//             steps, a non-seed after its descent) or to a local minimum r, and
//             takes r + 1. Nothing changes the forest any more.
// Path halving points a node at its grandparent, an ancestor in the same
// tree, so concurrent finds stay valid; it never writes a root.
//
// Every kernel gives a row to a wave, four consecutive columns to a lane, as one
// 16-byte access where rows and pointers allow it. On a 32 x 1012^2 membrane map
// with seeds below 0.05 (44 % of the voxels): ws_init 90 us, ws_union 220-234, ws_flat
// 55, ws_label 227; 1.57 ms in all when a row was a workgroup, one column a
// thread, and ws_label halved paths from every voxel (ws_init 228, ws_union 392,
// ws_label 944 us). ws_init moves 0.26 GB, the rate of a large copy; the other
// passes are chains of dependent loads and, in ws_union, 1.4 M compare-and-swaps.
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
// CU waits for: ws_union 268 us there, 217-234 here, and 259 against 111-128 on a
// volume of 2 M voxels in one component.)
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

// Columns per step of a wave.
constexpr int WC = 256;

// The last non-seed column before this lane's columns x .. x + 3 (m: which of
// them are seeds); carry: the last one before the wave's step, updated.
__device__ __forceinline__ int break_before(unsigned m, int x, int lane, int& carry) {
  // the last non-seed column of this lane's (columns past the row count as non-seeds)
  const int last = m == 15u ? -1 : x + 31 - __builtin_clz(~m & 15u);
  const uint64_t brk = __ballot(m != 15u);
  const uint64_t before = brk & ((1ull << lane) - 1);
  const int from = __shfl(last, before ? 63 - __builtin_clzll(before) : 0);
  const int lb = before ? from : carry;
  if (brk) carry = __shfl(last, 63 - __builtin_clzll(brk));
  return lb;
}

template <bool VEC>
__global__ __launch_bounds__(256) void ws_init(const float* __restrict__ p, Vol3 g, float t, int32_t* __restrict__ a) {
  const int HW = g.H * g.W, lane = threadIdx.x & 63;
  wave_rows((unsigned)(g.Z * g.H), [&](int row) __attribute__((always_inline)) {
    const int z = row / g.H, y = row - z * g.H, base = row * g.W;
    int carry = -1;  // the last non-seed column before the step
    for (int x0 = 0; x0 < g.W; x0 += WC) {
      const int x = x0 + 4 * lane, v = base + x, n = min(max(g.W - x, 0), 4);
      const f4 q = row4<VEC>(p, v, n);
      const f4 zm = row4<VEC>(p, z > 0 ? v - HW : v, n), zp = row4<VEC>(p, z < g.Z - 1 ? v + HW : v, n);
      const f4 ym = row4<VEC>(p, y > 0 ? v - g.W : v, n), yp = row4<VEC>(p, y < g.H - 1 ? v + g.W : v, n);
      float left = __shfl_up(q[3], 1), right = __shfl_down(q[0], 1);
      if (lane == 0 && x > 0) left = ld<float>(gin(p) + ((int64_t)v - 1) * 4);
      if (lane == 63 && x + 4 < g.W) right = ld<float>(gin(p) + ((int64_t)v + 4) * 4);
      const unsigned m = below4(q, n, t);
      int lb = break_before(m, x, lane, carry);
      i4 out;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (m >> k & 1) {
          out[k] = base + lb + 1;  // the run's first seed
        } else {
          lb = x + k;
          int best = v + k;
          float pb = q[k];
          // candidates in ascending index order: a later one wins only if strictly lower
          auto cand = [&](bool there, float pu, int u) __attribute__((always_inline)) {
            const bool take = there && (pu < pb || (pu == pb && u < best));
            pb = take ? pu : pb;
            best = take ? u : best;
          };
          cand(z > 0, zm[k], v + k - HW);
          cand(y > 0, ym[k], v + k - g.W);
          cand(x + k > 0, k > 0 ? q[k > 0 ? k - 1 : 0] : left, v + k - 1);
          cand(x + k < g.W - 1, k < 3 ? q[k < 3 ? k + 1 : 3] : right, v + k + 1);
          cand(y < g.H - 1, yp[k], v + k + g.W);
          cand(z < g.Z - 1, zp[k], v + k + HW);
          out[k] = best;
        }
      }
      if constexpr (VEC) {
        if (n > 0) st<i4>(gout(a) + (int64_t)v * 4, out);
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (k < n) st<int32_t>(gout(a) + ((int64_t)v + k) * 4, out[k]);
      }
    }
  });
}

// Root of r with path halving (any node may be passed; roots are fixed points).
__device__ __forceinline__ int32_t ws_find(int32_t* a, int32_t r) {
  int32_t par = wa(a, r);
  while (par != r) {
    if (par < 0) return ~par;  // ws_flat has written the root here
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

__device__ __forceinline__ void ws_unite(int32_t* a, int32_t u, int32_t v) {
  int32_t ru = ws_find(a, u), rv = ws_find(a, v);
  while (ru != rv) {
    const int32_t hi = ru > rv ? ru : rv, lo = ru < rv ? ru : rv;
    const int32_t old = atomicCAS(a + hi, hi, lo);
    if (old == hi) return;  // hooked while hi was still a root
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
// (a few per wave and step): done where they are met, one lane in ten works while
// the wave waits. So a wave queues them in LDS and works them off 64 at a time
// (ws_flat 59 -> 55 us; ws_union, which waits for its atomics, the same).
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

template <bool VEC>
__global__ __launch_bounds__(256) void ws_union(const float* __restrict__ p, Vol3 g, float t, int32_t* a) {
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
    unsigned prevy = 0, prevz = 0;
    for (int x0 = 0; x0 < g.W; x0 += WC) {
      const int x = x0 + 4 * lane, v = base + x, n = min(max(g.W - x, 0), 4);
      const unsigned m = below4(row4<VEC>(p, v, n), n, t);
      const unsigned my = y < g.H - 1 ? below4(row4<VEC>(p, v + g.W, n), n, t) : 0u;
      const unsigned mz = z < g.Z - 1 ? below4(row4<VEC>(p, v + HW, n), n, t) : 0u;
      // first columns where the run of this row touches one of the next row / slice
      const unsigned sy = run_starts(m & my, lane, prevy), sz = run_starts(m & mz, lane, prevz);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        wq.push(sy >> k & 1, v + k);
        wq.push(sz >> k & 1, ~(v + k));
      }
      wq.drain(false, work);
    }
  });
  wq.drain(true, work);
}

template <bool VEC>
__global__ __launch_bounds__(256) void ws_flat(const float* __restrict__ p, Vol3 g, float t, int32_t* a) {
  __shared__ int queue[4][WQCAP];
  const int lane = threadIdx.x & 63;
  WaveQueue wq{queue[threadIdx.x >> 6], 0, lane};
  auto work = [&](int v) __attribute__((always_inline)) {
    const int32_t r = ws_find(a, v);
    __hip_atomic_store(a + v, ~r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  wave_rows((unsigned)(g.Z * g.H), [&](int row) __attribute__((always_inline)) {
    const int base = row * g.W;
    unsigned prev = 0;
    for (int x0 = 0; x0 < g.W; x0 += WC) {
      const int x = x0 + 4 * lane, v = base + x, n = min(max(g.W - x, 0), 4);
      const unsigned s = run_starts(below4(row4<VEC>(p, v, n), n, t), lane, prev);
#pragma unroll
      for (int k = 0; k < 4; ++k) wq.push(s >> k & 1, v + k);
      wq.drain(false, work);
    }
  });
  wq.drain(true, work);
}

template <bool VEC>
__global__ __launch_bounds__(256) void ws_label(Vol3 g, const int32_t* __restrict__ a, int32_t* out) {
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
    for (int k = 0; k < 4; ++k) par[k] = ld<int32_t>(ab + (int64_t)r[k] * 4);
  }
  // the four walks step together, so that their loads overlap
  auto open = [&](int k) __attribute__((always_inline)) { return par[k] >= 0 && par[k] != r[k]; };
  while (open(0) || open(1) || open(2) || open(3)) {
    i4 nx;
#pragma unroll
    for (int k = 0; k < 4; ++k) nx[k] = open(k) ? ld<int32_t>(ab + (int64_t)par[k] * 4) : par[k];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      r[k] = open(k) ? par[k] : r[k];
      par[k] = nx[k];
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = (par[k] < 0 ? ~par[k] : r[k]) + 1;
  if constexpr (VEC) {
    st<i4>(gout(out) + v * 4, r);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (v + k < g.N) st<int32_t>(gout(out) + (v + k) * 4, r[k]);
  }
}

// ws_flat and ws_label in one launch: every voxel finds its root, halving the path
// as it goes, one voxel a thread. For volumes whose time is their launches.
__global__ __launch_bounds__(256) void ws_label_small(Vol3 g, int32_t* a, int32_t* __restrict__ out) {
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v < (int)g.N) out[v] = ws_find(a, v) + 1;
}
// Voxels up to which it is used (us per call, three launches against four: 15.6
// against 20.1 on 2^12 voxels, 22 against 29 on 2^15, 31-33 against 33 on 2^17,
// 39 against 34 on 2^18).
constexpr int64_t kSmall = 1 << 17;

template <bool VEC>
static hipError_t ws_run(const float* p, const Vol3& g, float t, int32_t* labels, int32_t* work, hipStream_t st) {
  const int64_t groups = ((int64_t)g.Z * g.H + 3) / 4;  // of four rows
  // multiples of 8 (wave_rows); the kernels with a queue run persistent waves, which keep theirs filled
  const dim3 rows((unsigned)std::min<int64_t>((groups + 7) / 8 * 8, 1 << 20)), block(256);
  const dim3 few(std::min(rows.x, 2048u));
  hipLaunchKernelGGL(ws_init<VEC>, rows, block, 0, st, p, g, t, work);
  hipLaunchKernelGGL(ws_union<VEC>, few, block, 0, st, p, g, t, work);
  if (g.N <= kSmall) {
    hipLaunchKernelGGL(ws_label_small, dim3((unsigned)((g.N + 255) / 256)), block, 0, st, g, work, labels);
  } else {
    hipLaunchKernelGGL(ws_flat<VEC>, few, block, 0, st, p, g, t, work);
    hipLaunchKernelGGL(ws_label<VEC>, dim3((unsigned)((g.N + 1023) / 1024)), block, 0, st, g, work, labels);
  }
  return hipGetLastError();
}

}  // namespace emcnn

using namespace emcnn;

extern "C" int watershed_3d(const float* prob, const int64_t dims[3], float seed_threshold, int32_t* labels_out,
                            int32_t* work, void* stream) {
  clear_error();
  if (!prob || !dims || !labels_out || !work) return fail(CNN_EINVAL, "watershed_3d: null argument");
  const int64_t Z = dims[0], H = dims[1], W = dims[2];
  if (Z < 1 || H < 1 || W < 1 || Z > (1 << 30) || H > (1 << 30) || W > (1 << 30) || Z * H * W >= 2147483647ll)
    return fail(CNN_EINVAL, "watershed_3d: dims must be >= 1 with Z H W < 2^31 - 1");
  if (seed_threshold != seed_threshold) return fail(CNN_EINVAL, "watershed_3d: NaN threshold");
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  Vol3 g{(int)Z, (int)H, (int)W, Z * H * W};
  // 16-byte accesses where every row starts at one
  const bool vec = W % 4 == 0 && ((uintptr_t)prob | (uintptr_t)work | (uintptr_t)labels_out) % 16 == 0;
  const hipError_t e = vec ? ws_run<true>(prob, g, seed_threshold, labels_out, work, st)
                           : ws_run<false>(prob, g, seed_threshold, labels_out, work, st);
  if (e != hipSuccess) return hip_fail(e, "watershed_3d");
  return CNN_OK;
}
