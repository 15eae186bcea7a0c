// pair_sweep_kernel: the sweeps along x_3 and x_2 of a step in three
// dimensions in one pass over f.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>

#include "slmpp_internal.hpp"
#include "sweep_device.hpp"

namespace slmpp {
namespace {

// Bytes of consecutive velocities per row of a tile.  A copy of f in such
// tiles runs at 4.5 TB/s with 128 bytes per row and at 2.3-2.8 with 64
// (32^3 x 24^3 and 48^3 x 48^3 FP32: no faster there than two sweeps).
constexpr int kPairBytes = 128;
constexpr size_t kPairLds = 160 * 1024;
// Rows (x_2, x_3) of a tile at most.  FP32: as many as two workgroups per CU
// hold.  With 1024 rows, one workgroup of 16 wavefronts that waits at every
// barrier, the step took 6.07 against 5.94 ms with two sweeps (32^3 x 24^3,
// outflow) and 2.37 against 2.40 (32^3 x 16^3).  FP64: as many as a CU holds;
// its two sweeps hold only eight wavefronts per CU and lose more (32^6: 24.4
// against 25.5 ms per step).
constexpr int kPairRowsF32 = 576, kPairRowsF64 = 1024;
template <typename T>
constexpr int kPairSlots = sizeof(T) == 4 ? 9 : 8;  // 16-byte vectors per thread and tile at most
template <typename T>
constexpr int kPairMaxR = sizeof(T) == 4 ? 16 : 8;  // cells per thread and round at most

// advance_line() for a pencil without ghost cells: reads wrap around the
// pencil, whose next offset is the smaller of off and off -+ n rs as unsigned
// numbers, or (outflow) outside it go to a cell of zero.
template <typename T, int ORDER, bool PERIODIC, int MAXR>
__device__ __forceinline__ void advance_bare(const T* col, int rs, int n, const T* zero,
                                             const PencilEntry<T>& e, int m0, int R, T alpha,
                                             T* out) {
  constexpr int H = (ORDER == 7) ? 3 : 2;
  constexpr int WIN = 2 * H + 1;
  // cells read ahead of the flux: FP64 32^6 24.4 ms per step with four, 25.3
  // with none or eight (which spill more); FP32 18x20x24 x 30x36x42 5.57 with
  // none, 5.67 with four
  constexpr int DIST = sizeof(T) == 8 ? 4 : 0;
  int r = e.base + e.dir * (m0 - 1 - H);
  if (PERIODIC) {
    r %= n;
    if (r < 0) r += n;
  }
  const int step = e.dir * rs;
  const uint32_t len = (uint32_t)(n * rs), adj = e.dir > 0 ? 0u - len : len;
  uint32_t off = (uint32_t)(r * rs);
  const uint32_t zoff = (uint32_t)(zero - col);
  auto fetch = [&]() __attribute__((always_inline)) -> T {
    T v;
    if constexpr (PERIODIC) {
      v = col[off];
      off += (uint32_t)step;
      off = min(off, off + adj);
    } else {
      v = col[off < len ? off : zoff];
      off += (uint32_t)step;
    }
    return v;
  };
  T q[MAXR + WIN + DIST];
#pragma unroll
  for (int k = 0; k < WIN + DIST; ++k)
    if (k < WIN + R) q[k] = fetch();
  T f_left = face_flux<T, ORDER, SLMPP_LIM_MPP>(q, e.w, e.tz, alpha);
#pragma unroll
  for (int k = 0; k < MAXR; ++k) {
    if (k < R) {
      if (k + DIST < MAXR && k + DIST < R) q[k + WIN + DIST] = fetch();
      const T f_right = face_flux<T, ORDER, SLMPP_LIM_MPP>(q + k + 1, e.w, e.tz, alpha);
      out[k] = vfma(-e.z, f_right - f_left, q[k + 1 + H]);
      f_left = f_right;
    }
  }
}

// Persistent over tiles of all (x_2, x_3) of one x_1 and 128 bytes of
// velocities; the next tile is loaded into registers before the current one
// is advanced.  In LDS a tile has no ghost cells, and lane c of 128 bytes keeps
// to velocity c, so that neither sweep has bank conflicts.  A sweep runs in
// rounds of whole pencils of one segment per thread.  Both pencil tables stay
// in LDS.  The results equal the two separate sweeps cell for cell.
//   Bound by the instructions of the two sweeps and by 128-byte rows (4.5 TB/s
// for a copy); saves one pass over f and one launch per step.  18x20x24 x
// 30x36x42 FP32: 1.17 ms against 2 x 0.74, step 5.80 -> 5.60 ms; 32^6 FP64
// 25.4 -> 24.5; 16^3 x 24^3 FP32 0.704 -> 0.670; 24x24x20 x 16x18x17 FP64
// 2.28 -> 2.16; 8^3 x 12^3 FP64 112 -> 106 us.
template <typename T, int ORDER, bool PERIODIC>
__global__ void __attribute__((amdgpu_flat_work_group_size(1, 1024), amdgpu_waves_per_eu(4)))
pair_sweep_kernel(T* __restrict__ f, T alpha, PairPlan pl, const PencilEntry<T>* __restrict__ tabA,
                  const PencilEntry<T>* __restrict__ tabB) {
  extern __shared__ __align__(16) unsigned char smem[];
  using V = typename Vec<T>::type;
  using U = typename UVec<T>::type;
  constexpr int VN = Vec<T>::N;
  constexpr int C = kPairBytes / (int)sizeof(T);
  constexpr int CV = C / VN;
  constexpr int MAXR = kPairMaxR<T>;
  const int nA = pl.nA, nB = pl.nB, NT = blockDim.x, tid = threadIdx.x;
  const int rows = nA * nB;
  T* tile = reinterpret_cast<T*>(smem);
  T* zero = tile + rows * C;
  PencilEntry<T>* entA = reinterpret_cast<PencilEntry<T>*>(zero + VN);
  PencilEntry<T>* entB = entA + pl.nvA;
  for (int i = tid; i < pl.nvA; i += NT) entA[i] = tabA[i];
  for (int i = tid; i < pl.nvB; i += NT) entB[i] = tabB[i];
  if (tid == 0) *zero = T(0);
  // data map: vector k of the thread is tid + k NT of the tile, the same
  // place in LDS; row (tid + k NT) / CV, velocities VN ((tid + k NT) % CV) on
  const int cv = tid % CV;
  const int nslot = (rows * CV + NT - 1) / NT;
  const int64_t gstep = (int64_t)(NT / CV) * pl.inner;
  uint32_t goff = (uint32_t)((tid / CV) * pl.inner32 + cv * VN) * (uint32_t)sizeof(T);  // bytes
  const int nvec = rows * CV;
  // compute maps: velocity c, then segment s of pencil k of a round
  const int c = tid % C, g = tid / C;
  const int sA = g / pl.kA, jA = g - sA * pl.kA, mA = min(sA * pl.rA, nA - pl.rA);
  const int sB = g / pl.kB, jB = g - sB * pl.kB, mB = min(sB * pl.rB, nB - pl.rB);
  V pf[kPairSlots<T>];
  int wv = 0;  // velocities of the tile
  int64_t base = 0;
  int j0 = 0;
  auto place = [&](int t) __attribute__((always_inline)) {
    const int o = (int)pl.dch.div((uint32_t)t);
    j0 = (t - o * pl.nch) * C;
    wv = min(C, pl.inner32 - j0);
    base = (int64_t)o * rows * pl.inner + j0;
  };
  auto load = [&]() __attribute__((always_inline)) {
    const T* src = f + base;
    uint32_t vo = goff;
    asm volatile("" : "+v"(vo));  // (addresses formed here, not kept across the tile)
#pragma unroll
    for (int k = 0; k < kPairSlots<T>; ++k)
      if (k < nslot && tid + k * NT < nvec && cv * VN < wv)
        pf[k] = __builtin_nontemporal_load(
            (GlobalPtr<const U>)(reinterpret_cast<const char*>(src + k * gstep) + vo));
  };
  auto sweep = [&](const PencilEntry<T>& e, int n, int rs, int pstride, int other, int K, int S,
                   int s, int j, int m0, int R, bool in) __attribute__((always_inline)) {
    T out[MAXR];
    for (int p0 = 0; p0 < other; p0 += K) {
      // (a round's pencils are read and written by that round only: one
      // barrier, between its reads and its writes)
      const bool act = in && s < S && p0 + j < other;
      T* col = tile + (p0 + j) * pstride + c;
      if (act) advance_bare<T, ORDER, PERIODIC, MAXR>(col, rs, n, zero, e, m0, R, alpha, out);
      __syncthreads();
      if (act) {
        T* op = col + (e.dir > 0 ? m0 : n - 1 - m0) * rs;
        const int step = e.dir * rs;
#pragma unroll
        for (int k = 0; k < MAXR; ++k)
          if (k < R) {
            *op = out[k];
            op += step;
          }
      }
    }
    __syncthreads();
  };
  int t = blockIdx.x;
  if (t < pl.tiles) {
    place(t);
    load();
  }
  __syncthreads();
  for (; t < pl.tiles; t += gridDim.x) {
    const int64_t b = base;
    const int w = wv;
    const uint32_t jv = (uint32_t)(j0 + min(c, w - 1));
    int lv = tid;
    asm volatile("" : "+v"(lv));
#pragma unroll
    for (int k = 0; k < kPairSlots<T>; ++k)
      if (k < nslot && lv + k * NT < nvec && cv * VN < w)
        *reinterpret_cast<V*>(tile + VN * (lv + k * NT)) = pf[k];
    __syncthreads();
    if (t + (int)gridDim.x < pl.tiles) {
      place(t + gridDim.x);
      load();
    }
    {
      const uint32_t qb = pl.dvB.div(jv);
      const PencilEntry<T> e = entB[qb - pl.dnB.div(qb) * (uint32_t)pl.nvB];
      sweep(e, nB, C, nB * C, nA, pl.kB, pl.sB, sB, jB, mB, pl.rB, c < w);
    }
    {
      const uint32_t qa = pl.dvA.div(jv);
      const PencilEntry<T> e = entA[qa - pl.dnA.div(qa) * (uint32_t)pl.nvA];
      sweep(e, nA, nB * C, C, nB, pl.kA, pl.sA, sA, jA, mA, pl.rA, c < w);
    }
    T* dst = f + b;
    uint32_t vo = goff;
    asm volatile("" : "+v"(vo), "+v"(lv));
#pragma unroll
    for (int k = 0; k < kPairSlots<T>; ++k)
      if (k < nslot && lv + k * NT < nvec && cv * VN < w)
        __builtin_nontemporal_store((U)*reinterpret_cast<V*>(tile + VN * (lv + k * NT)),
                                    (GlobalPtr<U>)(reinterpret_cast<char*>(dst + k * gstep) + vo));
    // (no barrier: the next tile's first LDS writes are this thread's own
    // vectors)
  }
}

template <typename T, int ORDER, bool PERIODIC>
hipError_t launch_t(const SweepArgs& a, const PairPlan& p, const void* tabA, const void* tabB, hipStream_t s) {
  auto kern = pair_sweep_kernel<T, ORDER, PERIODIC>;
  const void* fn = reinterpret_cast<const void*>(kern);
  hipError_t e = hipSuccess;
  if (p.lds_bytes > 64 * 1024)
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds_bytes);
  int64_t grid = 0;
  if (e == hipSuccess) e = resident_grid(fn, p.threads, p.lds_bytes, p.tiles, INT_MAX, &grid);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(p.threads), p.lds_bytes, s,
                     reinterpret_cast<T*>(a.f), (T)a.alpha, p,
                     reinterpret_cast<const PencilEntry<T>*>(tabA),
                     reinterpret_cast<const PencilEntry<T>*>(tabB));
  return hipGetLastError();
}

template <typename T, int ORDER>
hipError_t launch_o(const SweepArgs& a, const PairPlan& p, const void* tabA, const void* tabB, hipStream_t s) {
  return a.bc == SLMPP_BC_PERIODIC ? launch_t<T, ORDER, true>(a, p, tabA, tabB, s)
                                   : launch_t<T, ORDER, false>(a, p, tabA, tabB, s);
}

}  // namespace

PairPlan plan_pair(int dtype, const SweepArgs& sA, const SweepArgs& sB, int64_t outer) {
  PairPlan p{};
  const int es = dtype == SLMPP_F64 ? 8 : 4, vn = 16 / es, C = kPairBytes / es;
  const int64_t inner = sB.inner, nA = sA.n, nB = sB.n, rows = nA * nB;
  const int64_t nch = (inner + C - 1) / C;
  if (sA.cmode != SPEED_FROM_VELOCITY || sB.cmode != SPEED_FROM_VELOCITY || sA.bc != sB.bc ||
      inner % vn != 0 || inner * es >= ((int64_t)1 << 24) || nA < 4 || nB < 4 ||
      rows > (es == 4 ? kPairRowsF32 : kPairRowsF64) || outer * nch >= ((int64_t)1 << 30))
    return p;
  const size_t lds = (size_t)rows * kPairBytes + 16 +
                     (size_t)(sA.nvl + sB.nvl) * (es == 4 ? sizeof(PencilEntry<float>) : sizeof(PencilEntry<double>));
  if (lds > kPairLds) return p;
  // segments: the fewest faces per thread over the rounds of a sweep; threads:
  // the fewest of them per tile and resident workgroup (16 wavefronts per CU)
  const int maxr = es == 4 ? kPairMaxR<float> : kPairMaxR<double>;
  const int slots = es == 4 ? kPairSlots<float> : kPairSlots<double>;
  auto segments = [maxr](int n, int other, int groups, int32_t& S, int32_t& R, int32_t& K) {
    int best = INT32_MAX;
    for (int s = (n + maxr - 1) / maxr; s <= std::min(groups, (n + 3) / 4); ++s) {
      const int r = (n + s - 1) / s, k = std::min(groups / s, other);
      const int cost = (other + k - 1) / k * (r + 2);
      if ((n + r - 1) / r == s && cost < best) {
        best = cost;
        S = s;
        R = r;
        K = k;
      }
    }
    return best;
  };
  double best = 1e30;
  for (int nt = 128; nt <= 1024; nt += 64) {
    if (rows * (kPairBytes / 16) > (int64_t)slots * nt) continue;
    PairPlan q{};
    const int a = segments((int)nA, (int)nB, nt / C, q.sA, q.rA, q.kA);
    const int b = segments((int)nB, (int)nA, nt / C, q.sB, q.rB, q.kB);
    if (a == INT32_MAX || b == INT32_MAX) continue;
    const int resident = std::max(1, std::min(16 / (nt / 64), (int)(kPairLds / lds)));
    if ((double)(a + b) / resident < best) {
      best = (double)(a + b) / resident;
      q.threads = nt;
      p = q;
    }
  }
  if (!p.threads) return PairPlan{};
  p.nA = (int)nA;
  p.nB = (int)nB;
  p.nvA = sA.nvl;
  p.nvB = sB.nvl;
  p.inner = inner;
  p.inner32 = (int)inner;
  p.nch = (int)nch;
  p.tiles = (int)(outer * nch);
  p.dch = FastDiv32::of((uint32_t)nch);
  p.dvA = FastDiv32::of((uint32_t)sA.vdiv);
  p.dvB = FastDiv32::of((uint32_t)sB.vdiv);
  p.dnA = FastDiv32::of((uint32_t)sA.nvl);
  p.dnB = FastDiv32::of((uint32_t)sB.nvl);
  p.lds_bytes = lds;
  return p;
}

hipError_t launch_pair(int dtype, int order, const SweepArgs& a, const PairPlan& p, const void* tabA,
                       const void* tabB, hipStream_t s) {
  if (p.lds_bytes == 0) return hipErrorInvalidValue;
  if (dtype == SLMPP_F64)
    return order == 7 ? launch_o<double, 7>(a, p, tabA, tabB, s) : launch_o<double, 5>(a, p, tabA, tabB, s);
  return order == 7 ? launch_o<float, 7>(a, p, tabA, tabB, s) : launch_o<float, 5>(a, p, tabA, tabB, s);
}

}  // namespace slmpp
