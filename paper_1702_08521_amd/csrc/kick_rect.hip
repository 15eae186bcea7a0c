// kick_rect_kernel: the sweeps along the last two velocity axes of a kick in
// one pass over f, for planes of any size (kick_plane_kernel holds those of
// 24^2, 32^2, 48^2 and 64^2 cells at compile time).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "slmpp_internal.hpp"
#include "sweep_device.hpp"

namespace slmpp {
namespace {

// Cells per thread in a sweep at most.  With 8 the kernel holds in 5 wavefronts
// per SIMD in FP32, 4 in FP64; 12 in FP32 (4 wavefronts per SIMD) measured 6.20
// against 5.84 ms per step on 18x20x24 x 30x36x42.
constexpr int kRectMaxR = 8;
constexpr int kRectThreads = 1024;  // threads per workgroup at most
constexpr int kRectFast = 1;        // integer shifts read directly
constexpr size_t kRectLds = 64 * 1024;
// The pass is taken for planes of at least kRectCells cells, and on grids of
// at most kRectSmall cells for any.
//   Large grids: a plane gives cells / 8 threads and five barriers, so small
// ones leave the tail of a workgroup idle where line_sweep_kernel packs
// pencils of many planes.  Steps with the pass against the two sweeps, in us:
// FP32 12^3 x 16x24x28 386 / 357, 16x28x28 484 / 459, 16x30x30 535 / 527, but
// 16^3 x 20x36x44 1817 / 2085; FP64 12^3 x 30^3 1713 / 1677, but 12^3 x
// 16x32x40 1097 / 1260, 16x36x36 1130 / 1240, 40^2 x 80x72 227 / 281.
//   Small grids are bound by launches, of which the pass saves one per kick:
// 32^2 x 16^2 FP32 56 / 70, 32^2 x 24x30 FP64 79 / 93.
constexpr int64_t kRectCells = 1024;
constexpr int64_t kRectSmall = (int64_t)1 << 21;

// One plane (x, v_1 .. v_{D-2}) of na x nb cells per tile, one contiguous
// piece of f, persistent, the next plane loaded into registers before the
// current one is advanced.  In LDS the plane lies inside a ring of G zero
// cells (outflow).  All its pencils along v_{D-1} share one table entry, and
// all along v_D another: scalar loads.  The results equal two separate sweeps
// cell for cell.
//   Bound by the instructions of the flux and the limiters in both sweeps and
// by the five barriers of a plane; saves one pass over f and one launch per
// kick.  A step of 30x37 x 54x61 in FP32 took 118 us with two
// sweeps, 90 with the pass; of 18x20x24 x 30x36x42 6.10 and 5.84 ms.
template <typename T, int ORDER>
__global__ void __attribute__((amdgpu_flat_work_group_size(1, kRectThreads), amdgpu_waves_per_eu(sizeof(T) == 4 ? 5 : 4)))
kick_rect_kernel(SweepArgs a, RectPlan pl, const PencilEntry<T>* __restrict__ tabA,
                 const PencilEntry<T>* __restrict__ tabB) {
  extern __shared__ __align__(16) unsigned char smem[];
  using V = typename Vec<T>::type;
  using U = typename UVec<T>::type;
  constexpr int VN = Vec<T>::N;
  constexpr int NS = kRectMaxR / VN;
  T* lds = reinterpret_cast<T*>(smem);
  T* f = reinterpret_cast<T*>(a.f);
  const T alpha = (T)a.alpha;
  const int na = pl.na, nb = pl.nb, G = pl.G, P = pl.pitch, NT = blockDim.x;
  const int tid = threadIdx.x;
  const int cells = na * nb;
  const int nslot = (cells + VN * NT - 1) / (VN * NT);
  // data map: vector k is elements VN (tid + k NT) of the plane, at loff[k] in
  // LDS; with rows that are no whole number of vectors its elements from
  // number cross on lie in the next row
  const bool split = nb % VN != 0;
  int loff[NS], cross[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    const int e = VN * (tid + k * NT);
    const int ia = e / nb, ib = e - ia * nb;
    loff[k] = (ia + G) * P + G + ib;
    cross[k] = nb - ib;
  }
  const int gap = P - nb;  // from the end of a row to the next
  for (int e = tid; e < (na + 2 * G) * P; e += NT) lds[e] = T(0);
  __syncthreads();
  // compute maps: segment-major, the last segment moved back to the end
  const int sa = tid / nb, ja = tid - sa * nb, ma = min(sa * pl.ra, na - pl.ra);
  const int sb = tid / na, jb = tid - sb * na, mb = min(sb * pl.rb, nb - pl.rb);
  const bool actA = sa < pl.sa, actB = sb < pl.sb;
  T* colA = lds + G * P + G + ja;
  T* colB = lds + (G + jb) * P + G;
  // elements of the plane from vector k on (not positive: none); the last
  // plane is read element by element where f itself may end within a vector
  auto exist = [&](int k) __attribute__((always_inline)) -> int { return cells - VN * (tid + k * NT); };
  const bool tail = cells % VN != 0;
  V pf[NS];
  auto load = [&](int64_t t) __attribute__((always_inline)) {
    if (tail && t + 1 == pl.planes) return;
    const T* src = f + t * cells + VN * tid;
#pragma unroll
    for (int k = 0; k < NS; ++k)
      if (k < nslot && exist(k) > 0)
        pf[k] = __builtin_nontemporal_load((GlobalPtr<const U>)(src + k * VN * NT));
  };
  auto advance2 = [&](const T* col, int rs, int n, const PencilEntry<T>& e, int m0, int R, T* out)
      __attribute__((always_inline)) {
    if (e.absN <= kRectFast)
      advance_line<T, ORDER, SLMPP_LIM_MPP, false, kRectMaxR>(col, rs, n, G, 0, e, m0, R, alpha, out);
    else
      advance_line<T, ORDER, SLMPP_LIM_MPP, true, kRectMaxR>(col, rs, n, G, 0, e, m0, R, alpha, out);
  };
  auto keep = [&](T* col, int rs, int n, int dir, int m0, int R, const T* out) __attribute__((always_inline)) {
    T* op = col + (dir > 0 ? m0 : (n - 1 - m0)) * rs;
    const int step = dir * rs;
#pragma unroll
    for (int k = 0; k < kRectMaxR; ++k)
      if (k < R) {
        *op = out[k];
        op += step;
      }
  };
  int64_t t = blockIdx.x;
  if (t < pl.planes) load(t);
  for (; t < pl.planes; t += gridDim.x) {
    const uint32_t ix = pl.vdiv.div((uint32_t)t);
    const PencilEntry<T> eA = load_entry_uniform(tabA + ix);
    const PencilEntry<T> eB = load_entry_uniform(tabB + ix);
    if (tail && t + 1 == pl.planes) {
      const T* src = f + t * cells;
      for (int e = tid; e < cells; e += NT) {
        const int ia = e / nb;
        lds[(ia + G) * P + G + e - ia * nb] = src[e];
      }
    } else {
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (k < nslot && exist(k) > 0) {
          if (!split) {
            put(lds + loff[k], pf[k]);
          } else {
#pragma unroll
            for (int c = 0; c < VN; ++c)
              if (c < exist(k)) lds[loff[k] + c + (c >= cross[k] ? gap : 0)] = pf[k][c];
          }
        }
      }
    }
    __syncthreads();
    if (t + gridDim.x < pl.planes) load(t + gridDim.x);
    T out[kRectMaxR];
    if (actA) advance2(colA, P, na, eA, ma, pl.ra, out);
    __syncthreads();
    if (actA) keep(colA, P, na, eA.dir, ma, pl.ra, out);
    __syncthreads();
    if (actB) advance2(colB, 1, nb, eB, mb, pl.rb, out);
    __syncthreads();
    if (actB) keep(colB, 1, nb, eB.dir, mb, pl.rb, out);
    __syncthreads();
    T* dst = f + t * cells;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      if (k < nslot) {
        const int c1 = exist(k);
        if (c1 > 0) {
          V v;
          if (!split) {
            get(lds + loff[k], v);
          } else {
#pragma unroll
            for (int c = 0; c < VN; ++c)
              if (c < c1) v[c] = lds[loff[k] + c + (c >= cross[k] ? gap : 0)];
          }
          T* p = dst + VN * (tid + k * NT);
          if (c1 >= VN) {
            __builtin_nontemporal_store((U)v, (GlobalPtr<U>)p);
          } else {
#pragma unroll
            for (int c = 0; c < VN; ++c)
              if (c < c1) p[c] = v[c];
          }
        }
      }
    }
    // (no barrier: the next plane's first LDS writes are this thread's own
    // vectors; read element by element, they are not)
    if (tail && t + gridDim.x + 1 == pl.planes) __syncthreads();
  }
}

template <typename T, int ORDER>
hipError_t launch_t(const SweepArgs& a, const RectPlan& p, const void* tabA, const void* tabB, hipStream_t s) {
  auto kern = kick_rect_kernel<T, ORDER>;
  const void* fn = reinterpret_cast<const void*>(kern);
  // at most seven wavefronts per SIMD, as for the square planes
  int64_t grid = 0;
  const hipError_t e =
      resident_grid(fn, p.threads, p.lds_bytes, p.planes, std::max(1, 28 / ((p.threads + 63) / 64)), &grid);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(p.threads), p.lds_bytes, s, a, p,
                     reinterpret_cast<const PencilEntry<T>*>(tabA),
                     reinterpret_cast<const PencilEntry<T>*>(tabB));
  return hipGetLastError();
}

}  // namespace

RectPlan plan_kick_rect(int dtype, int order, int64_t na, int64_t nb, int64_t planes, int64_t vouter) {
  RectPlan p{};
  const int es = dtype == SLMPP_F64 ? 8 : 4;
  if (na < 8 || nb < 8 || na > 256 || nb > 256 || planes < 1 || planes >= ((int64_t)1 << 31) ||
      vouter < 1 || vouter >= ((int64_t)1 << 31))
    return p;
  if (na * nb < kRectCells && planes > kRectSmall / (na * nb)) return p;
  p.na = (int)na;
  p.nb = (int)nb;
  // segments: as long as they may be while a plane has two wavefronts, in
  // equal lengths
  constexpr int maxr = kRectMaxR;
  auto segments = [](int64_t n, int64_t pencils, int32_t& s, int32_t& r) {
    s = (int32_t)((n + maxr - 1) / maxr);
    while (s * pencils < 128 && n / (s + 1) >= 4) ++s;
    r = (int32_t)((n + s - 1) / s);
    s = (int32_t)((n + r - 1) / r);
  };
  segments(na, nb, p.sa, p.ra);
  segments(nb, na, p.sb, p.rb);
  int64_t nt = std::max<int64_t>(p.sa * nb, p.sb * na);
  nt = (nt + 63) / 64 * 64;
  if (nt > kRectThreads || na * nb > (int64_t)maxr * nt) return RectPlan{};
  p.threads = (int)nt;
  p.G = (order == 7 ? 4 : 3) + kRectFast;
  p.pitch = (int)(nb + 2 * p.G) | 1;
  p.planes = planes;
  p.vdiv = FastDiv32::of((uint32_t)vouter);
  const size_t lds = ((size_t)(na + 2 * p.G) * p.pitch * es + 15) & ~(size_t)15;
  if (lds > kRectLds) return RectPlan{};
  p.lds_bytes = lds;
  return p;
}

hipError_t launch_kick_rect(int dtype, int order, const SweepArgs& a, const RectPlan& p,
                            const void* tabA, const void* tabB, hipStream_t s) {
  if (p.lds_bytes == 0) return hipErrorInvalidValue;
  if (dtype == SLMPP_F64)
    return order == 7 ? launch_t<double, 7>(a, p, tabA, tabB, s) : launch_t<double, 5>(a, p, tabA, tabB, s);
  return order == 7 ? launch_t<float, 7>(a, p, tabA, tabB, s) : launch_t<float, 5>(a, p, tabA, tabB, s);
}

}  // namespace slmpp
