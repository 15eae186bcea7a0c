// line_sweep_kernel: one sweep of pencils of any length, stride, limiter and
// time integration (the sizes that no compile-time tile of sweep_fast_kernel
// divides).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <type_traits>

#include "slmpp_internal.hpp"
#include "sweep_device.hpp"

namespace slmpp {
namespace {

// cells per thread at most, and threads per workgroup at most: 128 VGPRs in
// both types, so that two workgroups of 512 threads share a CU.  TVD-RK stages
// keep a segment's old values as well and run 256 threads; so do FP64 block
// tiles, which have no rows to keep wide (10 x 12 x 9 x 20 x 21 x 22: 456
// against 497 us per step).
template <typename T>
constexpr int kLineMaxR = sizeof(T) == 4 ? 16 : 8;
constexpr int kLineThreads = 512, kLineThreadsSmall = 256;
constexpr size_t kLineLds = 40 * 1024;     // preferred LDS of a tile: four workgroups per CU
constexpr size_t kLineLdsMax = 80 * 1024;  // at most (long pencils)
// a workgroup of five wavefronts leaves the four SIMDs of a CU unevenly filled:
// its sweeps took as long as those of one-tile workgroups or longer, where four,
// seven or eight wavefronts took 0.6-0.8 of them (n 96, s 44, 1.3e8 cells FP64: 820 us,
// with two tiles of three wavefronts each 553)
constexpr int kUneven = 5;

// MODE of line_sweep_kernel: one sweep; all three TVD-RK stages; pl.reps
// sweeps of block tiles one after the other (the same kick twice, with one
// read and one write of f); one sweep of row tiles that leaves the row sums of
// the velocity moment (whose code took registers from the others: 24^6 FP32
// SL-MP7 sweeps 2.36 against 2.34 ms).  (Entries computed in the kernel instead of read
// from a table cost small grids more in registers than the launch for the
// table: 64 x 128 FP64, x sweep 9.0 -> 11.5 us.)
enum : int { LINE_ONE = 0, LINE_RK = 1, LINE_REPEAT = 2, LINE_SUMS = 3 };

// Persistent workgroups over tiles of whole pencils, the next tile's data
// loaded into registers before the current one is computed, as in
// sweep_fast_kernel, with every size a run-time value:
//  * row tiles (BLK false): W pencils of one block, staged [cell][pencil];
//  * block tiles (BLK true, blocks of few pencils and the contiguous axis): K
//    whole blocks, one contiguous piece of f, staged as it lies, each block
//    with its ghost cells around it.
// Thread t holds pencil t mod pw and segment t / pw; a pencil has S segments
// of R cells, the last one moved back to end at the pencil's end (the cells
// it shares with the one before are computed twice, to the same bits).  For
// the data movement it holds up to kLineMaxR elements in 16-byte vectors.
// LINE_RK: all three TVD-RK stages on the tile in LDS, one read and one write of
// f instead of eight passes.
//
// Bound by HBM on large grids (18 x 20 x 24 x 30 x 36 x 42 FP32 SL-MPP7, 3.1 GB
// per sweep: v sweeps 639 us, x sweeps 710-810 us, against 870-1640 us with
// one tile per workgroup, run-time segments through a second LDS tile and
// element-wise loads; the whole step 11.20 -> 6.42 ms), by its vector
// instructions at about 40 per cell where f stays in the caches (24^6 FP32
// SL-MP7: 414-523 us, was 650-700), by the latency of a tile on small grids
// (256 x 512: 5.4 and 6.9 us, was 9).  48^2 x 40^2 FP64 RK-MPP5 step: 495 ->
// 304 us.  What made it: registers for two workgroups per CU (one took
// 11.9 ms for that step), steps between a thread's vectors kept in scalar
// registers, and loads without a second path for partial vectors (whose
// merge made every load wait for the one before: 7.34 ms).
template <typename T, int ORDER, int LIM, bool BLK, int MODE, bool STREAM>
__global__ void __attribute__((amdgpu_flat_work_group_size(1, MODE == LINE_RK ? kLineThreadsSmall : kLineThreads),
                               amdgpu_waves_per_eu(MODE == LINE_RK ? 3 : (MODE == LINE_REPEAT ? 2 : 4))))
line_sweep_kernel(SweepArgs a, LinePlan pl, const PencilEntry<T>* __restrict__ table) {
  extern __shared__ __align__(16) unsigned char smem[];
  using V = typename Vec<T>::type;
  using U = typename UVec<T>::type;
  constexpr int VN = Vec<T>::N;
  constexpr int NS = kLineMaxR<T> / VN;
  T* tile = reinterpret_cast<T*>(smem);
  T* f = reinterpret_cast<T*>(a.f);
  const T alpha = (T)a.alpha;
  const int n = a.n, G = pl.G, R = pl.R, rs = pl.rs, bs = pl.bs, pw = pl.pw;
  const int inner = (int)a.inner;
  const int tid = threadIdx.x;
  const int nact = pw * pl.S;
  const bool periodic = a.bc == SLMPP_BC_PERIODIC;
  // compute map
  const int s = tid / pw, jj = tid - s * pw;
  const int cb = BLK ? jj / inner : 0, cj = BLK ? jj - cb * inner : jj;
  const int m0 = min(s * R, n - R);
  T* col = tile + cb * bs + G * rs + cj;
  const bool mine = tid < nact;
  // data map: vector k of the thread.  Row tiles: column ncol of row i0 + k di
  // (the steps between vectors are wave-uniform and stay in scalar registers);
  // block tiles: element VN (tid + k nact) of the piece, at loff[k] in LDS,
  // its elements from number cross[k] on in the next block
  int loff[NS], cross[NS];
  int ncol = 0, i0 = 0, di = 1, loff0 = 0;
  int64_t goff0 = 0, gstep = 0;
  uint32_t edge = 0;  // row tiles: bit k, k + 16: vector k is among the first, last G rows
  const int ni = BLK ? n * inner : 0;  // block tiles: elements of a block
  if constexpr (BLK) {
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const int e = VN * (tid + k * nact);
      const int b = e / ni, rem = e - b * ni;
      loff[k] = b * bs + G * rs + rem;
      cross[k] = ni - rem;
    }
    goff0 = VN * tid;
    gstep = VN * nact;
  } else {
    const int cpr = pw / VN;
    i0 = tid / cpr;
    ncol = (tid - i0 * cpr) * VN;
    di = VN * pl.S;
    loff0 = (i0 + G) * rs + ncol;
    goff0 = (int64_t)i0 * inner + ncol;
    gstep = (int64_t)di * inner;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const int i = i0 + k * di;
      if (i < G) edge |= 1u << k;
      if (i >= n - G) edge |= 0x10000u << k;
    }
    if (!mine) i0 = n;
  }
  const int nslot = (n + VN * pl.S - 1) / (VN * pl.S);
  const bool wrap_rows = !BLK && periodic && G <= n;
  // zero the LDS once: ghost cells of outflow axes stay zero (the data
  // never touch them), and so do pencils a short last tile does not fill
  for (int e = tid; e < pl.lds_elems; e += blockDim.x) tile[e] = T(0);
  __syncthreads();

  // tile t: first element in f, number of valid pencils (row tiles) or
  // elements (block tiles), first pencil index and block
  struct Where {
    int64_t base;
    int valid, j0, ob;
  };
  auto where = [&](int64_t t) -> Where {
    Where w;
    if constexpr (BLK) {
      const int64_t b0 = t * pl.K;
      w.base = b0 * ni;
      w.valid = (int)min<int64_t>(pl.K, pl.blocks - b0) * ni;
      w.j0 = 0;
      w.ob = (int)b0;
    } else {
      w.ob = (int)pl.dtpb.div((uint32_t)t);
      w.j0 = ((int)t - w.ob * pl.tpb) * pl.W;
      w.valid = min(pl.W, pl.blen - w.j0);
      w.base = (int64_t)w.ob * pl.bstride + w.j0;
    }
    return w;
  };
  // elements of vector k that exist (not positive: none)
  auto exist = [&](const Where& w, int k) __attribute__((always_inline)) -> int {
    if constexpr (BLK)
      return mine ? w.valid - VN * (tid + k * nact) : 0;
    else
      return i0 < n - k * di ? w.valid - ncol : 0;
  };
  // LDS element of the first component of vector k
  auto lds_at = [&](int k) __attribute__((always_inline)) -> int {
    if constexpr (BLK)
      return loff[k];
    else
      return loff0 + k * di * rs;
  };
  // The last vector of a row or piece may hold fewer than VN elements of the
  // tile; it is loaded whole (what lies beyond belongs to other pencils and
  // is not used), except where f itself may end within it: the last tile is
  // then read element by element, past the registers.
  V pf[NS];
  auto by_element = [&](int64_t t, const Where& w) { return t + 1 == pl.tiles && w.valid % VN != 0; };
  auto load = [&](const Where& w) __attribute__((always_inline)) {
    const T* src = f + w.base;
#pragma unroll
    for (int k = 0; k < NS; ++k)
      if (k < nslot && exist(w, k) > 0) {
        const GlobalPtr<const U> q = (GlobalPtr<const U>)(src + k * gstep + goff0);
        pf[k] = STREAM ? __builtin_nontemporal_load(q) : *q;
      }
  };
  // LDS element of component c of vector k
  auto at = [&](int k, int c) -> int {
    return loff[k] + c + (c >= cross[k] ? bs - ni : 0);
  };
  // ghost cells of a periodic axis from the pencils in LDS
  auto fill_ghosts = [&]() {
    for (int e = tid; e < 2 * G * pw; e += blockDim.x) {
      const int g = e / pw, p = e - g * pw;
      const int b = BLK ? p / inner : 0, j = BLK ? p - b * inner : p;
      T* c0 = tile + b * bs + G * rs + j;
      const int pr = g < G ? g - G : n + (g - G);
      int sp = pr < 0 ? pr + n : (pr >= n ? pr - n : pr);
      if (G > n) {
        sp = pr % n;
        if (sp < 0) sp += n;
      }
      c0[pr * rs] = c0[sp * rs];
    }
  };
  int64_t t = blockIdx.x;
  Where next{};
  if (t < pl.tiles) {
    next = where(t);
    if (!by_element(t, next)) load(next);
  }
  for (; t < pl.tiles; t += gridDim.x) {
    const Where w = next;
    // the pencil's entry, requested before the tile goes to LDS
    PencilEntry<T> e{};
    const bool act = BLK ? mine && jj * n < w.valid : mine && jj < w.valid;
    if (act) {
      uint32_t idx;
      if (a.cmode == SPEED_FROM_VELOCITY) {
        const uint32_t j = BLK ? (uint32_t)cj : (uint32_t)((int64_t)w.ob * (pl.blen == inner ? 0 : pl.blen) + w.j0 + jj);
        const uint32_t d = pl.dvdiv.div(j);
        idx = d - pl.dnvl.div(d) * (uint32_t)a.nvl;
      } else {
        idx = pl.dxdiv.div((uint32_t)(w.ob + cb));
      }
      e = table[idx];
    }
    // ---- prefetched data -> LDS ----
    // (opaque here: tests on them would otherwise be kept as lane masks, and
    // addresses formed from them, in registers over the whole loop)
    if constexpr (!BLK) asm volatile("" : "+v"(edge), "+v"(i0), "+v"(loff0));
    if (by_element(t, w)) {
      const T* src = f + w.base;
#pragma unroll 1
      for (int k = 0; k < nslot; ++k) {
        const int c1 = exist(w, k);
        for (int c = 0; c < VN && c < c1; ++c) {
          const T v = src[k * gstep + goff0 + c];
          if constexpr (BLK) {
            const int e = VN * (tid + k * nact) + c, eb = e / ni;
            tile[eb * bs + G * rs + e - eb * ni] = v;
          } else {
            const int l = loff0 + k * di * rs + c, i = i0 + k * di;
            tile[l] = v;
            if (wrap_rows && i < G) tile[l + n * rs] = v;
            if (wrap_rows && i >= n - G) tile[l - n * rs] = v;
          }
        }
      }
    } else {
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (k < nslot && exist(w, k) > 0) {
          if constexpr (BLK) {
            if (ni % VN == 0) {
              put(tile + loff[k], pf[k]);
            } else {
#pragma unroll
              for (int c = 0; c < VN; ++c)
                if (c < exist(w, k)) tile[at(k, c)] = pf[k][c];
            }
          } else {
            *reinterpret_cast<V*>(tile + lds_at(k)) = pf[k];
            if (wrap_rows) {
              if (edge & (1u << k)) *reinterpret_cast<V*>(tile + lds_at(k) + n * rs) = pf[k];
              if (edge & (0x10000u << k)) *reinterpret_cast<V*>(tile + lds_at(k) - n * rs) = pf[k];
            }
          }
        }
      }
    }
    __syncthreads();
    if (periodic && !wrap_rows) {
      fill_ghosts();
      __syncthreads();
    }
    // the entry has arrived: what follows must not be waited for with it
#pragma unroll
    for (int k = 0; k < ORDER; ++k) asm volatile("" : "+v"(e.w[k]) : : "memory");
    if (t + gridDim.x < pl.tiles) {
      next = where(t + gridDim.x);
      if (!by_element(t + gridDim.x, next)) load(next);
    }
    T out[kLineMaxR<T>];
    const bool safe = __any(act && e.absN > a.nfast);
    auto sweep_once = [&]() __attribute__((always_inline)) {
      if (act) {
        if (!safe)
          advance_line<T, ORDER, LIM, false, kLineMaxR<T>>(col, rs, n, G, periodic, e, m0, R, alpha, out);
        else
          advance_line<T, ORDER, LIM, true, kLineMaxR<T>>(col, rs, n, G, periodic, e, m0, R, alpha, out);
      }
    };
    auto keep = [&]() __attribute__((always_inline)) {
      if (act) {
        T* op = col + ((e.dir > 0) ? m0 : (n - 1 - m0)) * rs;
        const int step = e.dir * rs;
#pragma unroll
        for (int k = 0; k < kLineMaxR<T>; ++k)
          if (k < R) {
            *op = out[k];
            op += step;
          }
      }
    };
    if constexpr (MODE != LINE_RK) {
      sweep_once();
      __syncthreads();
      keep();
      if constexpr (MODE == LINE_REPEAT) {
        // the closing half-kick of a step and the opening one of the next
#pragma unroll 1
        for (int rep = 1; rep < pl.reps; ++rep) {
          __syncthreads();
          if (periodic) {
            fill_ghosts();
            __syncthreads();
          }
          sweep_once();
          __syncthreads();
          keep();
        }
      }
    } else {
      // f1 = S(f), f2 = 3/4 f + 1/4 S(f1), 1/3 f + 2/3 S(f2)  (Eq. (RK))
      T fn[kLineMaxR<T>];
      if (act) {
        const T* p = col + ((e.dir > 0) ? m0 : (n - 1 - m0)) * rs;
        const int step = e.dir * rs;
#pragma unroll
        for (int k = 0; k < kLineMaxR<T>; ++k)
          if (k < R) {
            fn[k] = *p;
            p += step;
          }
      }
#pragma unroll 1
      for (int stage = 0; stage < 3; ++stage) {
        sweep_once();
        if (stage > 0) {
          const T wf = stage == 1 ? T(0.75) : T(1.0 / 3.0), ws = stage == 1 ? T(0.25) : T(2.0 / 3.0);
#pragma unroll
          for (int k = 0; k < kLineMaxR<T>; ++k)
            if (k < R) out[k] = vfma(wf, fn[k], ws * out[k]);
        }
        __syncthreads();
        keep();
        if (stage < 2) {
          __syncthreads();
          if (periodic) {
            fill_ghosts();
            __syncthreads();
          }
        }
      }
    }
    __syncthreads();
    // ---- stream the results out ----
    T* dst = f + w.base;
    const bool whole = w.valid % VN == 0;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      if (k < nslot) {
        const int c1 = exist(w, k);
        if (c1 > 0) {
          V v;
          if constexpr (BLK) {
            if (ni % VN == 0) {
              get(tile + lds_at(k), v);
            } else {
#pragma unroll
              for (int c = 0; c < VN; ++c)
                if (c < c1) v[c] = tile[at(k, c)];
            }
          } else {
            v = *reinterpret_cast<const V*>(tile + lds_at(k));
          }
          T* p = dst + k * gstep + goff0;
          if (whole || c1 >= VN) {
            if constexpr (STREAM)
              __builtin_nontemporal_store((U)v, (GlobalPtr<U>)p);
            else
              *(GlobalPtr<U>)p = (U)v;
          } else {
#pragma unroll
            for (int c = 0; c < VN; ++c)
              if (c < c1) p[c] = v[c];
          }
        }
      }
    }
    if constexpr (MODE == LINE_SUMS) {
      // row sums for the velocity moment: L lanes per tile row, as few as give
      // every thread a row (fewer lanes add more and combine less), each its
      // vectors of the row in double, compensated, combined in a fixed order
      auto row_sums = [&](auto lanes) {
        constexpr int L = decltype(lanes)::value;
        const int q = tid % L;
        for (int i = tid / L; i < n; i += blockDim.x / L) {
          const T* row = tile + (i + G) * rs;
          KSum v{0.0, 0.0};
          auto add = [&](int c0, int c1) {
            for (int c = c0; c < c1; c += L * VN) {
              const V x = *reinterpret_cast<const V*>(row + c);
              if (c + VN <= w.valid) {
                kadd(v, vsum(x));
              } else {
#pragma unroll
                for (int m = 0; m < VN; ++m)
                  if (c + m < w.valid) kadd(v, (double)x[m]);
              }
            }
          };
          // neighbouring rows begin at different vectors, on different banks
          const int first = L < 16 && w.valid > 4 * L * VN ? (i & 3) * L * VN : 0;
          add(first + q * VN, w.valid);
          if (L < 16) add(q * VN, first);
          if (L > 8) merge_dpp<kRowMirror>(v);
          if (L > 4) merge_dpp<kHalfMirror>(v);
          merge_dpp<kQuadReverse>(v);
          merge_dpp<kPairSwap>(v);
          if (q == 0) *reinterpret_cast<double2*>(a.mom + 2 * (t * n + i)) = make_double2(v.s, v.c);
        }
      };
      if (4 * n >= (int)blockDim.x)
        row_sums(std::integral_constant<int, 4>{});
      else if (8 * n >= (int)blockDim.x)
        row_sums(std::integral_constant<int, 8>{});
      else
        row_sums(std::integral_constant<int, 16>{});
      __syncthreads();
    }
    // (otherwise no barrier: the next tile first writes this thread's own
    // vectors, at the offsets it has just read, and ghost cells)
  }
}

template <typename T, int ORDER, int LIM, bool BLK, int MODE, bool STREAM = true>
hipError_t launch_t(const SweepArgs& a, const LinePlan& p, const void* table, hipStream_t s) {
  auto kern = line_sweep_kernel<T, ORDER, LIM, BLK, MODE, STREAM>;
  const void* fn = reinterpret_cast<const void*>(kern);
  hipError_t e = hipSuccess;
  if (p.lds_bytes > 64 * 1024)
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds_bytes);
  int64_t grid = 0;
  if (e == hipSuccess) e = resident_grid(fn, p.threads, p.lds_bytes, p.tiles, INT_MAX, &grid);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(p.threads), p.lds_bytes, s, a, p,
                     reinterpret_cast<const PencilEntry<T>*>(table));
  return hipGetLastError();
}

template <typename T, int ORDER, int LIM>
hipError_t launch_l(const SweepArgs& a, const LinePlan& p, const void* table, hipStream_t s) {
  if (a.rk) {
    if (p.K) return launch_t<T, ORDER, LIM, true, LINE_RK>(a, p, table, s);
    return p.stream ? launch_t<T, ORDER, LIM, false, LINE_RK>(a, p, table, s)
                    : launch_t<T, ORDER, LIM, false, LINE_RK, false>(a, p, table, s);
  }
  if (p.K && p.reps > 1) return launch_t<T, ORDER, LIM, true, LINE_REPEAT>(a, p, table, s);
  if (p.K) return launch_t<T, ORDER, LIM, true, LINE_ONE>(a, p, table, s);
  if (a.mom)
    return p.stream ? launch_t<T, ORDER, LIM, false, LINE_SUMS>(a, p, table, s)
                    : launch_t<T, ORDER, LIM, false, LINE_SUMS, false>(a, p, table, s);
  return p.stream ? launch_t<T, ORDER, LIM, false, LINE_ONE>(a, p, table, s)
                  : launch_t<T, ORDER, LIM, false, LINE_ONE, false>(a, p, table, s);
}

template <typename T, int ORDER>
hipError_t launch_o(int limiter, const SweepArgs& a, const LinePlan& p, const void* table, hipStream_t s) {
  switch (limiter) {
    case SLMPP_LIM_NONE: return launch_l<T, ORDER, SLMPP_LIM_NONE>(a, p, table, s);
    case SLMPP_LIM_MP: return launch_l<T, ORDER, SLMPP_LIM_MP>(a, p, table, s);
    default: return launch_l<T, ORDER, SLMPP_LIM_MPP>(a, p, table, s);
  }
}

}  // namespace

LinePlan plan_line(int dtype, int order, const SweepArgs& a, int64_t moment_block) {
  LinePlan p{};
  const int es = dtype == SLMPP_F64 ? 8 : 4, vn = 16 / es;
  const int64_t n = a.n, inner = a.inner, outer = a.npen / a.inner;
  // 32-bit index arithmetic in the kernel; whole vectors per block
  if (a.npen >= ((int64_t)1 << 31) || inner >= ((int64_t)1 << 31) || n * inner < vn ||
      a.fmulti != nullptr || a.fout != nullptr || a.fblend != nullptr)
    return p;
  p.G = (order == 7 ? 4 : 3) + a.nfast;
  const int maxr = es == 4 ? kLineMaxR<float> : kLineMaxR<double>;
  // cells per thread: as many as the kernel takes where there are threads
  // enough, fewer on small grids, whose time is the latency of one thread's
  // segment
  const int64_t cells = a.npen * n;
  const int Rt = cells >= ((int64_t)1 << 22) ? maxr
                 : (cells >= ((int64_t)1 << 19) || moment_block > 0 ? 8 : 4);
  const int64_t percell = (n + 2 * p.G) * es;  // LDS bytes per pencil
  int S = 0, pwmax = 0;
  auto tile_of = [&](int threads, int rt) {
    S = (int)((n + rt - 1) / rt);
    if (S > threads / vn) S = (int)((n + maxr - 1) / maxr);
    if (S > threads / vn) return false;
    p.R = (int)((n + S - 1) / S);
    S = (int)((n + p.R - 1) / p.R);
    p.S = S;
    pwmax = std::min<int>(threads / S, (int)std::max<int64_t>(kLineLds / percell, 1));
    return true;
  };
  auto waves = [&](int64_t pencils) { return (int)((pencils * S + 63) / 64); };
  int threads = a.rk ? kLineThreadsSmall : kLineThreads;
  if (!tile_of(threads, Rt)) return p;
  // block tiles: whole blocks of few pencils; row tiles where one block needs
  // more threads than there are, overflows the LDS, or is of many pencils and
  // fills five wavefronts
  const bool blk = moment_block <= 0 && inner <= std::max(pwmax, 48) && inner * S <= threads &&
                   inner * percell + 32 * es <= (int64_t)kLineLdsMax && !(inner > 48 && waves(inner) == kUneven);
  // row tiles narrower than 64 bytes take longer segments
  if (!blk && pwmax * es < 64 && Rt == 8 && maxr > 8 && cells >= ((int64_t)1 << 19) && !tile_of(threads, maxr))
    return LinePlan{};
  if (blk && es == 8 && !a.rk) {
    const LinePlan wide = p;
    const int S0 = S, pw0 = pwmax;
    if (tile_of(kLineThreadsSmall, Rt) && pwmax >= inner) {
      threads = kLineThreadsSmall;
    } else {
      p = wide;
      S = S0;
      pwmax = pw0;
    }
  }
  // workgroups wanted before tiles grow: two per CU
  constexpr int64_t kWant = 512;
  if (blk) {
    p.K = (int)std::max<int64_t>(1, pwmax / inner);
    while (p.K > 1 && (outer + p.K - 1) / p.K < kWant && p.K * inner * S > 64) p.K = (p.K + 1) / 2;
    p.pw = (int)(p.K * inner);
    p.rs = (int)inner;
    p.bs = (int)((n + 2 * p.G) * inner);
    if (inner == 1) {
      p.bs |= 1;  // the lanes of a wavefront on distinct banks
    } else {
      while (p.bs % 32 != (int)inner % 32) ++p.bs;
    }
    if ((int64_t)p.pw * S > threads) return LinePlan{};
    p.blocks = outer;
    p.tiles = (outer + p.K - 1) / p.K;
    p.lds_elems = p.K * p.bs;
    p.W = p.pw;
    p.blen = (int)inner;
    p.tpb = 1;
  } else {
    p.blen = (int)(moment_block > 0 ? moment_block : inner);
    p.blocks = a.npen / p.blen;
    p.bstride = moment_block > 0 ? moment_block : n * inner;
    // rows of whole 64-byte pieces where every row starts on one
    const int line = 64 / es;
    const bool lines = inner % line == 0 && p.blen % line == 0 &&
                       (moment_block <= 0 || cells * es > ((int64_t)1 << 25));
    int w = std::max(vn, pwmax / vn * vn);
    if (lines && w >= line) w = w / line * line;
    int64_t tpb = (p.blen + w - 1) / w;
    auto width = [&](int64_t tb) {
      const int x = (int)(((p.blen + tb - 1) / tb + vn - 1) / vn * vn);
      return lines && x > line ? (x + line - 1) / line * line : x;
    };
    // (row sums: fewer, wider tiles, whose sums the field solve adds up)
    const int least = moment_block > 0 ? 64 : (Rt > 4 ? line : 8);
    while (tpb * p.blocks < kWant && width(2 * tpb) >= least && width(2 * tpb) * S >= 64) tpb *= 2;
    if (waves(width(tpb)) == kUneven)
      while (width(tpb) > least && waves(width(tpb)) >= kUneven) ++tpb;
    p.W = width(tpb);
    p.tpb = (int)((p.blen + p.W - 1) / p.W);
    p.pw = p.W;
    p.rs = p.W;
    p.tiles = (int64_t)p.tpb * p.blocks;
    p.lds_elems = (int)((n + 2 * p.G) * p.W);
    if (p.tiles >= ((int64_t)1 << 31)) return LinePlan{};
    p.dtpb = FastDiv32::of((uint32_t)p.tpb);
  }
  p.threads = (p.pw * S + 63) / 64 * 64;
  const size_t lds = ((size_t)p.lds_elems * es + 15) & ~(size_t)15;
  if (lds > kLineLdsMax || p.threads > threads) return LinePlan{};
  p.dvdiv = FastDiv32::of((uint32_t)std::max<int64_t>(1, std::min<int64_t>(a.vdiv, 0x7fffffff)));
  p.dnvl = FastDiv32::of((uint32_t)std::max(1, a.nvl));
  p.dxdiv = FastDiv32::of((uint32_t)std::max<int64_t>(1, std::min<int64_t>(a.xdiv, 0x7fffffff)));
  // Nontemporal accesses, but for rows that share lines with the rows of the
  // next tile, on grids beyond the L2: those lines would be fetched and written
  // twice (n 64, s 250, 3e7 cells FP32: 80 us nontemporal, 60 through the caches;
  // 1000-cell pencils, s 64, FP64 TVD-RK 237 / 136; 30x37 x 54x61 FP32, in L2,
  // 84 / 86 per step).
  p.stream = cells * es <= ((int64_t)1 << 25) || p.W * es >= 512;
  p.reps = 1;
  p.lds_bytes = lds;
  return p;
}

hipError_t launch_line_sweep(int dtype, int order, int limiter, const SweepArgs& a,
                             const LinePlan& p, const void* table, hipStream_t s) {
  if (p.lds_bytes == 0) return hipErrorInvalidValue;
  if (dtype == SLMPP_F64)
    return order == 7 ? launch_o<double, 7>(limiter, a, p, table, s) : launch_o<double, 5>(limiter, a, p, table, s);
  return order == 7 ? launch_o<float, 7>(limiter, a, p, table, s) : launch_o<float, 5>(limiter, a, p, table, s);
}

}  // namespace slmpp
