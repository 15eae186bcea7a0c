// Sweep kernels of one storage type and their launches (see sweep.hip); the
// translation units sweep_f32.hip and sweep_f64.hip each instantiate one
// SweepLaunch, so that the two compile side by side.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>

#include "slmpp_internal.hpp"
#include "sweep_device.hpp"
#include "sweep_launch.hpp"

namespace slmpp {
namespace {

// Result vector v of the elements at offset off from f: blended with
// fblend and stored to fout or f (see SweepArgs; STAGE false: plain store
// to f, for kernels that never run a TVD-RK stage); 16-byte aligned.
template <bool STAGE = true, typename T, typename V>
__device__ __forceinline__ void emit_vec(const SweepArgs& a, T* f, int64_t off, V v) {
  constexpr int VN = sizeof(V) / sizeof(T);
  if (!STAGE) {
    __builtin_nontemporal_store(v, reinterpret_cast<V*>(f + off));
    return;
  }
  if (a.fblend) {
    const T cb = (T)a.cb, cf = (T)a.cf;
    const V b = __builtin_nontemporal_load(
        reinterpret_cast<const V*>(reinterpret_cast<const T*>(a.fblend) + off));
#pragma unroll
    for (int c = 0; c < VN; ++c) v[c] = vfma(cb, b[c], cf * v[c]);
  }
  T* dst = a.fout ? reinterpret_cast<T*>(a.fout) : f;
  __builtin_nontemporal_store(v, reinterpret_cast<V*>(dst + off));
}
// emit_vec for the vector `lane` of a row at the wave-uniform element
// offset uoff
template <typename T, typename V>
__device__ __forceinline__ void emit_vec_row(const SweepArgs& a, T* f, int64_t uoff, int lane, V v) {
  constexpr int VN = sizeof(V) / sizeof(T);
  if (a.fblend) {
    const T cb = (T)a.cb, cf = (T)a.cf;
    const V b = global_load_nt(reinterpret_cast<const V*>(reinterpret_cast<const T*>(a.fblend) + uoff) + lane);
#pragma unroll
    for (int c = 0; c < VN; ++c) v[c] = vfma(cb, b[c], cf * v[c]);
  }
  T* dst = a.fout ? reinterpret_cast<T*>(a.fout) : f;
  global_store_nt(v, reinterpret_cast<V*>(dst + uoff) + lane);
}
template <bool STAGE = true, typename T>
__device__ __forceinline__ void emit_one(const SweepArgs& a, T* f, int64_t off, T v) {
  if (!STAGE) {
    f[off] = v;
    return;
  }
  if (a.fblend) v = vfma((T)a.cb, reinterpret_cast<const T*>(a.fblend)[off], (T)a.cf * v);
  (a.fout ? reinterpret_cast<T*>(a.fout) : f)[off] = v;
}

// a / b for non-negative 64-bit values, in 32-bit arithmetic when both fit
__device__ __forceinline__ int64_t udiv(int64_t a, int64_t b) {
  if (((a | b) >> 31) == 0) return (int64_t)((uint32_t)a / (uint32_t)b);
  return a / b;
}

// LDS tile layouts.  Strided axis: row-major [cell][pencil] with pitch W
// (a tile row is W consecutive elements of f; lanes of a wave read W
// different pencils of one row, so every bank is distinct).  Contiguous
// axis: pencil-major [pencil][cell] with an odd pitch (W pencils are W*n
// consecutive elements of f; lanes reading cell r of W pencils hit
// distinct banks).  Both layouts carry G ghost cells before and after each
// pencil.
// RC: cells per thread (0: runtime segment length).  WT: pencils per tile
// as a compile-time constant (0: runtime), which turns the thread -> (pencil,
// segment) and vector -> (row, column) maps into shifts and multiplies.
template <typename T, int ORDER, int LIM, int RC, int WT, bool STAGE = true>
__device__ __forceinline__ void sweep_tile(const SweepArgs& a, const SweepPlan& pl,
                                           const PencilEntry<T>* __restrict__ table,
                                           int64_t tile_index, unsigned char* smem) {
  using V = typename Vec<T>::type;
  constexpr int VN = Vec<T>::N;
  const int n = a.n, G = pl.G, P = pl.pitch;
  const int W = WT > 0 ? WT : pl.W;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const bool periodic = a.bc == SLMPP_BC_PERIODIC;
  const bool contiguous = a.inner == 1;
  // element offset of ghost-extended cell g (0 <= g < n+2G) of pencil jj
  // in the tile: contiguous jj*P + g, strided g*W + jj
  const int cstride = contiguous ? 1 : W;  // between cells of a pencil
  const int pstride = contiguous ? P : 1;  // between pencils
  const int tile_elems = contiguous ? W * P : (n + 2 * G) * W;
  T* tile = reinterpret_cast<T*>(smem);
  const size_t tile_bytes = ((size_t)tile_elems * sizeof(T) + 15) & ~(size_t)15;
  PencilEntry<T>* ent = reinterpret_cast<PencilEntry<T>*>(smem + tile_bytes);
  T* tout = reinterpret_cast<T*>(ent + W);  // RC == 0 only: tile_elems
  T* f = reinterpret_cast<T*>(a.f);
  const T alpha = (T)a.alpha;

  const int64_t p0 = tile_index * W;
  const int wv = (int)min<int64_t>(W, a.npen - p0);
  const bool block = !contiguous && (a.inner % W == 0);
  int64_t gbase = 0, o0 = 0, j0 = 0;
  if (contiguous) {
    gbase = p0 * n;
  } else if (block) {
    o0 = udiv(p0, a.inner);
    j0 = p0 - o0 * a.inner;
    gbase = o0 * (int64_t)n * a.inner + j0;
  }

  // ---- per-pencil table entry ------------------------------------------
  int need_safe = 0;
  for (int jj = tid; jj < W; jj += nthr) {
    if (jj < wv) {
      const int64_t p = p0 + jj;
      int64_t o, j;
      if (contiguous) {
        o = p;
        j = 0;
      } else if (block) {
        o = o0;
        j = j0 + jj;
      } else {
        o = udiv(p, a.inner);
        j = p - o * a.inner;
      }
      const int64_t idx = a.cmode == SPEED_FROM_VELOCITY ? udiv(j, a.vdiv) % a.nvl : udiv(o, a.xdiv);
      const PencilEntry<T>* src = table + idx;
      ent[jj] = *src;
      need_safe |= src->absN > a.nfast;
    } else {
      ent[jj].z = T(0);
      ent[jj].tz = T(0);
      ent[jj].base = 0;
      ent[jj].dir = 1;
      ent[jj].absN = 0;
    }
  }

  // ---- stream the tile in: global -> LDS ------------------------------------
  // Loads are issued in batches of KB vectors per thread before any of them
  // is written to LDS, so each thread keeps KB requests in flight.  Whole
  // vectors of f are loaded and stored nontemporally (read and written once).
  constexpr int KB = 6;
  const bool vec_strided = block && (W % VN) == 0 && (a.inner % VN) == 0 && (gbase % VN) == 0 &&
                           (nthr % (W / VN)) == 0;
  // strided periodic tiles with G <= n fill their ghost rows while staging
  // (the generic strided path needs every pencil column loaded: nthr % W == 0)
  const bool wrap_rows = !contiguous && periodic && G <= n && (vec_strided || (nthr % W) == 0);
  if (contiguous) {
    const int total = wv * n;
    if ((n % VN) == 0) {
      // vector e4 holds cells i..i+VN-1 of pencil jj (n % VN == 0: never split)
      const int nvec = total / VN;
      const int stepE = nthr * VN;
      const int dj = stepE / n, di = stepE - dj * n;
      int jj = (tid * VN) / n, i = tid * VN - jj * n;
      const V* src = reinterpret_cast<const V*>(f + gbase);
      for (int b0 = tid; b0 < nvec; b0 += KB * nthr) {
        V buf[KB];
#pragma unroll
        for (int k = 0; k < KB; ++k)
          if (b0 + k * nthr < nvec) buf[k] = __builtin_nontemporal_load(src + b0 + k * nthr);
#pragma unroll
        for (int k = 0; k < KB; ++k) {
          if (b0 + k * nthr < nvec) {
            put(tile + jj * P + G + i, buf[k]);
            i += di;
            jj += dj;
            if (i >= n) {
              i -= n;
              ++jj;
            }
          }
        }
      }
    } else {
      for (int e2 = tid; e2 < total; e2 += nthr) {
        const int jj = e2 / n, i = e2 - jj * n;
        tile[jj * P + G + i] = f[gbase + e2];
      }
    }
  } else if (vec_strided) {
    const int cpr = W / VN;  // vectors per row; nthr % cpr == 0
    const int c = tid % cpr;
    const int di = nthr / cpr;
    const int i0 = tid / cpr;
    const T* gp = f + gbase + (int64_t)i0 * a.inner + c * VN;
    const int64_t gstep = (int64_t)di * a.inner;
    for (int ib = i0; ib < n; ib += KB * di, gp += KB * gstep) {
      V buf[KB];
#pragma unroll
      for (int k = 0; k < KB; ++k)
        if (ib + k * di < n)
          buf[k] = __builtin_nontemporal_load(reinterpret_cast<const V*>(gp + k * gstep));
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        if (ib + k * di < n) {
          const int i = ib + k * di;
          V* dst = reinterpret_cast<V*>(tile + (i + G) * W + c * VN);
          *dst = buf[k];
          if (wrap_rows) {
            if (i < G) *reinterpret_cast<V*>(tile + (i + G + n) * W + c * VN) = buf[k];
            if (i >= n - G) *reinterpret_cast<V*>(tile + (i + G - n) * W + c * VN) = buf[k];
          }
        }
      }
    }
  } else {
    // generic strided tile: thread -> fixed pencil column, rows stepped
    const int jj = tid % W;
    if (jj < wv && (nthr % W) == 0) {
      const int64_t p = p0 + jj;
      const int64_t o = udiv(p, a.inner);
      const T* gp = f + o * (int64_t)n * a.inner + (p - o * a.inner);
      const int di = nthr / W;
      for (int ib = tid / W; ib < n; ib += KB * di) {
        T buf[KB];
#pragma unroll
        for (int k = 0; k < KB; ++k)
          if (ib + k * di < n) buf[k] = gp[(int64_t)(ib + k * di) * a.inner];
#pragma unroll
        for (int k = 0; k < KB; ++k) {
          if (ib + k * di < n) {
            const int i = ib + k * di;
            tile[(i + G) * W + jj] = buf[k];
            if (wrap_rows) {
              if (i < G) tile[(i + G + n) * W + jj] = buf[k];
              if (i >= n - G) tile[(i + G - n) * W + jj] = buf[k];
            }
          }
        }
      }
    }
  }
  // zero ghost cells (outflow); periodic images are copied after the barrier
  if (!periodic) {
    for (int e2 = tid; e2 < 2 * G * W; e2 += nthr) {
      const int g = e2 / W, jj = e2 - g * W;
      tile[jj * pstride + (g < G ? g : n + g) * cstride] = T(0);
    }
  }
  const bool safe = __syncthreads_or(need_safe) != 0;
  if (periodic && G > 0 && !wrap_rows) {
    for (int e2 = tid; e2 < 2 * G * W; e2 += nthr) {
      const int g = e2 / W, jj = e2 - g * W;
      const int pr = g < G ? g - G : n + (g - G);  // physical cell of the ghost
      int sp = pr < 0 ? pr + n : (pr >= n ? pr - n : pr);
      if (G > n) {  // pencils shorter than the ghost width
        sp = pr % n;
        if (sp < 0) sp += n;
      }
      tile[jj * pstride + (g < G ? g : n + g) * cstride] = tile[jj * pstride + (sp + G) * cstride];
    }
    __syncthreads();
  }

  // ---- compute: thread -> (pencil jj, segment s) -------------------------
  const int jj = tid % W;
  const int s = tid / W;
  const PencilEntry<T> e = ent[jj];
  const T* col = tile + jj * pstride + G * cstride;  // physical cell 0
  if constexpr (RC > 0) {
    T out[RC > 0 ? RC : 1];
    const int m0 = s * RC;
    const bool act = jj < wv && m0 < n;
    if (act) {
      if (!safe)
        advance<T, ORDER, LIM, READ_DIRECT, RC>(col, cstride, n, G, periodic, e, m0, RC, alpha,
                                                out, nullptr);
      else
        advance<T, ORDER, LIM, READ_SAFE, RC>(col, cstride, n, G, periodic, e, m0, RC, alpha, out,
                                              nullptr);
    }
    __syncthreads();
    if (act) {
      T* op = tile + jj * pstride + (G + ((e.dir > 0) ? m0 : (n - 1 - m0))) * cstride;
      const int ostep = e.dir * cstride;
#pragma unroll
      for (int k = 0; k < RC; ++k) {
        *op = out[k];
        op += ostep;
      }
    }
  } else {
    const int S = nthr / W;
    const int R = (n + S - 1) / S;
    const int m0 = s * R;
    const int cnt = min(n, m0 + R) - m0;
    if (jj < wv && cnt > 0) {
      T* ocol = tout + jj * pstride + G * cstride;
      if (!safe)
        advance<T, ORDER, LIM, READ_DIRECT, 0>(col, cstride, n, G, periodic, e, m0, cnt, alpha,
                                               nullptr, ocol);
      else
        advance<T, ORDER, LIM, READ_SAFE, 0>(col, cstride, n, G, periodic, e, m0, cnt, alpha,
                                             nullptr, ocol);
    }
  }
  __syncthreads();
  const T* res = RC > 0 ? tile : tout;  // same geometry as the tile

  // ---- fused velocity moment (batched 1D1V x_1 sweeps: the pencils of a
  // tile are consecutive velocity cells): each lane adds 8 consecutive
  // results of a tile row in double and stores that chunk sum at
  // mom[(p0 / 8 + chunk) n + i]; chunks of 8 for every tile width, so the
  // moment does not depend on W (W and the number of velocity cells are
  // multiples of 8 here, hence so is wv)
  if (!contiguous && a.mom != nullptr) {
    const int CPR = W / 8;
    const int q = tid % CPR;
    if (8 * q < wv) {
      for (int i = tid / CPR; i < n; i += nthr / CPR) {
        const T* row = res + (i + G) * W + 8 * q;
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k) v += (double)row[k];
        a.mom[(p0 / 8 + q) * n + i] = v;
      }
    }
  }

  // ---- stream the tile out in place ---------------------------------------
  if (contiguous) {
    const int total = wv * n;
    if ((n % VN) == 0) {
      const int nvec = total / VN;
      const int stepE = nthr * VN;
      const int dj = stepE / n, di = stepE - dj * n;
      int c = (tid * VN) / n, i = tid * VN - c * n;
      for (int b0 = tid; b0 < nvec; b0 += KB * nthr) {
        V buf[KB];
#pragma unroll
        for (int k = 0; k < KB; ++k) {
          if (b0 + k * nthr < nvec) {
            get(res + c * P + G + i, buf[k]);
            i += di;
            c += dj;
            if (i >= n) {
              i -= n;
              ++c;
            }
          }
        }
#pragma unroll
        for (int k = 0; k < KB; ++k)
          if (b0 + k * nthr < nvec) emit_vec<STAGE>(a, f, gbase + (int64_t)(b0 + k * nthr) * VN, buf[k]);
      }
    } else {
      for (int e2 = tid; e2 < total; e2 += nthr) {
        const int c = e2 / n, i = e2 - c * n;
        emit_one<STAGE>(a, f, gbase + e2, res[c * P + G + i]);
      }
    }
  } else if (vec_strided) {
    const int cpr = W / VN;
    const int c = tid % cpr;
    const int di = nthr / cpr;
    const int i0 = tid / cpr;
    int64_t go = gbase + (int64_t)i0 * a.inner + c * VN;
    const int64_t gstep = (int64_t)di * a.inner;
    for (int ib = i0; ib < n; ib += KB * di, go += KB * gstep) {
      V buf[KB];
#pragma unroll
      for (int k = 0; k < KB; ++k)
        if (ib + k * di < n) buf[k] = *reinterpret_cast<const V*>(res + (ib + k * di + G) * W + c * VN);
#pragma unroll
      for (int k = 0; k < KB; ++k)
        if (ib + k * di < n) emit_vec<STAGE>(a, f, go + k * gstep, buf[k]);
    }
  } else {
    const int c = tid % W;
    if (c < wv && (nthr % W) == 0) {
      const int64_t p = p0 + c;
      const int64_t o = udiv(p, a.inner);
      const int64_t go = o * (int64_t)n * a.inner + (p - o * a.inner);
      for (int i = tid / W; i < n; i += nthr / W)
        emit_one<STAGE>(a, f, go + (int64_t)i * a.inner, res[(i + G) * W + c]);
    }
  }
}

// One tile per workgroup: pencils in segments of RC cells, or (RC 0) of a
// run-time length (see line_preferred in api.hip for the sizes).
template <typename T, int ORDER, int LIM, int RC>
__global__ void __launch_bounds__(256) sweep_kernel(SweepArgs a, SweepPlan pl,
                                                    const PencilEntry<T>* __restrict__ table) {
  extern __shared__ __align__(16) unsigned char smem[];
  sweep_tile<T, ORDER, LIM, RC, 0>(a, pl, table, (int64_t)blockIdx.x, smem);
}

// Fast path: persistent workgroups over whole tiles with software prefetch.
// f is streamed with nontemporal loads and stores (each element is read and
// written once per sweep; measured 4-5% faster than cached accesses).
// Each thread owns RC cells of one pencil and, for the data movement, RC
// elements of the tile (RC/VN vectors at fixed offsets, the same for every
// tile), so the loads of the next tile can be issued into registers before
// the current tile is computed.  Requirements checked on the host: SL-MPP,
// W divides `inner` (strided) or inner == 1 (contiguous), RC divides n,
// VN divides RC (and n when contiguous), and all pencil / cell counts of a
// block fit in 32 bits.
// Strided 256-pencil tiles (48-cell FP32 pencils) run 512 threads in two
// segments with at most 128 VGPRs, so that two workgroups share a CU: the
// register bound costs a few spilled values per tile, and the wider rows
// (1 KiB per row and tile) and the loads of two tiles in flight per CU
// make these sweeps 4-14% faster than 128-pencil tiles at 48^3 x 48^3.
template <typename T, int ORDER, int RC, int WT, bool CONTIG, bool MOM>
__global__ void __attribute__((amdgpu_flat_work_group_size(1, WT == 256 ? 512 : 256),
                               amdgpu_waves_per_eu(WT == 256 ? 4 : 1)))
sweep_fast_kernel(SweepArgs a, SweepPlan pl,
                                                         const PencilEntry<T>* __restrict__ table) {
  extern __shared__ __align__(16) unsigned char smem[];
  using V = typename Vec<T>::type;
  constexpr int VN = Vec<T>::N;
  constexpr int NV = RC / VN;  // vectors per thread and tile
  constexpr int W = WT;
  static_assert(RC % VN == 0, "segment length must be a multiple of the vector width");
  const int n = a.n, G = pl.G, P = pl.pitch;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int S = WT == 256 ? 2 : nthr / W;
  const bool periodic = a.bc == SLMPP_BC_PERIODIC;
  const int cstride = CONTIG ? 1 : W;
  const int pstride = CONTIG ? P : 1;
  const int tile_elems = CONTIG ? W * P : (n + 2 * G) * W;
  T* tile = reinterpret_cast<T*>(smem);
  const size_t tile_bytes = ((size_t)tile_elems * sizeof(T) + 15) & ~(size_t)15;
  PencilEntry<T>* ent = reinterpret_cast<PencilEntry<T>*>(smem + tile_bytes);
  T* f = reinterpret_cast<T*>(a.f);
  const T alpha = (T)a.alpha;
  const uint32_t inner = (uint32_t)a.inner;

  // per-thread element map of the data movement (identical for every tile)
  int loff[NV];       // LDS element offset of vector k
  int64_t goff0;      // global element offset of vector 0 relative to the tile
  int64_t gstep;      // between consecutive vectors of the thread
  // strided 256-pencil tiles: a row of the tile is the 64 vectors of one
  // wavefront, so the row part of each address is wave-uniform
  constexpr bool ROWWAVE = !CONTIG && W / VN == 64;
  int64_t urow = 0;   // wave-uniform row offset of vector 0
  int vlane = 0;      // vector of the lane within its row
  int vlim[NV];       // vector k exists when the tile has more than vlim[k] valid pencils
  if constexpr (CONTIG) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int e = VN * (tid + k * nthr);
      const int pj = e / n;
      loff[k] = pj * P + G + (e - pj * n);
      vlim[k] = pj;
    }
    goff0 = (int64_t)VN * tid;
    gstep = (int64_t)VN * nthr;
  } else {
    constexpr int cpr = W / VN;
    const int c = tid % cpr, i0 = tid / cpr;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      loff[k] = (i0 + k * S * VN + G) * W + c * VN;
      vlim[k] = c * VN;
    }
    goff0 = (int64_t)i0 * inner + c * VN;
    gstep = (int64_t)S * VN * inner;
    if constexpr (ROWWAVE) {
      urow = (int64_t)__builtin_amdgcn_readfirstlane(i0) * inner;
      vlane = c;
    }
  }
  // strided periodic tiles with G <= n fill their ghost rows while staging
  const bool wrap_rows = !CONTIG && periodic && G <= n;
  int i0s = 0;  // first physical row of this thread's vectors (strided)
  if constexpr (!CONTIG) i0s = tid / (W / VN);
  // zero ghost cells once: interior writes never touch them
  if (!periodic) {
    for (int e2 = tid; e2 < 2 * G * W; e2 += nthr) {
      const int g = e2 / W, c = e2 - g * W;
      tile[c * pstride + (g < G ? g : n + g) * cstride] = T(0);
    }
  }
  const int jj = tid % W;
  const int s = tid / W;
  const int m0 = s * RC;

  auto tile_base = [&](int64_t t, int& wv) -> int64_t {
    const int64_t p0 = t * W;
    wv = (int)min<int64_t>(W, a.npen - p0);
    if constexpr (CONTIG) {
      return p0 * n;
    } else {
      const uint32_t o0 = (uint32_t)p0 / inner;
      const uint32_t j0 = (uint32_t)p0 - o0 * inner;
      return (int64_t)o0 * n * inner + j0;
    }
  };

  // run and local tile of global tile tt (several runs: see SweepArgs)
  auto locate = [&](int64_t tt, int64_t& lt) -> int {
    if (a.fmulti == nullptr) {
      lt = tt;
      return 0;
    }
    const int r = (int)(tt / a.tpr);
    lt = tt - (int64_t)r * a.tpr;
    return r;
  };

  auto load_vec = [&](const T* fb, int64_t gb, int k) -> V {
    if constexpr (ROWWAVE)
      return global_load_nt(reinterpret_cast<const V*>(fb + (gb + urow + k * gstep)) + vlane);
    else
      return global_load_nt(reinterpret_cast<const V*>(fb + gb + goff0 + k * gstep));
  };

  V pf[NV];
  int64_t t = blockIdx.x;
  int wv_next = 0;
  int64_t gb_next = 0, lt_next = 0;
  int r_next = 0;
  T* f_next = f;
  if (t < pl.tiles) {
    r_next = locate(t, lt_next);
    if (a.fmulti) f_next = reinterpret_cast<T*>(a.fmulti[r_next]);
    gb_next = tile_base(lt_next, wv_next);
#pragma unroll
    for (int k = 0; k < NV; ++k)
      if (!CONTIG || vlim[k] < wv_next)
        pf[k] = load_vec(f_next, gb_next, k);
  }
  for (; t < pl.tiles; t += gridDim.x) {
    const int wv = wv_next;
    const int64_t gbase = gb_next;
    const int64_t p0 = lt_next * W;
    T* const fc = f_next;
    const PencilEntry<T>* tabc =
        a.fmulti ? reinterpret_cast<const PencilEntry<T>*>(a.tmulti[r_next]) : table;
    // ---- pencil entries of this tile ----
    int need_safe = 0;
    if (tid < W) {
      if (tid < wv) {
        uint32_t idx;
        if constexpr (CONTIG) {
          const uint32_t o = (uint32_t)(p0 + tid);
          idx = a.cmode == SPEED_FROM_VELOCITY ? 0u : o / (uint32_t)a.xdiv;
        } else {
          const uint32_t o0 = (uint32_t)p0 / inner;
          const uint32_t j = (uint32_t)p0 - o0 * inner + tid;
          idx = a.cmode == SPEED_FROM_VELOCITY ? (j / (uint32_t)a.vdiv) % (uint32_t)a.nvl
                                               : o0 / (uint32_t)a.xdiv;
        }
        const PencilEntry<T>* src = tabc + idx;
        ent[tid] = *src;
        need_safe = src->absN > a.nfast;
      } else {
        ent[tid].z = T(0);
        ent[tid].tz = T(0);
        ent[tid].base = 0;
        ent[tid].dir = 1;
        ent[tid].absN = 0;
      }
    }
    // ---- prefetched data -> LDS ----
    // (strided periodic tiles also write the first and last G rows into the
    // ghost rows on the other side, which saves a copy pass and a barrier)
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      if (!CONTIG || vlim[k] < wv) {
        put(tile + loff[k], pf[k]);
        if constexpr (!CONTIG) {
          if (wrap_rows) {
            const int i = i0s + k * S * VN;  // physical row of vector k
            if (i < G) put(tile + loff[k] + n * W, pf[k]);
            if (i >= n - G) put(tile + loff[k] - n * W, pf[k]);
          }
        }
      }
    }
    const bool safe = __syncthreads_or(need_safe) != 0;
    if (periodic && !wrap_rows) {
      for (int e2 = tid; e2 < 2 * G * W; e2 += nthr) {
        const int g = e2 / W, c = e2 - g * W;
        const int pr = g < G ? g - G : n + (g - G);
        int sp = pr < 0 ? pr + n : (pr >= n ? pr - n : pr);
        if (G > n) {
          sp = pr % n;
          if (sp < 0) sp += n;
        }
        tile[c * pstride + (g < G ? g : n + g) * cstride] = tile[c * pstride + (sp + G) * cstride];
      }
      __syncthreads();
    }
    // ---- issue the loads of the next tile ----
    if (t + gridDim.x < pl.tiles) {
      r_next = locate(t + gridDim.x, lt_next);
      if (a.fmulti) f_next = reinterpret_cast<T*>(a.fmulti[r_next]);
      gb_next = tile_base(lt_next, wv_next);
#pragma unroll
      for (int k = 0; k < NV; ++k)
        if (!CONTIG || vlim[k] < wv_next)
          pf[k] = load_vec(f_next, gb_next, k);
    }
    // ---- compute ----
    const PencilEntry<T> e = ent[jj];
    const bool act = !CONTIG || jj < wv;
    T out[RC];
    const T* col = tile + jj * pstride + G * cstride;
    if (act) {
      if (!safe)
        advance<T, ORDER, SLMPP_LIM_MPP, READ_DIRECT, RC>(col, cstride, n, G, periodic, e, m0, RC,
                                                          alpha, out, nullptr);
      else
        advance<T, ORDER, SLMPP_LIM_MPP, READ_SAFE, RC>(col, cstride, n, G, periodic, e, m0, RC,
                                                        alpha, out, nullptr);
    }
    __syncthreads();
    if (act) {
      T* op = tile + jj * pstride + (G + ((e.dir > 0) ? m0 : (n - 1 - m0))) * cstride;
      const int ostep = e.dir * cstride;
#pragma unroll
      for (int k = 0; k < RC; ++k) {
        *op = out[k];
        op += ostep;
      }
    }
    __syncthreads();
    // ---- stream the results out ----
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      if (!CONTIG || vlim[k] < wv) {
        V v;
        get(tile + loff[k], v);
        if constexpr (ROWWAVE)
          emit_vec_row(a, fc, gbase + urow + k * gstep, vlane, v);
        else
          emit_vec(a, fc, gbase + goff0 + k * gstep, v);
      }
    }
    if constexpr (MOM) {
      // fused velocity moment (strided tiles of 64, 128 or 256 pencils within
      // one velocity block): LPR lanes per tile row each add 16 of the
      // row's pencils in double (16-byte reads, start rotated by the row so
      // the lanes of a wavefront spread over the LDS banks), then the
      // partial sums are combined in a fixed order and stored per tile and
      // row
      static_assert(!CONTIG && (WT == 64 || WT == 128 || WT == 256), "fused moment needs wide strided tiles");
      constexpr int LPR = WT / 16;
      const int q = tid % LPR;
      for (int i = tid / LPR; i < n; i += nthr / LPR) {
        const T* row = tile + (i + G) * W;
        double v = 0.0;
#pragma unroll
        for (int r = 0; r < 16 / VN; ++r) {
          V x;
          get(row + ((q * 16 + r * VN + 4 * i) & (WT - 1)), x);
          v += vsum(x);
        }
#pragma unroll
        for (int off = 1; off < LPR; off <<= 1) v += __shfl_xor(v, off, LPR);
        if (q == 0) a.mom[t * n + i] = v;
      }
    }
    // the row sums read every thread's vectors: the next tile's LDS writes
    // wait for them.  Without them no barrier is needed here: the next
    // tile first writes this thread's own data-movement vectors (at the
    // offsets it has just read), ghost rows and pencil entries, none of
    // which another thread reads before the next barrier.
    if constexpr (MOM) __syncthreads();
  }
}

// The last two velocity axes of a kick in one pass.  The acceleration
// depends on x only, so all pencils along v_{D-1} of a plane
// (x, v_1..v_{D-2}) share one shift and one set of weights, and so do all
// pencils along v_D; and a plane of N x N cells is one contiguous block of
// f.  A workgroup stages PB planes at a time in LDS, each inside a ring of
// G zero cells (outflow), advances the v_{D-1} pencils, writes the results
// back into the plane, advances the v_D pencils of the updated plane and
// streams the planes out: the two sweeps one after the other, cell for
// cell, for one read and one write of f.  Persistent over tiles of PB
// consecutive planes; the next tile's data are loaded into registers
// before the current tile is computed (as in sweep_fast_kernel).
//
// Threads are segment-major: thread t advances cells s R .. s R + R - 1 of
// pencil u = t mod (PB N) (plane u / N, pencil u mod N) with s = t / (PB N),
// so that where PB N is 64 (32^2 planes in pairs, 64^2 planes) every
// wavefront holds one segment and the wave-uniform skip of the MP bounds
// (App. A steps 4-7) is lost only in the wavefronts whose segment contains
// a rejecting face.  With UNI the PB planes of a tile belong to one spatial
// cell (vouter a multiple of PB): the two pencil entries are uniform over
// the workgroup and live in scalar registers.  (Four 48^2 planes per
// workgroup with one segment per wavefront were measured slower than one
// plane per workgroup: 33-38 ms against 25 ms per pass at 48^3 x 48^3, for
// want of wavefronts per CU.)
// FP64 48^2 planes are held to 128 VGPRs (132 without): LDS fits four
// workgroups of three wavefronts per CU, and with only three wavefronts per
// SIMD their twelve fill the CU exactly, where some launches placed but three
// workgroups and ran the fourth after them (48^3 x 48^3: 78 ms in such
// launches, 51 in others; held to 128: 49 in all).
template <typename T, int ORDER, int N, int PLANES, bool UNI>
__global__ void __attribute__((amdgpu_flat_work_group_size(1, PlaneShape<T, ORDER, N, PLANES>::threads),
                               amdgpu_waves_per_eu(N == 48 && sizeof(T) == 8 ? 4 : 1)))
    kick_plane_kernel(SweepArgs a, PlanePlan pl, const PencilEntry<T>* __restrict__ tabA,
                      const PencilEntry<T>* __restrict__ tabB) {
  extern __shared__ __align__(16) unsigned char smem[];
  using V = typename Vec<T>::type;
  using Sh = PlaneShape<T, ORDER, N, PLANES>;
  constexpr int VN = Vec<T>::N;
  constexpr int R = Sh::R, S = Sh::S, PB = Sh::PB, NT = Sh::threads;
  constexpr int G = Sh::G, P = Sh::P, PS = Sh::PS;
  constexpr int NN = N * N;
  constexpr int PN = PB * N;                // pencils of one segment row of the tile
  constexpr int NVEC = PB * NN / VN;       // 16-byte vectors per tile
  constexpr int NV = (NVEC + NT - 1) / NT;  // per thread
  static_assert(N % VN == 0 && N % R == 0 && PB >= 1 && NT <= 1024, "plane shape");
  const int tid = threadIdx.x;
  T* lds = reinterpret_cast<T*>(smem);
  T* f = reinterpret_cast<T*>(a.f);
  const T alpha = (T)a.alpha;
  // zero the planes with their rings once (interior writes never touch the
  // rings); the barrier orders these stores before the first tile's data
  for (int e = tid; e < PB * PS; e += NT) lds[e] = T(0);
  __syncthreads();
  // data movement map: vector k of this thread is tile vector tid + NT k, in
  // plane plane_of(k) (PB: none) at LDS offset off_of(k).  Where NT vectors
  // are whole rows and planes whole multiples of them, both follow from k at
  // compile time and one register holds the map: FP64 48^2 planes 53.2 -> 49.3
  // ms at 48^3 x 48^3 (no values spilled under their bound of 128 VGPRs,
  // instead of 8), 64^2 562 -> 455 us at 12^3 x 20x64^2 and FP32 230 -> 212,
  // FP64 32^2 605 -> 530 at 20^3 x 20x32^2.  FP32 32^2 and 48^2 planes, whose
  // registers do not bound them, are 3-8% slower so (262 against 243 us).
  constexpr bool STEP = (sizeof(T) == 8 || N == 64) && NN % (VN * NT) == 0 && (VN * NT) % N == 0;
  int loff[STEP ? 1 : NV], vq[STEP ? 1 : NV];
#pragma unroll
  for (int k = 0; k < (STEP ? 1 : NV); ++k) {
    const int v = tid + NT * k;
    if (v < NVEC) {
      const int e = v * VN;
      const int q = e / NN, rem = e - q * NN;
      const int ia = rem / N, ib = rem - ia * N;
      loff[k] = q * PS + (ia + G) * P + G + ib;
      vq[k] = q;
    } else {
      loff[k] = 0;
      vq[k] = PB;
    }
  }
  auto plane_of = [&](int k) __attribute__((always_inline)) -> int {
    return STEP ? k * VN * NT / NN : vq[STEP ? 0 : k];
  };
  auto off_of = [&](int k) __attribute__((always_inline)) -> int {
    return STEP ? loff[0] + k * VN * NT / NN * PS + k * VN * NT % NN / N * P : loff[STEP ? 0 : k];
  };
  // compute map (segment-major): plane cq, pencil cj, cells m0 .. m0 + R - 1
  // of segment s.  With four segments and a wavefront holding parts of two,
  // the segments are laid out in the order 2, 0, 3, 1 (wavefronts hold
  // segments 2 and 0, 0 and 3, 3 and 1), so that a wavefront's lanes fail
  // the early MP accept at few distinct processing positions for a profile
  // with its extremum at the pencil's centre and zero ghost cells at both
  // ends: segment 2 (starting at the centre) fails at its first two faces,
  // segment 0 (inflow) at its first, segment 1 (ending at the centre) at its
  // last, segment 3 (outflow) rarely.  Which lane computes which
  // (segment, pencil) does not change any result.
  const int sl = tid / PN;
  const int s = S == 4 ? (0x1302 >> (4 * sl)) & 15 : sl;
  const int u = tid - sl * PN;
  const int cq = u / N;
  const int cj = u - cq * N;
  const int m0 = s * R;
  const T* colA = lds + cq * PS + G * P + G + cj;    // along v_{D-1}: stride P
  const T* colB = lds + cq * PS + (G + cj) * P + G;  // along v_D: stride 1

  V pf[NV];
  // several runs of one geometry (batched ensembles): tile tt belongs to
  // run tt / tpr with f fmulti[r] and tables tmulti[r] (v_{D-1}) and
  // tmulti[nrun + r] (v_D); pl.planes counts the planes of one run
  const int64_t nrun = a.fmulti ? pl.tiles / a.tpr : 1;
  int np_next = 0;
  int64_t p0_next = 0;
  T* f_next = f;
  const PencilEntry<T>* ta_next = tabA;
  const PencilEntry<T>* tb_next = tabB;
  auto issue = [&](int64_t tt) __attribute__((always_inline)) {
    int64_t lt = tt;
    ta_next = tabA;
    tb_next = tabB;
    if (a.fmulti) {
      const int64_t r = tt / a.tpr;
      lt = tt - r * a.tpr;
      f_next = reinterpret_cast<T*>(load_ptr_uniform(a.fmulti + r));
      ta_next = reinterpret_cast<const PencilEntry<T>*>(load_ptr_uniform(a.tmulti + r));
      tb_next = reinterpret_cast<const PencilEntry<T>*>(load_ptr_uniform(a.tmulti + nrun + r));
    }
    p0_next = lt * PB;
    np_next = (int)min<int64_t>(PB, pl.planes - p0_next);
    const V* src = reinterpret_cast<const V*>(f_next + p0_next * NN);
#pragma unroll
    for (int k = 0; k < NV; ++k)
      if (plane_of(k) < np_next) pf[k] = __builtin_nontemporal_load(src + tid + NT * k);
  };
  int64_t t = blockIdx.x;
  if (t < pl.tiles) issue(t);
  for (; t < pl.tiles; t += gridDim.x) {
    const int np = np_next;
    const int64_t p0 = p0_next;
    T* const fc = f_next;
    const bool act = cq < np;
    // the two pencil entries of this thread's plane (with UNI: of every
    // plane of the tile, read with scalar loads), requested before the
    // tile's data go to LDS
    PencilEntry<T> eA{}, eB{};
    if (UNI || act) {
      const int64_t pp = UNI ? p0 : p0 + cq;
      const int64_t ix = pl.vdiv.m ? (int64_t)pl.vdiv.div((uint32_t)pp) : udiv(pp, pl.vouter);
      eA = load_entry_uniform(ta_next + ix);
      eB = load_entry_uniform(tb_next + ix);
    }
#pragma unroll
    for (int k = 0; k < NV; ++k)
      if (plane_of(k) < np) put(lds + off_of(k), pf[k]);
    __syncthreads();
    if (t + gridDim.x < pl.tiles) issue(t + gridDim.x);
    T out[R];
    // v_{D-1}
    if (act) {
      if (eA.absN <= kPlaneFast) {
        if (eA.dir > 0)
          advance_ct<T, ORDER, R, P, 1>(colA, eA, m0, alpha, out);
        else
          advance_ct<T, ORDER, R, P, -1>(colA, eA, m0, alpha, out);
      } else {
        advance<T, ORDER, SLMPP_LIM_MPP, READ_SAFE, R>(colA, P, N, G, 0, eA, m0, R, alpha, out,
                                                        nullptr);
      }
    }
    __syncthreads();
    if (act) {
      if (eA.dir > 0)
        store_ct<T, R, P, 1>(const_cast<T*>(colA), N, m0, out);
      else
        store_ct<T, R, P, -1>(const_cast<T*>(colA), N, m0, out);
    }
    __syncthreads();
    // v_D on the updated plane
    if (act) {
      if (eB.absN <= kPlaneFast) {
        if (eB.dir > 0)
          advance_ct<T, ORDER, R, 1, 1>(colB, eB, m0, alpha, out);
        else
          advance_ct<T, ORDER, R, 1, -1>(colB, eB, m0, alpha, out);
      } else {
        advance<T, ORDER, SLMPP_LIM_MPP, READ_SAFE, R>(colB, 1, N, G, 0, eB, m0, R, alpha, out,
                                                        nullptr);
      }
    }
    __syncthreads();
    if (act) {
      if (eB.dir > 0)
        store_ct<T, R, 1, 1>(const_cast<T*>(colB), N, m0, out);
      else
        store_ct<T, R, 1, -1>(const_cast<T*>(colB), N, m0, out);
    }
    __syncthreads();
    V* dst = reinterpret_cast<V*>(fc + p0 * NN);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      if (plane_of(k) < np) {
        V v;
        get(lds + off_of(k), v);
        __builtin_nontemporal_store(v, dst + tid + NT * k);
      }
    }
    // no barrier before the next tile: its first LDS writes are this
    // thread's own data-movement vectors, at the offsets it has just read
  }
}

// The tables of several sweeps in one launch (grid.y = table).
template <typename T, int ORDER>
__global__ void __launch_bounds__(128) pencil_table_kernel(TableJobs jobs) {
  const int y = blockIdx.y;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < jobs.count[y])
    reinterpret_cast<PencilEntry<T>*>(jobs.tab[y])[idx] = pencil_entry<T, ORDER>(jobs.a[y], idx);
}

template <typename T, int ORDER, int LIM, int RC>
hipError_t launch_k(const SweepArgs& a, const SweepPlan& p, const void* table, hipStream_t s) {
  auto kern = sweep_kernel<T, ORDER, LIM, RC>;
  if (p.lds_bytes > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)p.lds_bytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)p.tiles), dim3(p.threads), p.lds_bytes, s, a, p,
                     reinterpret_cast<const PencilEntry<T>*>(table));
  return hipGetLastError();
}

template <typename T, int ORDER, int RC, int WT, bool CONTIG, bool MOM = false>
hipError_t launch_fast(const SweepArgs& a, const SweepPlan& p, const void* table, hipStream_t s) {
  auto kern = sweep_fast_kernel<T, ORDER, RC, WT, CONTIG, MOM>;
  if (p.lds_bytes > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)p.lds_bytes);
    if (e != hipSuccess) return e;
  }
  int64_t grid = 0;
  const hipError_t e =
      resident_grid(reinterpret_cast<const void*>(kern), p.threads, p.lds_bytes, p.tiles, INT_MAX, &grid);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(p.threads), p.lds_bytes, s, a, p,
                     reinterpret_cast<const PencilEntry<T>*>(table));
  return hipGetLastError();
}

// SL-MPP sweeps in segments of RC cells: the persistent kernel with the plan's
// width, or one tile per workgroup
template <typename T, int ORDER, int RC>
hipError_t launch_w(const SweepArgs& a, const SweepPlan& p, const void* table, hipStream_t s) {
  if constexpr (RC == 32) {  // strided 128-pencil tiles of 64-cell pencils only
    if (!p.fast || a.inner == 1 || p.W != 128) return hipErrorInvalidValue;
    if (a.mom) return launch_fast<T, ORDER, RC, 128, false, true>(a, p, table, s);
    return launch_fast<T, ORDER, RC, 128, false>(a, p, table, s);
  } else {
    if (!p.fast) return launch_k<T, ORDER, SLMPP_LIM_MPP, RC>(a, p, table, s);
    if (a.inner == 1) return launch_fast<T, ORDER, RC, 64, true>(a, p, table, s);
    switch (p.W) {
      case 256:
        if constexpr (RC == 24 && ORDER == 7 && sizeof(T) == 4) {
          if (a.mom) return launch_fast<T, ORDER, RC, 256, false, true>(a, p, table, s);
          return launch_fast<T, ORDER, RC, 256, false>(a, p, table, s);
        }
        break;
      case 128:
        if (a.mom) return launch_fast<T, ORDER, RC, 128, false, true>(a, p, table, s);
        return launch_fast<T, ORDER, RC, 128, false>(a, p, table, s);
      case 64:
        if (a.mom) return launch_fast<T, ORDER, RC, 64, false, true>(a, p, table, s);
        return launch_fast<T, ORDER, RC, 64, false>(a, p, table, s);
      case 48: return launch_fast<T, ORDER, RC, 48, false>(a, p, table, s);
      case 32: return launch_fast<T, ORDER, RC, 32, false>(a, p, table, s);
      default: break;
    }
    return hipErrorInvalidValue;
  }
}

template <typename T, int ORDER, int LIM>
hipError_t launch_r(const SweepArgs& a, const SweepPlan& p, const void* table, hipStream_t s) {
  if constexpr (LIM == SLMPP_LIM_MPP) {
    switch (p.R) {
      case 12: return launch_w<T, ORDER, 12>(a, p, table, s);
      case 16: return launch_w<T, ORDER, 16>(a, p, table, s);
      case 24: return launch_w<T, ORDER, 24>(a, p, table, s);
      case 32:  // planned for FP32 only
        if constexpr (sizeof(T) == 4) return launch_w<T, ORDER, 32>(a, p, table, s);
        return hipErrorInvalidValue;
      default: break;
    }
  }
  return launch_k<T, ORDER, LIM, 0>(a, p, table, s);
}

template <typename T, int ORDER>
hipError_t launch_o(int limiter, const SweepArgs& a, const SweepPlan& p, const void* table,
                    hipStream_t s) {
  if (p.tiles <= 0) return hipSuccess;
  switch (limiter) {
    case SLMPP_LIM_NONE: return launch_r<T, ORDER, SLMPP_LIM_NONE>(a, p, table, s);
    case SLMPP_LIM_MP: return launch_r<T, ORDER, SLMPP_LIM_MP>(a, p, table, s);
    default: return launch_r<T, ORDER, SLMPP_LIM_MPP>(a, p, table, s);
  }
}

// ---- grouped launches over many independent runs ----------------------
template <typename T>
__global__ void batch_table_kernel(const BatchSweep* __restrict__ sweeps) {
  const BatchSweep& b = sweeps[blockIdx.y];
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= b.count) return;
  PencilEntry<T>* tab = reinterpret_cast<PencilEntry<T>*>(b.table);
  tab[idx] = b.order == 7 ? pencil_entry<T, 7>(b.a, idx) : pencil_entry<T, 5>(b.a, idx);
}

// Persistent over work items; every item is one tile of one run's sweep,
// with its own shape, plan (256 threads) and order.  Segments of 8, 12 or
// 16 cells per thread (pl.R) take the compile-time variants, which keep a
// segment's outputs in registers; other lengths take the runtime one.
template <typename T>
__global__ void __launch_bounds__(256) batch_sweep_kernel(const BatchSweep* __restrict__ sweeps,
                                                          const BatchItem* __restrict__ items,
                                                          int nitems) {
  extern __shared__ __align__(16) unsigned char smem[];
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const BatchItem item = items[it];
    const BatchSweep& b = sweeps[item.sweep];
    const SweepArgs a = b.a;
    const SweepPlan pl = b.p;
    const PencilEntry<T>* tab = reinterpret_cast<const PencilEntry<T>*>(b.table);
    const int64_t t = item.tile;
    switch (b.order * 100 + pl.R) {
      case 508: sweep_tile<T, 5, SLMPP_LIM_MPP, 8, 0, false>(a, pl, tab, t, smem); break;
      case 512: sweep_tile<T, 5, SLMPP_LIM_MPP, 12, 0, false>(a, pl, tab, t, smem); break;
      case 516: sweep_tile<T, 5, SLMPP_LIM_MPP, 16, 0, false>(a, pl, tab, t, smem); break;
      case 708: sweep_tile<T, 7, SLMPP_LIM_MPP, 8, 0, false>(a, pl, tab, t, smem); break;
      case 712: sweep_tile<T, 7, SLMPP_LIM_MPP, 12, 0, false>(a, pl, tab, t, smem); break;
      case 716: sweep_tile<T, 7, SLMPP_LIM_MPP, 16, 0, false>(a, pl, tab, t, smem); break;
      case 700: sweep_tile<T, 7, SLMPP_LIM_MPP, 0, 0, false>(a, pl, tab, t, smem); break;
      default: sweep_tile<T, 5, SLMPP_LIM_MPP, 0, 0, false>(a, pl, tab, t, smem); break;
    }
    __syncthreads();
  }
}

template <typename T, int ORDER, int N, int PB, bool UNI>
hipError_t launch_plane_u(const SweepArgs& a, const PlanePlan& p, const void* tabA,
                          const void* tabB, hipStream_t s) {
  auto kern = kick_plane_kernel<T, ORDER, N, PB, UNI>;
  if (p.lds_bytes > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)p.lds_bytes);
    if (e != hipSuccess) return e;
  }
  constexpr int NT = PlaneShape<T, ORDER, N, PB>::threads;
  // at most seven wavefronts per SIMD: with all eight slots taken the 24^2
  // planes in twos took 390 against 319 us (24^3 x 20x24^2 FP32) and the 64^2
  // planes 207 against 180 us (15 runs of 32^2 x 64^2); 48^2 planes 20.8 ms
  // either way
  constexpr int kWaves = (NT + 63) / 64;
  int64_t grid = 0;
  const hipError_t e =
      resident_grid(reinterpret_cast<const void*>(kern), NT, p.lds_bytes, p.tiles, std::max(1, 28 / kWaves), &grid);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NT), p.lds_bytes, s, a, p,
                     reinterpret_cast<const PencilEntry<T>*>(tabA),
                     reinterpret_cast<const PencilEntry<T>*>(tabB));
  return hipGetLastError();
}

template <typename T, int ORDER>
hipError_t launch_plane_o(const SweepArgs& a, const PlanePlan& p, const void* tabA,
                          const void* tabB, hipStream_t s) {
  constexpr bool f32 = sizeof(T) == 4;
  switch (p.N * 10 + p.PB) {
    case 244:
      if constexpr (f32) return launch_plane_u<T, ORDER, 24, 4, true>(a, p, tabA, tabB, s);
      break;
    case 242:
      return p.uni ? launch_plane_u<T, ORDER, 24, 2, true>(a, p, tabA, tabB, s)
                   : launch_plane_u<T, ORDER, 24, 2, false>(a, p, tabA, tabB, s);
    case 322:
      if (p.uni) return launch_plane_u<T, ORDER, 32, 2, true>(a, p, tabA, tabB, s);
      if constexpr (f32) return launch_plane_u<T, ORDER, 32, 2, false>(a, p, tabA, tabB, s);
      break;
    case 321:
      if constexpr (!f32) return launch_plane_u<T, ORDER, 32, 1, true>(a, p, tabA, tabB, s);
      break;
    case 481: return launch_plane_u<T, ORDER, 48, 1, true>(a, p, tabA, tabB, s);
    case 641: return launch_plane_u<T, ORDER, 64, 1, true>(a, p, tabA, tabB, s);
    default: break;
  }
  return hipErrorInvalidValue;
}

}  // namespace

template <typename T>
hipError_t SweepLaunch<T>::tables(int order, const TableJobs& jobs, hipStream_t s) {
  int most = 0;
  for (int k = 0; k < jobs.n; ++k) most = std::max(most, jobs.count[k]);
  if (most <= 0) return hipSuccess;
  const dim3 grid((most + 127) / 128, jobs.n);
  if (order == 7)
    hipLaunchKernelGGL((pencil_table_kernel<T, 7>), grid, dim3(128), 0, s, jobs);
  else
    hipLaunchKernelGGL((pencil_table_kernel<T, 5>), grid, dim3(128), 0, s, jobs);
  return hipGetLastError();
}

template <typename T>
hipError_t SweepLaunch<T>::sweep(int order, int limiter, const SweepArgs& a, const SweepPlan& p,
                                 const void* tab, hipStream_t s) {
  return order == 7 ? launch_o<T, 7>(limiter, a, p, tab, s) : launch_o<T, 5>(limiter, a, p, tab, s);
}

template <typename T>
hipError_t SweepLaunch<T>::kick_plane(int order, const SweepArgs& a, const PlanePlan& p,
                                      const void* tabA, const void* tabB, hipStream_t s) {
  return order == 7 ? launch_plane_o<T, 7>(a, p, tabA, tabB, s) : launch_plane_o<T, 5>(a, p, tabA, tabB, s);
}

template <typename T>
hipError_t SweepLaunch<T>::batch_tables(const BatchSweep* sweeps, int nsweeps, int max_count,
                                        hipStream_t s) {
  hipLaunchKernelGGL(batch_table_kernel<T>, dim3((max_count + 127) / 128, nsweeps), dim3(128), 0, s,
                     sweeps);
  return hipGetLastError();
}

template <typename T>
hipError_t SweepLaunch<T>::prepare_batch(size_t lds_bytes) {
  if (lds_bytes > 64 * 1024)
    return hipFuncSetAttribute(reinterpret_cast<const void*>(batch_sweep_kernel<T>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  return hipSuccess;
}

template <typename T>
int SweepLaunch<T>::batch_blocks_per_cu(size_t lds_bytes) {
  int per_cu = 0;
  (void)prepare_batch(lds_bytes);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &per_cu, reinterpret_cast<const void*>(batch_sweep_kernel<T>), 256, lds_bytes) != hipSuccess)
    return 1;
  return per_cu > 0 ? per_cu : 1;
}

template <typename T>
hipError_t SweepLaunch<T>::batch_sweeps(const BatchSweep* sweeps, const BatchItem* items, int nitems,
                                        size_t lds_bytes, int grid, hipStream_t s) {
  hipLaunchKernelGGL(batch_sweep_kernel<T>, dim3(grid), dim3(256), lds_bytes, s, sweeps, items, nitems);
  return hipGetLastError();
}

}  // namespace slmpp
