// Field kernels: velocity moment, periodic Poisson solve with high-order
// Green functions and forces (Sec. 2.2, App. C), initialisation, and
// reductions for diagnostics.  All field arithmetic is double precision.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "slmpp_internal.hpp"

namespace slmpp {
namespace {

// ---- compensated (Neumaier) accumulation ------------------------------
struct KSum {
  double s, c;
};
__device__ __forceinline__ void kadd(KSum& a, double x) {
  const double t = a.s + x;
  if (fabs(a.s) >= fabs(x))
    a.c += (a.s - t) + x;
  else
    a.c += (x - t) + a.s;
  a.s = t;
}
__device__ __forceinline__ void kmerge(KSum& a, const KSum& b) {
  kadd(a, b.s);
  a.c += b.c;
}

template <int NT>
__device__ KSum block_ksum(KSum v) {
  __shared__ double ss[NT], sc[NT];
  ss[threadIdx.x] = v.s;
  sc[threadIdx.x] = v.c;
  __syncthreads();
  for (int off = NT / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) {
      KSum a{ss[threadIdx.x], sc[threadIdx.x]};
      KSum b{ss[threadIdx.x + off], sc[threadIdx.x + off]};
      kmerge(a, b);
      ss[threadIdx.x] = a.s;
      sc[threadIdx.x] = a.c;
    }
    __syncthreads();
  }
  KSum r{ss[0], sc[0]};
  __syncthreads();
  return r;
}

// rho[ix] = dvol * sum over the contiguous velocity block of cell ix.
// One workgroup per spatial cell; fixed reduction order (deterministic).
// When the block is a whole number of 16-byte vectors, each thread reads
// vectors (four loads in flight), adds a vector's components in double and
// feeds the sum to one of two compensated accumulators.
template <typename T>
struct MomVec;
template <>
struct MomVec<float> {
  typedef float type __attribute__((ext_vector_type(4)));
  static constexpr int N = 4;
  __device__ static double sum(type v) {
    return ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w);
  }
};
template <>
struct MomVec<double> {
  typedef double type __attribute__((ext_vector_type(2)));
  static constexpr int N = 2;
  __device__ static double sum(type v) { return v.x + v.y; }
};

template <typename T, int NT>
__global__ void __launch_bounds__(NT) moment_kernel(const T* __restrict__ f, int64_t nvs,
                                                    double dvol, double* __restrict__ rho) {
  using MV = MomVec<T>;
  using V = typename MV::type;
  const T* b = f + (int64_t)blockIdx.x * nvs;
  KSum acc0{0.0, 0.0}, acc1{0.0, 0.0};
  if (nvs % MV::N == 0) {
    const V* bv = reinterpret_cast<const V*>(b);
    const int64_t nv = nvs / MV::N;
    constexpr int U = 4;
    int64_t k = threadIdx.x;
    for (; k + (U - 1) * NT < nv; k += U * NT) {
      V x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = bv[k + u * NT];
#pragma unroll
      for (int u = 0; u < U; u += 2) {
        kadd(acc0, MV::sum(x[u]));
        kadd(acc1, MV::sum(x[u + 1]));
      }
    }
    for (; k < nv; k += NT) kadd(acc0, MV::sum(bv[k]));
  } else {
    for (int64_t k = threadIdx.x; k < nvs; k += NT) kadd(acc0, (double)b[k]);
  }
  kmerge(acc0, acc1);
  KSum tot = block_ksum<NT>(acc0);
  if (threadIdx.x == 0) rho[blockIdx.x] = dvol * (tot.s + tot.c);
}

// Exact addition: a.s + x as s plus its rounding error in c (Knuth's
// two-sum, no comparison of the magnitudes).
__device__ __forceinline__ void kadd2(KSum& a, double x) {
  const double t = a.s + x;
  const double b = t - a.s;
  a.c += (a.s - (t - b)) + (x - b);
  a.s = t;
}
__device__ __forceinline__ void kmerge2(KSum& a, const KSum& b) {
  kadd2(a, b.s);
  a.c += b.c;
}
__device__ __forceinline__ KSum shfl_ksum(const KSum& v, int off) {
  return {__shfl_xor(v.s, off, 64), __shfl_xor(v.c, off, 64)};
}
// Sum over each row of 16 lanes, in all of them: pairs by data-parallel
// permutes of the row (mirrored, its halves mirrored, its quads reversed, its
// pairs swapped), which take a few cycles where a shuffle goes through the LDS.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const int64_t b = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
}
template <int CTRL>
__device__ __forceinline__ void merge_dpp(KSum& v) {
  const KSum o{dpp<CTRL>(v.s), dpp<CTRL>(v.c)};
  kmerge2(v, o);
}
constexpr int kRowMirror = 0x140, kHalfMirror = 0x141, kQuadReverse = 0x1b, kPairSwap = 0xb1;
__device__ __forceinline__ void sum_rows(KSum& v) {
  merge_dpp<kRowMirror>(v);
  merge_dpp<kHalfMirror>(v);
  merge_dpp<kQuadReverse>(v);
  merge_dpp<kPairSwap>(v);
}
__device__ __forceinline__ double sum_rows(double v) {
  v += dpp<kRowMirror>(v);
  v += dpp<kHalfMirror>(v);
  v += dpp<kQuadReverse>(v);
  v += dpp<kPairSwap>(v);
  return v;
}

// 16-byte vectors at element-aligned addresses (the hardware takes global
// vector accesses at any 4-byte address)
template <typename T>
struct UVec;
template <>
struct UVec<float> {
  typedef float type __attribute__((ext_vector_type(4), aligned(4)));
  static constexpr int N = 4;
};
template <>
struct UVec<double> {
  typedef double type __attribute__((ext_vector_type(2), aligned(8)));
  static constexpr int N = 2;
};
// the vector at p, of which only the first `valid` elements exist (zeros for the rest)
template <typename T>
__device__ __forceinline__ typename UVec<T>::type load_part(const T* p, int64_t valid) {
  using V = typename UVec<T>::type;
  constexpr int VN = UVec<T>::N;
  if (valid >= VN) return __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
  V v{};
#pragma unroll
  for (int c = 0; c < VN; ++c)
    if (c < valid) v[c] = p[c];
  return v;
}

// Velocity moments of one spatial cell per workgroup (Sec. 2.3): density,
// mean velocity and dispersion per velocity axis, from one read of the
// cell's velocity block.  The block [n1][n2][n3] (n3 = 1 for two velocity
// axes) is summed to its marginals M_l(j_l) in LDS, and mean
// and dispersion of axis l come from M_l alone (two passes over n_l numbers,
// so nothing cancels that did not cancel in two passes over f).
//
// Bound by the read of f (and, with short planes, by the latency of its
// bursts of loads): one pass instead of two, 16-byte loads and sums without
// index arithmetic took 24^3 x 40^3 FP32 (3.5 GB) from 2414 to 868 us.
// A wavefront takes whole planes j1, its lanes the plane's 16-byte vectors
// (kMomVec per lane; what is left of a plane, or a plane narrower than a
// wavefront, is taken several j1 at a time) and kMomPlanes planes per burst
// of loads: the plane sums go to M_1(j1), and the lanes' running sums over j1
// give the marginal over (j2, j3) of the chunk, which is folded into M_2 and
// M_3.  A lane adds at most eight values plainly; every sum above that is a
// compensated pair (plain sums took 822 us of 24^3 x 40^3 FP32, these 942).
// Held to 128 VGPRs: at three wavefronts per SIMD instead of four it took 958 us; four
// vectors per lane and two planes per burst 970 us, the wavefronts of a
// workgroup sharing one spatial cell 1118 us.
// GLOB: the marginals in `marg` instead of LDS (axes too long for it).
constexpr int kMomVec = 2;
constexpr int kMomPlanes = 4;
template <typename T, int NT, bool GLOB>
__global__ void __attribute__((amdgpu_flat_work_group_size(1, NT), amdgpu_waves_per_eu(4)))
velocity_moments_kernel(const T* __restrict__ f, int D, int n1,
                                                              int n2, int n3, double3 vlo, double3 dv,
                                                              double dvol, int64_t nxs, int64_t cell0,
                                                              double* __restrict__ rho,
                                                              double* __restrict__ mean,
                                                              double* __restrict__ disp,
                                                              KSum* __restrict__ marg) {
  using V = typename UVec<T>::type;
  const int64_t cell = cell0 + blockIdx.x;
  constexpr int VN = UVec<T>::N;
  constexpr int NW = NT / 64;
  constexpr int CH = 64 * VN * kMomVec;  // plane elements of a full chunk
  extern __shared__ __align__(16) unsigned char mom_smem[];
  // LDS: the wavefronts' marginals over (j2, j3) of the current chunk, the
  // parts of M_3 of that chunk, and the marginals M_l
  const int cl = min(CH, n2 * n3);
  double* W = reinterpret_cast<double*>(mom_smem);
  KSum* Q = reinterpret_cast<KSum*>(W + NW * cl);
  KSum* M1 = Q + max(NT, n3);
  if constexpr (GLOB) M1 = marg + (int64_t)blockIdx.x * (n1 + n2 + n3);
  KSum* M2 = M1 + n1;
  KSum* M3 = M2 + n2;
  const int np = n2 * n3;
  const T* b = f + cell * n1 * np;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int k = tid; k < n1 + n2 + n3; k += NT) M1[k] = KSum{0.0, 0.0};
  __syncthreads();
  for (int c0 = 0; c0 < np; c0 += CH) {
    // lanes per plane (a power of two) and planes per wavefront pass
    int lpp = 64;
    while (lpp > 1 && (lpp / 2) * VN * kMomVec >= np - c0) lpp >>= 1;
    const int sub = 64 / lpp, sl = lane / lpp, pl = lane & (lpp - 1);
    KSum acc[kMomVec][VN];
#pragma unroll
    for (int k = 0; k < kMomVec; ++k)
#pragma unroll
      for (int c = 0; c < VN; ++c) acc[k][c] = KSum{0.0, 0.0};
    // (loads are unconditional, from the last whole vector of the plane at
    // most; off[k] says by how many elements vector k was moved down, VN or
    // more where it has no element of the plane)
    int ek[kMomVec], off_[kMomVec];
#pragma unroll
    for (int k = 0; k < kMomVec; ++k) {
      const int e = c0 + (pl + k * lpp) * VN;
      ek[k] = max(0, min(e, np - VN));
      off_[k] = e - ek[k];
    }
    const bool tails = np % VN != 0;
    for (int j0 = wave * sub + sl; j0 - sl < n1; j0 += kMomPlanes * NW * sub) {
      // kMomPlanes planes: their loads first, then each element's plain sum
      // over them into its compensated one
      V x[kMomPlanes][kMomVec];
#pragma unroll
      for (int g = 0; g < kMomPlanes; ++g) {
        const T* row = b + (int64_t)min(j0 + g * NW * sub, n1 - 1) * np;
#pragma unroll
        for (int k = 0; k < kMomVec; ++k) {
          if (np >= VN)
            x[g][k] = __builtin_nontemporal_load(reinterpret_cast<const V*>(row + ek[k]));
          else
            x[g][k] = load_part(row, np);
        }
      }
      if (tails) {
#pragma unroll
        for (int g = 0; g < kMomPlanes; ++g)
#pragma unroll
          for (int k = 0; k < kMomVec; ++k)
#pragma unroll
            for (int c = 0; c < VN; ++c) {
              T v = T(0);
#pragma unroll
              for (int q = c; q < VN; ++q) v = off_[k] == q - c ? x[g][k][q] : v;
              x[g][k][c] = v;
            }
      }
      double rs[kMomPlanes];
#pragma unroll
      for (int g = 0; g < kMomPlanes; ++g) {
        rs[g] = 0.0;
#pragma unroll
        for (int k = 0; k < kMomVec; ++k)
          if (off_[k] >= VN || j0 + g * NW * sub >= n1) x[g][k] = V{};
      }
#pragma unroll
      for (int k = 0; k < kMomVec; ++k)
#pragma unroll
        for (int c = 0; c < VN; ++c) {
          double v[kMomPlanes];
#pragma unroll
          for (int g = 0; g < kMomPlanes; ++g) {
            v[g] = (double)x[g][k][c];
            rs[g] += v[g];
          }
          kadd2(acc[k][c], (v[0] + v[1]) + (v[2] + v[3]));
        }
      // the planes' sums over the lanes; this wavefront's own M_1(j1)
      if (lpp == 64) {
        // four sums at once: halves of the wavefront swap pairs, quarters
        // single sums, and 16 lanes add up one plane each
        const bool h = lane & 32, q = lane & 16;
        KSum u0{h ? rs[2] : rs[0], 0.0}, u1{h ? rs[3] : rs[1], 0.0};
        kadd2(u0, __shfl_xor(h ? rs[0] : rs[2], 32, 64));
        kadd2(u1, __shfl_xor(h ? rs[1] : rs[3], 32, 64));
        KSum u = q ? u1 : u0;
        const KSum o = shfl_ksum(q ? u0 : u1, 16);
        kmerge2(u, o);
        sum_rows(u);
        const int j1 = j0 + ((h ? 2 : 0) + (q ? 1 : 0)) * NW;
        if ((lane & 15) == 0 && j1 < n1) kmerge2(M1[j1], u);
      } else {
#pragma unroll
        for (int g = 0; g < kMomPlanes; ++g) {
          KSum u{rs[g], 0.0};
          if (lpp >= 16) {
            sum_rows(u);
            for (int off = 16; off < lpp; off <<= 1) kmerge2(u, shfl_ksum(u, off));
          } else {
            for (int off = 1; off < lpp; off <<= 1) kmerge2(u, shfl_ksum(u, off));
          }
          const int j1 = j0 + g * NW * sub;
          if (pl == 0 && j1 < n1) kmerge2(M1[j1], u);
        }
      }
    }
    // the planes of a wavefront pass, in a fixed order
    for (int off = lpp; off < 64; off <<= 1)
#pragma unroll
      for (int k = 0; k < kMomVec; ++k)
#pragma unroll
        for (int c = 0; c < VN; ++c) kmerge2(acc[k][c], shfl_ksum(acc[k][c], off));
    const int ce = min(CH, np - c0);
    const int r0 = c0 / n3, rows = (c0 + ce - 1) / n3 - r0 + 1;
    const int parts = n3 < NT ? NT / n3 : 1;
    auto to_lds = [&](auto&& value) {  // the wavefronts' marginals of the chunk
      if (sl == 0) {
#pragma unroll
        for (int k = 0; k < kMomVec; ++k)
#pragma unroll
          for (int c = 0; c < VN; ++c) {
            const int e = (pl + k * lpp) * VN + c;
            if (e < ce) W[wave * cl + e] = value(acc[k][c]);
          }
      }
      __syncthreads();
    };
    // M_2: 16 lanes per row of the chunk; M_3: the rows dealt to as many
    // parts as there are threads for, then the parts in order.  First the
    // sums, compensated, then their errors, plainly into the errors.
    const int rows16 = (rows + NT / 16 - 1) / (NT / 16) * (NT / 16);
    auto row_lo = [&](int q) { return max((r0 + q) * n3, c0) - c0; };
    auto row_hi = [&](int q) { return min((r0 + q + 1) * n3, c0 + ce) - c0; };
    to_lds([](const KSum& v) { return v.s; });
    for (int q = tid / 16; q < rows16; q += NT / 16) {
      KSum m{0.0, 0.0};
      if (q < rows)
        for (int e = row_lo(q) + (tid & 15); e < row_hi(q); e += 16)
#pragma unroll
          for (int w = 0; w < NW; ++w) kadd2(m, W[w * cl + e]);
      sum_rows(m);
      if ((tid & 15) == 0 && q < rows) kmerge2(M2[r0 + q], m);
    }
    for (int j = tid; j < parts * n3; j += NT) {
      const int j3 = j % n3;
      KSum m{0.0, 0.0};
      for (int r = r0 + j / n3; r < r0 + rows; r += parts) {
        const int e = r * n3 + j3 - c0;
        if (e >= 0 && e < ce)
#pragma unroll
          for (int w = 0; w < NW; ++w) kadd2(m, W[w * cl + e]);
      }
      Q[j] = m;
    }
    __syncthreads();
    to_lds([](const KSum& v) { return v.c; });
    for (int q = tid / 16; q < rows16; q += NT / 16) {
      double v = 0.0;
      if (q < rows)
        for (int e = row_lo(q) + (tid & 15); e < row_hi(q); e += 16)
#pragma unroll
          for (int w = 0; w < NW; ++w) v += W[w * cl + e];
      v = sum_rows(v);
      if ((tid & 15) == 0 && q < rows) M2[r0 + q].c += v;
    }
    for (int j = tid; j < parts * n3; j += NT) {
      const int j3 = j % n3;
      double v = 0.0;
      for (int r = r0 + j / n3; r < r0 + rows; r += parts) {
        const int e = r * n3 + j3 - c0;
        if (e >= 0 && e < ce)
#pragma unroll
          for (int w = 0; w < NW; ++w) v += W[w * cl + e];
      }
      Q[j].c += v;
    }
    __syncthreads();
    for (int j3 = tid; j3 < n3; j3 += NT) {
      KSum m = M3[j3];
      for (int q = 0; q < parts; ++q) kmerge2(m, Q[q * n3 + j3]);
      M3[j3] = m;
    }
  }
  __syncthreads();
  // density, then mean and dispersion per axis, axes dealt to the wavefronts;
  // one density for all of them
  auto marginal = [&](int ax) { return ax == 0 ? M1 : ax == 1 ? M2 : M3; };
  auto cells_of = [&](int ax) { return ax == 0 ? n1 : ax == 1 ? n2 : n3; };
  auto wave_sum = [&](KSum v) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) kmerge2(v, shfl_ksum(v, off));
    return __shfl(v.s + v.c, 0, 64);
  };
  KSum s0{0.0, 0.0};
  for (int j = lane; j < cells_of(0); j += 64) kmerge2(s0, marginal(0)[j]);
  const double m0 = wave_sum(s0);
  for (int ax = wave; ax < D; ax += NW) {
    const KSum* M = marginal(ax);
    const int n = cells_of(ax);
    const double lo = ax == 0 ? vlo.x : ax == 1 ? vlo.y : vlo.z;
    const double h = ax == 0 ? dv.x : ax == 1 ? dv.y : dv.z;
    KSum s1{0.0, 0.0}, s2{0.0, 0.0};
    for (int j = lane; j < n; j += 64) {
      const double v = lo + ((double)j + 0.5) * h;
      kadd2(s1, M[j].s * v);
      s1.c += M[j].c * v;
    }
    const double u = m0 != 0.0 ? wave_sum(s1) / m0 : 0.0;
    for (int j = lane; j < n; j += 64) {
      const double d = lo + ((double)j + 0.5) * h - u;
      kadd2(s2, M[j].s * d * d);
      s2.c += M[j].c * d * d;
    }
    const double m2 = wave_sum(s2);
    if (lane == 0) {
      mean[(int64_t)ax * nxs + cell] = u;
      disp[(int64_t)ax * nxs + cell] = m0 != 0.0 ? m2 / m0 : 0.0;
      if (ax == 0) rho[cell] = dvol * m0;
    }
  }
}

// The same for one velocity axis and for small velocity blocks: two passes over
// the cell's contiguous velocity block (the second re-reads it from cache);
// compensated double sums of plain sums over groups of eight elements.  Bound
// by the latency of the passes, or on large blocks by the arithmetic of every
// element, which the marginals save.
template <typename T, int NT, int D>  // D: velocity axes (a constant: the loops over
                                      // axes unroll and every accumulator stays in registers)
__global__ void __launch_bounds__(NT) velocity_moments_direct_kernel(const T* __restrict__ f,
                                                              int64_t nvs, int3 nv, double3 vlo,
                                                              double3 dv, double dvol, int64_t nxs,
                                                              double* __restrict__ rho,
                                                              double* __restrict__ mean,
                                                              double* __restrict__ disp) {
  const T* b = f + (int64_t)blockIdx.x * nvs;
  const int n[3] = {nv.x, nv.y, nv.z};
  const double lo[3] = {vlo.x, vlo.y, vlo.z}, h[3] = {dv.x, dv.y, dv.z};
  // velocity index of element k as digits (last axis fastest): the digits
  // of this thread's first element and of the stride NT, then a digit-wise
  // add with carries per step instead of a division per element
  int j0[3] = {0, 0, 0}, st[3] = {0, 0, 0};
  {
    int64_t rem = threadIdx.x, str = NT;
    for (int l = D - 1; l >= 0; --l) {
      j0[l] = (int)(rem % n[l]);
      rem /= n[l];
      st[l] = (int)(str % n[l]);
      str /= n[l];
    }
  }
  int j[3];
  auto restart = [&]() {
    for (int l = 0; l < 3; ++l) j[l] = j0[l];
  };
  auto centres = [&](double* v) {
    for (int l = 0; l < D; ++l) v[l] = lo[l] + ((double)j[l] + 0.5) * h[l];
  };
  auto next = [&]() {  // j += st; past the last element the digits are unused
    int carry = 0;
    for (int l = D - 1; l >= 0; --l) {
      j[l] += st[l] + carry;
      carry = j[l] >= n[l];
      if (carry) j[l] -= n[l];
    }
  };
  // each thread adds groups of up to kGroup of its elements plainly and
  // feeds the group sums to the compensated accumulators
  constexpr int kGroup = 8;
  KSum s0{0.0, 0.0}, s1[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
  double p0 = 0.0, p1[3] = {0.0, 0.0, 0.0};
  int cnt = 0;
  restart();
  for (int64_t k = threadIdx.x; k < nvs; k += NT, next()) {
    double v[3];
    centres(v);
    const double x = (double)b[k];
    p0 += x;
    for (int l = 0; l < D; ++l) p1[l] += x * v[l];
    if (++cnt == kGroup) {
      kadd(s0, p0);
      for (int l = 0; l < D; ++l) kadd(s1[l], p1[l]);
      p0 = 0.0;
      for (int l = 0; l < D; ++l) p1[l] = 0.0;
      cnt = 0;
    }
  }
  kadd(s0, p0);
  for (int l = 0; l < D; ++l) kadd(s1[l], p1[l]);
  const KSum t0 = block_ksum<NT>(s0);
  const double m0 = t0.s + t0.c;
  double u[3] = {0.0, 0.0, 0.0};
  for (int l = 0; l < D; ++l) {
    const KSum t1 = block_ksum<NT>(s1[l]);
    u[l] = m0 != 0.0 ? (t1.s + t1.c) / m0 : 0.0;
  }
  KSum s2[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
  double p2[3] = {0.0, 0.0, 0.0};
  cnt = 0;
  restart();
  for (int64_t k = threadIdx.x; k < nvs; k += NT, next()) {
    double v[3];
    centres(v);
    const double x = (double)b[k];
    for (int l = 0; l < D; ++l) {
      const double d = v[l] - u[l];
      p2[l] += x * d * d;
    }
    if (++cnt == kGroup) {
      for (int l = 0; l < D; ++l) {
        kadd(s2[l], p2[l]);
        p2[l] = 0.0;
      }
      cnt = 0;
    }
  }
  for (int l = 0; l < D; ++l) kadd(s2[l], p2[l]);
  for (int l = 0; l < D; ++l) {
    const KSum t2 = block_ksum<NT>(s2[l]);
    if (threadIdx.x == 0) {
      mean[(int64_t)l * nxs + blockIdx.x] = u[l];
      disp[(int64_t)l * nxs + blockIdx.x] = m0 != 0.0 ? (t2.s + t2.c) / m0 : 0.0;
    }
  }
  if (threadIdx.x == 0) rho[blockIdx.x] = dvol * m0;
}

// F[k] = xvol * sum_x f[x][k]: a thread walks the spatial cells of its
// share (grid.y shares) for one 16-byte vector of velocity cells, eight rows
// in flight, every velocity cell's sum compensated.  With one share the
// thread writes F; with several, each writes its sums to part[share][k] and
// distribution_sum_kernel adds them in order.  (One share only was bound by
// the few workgroups of a small velocity grid: 16 for 64^2 velocity cells;
// 24^3 x 40^3 FP32 took 789 us, now 574 + 13 us.)
template <typename T>
__global__ void __launch_bounds__(256) velocity_distribution_kernel(const T* __restrict__ f,
                                                                    int64_t nxs, int64_t nvs,
                                                                    double xvol,
                                                                    double* __restrict__ F,
                                                                    KSum* __restrict__ part) {
  using V = typename UVec<T>::type;
  constexpr int VN = UVec<T>::N, U = 8;
  const int64_t per = (nxs + gridDim.y - 1) / gridDim.y;
  const int64_t x0 = blockIdx.y * per, x1 = min(nxs, x0 + per);
  const int64_t nvec = (nvs + VN - 1) / VN;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nvec;
       q += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = q * VN;
    const T* col = f + k;
    KSum a[VN];
#pragma unroll
    for (int c = 0; c < VN; ++c) a[c] = KSum{0.0, 0.0};
    int64_t ix = x0;
    if (nvs - k >= VN) {
      for (; ix + U <= x1; ix += U) {
        V x[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          x[u] = __builtin_nontemporal_load(reinterpret_cast<const V*>(col + (ix + u) * nvs));
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int c = 0; c < VN; ++c) kadd2(a[c], (double)x[u][c]);
      }
    }
    for (; ix < x1; ++ix) {
      const V x = load_part(col + ix * nvs, nvs - k);
#pragma unroll
      for (int c = 0; c < VN; ++c) kadd2(a[c], (double)x[c]);
    }
#pragma unroll
    for (int c = 0; c < VN; ++c)
      if (k + c < nvs) {
        if (part)
          part[blockIdx.y * nvs + k + c] = a[c];
        else
          F[k + c] = xvol * (a[c].s + a[c].c);
      }
  }
}
// The same for few spatial cells: one thread per velocity cell.  Few threads
// walk long columns here (one per velocity cell), so each keeps 16 loads in
// flight: rows x = 16 m + r go to accumulator r % 4, merged in a fixed order.
template <typename T>
__global__ void __launch_bounds__(256) velocity_distribution_direct_kernel(const T* __restrict__ f,
                                                                    int64_t nxs, int64_t nvs,
                                                                    double xvol,
                                                                    double* __restrict__ F) {
  constexpr int U = 16;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nvs;
       k += (int64_t)gridDim.x * blockDim.x) {
    KSum a[4] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
    const T* col = f + k;
    int64_t ix = 0;
    for (; ix + U <= nxs; ix += U) {
      T x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = col[(ix + u) * nvs];
#pragma unroll
      for (int u = 0; u < U; ++u) kadd(a[u % 4], (double)x[u]);
    }
    for (; ix < nxs; ++ix) kadd(a[0], (double)col[ix * nvs]);
    kmerge(a[0], a[1]);
    kmerge(a[2], a[3]);
    kmerge(a[0], a[2]);
    F[k] = xvol * (a[0].s + a[0].c);
  }
}

__global__ void __launch_bounds__(256) distribution_sum_kernel(const KSum* __restrict__ part,
                                                               int shares, int64_t nvs, double xvol,
                                                               double* __restrict__ F) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nvs) return;
  KSum a{0.0, 0.0};
  for (int y = 0; y < shares; ++y) kmerge2(a, part[y * nvs + k]);
  F[k] = xvol * (a.s + a.c);
}

// rho[i * ncol + c] = dvol * sum_q part[(c * nsub + q) * n + i]; thread
// (c, i) adds the nsub tile-row sums of its cell in tile order (compensated).
__global__ void __launch_bounds__(256) moment_reduce_kernel(const double* __restrict__ part,
                                                            bool pairs, int n,
                                                            int64_t ncol, int64_t nsub, double dvol,
                                                            double* __restrict__ rho) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= ncol * n) return;
  const int64_t c = g / n;
  const int i = (int)(g - c * n);
  const int64_t at = c * nsub * n + i;
  auto get = [&](int64_t q) {
    return pairs ? reinterpret_cast<const double2*>(part)[at + q * n] : make_double2(part[at + q * n], 0.0);
  };
  KSum acc0{0.0, 0.0}, acc1{0.0, 0.0};
  int64_t q = 0;
  for (; q + 1 < nsub; q += 2) {
    const double2 x0 = get(q), x1 = get(q + 1);
    kadd(acc0, x0.x);
    kadd(acc1, x1.x);
    acc0.c += x0.y;
    acc1.c += x1.y;
  }
  if (q < nsub) {
    const double2 x0 = get(q);
    kadd(acc0, x0.x);
    acc0.c += x0.y;
  }
  kmerge(acc0, acc1);
  rho[(int64_t)i * ncol + c] = dvol * (acc0.s + acc0.c);
}

// ---- discrete Fourier transform along one axis ------------------------
// out[o, k, j] = sum_m in[o, m, j] * tw[(m k) mod n]^sign, tw[q] = exp(-2 pi i q / n)
__global__ void dft_axis_kernel(const double2* __restrict__ in, double2* __restrict__ out,
                                int64_t total, int64_t n, int64_t inner,
                                const double2* __restrict__ tw, int conj) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= total) return;
  const int64_t j = t % inner;
  const int64_t k = (t / inner) % n;
  const int64_t o = t / (inner * n);
  const double2* src = in + o * n * inner + j;
  double sr = 0.0, si = 0.0;
  int64_t q = 0;
  for (int64_t m = 0; m < n; ++m) {
    const double2 x = src[m * inner];
    const double2 w = tw[q];
    const double wi = conj ? -w.y : w.y;
    sr += x.x * w.x - x.y * wi;
    si += x.x * wi + x.y * w.x;
    q += k;
    if (q >= n) q -= n;
  }
  out[t] = make_double2(sr, si);
}

__global__ void real_to_complex_kernel(const double* __restrict__ r, double2* __restrict__ c,
                                       int64_t n) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) c[t] = make_double2(r[t], 0.0);
}

__global__ void green_kernel(double2* __restrict__ c, const double* __restrict__ g, int64_t n) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) {
    const double2 v = c[t];
    c[t] = make_double2(v.x * g[t], v.y * g[t]);
  }
}

__global__ void complex_to_real_kernel(const double2* __restrict__ c, double* __restrict__ r,
                                       int64_t n, double scale) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) r[t] = c[t].x * scale;
}

// accel_l = -dphi/dx_l by the periodic 2-, 4- or 6-point FDA (App. C)
__global__ void fda_kernel(const double* __restrict__ phi, double* __restrict__ accel,
                           int64_t total, int64_t n, int64_t inner, double h, int order) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= total) return;
  const int64_t i = (t / inner) % n;
  const double* base = phi + (t - i * inner);
  auto P = [&](int64_t k) {
    int64_t r = (i + k) % n;
    if (r < 0) r += n;
    return base[r * inner];
  };
  double d;
  if (order == 2)
    d = (P(1) - P(-1)) / (2.0 * h);
  else if (order == 4)
    d = (8.0 * (P(1) - P(-1)) - (P(2) - P(-2))) / (12.0 * h);
  else
    d = (45.0 * (P(1) - P(-1)) - 9.0 * (P(2) - P(-2)) + (P(3) - P(-3))) / (60.0 * h);
  accel[t] = -d;
}

// ---- isolated boundaries (doubling-up method) -----------------------------
// the density in the low corner of the doubled grid, zero elsewhere
__global__ void iso_pad_kernel(const double* __restrict__ rho, double2* __restrict__ out, int3 n,
                               int3 m, int64_t ms) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < ms;
       q += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(q % m.z);
    const int j = (int)((q / m.z) % m.y);
    const int i = (int)(q / ((int64_t)m.y * m.z));
    double v = 0.0;
    if (i < n.x && j < n.y && k < n.z) v = rho[((int64_t)i * n.y + j) * n.z + k];
    out[q] = make_double2(v, 0.0);
  }
}

__global__ void real_part_kernel(const double2* __restrict__ c, double* __restrict__ r, int64_t n) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
       q += (int64_t)gridDim.x * blockDim.x)
    r[q] = c[q].x;
}

// potential of the physical cells and the FDA force from the doubled
// potential (its values beyond the physical cells are the isolated
// potential there); pd holds the unnormalised inverse DFT
__global__ void iso_force_kernel(const double2* __restrict__ pd, int3 n, int3 m, double scale,
                                 double3 h, int order, double* __restrict__ phi,
                                 double* __restrict__ accel, int64_t nxs) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < nxs;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(t % n.z);
    const int j = (int)((t / n.z) % n.y);
    const int i = (int)(t / ((int64_t)n.y * n.z));
    const int64_t q = ((int64_t)i * m.y + j) * m.z + k;
    phi[t] = pd[q].x * scale;
    const int pos[3] = {i, j, k};
    const int mm[3] = {m.x, m.y, m.z};
    const int64_t inner[3] = {(int64_t)m.y * m.z, (int64_t)m.z, 1};
    const double hh[3] = {h.x, h.y, h.z};
    for (int l = 0; l < 3; ++l) {
      const double2* base = pd + (q - (int64_t)pos[l] * inner[l]);
      auto P = [&](int kk) {
        int r = (pos[l] + kk) % mm[l];
        if (r < 0) r += mm[l];
        return base[(int64_t)r * inner[l]].x * scale;
      };
      double d;
      if (order == 2)
        d = (P(1) - P(-1)) / (2.0 * hh[l]);
      else if (order == 4)
        d = (8.0 * (P(1) - P(-1)) - (P(2) - P(-2))) / (12.0 * hh[l]);
      else
        d = (45.0 * (P(1) - P(-1)) - 9.0 * (P(2) - P(-2)) + (P(3) - P(-3))) / (60.0 * hh[l]);
      accel[(int64_t)l * nxs + t] = -d;
    }
  }
}

// ---- initialisation and conversions -----------------------------------
template <typename T>
__global__ void init_separable_kernel(T* __restrict__ f, const double* __restrict__ s,
                                      const double* __restrict__ g1, const double* __restrict__ g2,
                                      const double* __restrict__ g3, int D, int64_t nv1,
                                      int64_t nv2, int64_t nv3, int64_t nvs, int64_t total) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t ix = t / nvs;
    int64_t iv = t - ix * nvs;
    double v = s[ix];
    if (D == 1) {
      v = v * g1[iv];
    } else if (D == 2) {
      const int64_t j2 = iv % nv2, j1 = iv / nv2;
      v = v * g1[j1];
      v = v * g2[j2];
    } else {
      const int64_t j3 = iv % nv3;
      iv /= nv3;
      const int64_t j2 = iv % nv2, j1 = iv / nv2;
      v = v * g1[j1];
      v = v * g2[j2];
      v = v * g3[j3];
    }
    f[t] = (T)v;
  }
  (void)nv1;
}

template <typename T>
__global__ void from_double_kernel(T* __restrict__ f, const double* __restrict__ src, int64_t n) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n;
       t += (int64_t)gridDim.x * blockDim.x)
    f[t] = (T)src[t];
}

template <typename T>
__global__ void to_double_kernel(const T* __restrict__ f, double* __restrict__ dst, int64_t n) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n;
       t += (int64_t)gridDim.x * blockDim.x)
    dst[t] = (double)f[t];
}

// ---- diagnostics --------------------------------------------------------
// partials[b*5 + 0..4] = (sum, compensation, min, max, number of non-finite
// values) of block b; non-finite values enter nothing else.  Bound by the
// read of f: 16-byte loads, four in flight per thread (one 4-byte load at a
// time read 24^3 x 40^3 FP32 at 1.8 TB/s in 1989 us; now 609 us,
// 5.8 TB/s).  A
// vector's elements are tested together through their sum, and one by one
// only where that is not finite.
template <typename T, int NT>
__global__ void __launch_bounds__(NT) diag_f_kernel(const T* __restrict__ f, int64_t n,
                                                    double* __restrict__ partials) {
  using V = typename UVec<T>::type;
  constexpr int VN = UVec<T>::N, U = 4;
  KSum acc{0.0, 0.0};
  T mn = (T)INFINITY, mx = -(T)INFINITY;
  double bad = 0.0;
  auto one = [&](T x) {
    if (!isfinite(x)) {
      bad += 1.0;
      return;
    }
    kadd2(acc, (double)x);
    mn = x < mn ? x : mn;
    mx = x > mx ? x : mx;
  };
  auto vec = [&](V x) {
    double t = (double)x[0];
#pragma unroll
    for (int c = 1; c < VN; ++c) t += (double)x[c];
    if (!isfinite(t)) {
#pragma unroll
      for (int c = 0; c < VN; ++c) one(x[c]);
      return;
    }
#pragma unroll
    for (int c = 0; c < VN; ++c) kadd2(acc, (double)x[c]);
#pragma unroll
    for (int c = 0; c < VN; ++c) {
      mn = x[c] < mn ? x[c] : mn;
      mx = x[c] > mx ? x[c] : mx;
    }
  };
  const int64_t nvec = n / VN, step = (int64_t)gridDim.x * NT;
  const V* fv = reinterpret_cast<const V*>(f);
  int64_t t = (int64_t)blockIdx.x * NT + threadIdx.x;
  for (; t + (U - 1) * step < nvec; t += U * step) {
    V x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = __builtin_nontemporal_load(fv + t + u * step);
#pragma unroll
    for (int u = 0; u < U; ++u) vec(x[u]);
  }
  for (; t < nvec; t += step) vec(fv[t]);
  if (blockIdx.x == 0 && (int64_t)threadIdx.x < n - nvec * VN) one(f[nvec * VN + threadIdx.x]);
  KSum tot = block_ksum<NT>(acc);
  __shared__ double smn[NT], smx[NT], sbad[NT];
  smn[threadIdx.x] = (double)mn;
  smx[threadIdx.x] = (double)mx;
  sbad[threadIdx.x] = bad;
  __syncthreads();
  for (int off = NT / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) {
      smn[threadIdx.x] = fmin(smn[threadIdx.x], smn[threadIdx.x + off]);
      smx[threadIdx.x] = fmax(smx[threadIdx.x], smx[threadIdx.x + off]);
      sbad[threadIdx.x] += sbad[threadIdx.x + off];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double* p = partials + (int64_t)blockIdx.x * 5;
    p[0] = tot.s;
    p[1] = tot.c;
    p[2] = smn[0];
    p[3] = smx[0];
    p[4] = sbad[0];
  }
}

// Per block b: partials[b*6 + 0..5] = sum |a|^2 over all components and
// cells, and real and imaginary part of sum_x a_1(x) exp(-2 pi i x1_index /
// nx1), each as (sum, compensation).  (One block took 96 us at 24^3 cells, now 6 us.)
template <int NT>
__global__ void __launch_bounds__(NT) diag_field_kernel(const double* __restrict__ accel, int D,
                                                        int64_t nxs, int64_t nx1, int64_t inner1,
                                                        double* __restrict__ partials) {
  KSum e{0.0, 0.0}, cr{0.0, 0.0}, ci{0.0, 0.0};
  const int64_t t0 = (int64_t)blockIdx.x * NT + threadIdx.x, step = (int64_t)gridDim.x * NT;
  for (int64_t t = t0; t < (int64_t)D * nxs; t += step) {
    const double a = accel[t];
    kadd2(e, a * a);
  }
  for (int64_t t = t0; t < nxs; t += step) {
    double sn, cs;
    sincospi(-2.0 * (double)(t / inner1) / (double)nx1, &sn, &cs);
    kadd2(cr, accel[t] * cs);
    kadd2(ci, accel[t] * sn);
  }
  const KSum te = block_ksum<NT>(e), tr = block_ksum<NT>(cr), ti = block_ksum<NT>(ci);
  if (threadIdx.x == 0) {
    double* p = partials + (int64_t)blockIdx.x * 6;
    p[0] = te.s;
    p[1] = te.c;
    p[2] = tr.s;
    p[3] = tr.c;
    p[4] = ti.s;
    p[5] = ti.c;
  }
}

// out[0..6] = sum of f, min, max, non-finite count, sum |a|^2, real and
// imaginary part of the first mode, from the block results in block order.
template <int NT>
__global__ void __launch_bounds__(NT) diag_sum_kernel(const double* __restrict__ pf, int nf,
                                                      const double* __restrict__ pa, int na,
                                                      double* __restrict__ out) {
  KSum s[4] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
  double mn = INFINITY, mx = -INFINITY, bad = 0.0;
  for (int b = threadIdx.x; b < nf; b += NT) {
    const double* p = pf + (int64_t)b * 5;
    kmerge2(s[0], KSum{p[0], p[1]});
    mn = fmin(mn, p[2]);
    mx = fmax(mx, p[3]);
    bad += p[4];
  }
  for (int b = threadIdx.x; b < na; b += NT)
#pragma unroll
    for (int q = 0; q < 3; ++q) kmerge2(s[1 + q], KSum{pa[b * 6 + 2 * q], pa[b * 6 + 2 * q + 1]});
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const KSum r = block_ksum<NT>(s[q]);
    if (threadIdx.x == 0) out[q == 0 ? 0 : 3 + q] = r.s + r.c;
  }
  __shared__ double smn[NT], smx[NT], sbad[NT];
  smn[threadIdx.x] = mn;
  smx[threadIdx.x] = mx;
  sbad[threadIdx.x] = bad;
  __syncthreads();
  for (int off = NT / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) {
      smn[threadIdx.x] = fmin(smn[threadIdx.x], smn[threadIdx.x + off]);
      smx[threadIdx.x] = fmax(smx[threadIdx.x], smx[threadIdx.x + off]);
      sbad[threadIdx.x] += sbad[threadIdx.x + off];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[1] = smn[0];
    out[2] = smx[0];
    out[3] = sbad[0];
  }
}

__global__ void copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int64_t n) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n;
       t += (int64_t)gridDim.x * blockDim.x)
    dst[t] = src[t];
}

inline unsigned blocks_for(int64_t n, int nt) { return (unsigned)((n + nt - 1) / nt); }
inline unsigned grid_capped(int64_t n, int nt) {
  int64_t b = (n + nt - 1) / nt;
  return (unsigned)(b > 65536 ? 65536 : (b < 1 ? 1 : b));
}

}  // namespace

hipError_t launch_moment(int dtype, const void* f, int64_t nxs, int64_t nvs, double dvol,
                         double* rho, hipStream_t s) {
  if (nxs <= 0) return hipSuccess;
  constexpr int NT = 256;
  if (dtype == SLMPP_F64)
    hipLaunchKernelGGL((moment_kernel<double, NT>), dim3((unsigned)nxs), dim3(NT), 0, s,
                       (const double*)f, nvs, dvol, rho);
  else
    hipLaunchKernelGGL((moment_kernel<float, NT>), dim3((unsigned)nxs), dim3(NT), 0, s,
                       (const float*)f, nvs, dvol, rho);
  return hipGetLastError();
}

hipError_t launch_moment_reduce(const double* part, bool pairs, int n, int64_t ncol, int64_t nsub,
                                double dvol, double* rho, hipStream_t s) {
  const int64_t total = ncol * n;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(moment_reduce_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                     part, pairs, n, ncol, nsub, dvol, rho);
  return hipGetLastError();
}

hipError_t launch_poisson(const double* rho, double* phi, double* accel, double2* bufA,
                          double2* bufB, const double2* twiddles, const int64_t* tw_off,
                          const double* green, int D, const int64_t* nx, const double* h,
                          int order, hipStream_t s) {
  int64_t nxs = 1;
  for (int l = 0; l < D; ++l) nxs *= nx[l];
  constexpr int NT = 256;
  hipLaunchKernelGGL(real_to_complex_kernel, dim3(blocks_for(nxs, NT)), dim3(NT), 0, s, rho, bufA,
                     nxs);
  double2* cur = bufA;
  double2* oth = bufB;
  for (int pass = 0; pass < 2; ++pass) {
    for (int l = 0; l < D; ++l) {
      int64_t inner = 1;
      for (int k = l + 1; k < D; ++k) inner *= nx[k];
      hipLaunchKernelGGL(dft_axis_kernel, dim3(blocks_for(nxs, NT)), dim3(NT), 0, s, cur, oth,
                         nxs, nx[l], inner, twiddles + tw_off[l], pass);
      double2* t = cur;
      cur = oth;
      oth = t;
    }
    if (pass == 0)
      hipLaunchKernelGGL(green_kernel, dim3(blocks_for(nxs, NT)), dim3(NT), 0, s, cur, green, nxs);
  }
  hipLaunchKernelGGL(complex_to_real_kernel, dim3(blocks_for(nxs, NT)), dim3(NT), 0, s, cur, phi,
                     nxs, 1.0 / (double)nxs);
  for (int l = 0; l < D; ++l) {
    int64_t inner = 1;
    for (int k = l + 1; k < D; ++k) inner *= nx[k];
    hipLaunchKernelGGL(fda_kernel, dim3(blocks_for(nxs, NT)), dim3(NT), 0, s, phi,
                       accel + (int64_t)l * nxs, nxs, nx[l], inner, h[l], order);
  }
  return hipGetLastError();
}

// Three DFT passes over the doubled grid (sizes m, twiddles per axis at
// tw + tw_off[l]); returns the buffer holding the result.
static double2* dft3(double2* a, double2* b, const int64_t* m, const double2* tw,
                     const int64_t* tw_off, int conj, hipStream_t s) {
  const int64_t ms = m[0] * m[1] * m[2];
  constexpr int NT = 256;
  double2* cur = a;
  double2* oth = b;
  for (int l = 0; l < 3; ++l) {
    int64_t inner = 1;
    for (int k = l + 1; k < 3; ++k) inner *= m[k];
    hipLaunchKernelGGL(dft_axis_kernel, dim3(blocks_for(ms, NT)), dim3(NT), 0, s, cur, oth, ms,
                       m[l], inner, tw + tw_off[l], conj);
    double2* t = cur;
    cur = oth;
    oth = t;
  }
  return cur;
}

hipError_t launch_iso_green(double2* a, double2* b, const double2* tw, const int64_t* tw_off,
                            const int64_t* m, double* ghat, hipStream_t s) {
  const int64_t ms = m[0] * m[1] * m[2];
  double2* res = dft3(a, b, m, tw, tw_off, 0, s);
  hipLaunchKernelGGL(real_part_kernel, dim3(grid_capped(ms, 256)), dim3(256), 0, s, res, ghat, ms);
  return hipGetLastError();
}

hipError_t launch_poisson_isolated(const double* rho, double* phi, double* accel, double2* a,
                                   double2* b, const double2* tw, const int64_t* tw_off,
                                   const double* ghat, const int64_t* nx, const double* h,
                                   int order, hipStream_t s) {
  const int64_t m[3] = {2 * nx[0], 2 * nx[1], 2 * nx[2]};
  const int64_t ms = m[0] * m[1] * m[2], nxs = nx[0] * nx[1] * nx[2];
  const int3 n3 = make_int3((int)nx[0], (int)nx[1], (int)nx[2]);
  const int3 m3 = make_int3((int)m[0], (int)m[1], (int)m[2]);
  hipLaunchKernelGGL(iso_pad_kernel, dim3(grid_capped(ms, 256)), dim3(256), 0, s, rho, a, n3, m3,
                     ms);
  double2* fwd = dft3(a, b, m, tw, tw_off, 0, s);
  hipLaunchKernelGGL(green_kernel, dim3(blocks_for(ms, 256)), dim3(256), 0, s, fwd, ghat, ms);
  double2* other = fwd == a ? b : a;
  double2* inv = dft3(fwd, other, m, tw, tw_off, 1, s);
  hipLaunchKernelGGL(iso_force_kernel, dim3(grid_capped(nxs, 256)), dim3(256), 0, s, inv, n3, m3,
                     1.0 / (double)ms, make_double3(h[0], h[1], h[2]), order, phi, accel, nxs);
  return hipGetLastError();
}

hipError_t launch_init_separable(int dtype, void* f, const double* sx, const double* g1,
                                 const double* g2, const double* g3, int D, const int64_t* nv,
                                 int64_t nxs, int64_t nvs, hipStream_t st) {
  const int64_t total = nxs * nvs;
  constexpr int NT = 256;
  const unsigned grid = grid_capped(total, NT);
  const int64_t n1 = nv[0], n2 = D > 1 ? nv[1] : 1, n3 = D > 2 ? nv[2] : 1;
  if (dtype == SLMPP_F64)
    hipLaunchKernelGGL(init_separable_kernel<double>, dim3(grid), dim3(NT), 0, st, (double*)f, sx,
                       g1, g2, g3, D, n1, n2, n3, nvs, total);
  else
    hipLaunchKernelGGL(init_separable_kernel<float>, dim3(grid), dim3(NT), 0, st, (float*)f, sx,
                       g1, g2, g3, D, n1, n2, n3, nvs, total);
  return hipGetLastError();
}

hipError_t launch_from_double(int dtype, void* f, const double* src, int64_t n, hipStream_t s) {
  constexpr int NT = 256;
  if (dtype == SLMPP_F64)
    hipLaunchKernelGGL(from_double_kernel<double>, dim3(grid_capped(n, NT)), dim3(NT), 0, s,
                       (double*)f, src, n);
  else
    hipLaunchKernelGGL(from_double_kernel<float>, dim3(grid_capped(n, NT)), dim3(NT), 0, s,
                       (float*)f, src, n);
  return hipGetLastError();
}

hipError_t launch_to_double(int dtype, const void* f, double* dst, int64_t n, hipStream_t s) {
  constexpr int NT = 256;
  if (dtype == SLMPP_F64)
    hipLaunchKernelGGL(to_double_kernel<double>, dim3(grid_capped(n, NT)), dim3(NT), 0, s,
                       (const double*)f, dst, n);
  else
    hipLaunchKernelGGL(to_double_kernel<float>, dim3(grid_capped(n, NT)), dim3(NT), 0, s,
                       (const float*)f, dst, n);
  return hipGetLastError();
}

hipError_t launch_diag(int dtype, const void* f, int64_t n, const double* accel, int D, int64_t nxs,
                       int64_t nx1, int64_t inner1, double* partials, double* out, hipStream_t s) {
  constexpr int NT = 256;
  const int nf = (int)std::max<int64_t>(1, std::min<int64_t>(kDiagBlocks, (n + 16 * NT - 1) / (16 * NT)));
  const int na = (int)std::max<int64_t>(1, std::min<int64_t>(kDiagFieldBlocks, (nxs + NT - 1) / NT));
  double* pa = partials + (int64_t)kDiagBlocks * 5;
  if (dtype == SLMPP_F64)
    hipLaunchKernelGGL((diag_f_kernel<double, NT>), dim3(nf), dim3(NT), 0, s, (const double*)f, n,
                       partials);
  else
    hipLaunchKernelGGL((diag_f_kernel<float, NT>), dim3(nf), dim3(NT), 0, s, (const float*)f, n,
                       partials);
  hipLaunchKernelGGL((diag_field_kernel<NT>), dim3(na), dim3(NT), 0, s, accel, D, nxs, nx1, inner1, pa);
  hipLaunchKernelGGL((diag_sum_kernel<NT>), dim3(1), dim3(NT), 0, s, partials, nf, pa, na, out);
  return hipGetLastError();
}

hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const int64_t n = (int64_t)(bytes / 16);
  constexpr int NT = 256;
  const int64_t blocks = std::min<int64_t>((n + NT - 1) / NT, 256 * 64);
  if (n > 0)
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)std::max<int64_t>(blocks, 1)), dim3(NT), 0, s,
                       (const uint4*)src, (uint4*)dst, n);
  return hipGetLastError();
}

namespace {
// spatial cells from which one wavefront each takes the marginals
constexpr int64_t kMomMany = 2048;
// Whether the moments of a velocity block [n1][plane] are taken directly rather
// than through the marginals, whose folds and barriers cost more than they save
// where there is little to add up.  us, directly / through the marginals:
//   one axis (a plane of one element each): 1024 x 4096 FP32 11 / 850;
//   two axes, few cells: 17^2 x 54x61 11 / 32, 8^2 x 128^2 FP64 29 / 31, 4^2 x
// 200x210 63 / 41; many: 142^2 x 54x61 FP32 167 / 205, FP64 218 / 177, 64^2 x
// 128^2 138 / 105;
//   three axes, few cells: 12^3 x 8^3 16 / 27, 8^3 x 12^3 FP64 12 / 9; many: 37^3 x
// 9x11x13 329 / 290;
//   few large planes (a fold after each few): 5^3 x 4x40x40 18 / 30, 129^2 x
// 2x2000 161 / 5245; small planes (many lanes' sums each): 129^2 x 2000x2 162 / 566.
bool moments_direct(bool f64, int D, int64_t nxs, int n1, int64_t plane) {
  const bool many = nxs >= kMomMany;
  const int64_t nvs = n1 * plane;
  if (D == 1 || plane < 32 || (plane >= 256 && n1 < (many ? 4 : 8))) return true;
  if (D == 2) return nvs < (!many ? 16384 : f64 ? 2048 : 9216);
  return !many && nvs < (f64 ? 768 : 2048);
}
}  // namespace

hipError_t launch_velocity_moments(int dtype, const void* f, int D, const int64_t* nv,
                                   const double* vlo, const double* dv, int64_t nxs,
                                   double* rho, double* mean, double* disp, double* scratch,
                                   int64_t scratch_doubles, hipStream_t s) {
  if (D < 1 || D > 3) return hipErrorInvalidValue;
  double dvol = 1.0;
  int64_t nvs = 1;
  for (int l = 0; l < D; ++l) {
    dvol *= dv[l];
    nvs *= nv[l];
  }
  const int n1 = (int)nv[0], n2 = D > 1 ? (int)nv[1] : 1, n3 = D > 2 ? (int)nv[2] : 1;
  const double3 lo3 = make_double3(vlo[0], D > 1 ? vlo[1] : 0.0, D > 2 ? vlo[2] : 0.0);
  const double3 dv3 = make_double3(dv[0], D > 1 ? dv[1] : 1.0, D > 2 ? dv[2] : 1.0);
  if (moments_direct(dtype == SLMPP_F64, D, nxs, n1, (int64_t)n2 * n3)) {
    auto direct = [&](auto tag, auto axes) {
      using T = decltype(tag);
      constexpr int NT = 256;
      hipLaunchKernelGGL((velocity_moments_direct_kernel<T, NT, decltype(axes)::value>), dim3((unsigned)nxs),
                         dim3(NT), 0, s, (const T*)f, nvs, make_int3(n1, n2, n3), lo3, dv3, dvol, nxs, rho,
                         mean, disp);
      return hipGetLastError();
    };
    auto axes = [&](auto tag) {
      return D == 1   ? direct(tag, std::integral_constant<int, 1>{})
             : D == 2 ? direct(tag, std::integral_constant<int, 2>{})
                      : direct(tag, std::integral_constant<int, 3>{});
    };
    return dtype == SLMPP_F64 ? axes(0.0) : axes(0.0f);
  }
  auto go = [&](auto tag, auto width) -> hipError_t {
    using T = decltype(tag);
    constexpr int NT = decltype(width)::value;
    const int64_t ch = 64 * UVec<T>::N * kMomVec;
    const int64_t axes = n1 + n2 + n3;
    size_t lds = sizeof(double) * (size_t)(NT / 64) * std::min<int64_t>(ch, (int64_t)n2 * n3) +
                 sizeof(KSum) * std::max(NT, n3);
    // axes of several thousand cells each: the scratch holds the marginals of
    // as many spatial cells at a time as fit it
    KSum* marg = nullptr;
    int64_t per = nxs;
    if (lds + sizeof(KSum) * axes > 160 * 1024) {
      per = std::min(nxs, scratch_doubles / (2 * axes));
      if (per < 1) return hipErrorInvalidValue;
      marg = reinterpret_cast<KSum*>(scratch);
    } else {
      lds += sizeof(KSum) * axes;
    }
    auto kern = marg ? velocity_moments_kernel<T, NT, true> : velocity_moments_kernel<T, NT, false>;
    if (lds > 64 * 1024) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    for (int64_t cell0 = 0; cell0 < nxs; cell0 += per)
      hipLaunchKernelGGL(kern, dim3((unsigned)std::min(per, nxs - cell0)), dim3(NT), lds, s, (const T*)f, D,
                         n1, n2, n3, lo3, dv3, dvol, nxs, cell0, rho, mean, disp, marg);
    return hipGetLastError();
  };
  // one wavefront per spatial cell where there are enough cells to fill the
  // GPU with them (no barriers, long runs of loads between two folds), four
  // where there are not
  using One = std::integral_constant<int, 64>;
  using Four = std::integral_constant<int, 256>;
  if (nxs >= kMomMany) return dtype == SLMPP_F64 ? go(0.0, One{}) : go(0.0f, One{});
  return dtype == SLMPP_F64 ? go(0.0, Four{}) : go(0.0f, Four{});
}

hipError_t launch_velocity_distribution(int dtype, const void* f, int64_t nxs, int64_t nvs,
                                        double xvol, double* F, double* scratch,
                                        int64_t scratch_doubles, hipStream_t s) {
  // Few spatial cells, or enough velocity cells for a thread each: one launch
  // without shares.  us, directly / in vectors and shares: 64 x 8^2 x 128^2 FP32 3.8 /
  // 7.7, 7^2 x 30x41 FP64 4.0 / 6.8, 22^2 x 128^2 FP32 15.6 / 20.8, 10^3 x 40^3 FP32
  // 45 / 63, 12^3 x 32^3 FP64 101 / 90, 24^3 x 16x20x24 FP32 662 / 157.
  if (nxs <= (nvs >= 32768 ? 2048 : nvs >= 12288 ? 512 : dtype == SLMPP_F64 ? 128 : 256)) {
    const dim3 all((unsigned)std::min<int64_t>((nvs + 255) / 256, 4096));
    if (dtype == SLMPP_F64)
      hipLaunchKernelGGL(velocity_distribution_direct_kernel<double>, all, dim3(256), 0, s, (const double*)f,
                         nxs, nvs, xvol, F);
    else
      hipLaunchKernelGGL(velocity_distribution_direct_kernel<float>, all, dim3(256), 0, s, (const float*)f,
                         nxs, nvs, xvol, F);
    return hipGetLastError();
  }
  const int vn = dtype == SLMPP_F64 ? 2 : 4;
  const int64_t bx = std::min<int64_t>(((nvs + vn - 1) / vn + 255) / 256, 4096);
  // shares of the spatial cells: about 2048 workgroups in all, at least 16
  // cells each, within the scratch
  int64_t shares = std::min<int64_t>((2048 + bx - 1) / bx, (nxs + 15) / 16);
  shares = std::min<int64_t>(shares, scratch_doubles / (2 * nvs));
  shares = std::max<int64_t>(1, std::min<int64_t>(shares, 1024));
  KSum* part = shares > 1 ? reinterpret_cast<KSum*>(scratch) : nullptr;
  const dim3 grid((unsigned)bx, (unsigned)shares);
  if (dtype == SLMPP_F64)
    hipLaunchKernelGGL(velocity_distribution_kernel<double>, grid, dim3(256), 0, s, (const double*)f,
                       nxs, nvs, xvol, F, part);
  else
    hipLaunchKernelGGL(velocity_distribution_kernel<float>, grid, dim3(256), 0, s, (const float*)f,
                       nxs, nvs, xvol, F, part);
  if (part)
    hipLaunchKernelGGL(distribution_sum_kernel, dim3(blocks_for(nvs, 256)), dim3(256), 0, s, part,
                       (int)shares, nvs, xvol, F);
  return hipGetLastError();
}

}  // namespace slmpp
