// Device code shared by the sweep kernels: pencil-table entries, the interface
// flux (CSL polynomial, MP constraint, PP limiter) and the advance of one
// segment of a pencil held in LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "slmpp_internal.hpp"

namespace slmpp {
namespace {

template <typename T>
struct alignas(16) PencilEntry {
  T w[7];        // FIR weights of the CSL flux at |zeta| (first ORDER used)
  T z;           // |zeta|
  T tz;          // 2 |zeta| (exact), the factor of the PP half-updates
  int32_t base;  // physical row read at processing position 0
  int16_t dir;   // +1 forward, -1 mirrored (zeta < 0)
  int16_t absN;  // |N| after periodic reduction (at most n + 64 <= 4160)
};
static_assert(sizeof(PencilEntry<float>) == 48 && sizeof(PencilEntry<double>) == 80,
              "pencil entries are 16-byte multiples");

// CSL flux as an FIR filter: Phi_{i-1/2} = sum_k w_k(zeta) f_{i-h+k} with
// h = 3 (fifth order) or 4 (seventh order), w_k(zeta) = sum_j K[k][j] zeta^j.
// K is the transpose of the coefficient rows C_0..C_4 (D_0..D_6) of
// Sec. 2.1.2, each entry a numerator over the row's common denominator.
struct Frac {
  double num, den;
};
__device__ constexpr Frac kCsl5[5][5] = {
    // zeta^0      zeta^1       zeta^2       zeta^3       zeta^4
    {{2, 60}, {0, 24}, {-1, 24}, {0, 24}, {1, 120}},      // f_{i-3}
    {{-13, 60}, {-1, 24}, {6, 24}, {1, 24}, {-4, 120}},   // f_{i-2}
    {{47, 60}, {15, 24}, {-8, 24}, {-3, 24}, {6, 120}},   // f_{i-1}
    {{27, 60}, {-15, 24}, {2, 24}, {3, 24}, {-4, 120}},   // f_i
    {{-3, 60}, {1, 24}, {1, 24}, {-1, 24}, {1, 120}},     // f_{i+1}
};
__device__ constexpr Frac kCsl7[7][7] = {
    {{-3, 420}, {0, 360}, {7, 720}, {0, 144}, {-2, 720}, {0, 720}, {1, 5040}},        // f_{i-4}
    {{25, 420}, {2, 360}, {-57, 720}, {-1, 144}, {15, 720}, {1, 720}, {-6, 5040}},    // f_{i-3}
    {{-101, 420}, {-25, 360}, {210, 720}, {11, 144}, {-39, 720}, {-5, 720}, {15, 5040}},  // f_{i-2}
    {{319, 420}, {245, 360}, {-230, 720}, {-28, 144}, {46, 720}, {10, 720}, {-20, 5040}}, // f_{i-1}
    {{214, 420}, {-245, 360}, {15, 720}, {28, 144}, {-24, 720}, {-10, 720}, {15, 5040}},  // f_i
    {{-38, 420}, {25, 360}, {63, 720}, {-11, 144}, {3, 720}, {5, 720}, {-6, 5040}},   // f_{i+1}
    {{4, 420}, {-2, 360}, {-8, 720}, {1, 144}, {1, 720}, {-1, 720}, {1, 5040}},       // f_{i+2}
};

// Cell centre and departure offset with the rounding fixed (no FMA
// contraction), so that the integer split agrees with any other IEEE
// evaluation of the same expressions.
__device__ __forceinline__ double cell_center(double lo, double d, int64_t j) {
#pragma clang fp contract(off)
  return lo + ((double)j + 0.5) * d;
}
__device__ __forceinline__ double departure(double c, double dt, double h) {
#pragma clang fp contract(off)
  return (c * dt) / h;
}

__device__ __forceinline__ float vmin(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ float vmax(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ __forceinline__ double vmin(double a, double b) { return __builtin_fmin(a, b); }
__device__ __forceinline__ double vmax(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ float vfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double vfma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// middle value of three numbers
__device__ __forceinline__ float med3(float a, float b, float c) {
  return __builtin_amdgcn_fmed3f(a, b, c);
}
__device__ __forceinline__ double med3(double a, double b, double c) {
  return vmax(vmin(a, b), vmin(vmax(a, b), c));
}
template <typename T>
__device__ __forceinline__ T min3(T a, T b, T c) { return vmin(vmin(a, b), c); }
template <typename T>
__device__ __forceinline__ T max3(T a, T b, T c) { return vmax(vmax(a, b), c); }

// minmod of two / four numbers through the median with zero: for equal
// signs the median of (a, b, 0) is the argument of smaller magnitude,
// otherwise it is zero.
template <typename T>
__device__ __forceinline__ T minmod2(T a, T b) { return med3(a, b, T(0)); }
template <typename T>
__device__ __forceinline__ T minmod4(T a, T b, T c, T d) {
  return med3(minmod2(a, b), minmod2(c, d), T(0));
}

// 2 |zeta| phib as one rounded product (never fused into a later add)
template <typename T>
__device__ __forceinline__ T pp_product(T tz, T phib) {
#pragma clang fp contract(off)
  return tz * phib;
}

// (Inlined into its rare branch: as a function of its own, the calling
// convention left a kernel only half of its registers for values that live
// across the call.  Without the call the FP32 48^2 two-axis pass needs 72
// VGPRs instead of 91, seven wavefronts per SIMD instead of five, and takes
// 20.8 instead of 23.3 ms at 48^3 x 48^3; the FP64 64^2 one 161 instead of
// 193, and 72 instead of 89 us at 64^2 x 64^2.)
template <typename T>
__device__ __forceinline__ T pp_limit(T phib, T f0, T fp1, T tz, T p) {
  // theta = U^UP / (U^UP - U) on each side whose half-update is negative
  // (zero when the denominator is not positive), clamped to [0, 1]; the
  // flux moves toward the upwind value f0 by 1 - min(theta+, theta-).
  // p = 2 |zeta| phib (rounded); the half-updates and the limited flux are
  // formed without contraction, each operation rounded once.
#pragma clang fp contract(off)
  const T u_plus = f0 - p;
  const T u_minus = fp1 + p;
  T th = T(1);
  if (u_plus < T(0)) {
    const T up = f0 - tz * f0;
    const T den = up - u_plus;
    th = den > T(0) ? vmin(vmax(up / den, T(0)), T(1)) : T(0);
  }
  if (u_minus < T(0)) {
    const T up = fp1 + tz * f0;
    const T den = up - u_minus;
    th = vmin(th, den > T(0) ? vmin(vmax(up / den, T(0)), T(1)) : T(0));
  }
  return th * phib + (T(1) - th) * f0;
}

// App. A steps 4-7: the bounds f^min, f^max from the curvatures and the
// median of the flux with them.  The curvatures d_j = f_{j-1} + f_{j+1} -
// 2 f_j are formed as differences of the one-cell differences
// dll = f_{i-1} - f_{i-2}, dl = f_i - f_{i-1}, dr = f_{i+1} - f_i and
// drr = f_{i+2} - f_{i+1}, of which the face already holds dl and dr (and
// the previous face dll), so that nothing of these steps is computed
// outside the rare branch that needs them.
template <typename T>
__device__ __forceinline__ T mp_clamp(T phi, T dll, T dl, T dr, T drr, T f0, T fp1, T alpha) {
  const T dm1 = dl - dll;
  const T d0 = dr - dl;
  const T dp1 = drr - dr;
  const T dm4_plus = minmod4(vfma(T(4), d0, -dp1), vfma(T(4), dp1, -d0), d0, dp1);
  const T dm4_minus = minmod4(vfma(T(4), dm1, -d0), vfma(T(4), d0, -dm1), dm1, d0);
  const T f_ul = vfma(alpha, dl, f0);
  const T f_md = vfma(T(-0.5), dm4_plus, vfma(T(0.5), dr, f0));
  const T f_lc = vfma(T(4.0 / 3.0), dm4_minus, vfma(T(0.5), dl, f0));
  const T lo = vmax(min3(f0, fp1, f_md), min3(f0, f_ul, f_lc));
  const T hi = vmin(max3(f0, fp1, f_md), max3(f0, f_ul, f_lc));
  return med3(phi, lo, hi);
}

// Interface flux at the face between processing positions m and m+1
// (upwind cell m).  q holds r_{m-3}..r_{m+3} (seventh order) or
// r_{m-2}..r_{m+2} (fifth order); the MP constraint works on the five
// cells r_{m-2}..r_{m+2} in both cases.
template <typename T, int ORDER, int LIM>
__device__ __forceinline__ T face_flux(const T* q, const T* w, T tz, T alpha) {
  constexpr int o = (ORDER == 7) ? 1 : 0;  // offset of the MP stencil in q
  T phi = w[0] * q[0];
#pragma unroll
  for (int k = 1; k < ORDER; ++k) phi = vfma(w[k], q[k], phi);
  if constexpr (LIM == SLMPP_LIM_NONE) {
    return phi;
  } else {
    const T fm2 = q[o], fm1 = q[o + 1], f0 = q[o + 2], fp1 = q[o + 3], fp2 = q[o + 4];
    const T dl = f0 - fm1, dr = fp1 - f0;
    // App. A steps 2-3.  f* = f_i + minmod(f_{i+1} - f_i, alpha (f_i - f_{i-1}))
    // is the median of f_{i+1}, f^UL = f_i + alpha (f_i - f_{i-1}) and f_i
    // (adding f_i commutes with the median); it is formed that way, from
    // the same rounded f^UL that the bounds of step 6 use.  The flux is kept
    // when it lies between f_i and f*: f_i, f_{i+1} and f^UL each lie within
    // [f^min, f^max] (each bound is a min or max over sets holding f_i and
    // f_{i+1} or f_i and f^UL), so does every value between two of them, and
    // step 7 returns the flux unchanged there, in floating point as well.
    // The strict test of the text only sends the end points (a flux equal
    // to f_i, as in regions of zeros) through steps 4-7.
    const T fstar = med3(fp1, vfma(alpha, dl, f0), f0);
    const bool accept = med3(phi, f0, fstar) == phi;
    T phib = phi;
    // steps 4-7, skipped when every lane of the wavefront accepted (the
    // common case on smooth data)
    if (!__all(accept)) {
      // a zero the compiler cannot see through keeps the curvatures inside
      // this branch (it would otherwise form one per face for reuse by the
      // next face's branch: two instructions on every face)
      T zero = T(0);
      asm volatile("" : "+v"(zero));
      const T c = mp_clamp(phi, fm1 - fm2, dl + zero, dr + zero, fp2 - fp1, f0, fp1, alpha);
      phib = accept ? phi : c;
    }
    if constexpr (LIM == SLMPP_LIM_MPP) {
      // PP limiter, Sec. 2.1.1: keep both half-updates U+ = f_i - p and
      // U- = f_{i+1} + p (p = 2 |zeta| phib, rounded once) non-negative.
      // For floats a - b < 0 exactly when a < b, so the test needs only p.
      const T p = pp_product(tz, phib);
      if (p > f0 || -p > fp1) phib = pp_limit(phib, f0, fp1, tz, p);
    }
    return phib;
  }
}

enum : int32_t { READ_DIRECT = 0, READ_SAFE = 1 };

// Advance cells m0 .. m0+cnt-1 of one pencil (processing order).  `col`
// points at physical cell 0 of the pencil in the LDS tile; consecutive
// cells are `stride` elements apart and G ghost cells exist on both sides.
// READ_DIRECT assumes every read stays within the ghost cells; READ_SAFE
// wraps (periodic) or clamps onto the zero ghost cells (outflow).  With
// RC > 0 the segment length is RC and the results stay in out[]; with
// RC == 0 they are written to `ocol` (same geometry as col, no ghosts).
template <typename T, int ORDER, int LIM, int MODE, int RC>
__device__ __forceinline__ void advance(const T* __restrict__ col, int stride, int n, int G,
                                        int periodic, const PencilEntry<T>& e, int m0, int cnt,
                                        T alpha, T* out, T* __restrict__ ocol) {
  constexpr int H = (ORDER == 7) ? 3 : 2;  // window r_{m-H}..r_{m+H}
  constexpr int WIN = 2 * H + 1;
  T w[ORDER];
#pragma unroll
  for (int k = 0; k < ORDER; ++k) w[k] = e.w[k];
  const T z = e.z;
  const T tz = e.tz;
  const int dir = e.dir;
  int r = e.base + dir * (m0 - 1 - H);  // physical cell of r_{m0-1-H}
  const T* ptr = col + r * stride;      // READ_DIRECT walks a pointer
  const int step = dir * stride;
  auto fetch = [&]() -> T {
    T v;
    if constexpr (MODE == READ_DIRECT) {
      v = *ptr;
      ptr += step;
    } else {
      int rr = r;
      if (periodic) {
        rr %= n;
        if (rr < 0) rr += n;
      } else {
        rr = min(max(rr, -G), n + G - 1);  // ghost cells are zero
      }
      v = col[rr * stride];
      r += dir;
    }
    return v;
  };
  T q[WIN];
#pragma unroll
  for (int k = 0; k < WIN; ++k) q[k] = fetch();
  T f_left = face_flux<T, ORDER, LIM>(q, w, tz, alpha);
  if constexpr (RC > 0) {
#pragma unroll
    for (int k = 0; k < RC; ++k) {
#pragma unroll
      for (int j = 0; j < WIN - 1; ++j) q[j] = q[j + 1];
      q[WIN - 1] = fetch();
      const T f_right = face_flux<T, ORDER, LIM>(q, w, tz, alpha);
      out[k] = vfma(-z, f_right - f_left, q[H]);
      f_left = f_right;
    }
  } else {
    T* optr = ocol + ((dir > 0) ? m0 : (n - 1 - m0)) * stride;
    for (int k = 0; k < cnt; ++k) {
#pragma unroll
      for (int j = 0; j < WIN - 1; ++j) q[j] = q[j + 1];
      q[WIN - 1] = fetch();
      const T f_right = face_flux<T, ORDER, LIM>(q, w, tz, alpha);
      *optr = vfma(-z, f_right - f_left, q[H]);
      optr += step;
      f_left = f_right;
    }
  }
}

// advance() for READ_DIRECT with the stride and the processing direction
// known at compile time, so that the reads of a segment use fixed offsets
// from one address.  Same operations, same results.
template <typename T, int ORDER, int RC, int STRIDE, int DIR>
__device__ __forceinline__ void advance_ct(const T* __restrict__ col, const PencilEntry<T>& e,
                                           int m0, T alpha, T* out) {
  constexpr int H = (ORDER == 7) ? 3 : 2;
  constexpr int WIN = 2 * H + 1;
  constexpr int ST = DIR * STRIDE;
  T w[ORDER];
#pragma unroll
  for (int k = 0; k < ORDER; ++k) w[k] = e.w[k];
  const T z = e.z;
  const T tz = e.tz;
  const T* ptr = col + (e.base + DIR * (m0 - 1 - H)) * STRIDE;
  // the whole window of the segment is read before any flux is formed, so
  // that the LDS reads are in flight together (the branches of the MP and
  // PP steps would otherwise keep each read next to its first use)
  constexpr int NQ = RC + WIN;
  T q[NQ];
#pragma unroll
  for (int k = 0; k < NQ; ++k) q[k] = ptr[k * ST];
  T f_left = face_flux<T, ORDER, SLMPP_LIM_MPP>(q, w, tz, alpha);
#pragma unroll
  for (int k = 0; k < RC; ++k) {
    const T f_right = face_flux<T, ORDER, SLMPP_LIM_MPP>(q + k + 1, w, tz, alpha);
    out[k] = vfma(-z, f_right - f_left, q[k + 1 + H]);
    f_left = f_right;
  }
}

// Store the results of processing positions m0 .. m0 + RC - 1 of a pencil
// of n cells (physical cells m0 + k, or n - 1 - m0 - k when mirrored).
template <typename T, int RC, int STRIDE, int DIR>
__device__ __forceinline__ void store_ct(T* col, int n, int m0, const T* out) {
  T* op = col + ((DIR > 0) ? m0 : (n - 1 - m0)) * STRIDE;
#pragma unroll
  for (int k = 0; k < RC; ++k) op[k * DIR * STRIDE] = out[k];
}

// Compensated sums: s + c, each addition exact in s plus its rounding error in
// c (Knuth's two-sum, no comparison of the magnitudes).
struct KSum {
  double s, c;
};
__device__ __forceinline__ void kadd(KSum& a, double x) {
  const double t = a.s + x;
  const double b = t - a.s;
  a.c += (a.s - (t - b)) + (x - b);
  a.s = t;
}
__device__ __forceinline__ void kmerge(KSum& a, const KSum& b) {
  kadd(a, b.s);
  a.c += b.c;
}

// Adds to a pair that of another lane, which must be active, by a data-parallel
// permute: a few cycles where a shuffle goes through the LDS.  The row of 16
// lanes mirrored, its halves mirrored, its quads reversed and its pairs swapped,
// one after the other (the last m of them), sum over 16 lanes (over 2^m).
constexpr int kRowMirror = 0x140, kHalfMirror = 0x141, kQuadReverse = 0x1b, kPairSwap = 0xb1;
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const int64_t b = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
}
template <int CTRL>
__device__ __forceinline__ void merge_dpp(KSum& v) {
  const KSum o{dpp_move<CTRL>(v.s), dpp_move<CTRL>(v.c)};
  kmerge(v, o);
}

// 16-byte vectors as native clang vector types (kept in registers)
typedef float vf4 __attribute__((ext_vector_type(4)));
typedef double vd2 __attribute__((ext_vector_type(2)));
template <typename T>
struct Vec;
template <>
struct Vec<float> {
  using type = vf4;
  static constexpr int N = 4;
};
template <>
struct Vec<double> {
  using type = vd2;
  static constexpr int N = 2;
};

// scatter / gather the components of a 16-byte vector to / from
// consecutive elements (component access keeps the vector in registers)
// sum of a vector's components in double (fused moment)
__device__ __forceinline__ double vsum(const vf4& v) {
  return ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w);
}
__device__ __forceinline__ double vsum(const vd2& v) { return v.x + v.y; }

__device__ __forceinline__ void put(float* d, const vf4& v) {
  d[0] = v.x;
  d[1] = v.y;
  d[2] = v.z;
  d[3] = v.w;
}
__device__ __forceinline__ void put(double* d, const vd2& v) {
  d[0] = v.x;
  d[1] = v.y;
}
__device__ __forceinline__ void get(const float* s, vf4& v) {
  v.x = s[0];
  v.y = s[1];
  v.z = s[2];
  v.w = s[3];
}
__device__ __forceinline__ void get(const double* s, vd2& v) {
  v.x = s[0];
  v.y = s[1];
}

// f as global memory: global (not flat) loads and stores of the fast
// kernel, whose address may then keep a wave-uniform base in scalar
// registers
template <typename V>
using GlobalPtr = __attribute__((address_space(1))) V*;
template <typename V>
__device__ __forceinline__ V global_load_nt(const V* p) {
  return __builtin_nontemporal_load((GlobalPtr<const V>)p);
}
template <typename V>
__device__ __forceinline__ void global_store_nt(V v, V* p) {
  __builtin_nontemporal_store(v, (GlobalPtr<V>)p);
}

// 16-byte vectors at element-aligned addresses (rows and blocks of odd
// length start anywhere; the hardware takes any 4-byte address)
template <typename T>
struct UVec;
template <>
struct UVec<float> {
  typedef float type __attribute__((ext_vector_type(4), aligned(4)));
};
template <>
struct UVec<double> {
  typedef double type __attribute__((ext_vector_type(2), aligned(8)));
};

// Advance cells m0 .. m0 + R - 1 (processing order) of the pencil whose
// physical cell 0 is at col, cells rs elements apart; R <= MAXR, the
// same for the whole launch (the loop is unrolled with a scalar exit).
// SAFE: reads wrap (periodic) or stop at the zero ghost cells (outflow).
template <typename T, int ORDER, int LIM, bool SAFE, int MAXR>
__device__ __forceinline__ void advance_line(const T* __restrict__ col, int rs, int n, int G,
                                             int periodic, const PencilEntry<T>& e, int m0, int R,
                                             T alpha, T* out) {
  constexpr int H = (ORDER == 7) ? 3 : 2;
  constexpr int WIN = 2 * H + 1;
  int r = e.base + e.dir * (m0 - 1 - H);
  const T* ptr = col + r * rs;
  const int step = e.dir * rs;
  auto fetch = [&]() -> T {
    if constexpr (!SAFE) {
      const T v = *ptr;
      ptr += step;
      return v;
    } else {
      int rr = r;
      if (periodic) {
        rr %= n;
        if (rr < 0) rr += n;
      } else {
        rr = min(max(rr, -G), n + G - 1);
      }
      r += e.dir;
      return col[rr * rs];
    }
  };
  T q[MAXR + WIN];
#pragma unroll
  for (int k = 0; k < WIN; ++k) q[k] = fetch();
  T f_left = face_flux<T, ORDER, LIM>(q, e.w, e.tz, alpha);
#pragma unroll
  for (int k = 0; k < MAXR; ++k) {
    if (k < R) {
      q[k + WIN] = fetch();
      const T f_right = face_flux<T, ORDER, LIM>(q + k + 1, e.w, e.tz, alpha);
      out[k] = vfma(-e.z, f_right - f_left, q[k + 1 + H]);
      f_left = f_right;
    }
  }
}

// A pencil entry read through the constant address space: the tables are
// not written while a sweep runs, so where the address is uniform over the
// wavefront the compiler loads the entry with scalar loads and keeps it in
// scalar registers (its weights then enter the FMAs as scalar operands).
template <typename T>
__device__ __forceinline__ PencilEntry<T> load_entry_uniform(const PencilEntry<T>* p) {
  constexpr int NW = sizeof(PencilEntry<T>) / 4;
  using CW = const __attribute__((address_space(4))) uint32_t*;
  const CW q = (CW)(p);
  uint32_t w[NW];
#pragma unroll
  for (int i = 0; i < NW; ++i) w[i] = q[i];
  PencilEntry<T> e;
  __builtin_memcpy(&e, w, sizeof(e));
  return e;
}
template <typename P>
__device__ __forceinline__ P load_ptr_uniform(const P* p) {
  using CU = const __attribute__((address_space(4))) uint64_t*;
  return reinterpret_cast<P>(static_cast<uintptr_t>(*(CU)(p)));
}

// Pencil-table entry for speed c (see PencilEntry).
template <typename T, int ORDER>
__device__ __forceinline__ PencilEntry<T> pencil_entry_of(const SweepArgs& a, double c) {
  const double xi = departure(c, a.dt, a.h);
  const int n = a.n;
  double zeta;
  int64_t N;
  if (a.rk) {
    // TVD-RK stage (Sec. 2.1.1): no shift, the CFL number itself as zeta;
    // |nu| > 1 poisons the pencil
    N = 0;
    zeta = fabs(xi) <= 1.0 ? xi : __builtin_nan("");
  } else if (!(fabs(xi) < 4.0e18)) {  // non-finite or absurd offset: poison the pencil
    N = 0;
    zeta = __builtin_nan("");
  } else {
    const double Nd = floor(xi + 0.5);
    zeta = xi - Nd;
    N = (int64_t)Nd;
  }
  if (a.bc == SLMPP_BC_PERIODIC) {
    N %= n;
    if (N < 0) N += n;
    if (N > n / 2) N -= n;
  } else {
    const int64_t lim = (int64_t)n + 64;
    N = N < -lim ? -lim : (N > lim ? lim : N);
  }
  const bool mirror = zeta < 0.0;
  const double az = mirror ? -zeta : zeta;
  PencilEntry<T> e{};
  e.dir = mirror ? -1 : 1;
  e.base = (int32_t)((mirror ? (int64_t)(n - 1) : 0) - N);
  e.absN = (int16_t)(N < 0 ? -N : N);
  e.z = (T)az;
  e.tz = (T)(az + az);
  // an RK stage takes the interface interpolation itself: the flux
  // polynomial at zero Courant number
  const double zw = a.rk ? 0.0 : az;
#pragma unroll
  for (int k = 0; k < ORDER; ++k) {
    double acc = 0.0;
#pragma unroll
    for (int j = ORDER - 1; j >= 0; --j) {
      Frac fr;
      if constexpr (ORDER == 7) {
        fr = kCsl7[k][j];
      } else {
        fr = kCsl5[k][j];
      }
      acc = acc * zw + fr.num / fr.den;
    }
    e.w[k] = (T)acc;
  }
  return e;
}

// Entry for speed index idx: a velocity cell centre or a spatial cell.
template <typename T, int ORDER>
__device__ __forceinline__ PencilEntry<T> pencil_entry(const SweepArgs& a, int idx) {
  return pencil_entry_of<T, ORDER>(
      a, a.cmode == SPEED_FROM_VELOCITY ? cell_center(a.vlo, a.dv, idx) : a.accel[idx]);
}

}  // namespace
}  // namespace slmpp
