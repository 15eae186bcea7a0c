// The field solve in four launches: density and transform along x_1, the
// other axes with the Green function between forward and inverse, inverse
// along x_1, and forces by the FDA together with the pencil tables of the
// next velocity kick (Sec. 2.2, App. C).  Periodic boundaries and, on the
// doubled grid, isolated ones (D = 3).  Double precision throughout.
//
// One-dimensional transforms are direct sums over at most a few hundred
// points.  Where the length divides by 4 (or 2) the sum is taken in 4 (2)
// residue classes of the input index, from which 4 (2) outputs a quarter
// (half) of the length apart follow without further products:
//   X[k + q m / R] = sum_r exp(-2 pi i q r / R) S_r[k],
//   S_r[k] = sum_{j = r mod R} x_j exp(-2 pi i j k / m).
// Launches and the latency of the sums bound it, not bytes or operations:
// 64^2 cells took 11 launches and 75 us, now 28 us with the moment's row sums
// and the tables of the next kick; 32^3 cells isolated 13 launches (the doubled
// grid in full) and 165 us, now 72 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "slmpp_internal.hpp"
#include "sweep_device.hpp"

namespace slmpp {
namespace {

// The density of cell i from its nsub row sums, part[s n + i] (pairs: each the
// sum and its error), added in tile order.
__device__ __forceinline__ double sum_rows(const double* part, bool pairs, int64_t i, int nsub, int n, double dvol) {
  constexpr int U = 16;  // loads in flight
  KSum a{0.0, 0.0}, b{0.0, 0.0};
  for (int s = 0; s < nsub; s += U) {
    double v[U], e[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t at = (int64_t)min(s + u, nsub - 1) * n + i;
      if (pairs) {
        const double2 x = reinterpret_cast<const double2*>(part)[at];
        v[u] = x.x;
        e[u] = x.y;
      } else {
        v[u] = part[at];
        e[u] = 0.0;
      }
    }
#pragma unroll
    for (int u = 0; u < U; u += 2) {
      if (s + u < nsub) {
        kadd(a, v[u]);
        a.c += e[u];
      }
      if (s + u + 1 < nsub) {
        kadd(b, v[u + 1]);
        b.c += e[u + 1];
      }
    }
  }
  kadd(a, b.s);
  return dvol * (a.s + (a.c + b.c));
}

// S_r[k] (see above) of the nin inputs x(j), r = 0..R-1; tw[q] = exp(-2 pi i
// q / m), conjugated with inv.
template <int R, typename X>
__device__ __forceinline__ void residue_sums(X&& x, int nin, int m, int k, const double2* tw, bool inv,
                                             double2* S) {
#pragma unroll
  for (int r = 0; r < R; ++r) S[r] = make_double2(0.0, 0.0);
  int q = 0, j = 0;
  for (; j + R <= nin; j += R) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double2 w = tw[q], v = x(j + r);
      const double wi = inv ? -w.y : w.y;
      S[r].x += v.x * w.x - v.y * wi;
      S[r].y += v.x * wi + v.y * w.x;
      q += k;
      if (q >= m) q -= m;
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (j + r < nin) {
      const double2 w = tw[q], v = x(j + r);
      const double wi = inv ? -w.y : w.y;
      S[r].x += v.x * w.x - v.y * wi;
      S[r].y += v.x * wi + v.y * w.x;
      q += k;
      if (q >= m) q -= m;
    }
  }
}

// Outputs k + q m / R (q = 0..R-1) of one transform, handed to put(index, value).
template <int R, typename X, typename P>
__device__ __forceinline__ void transform_group(X&& x, int nin, int m, int k, const double2* tw, bool inv,
                                                P&& put) {
  double2 S[R];
  residue_sums<R>(x, nin, m, k, tw, inv, S);
  if constexpr (R == 1) {
    put(k, S[0]);
  } else if constexpr (R == 2) {
    put(k, make_double2(S[0].x + S[1].x, S[0].y + S[1].y));
    put(k + m / 2, make_double2(S[0].x - S[1].x, S[0].y - S[1].y));
  } else {
    const double2 a = make_double2(S[0].x + S[2].x, S[0].y + S[2].y);
    const double2 b = make_double2(S[0].x - S[2].x, S[0].y - S[2].y);
    const double2 c = make_double2(S[1].x + S[3].x, S[1].y + S[3].y);
    // (S_1 - S_3) times -i forward, +i inverse
    double2 d = make_double2(S[1].y - S[3].y, S[3].x - S[1].x);
    if (inv) d = make_double2(-d.x, -d.y);
    put(k, make_double2(a.x + c.x, a.y + c.y));
    put(k + m / 4, make_double2(b.x + d.x, b.y + d.y));
    put(k + m / 2, make_double2(a.x - c.x, a.y - c.y));
    put(k + 3 * (m / 4), make_double2(b.x - d.x, b.y - d.y));
  }
}

// All outputs wanted of `lines` transforms of length m, dealt to the threads
// of the workgroup: x(line, j) the inputs, put(line, index, value) for the
// outputs o0 .. o0 + nout - 1 (mod m).  Full transforms use the residue
// classes; part ones are summed output by output.
template <typename X, typename P>
__device__ __forceinline__ void transforms(X&& x, int lines, int nin, int m, int nout, int o0,
                                           const double2* tw, bool inv, P&& put) {
  const bool full = nout == m && o0 == 0;
  auto all = [&](auto rad) {
    constexpr int R = decltype(rad)::value;
    const int g = full ? m / R : nout;
    for (int t = threadIdx.x; t < lines * g; t += blockDim.x) {
      // consecutive threads take consecutive lines
      const int k = t / lines, l = t - k * lines;
      auto xl = [&](int j) { return x(l, j); };
      if (full) {
        transform_group<R>(xl, nin, m, k, tw, inv, [&](int o, double2 v) { put(l, o, v); });
      } else {
        int o = k + o0;
        o += o < 0 ? m : 0;
        o -= o >= m ? m : 0;
        transform_group<1>(xl, nin, m, o, tw, inv, [&](int, double2 v) { put(l, k, v); });
      }
    }
  };
  if (full && m % 4 == 0)
    all(std::integral_constant<int, 4>{});
  else if (full && m % 2 == 0)
    all(std::integral_constant<int, 2>{});
  else
    all(std::integral_constant<int, 1>{});
}

// Forward transform along x_1 of columns c (x_2..x_D) of the density, out
// [k1][c].  The density is rho[i][c], or the row sums of an x_1 sweep
// (part[(c nsub + q) n1 + i], added in tile order, compensated), which
// leaves rho as well.
__global__ void __launch_bounds__(256) field_forward_kernel(FieldPlan p, const double* __restrict__ part,
                                                            bool pairs, int nsub,
                                                            double dvol,
                                                            double* __restrict__ rho,
                                                            double2* __restrict__ out,
                                                            const double2* __restrict__ tw) {
  extern __shared__ __align__(16) unsigned char smem[];
  double2* t1 = reinterpret_cast<double2*>(smem);
  double* x = reinterpret_cast<double*>(t1 + p.m[0]);  // [column][i], odd pitch
  const int n1 = p.n[0], m1 = p.m[0], C = p.n[1] * p.n[2], pitch = n1 | 1;
  const int c0 = blockIdx.x * p.cols1, cols = min(p.cols1, C - c0);
  for (int t = threadIdx.x; t < m1; t += blockDim.x) t1[t] = tw[p.tw[0] + t];
  if (part) {
    for (int t = threadIdx.x; t < cols * n1; t += blockDim.x) {
      const int c = t / n1, i = t - c * n1;
      const int64_t at = ((int64_t)(c0 + c) * nsub) * n1 + i;
      const double r = sum_rows(part, pairs, at, nsub, n1, dvol);
      x[c * pitch + i] = r;
      rho[(int64_t)i * C + c0 + c] = r;
    }
  } else {
    for (int t = threadIdx.x; t < cols * n1; t += blockDim.x) {
      const int i = t / cols, c = t - i * cols;
      x[c * pitch + i] = rho[(int64_t)i * C + c0 + c];
    }
  }
  __syncthreads();
  transforms([&](int l, int j) { return make_double2(x[l * pitch + j], 0.0); }, cols, n1, m1, m1, 0, t1,
             false, [&](int l, int k, double2 v) { out[(int64_t)k * C + c0 + l] = v; });
}

// One k_1 per workgroup: forward along x_2 and x_3, the Green function,
// inverse along x_3 and x_2 (D = 2: x_2 alone, held as the plane's x_3).
// in [k1][n2][n3] -> out [k1][o2][o3].
__global__ void __launch_bounds__(512) field_planes_kernel(FieldPlan p, const double2* __restrict__ in,
                                                           double2* __restrict__ out,
                                                           const double* __restrict__ green,
                                                           const double2* __restrict__ tw) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int n2 = p.n[1], n3 = p.n[2], m2 = p.m[1], m3 = p.m[2], o2 = p.o[1], o3 = p.o[2];
  const int pitch = max(n3, o3) | 1;
  double2* t2 = reinterpret_cast<double2*>(smem);
  double2* t3 = t2 + m2;
  double2* B = t3 + m3;              // [k2][pitch]
  double2* chunk = B + m2 * pitch;   // some columns [c][n2 | 1], then some rows [r][m3 | 1]
  const int64_t k1 = blockIdx.x;
  for (int t = threadIdx.x; t < m2; t += blockDim.x) t2[t] = tw[p.tw[1] + t];
  for (int t = threadIdx.x; t < m3; t += blockDim.x) t3[t] = tw[p.tw[2] + t];
  const double2* src = in + k1 * n2 * n3;
  // forward along x_2
  if (n2 == 1) {
    for (int t = threadIdx.x; t < n3; t += blockDim.x) B[t] = src[t];
  } else {
    const int pc = n2 | 1;
    for (int c0 = 0; c0 < n3; c0 += p.cols2) {
      const int cols = min(p.cols2, n3 - c0);
      __syncthreads();
      for (int t = threadIdx.x; t < cols * n2; t += blockDim.x) {
        const int i = t / cols, c = t - i * cols;
        chunk[c * pc + i] = src[i * n3 + c0 + c];
      }
      __syncthreads();
      transforms([&](int l, int j) { return chunk[l * pc + j]; }, cols, n2, m2, m2, 0, t2, false,
                 [&](int l, int k, double2 v) { B[k * pitch + c0 + l] = v; });
    }
  }
  // rows k_2: forward along x_3, Green function, inverse
  const int pr = m3 | 1;
  for (int r0 = 0; r0 < m2; r0 += p.rows2) {
    const int rows = min(p.rows2, m2 - r0);
    __syncthreads();
    transforms([&](int l, int j) { return B[(r0 + l) * pitch + j]; }, rows, n3, m3, m3, 0, t3, false,
               [&](int l, int k, double2 v) {
                 const double g = green[(k1 * m2 + r0 + l) * m3 + k];
                 chunk[l * pr + k] = make_double2(v.x * g, v.y * g);
               });
    __syncthreads();
    transforms([&](int l, int j) { return chunk[l * pr + j]; }, rows, m3, m3, o3, -p.halo, t3, true,
               [&](int l, int k, double2 v) { B[(r0 + l) * pitch + k] = v; });
  }
  __syncthreads();
  // inverse along x_2
  double2* dst = out + k1 * o2 * o3;
  if (n2 == 1) {
    for (int t = threadIdx.x; t < o3; t += blockDim.x) dst[t] = B[t];
  } else {
    transforms([&](int l, int j) { return B[j * pitch + l]; }, o3, m2, m2, o2, -p.halo, t2, true,
               [&](int l, int k, double2 v) { dst[k * o3 + l] = v; });
  }
}

// Inverse along x_1 of columns c of [m1][o2 o3]; the real part, scaled, to
// phi [o1][o2 o3].
__global__ void __launch_bounds__(256) field_inverse_kernel(FieldPlan p, const double2* __restrict__ in,
                                                            double* __restrict__ phi, double scale,
                                                            const double2* __restrict__ tw) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int m1 = p.m[0], C = p.o[1] * p.o[2], pitch = m1 | 1;
  double2* t1 = reinterpret_cast<double2*>(smem);
  double2* x = t1 + m1;
  const int c0 = blockIdx.x * p.cols3, cols = min(p.cols3, C - c0);
  for (int t = threadIdx.x; t < m1; t += blockDim.x) t1[t] = tw[p.tw[0] + t];
  for (int t = threadIdx.x; t < cols * m1; t += blockDim.x) {
    const int i = t / cols, c = t - i * cols;
    x[c * pitch + i] = in[(int64_t)i * C + c0 + c];
  }
  __syncthreads();
  transforms([&](int l, int j) { return x[l * pitch + j]; }, cols, m1, m1, p.o[0], -p.halo, t1, true,
             [&](int l, int k, double2 v) { phi[(int64_t)k * C + c0 + l] = v.x * scale; });
}

__device__ __forceinline__ double fda(int order, double h, double a1, double b1, double a2, double b2,
                                      double a3, double b3) {
  if (order == 2) return (a1 - b1) / (2.0 * h);
  if (order == 4) return (8.0 * (a1 - b1) - (a2 - b2)) / (12.0 * h);
  return (45.0 * (a1 - b1) - 9.0 * (a2 - b2) + (a3 - b3)) / (60.0 * h);
}

// accel_l = -dphi/dx_l (App. C) of every cell and component (grid.y), from
// phi [o1][o2][o3] (with a halo of p.halo cells, or wrapping); with tab[l]
// the pencil-table entries of a velocity sweep along v_l as well.
template <typename T, int ORDER>
__global__ void __launch_bounds__(128) field_force_kernel(FieldPlan p, const double* __restrict__ phi,
                                                          double* __restrict__ phi_out,
                                                          double* __restrict__ accel, FieldTables tabs) {
  const int64_t nxs = (int64_t)p.n[0] * p.n[1] * p.n[2];
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nxs) return;
  const int i3 = (int)(t % p.n[2]);
  const int i2 = (int)((t / p.n[2]) % p.n[1]);
  const int i1 = (int)(t / ((int64_t)p.n[1] * p.n[2]));
  const int H = p.halo;
  const int h2 = p.n[1] > 1 ? H : 0;
  const int64_t q = ((int64_t)(i1 + H) * p.o[1] + (i2 + h2)) * p.o[2] + (i3 + H);
  const int l = blockIdx.y;  // component
  // array axis of component l: D = 2 holds x_2 as the third axis
  const int ax = l == 0 ? 0 : (p.D == 2 ? 2 : l);
  const int i = ax == 0 ? i1 : (ax == 1 ? i2 : i3);
  const int n = p.n[ax];
  const int64_t st = ax == 0 ? (int64_t)p.o[1] * p.o[2] : (ax == 1 ? p.o[2] : 1);
  auto P = [&](int k) {
    if (H) return phi[q + k * st];
    int r = (i + k) % n;
    if (r < 0) r += n;
    return phi[q + (int64_t)(r - i) * st];
  };
  const bool far2 = p.order > 2, far3 = p.order > 4;
  const double a = -fda(p.order, p.h[l], P(1), P(-1), far2 ? P(2) : 0.0, far2 ? P(-2) : 0.0,
                        far3 ? P(3) : 0.0, far3 ? P(-3) : 0.0);
  accel[(int64_t)l * nxs + t] = a;
  if (l == 0 && phi_out) phi_out[t] = phi[q];
  if (tabs.tab[l]) {
    SweepArgs s{};
    s.dt = tabs.dt;
    s.h = tabs.h[l];
    s.n = tabs.n[l];
    s.bc = tabs.bc;
    s.rk = tabs.rk;
    reinterpret_cast<PencilEntry<T>*>(tabs.tab[l])[t] = pencil_entry_of<T, ORDER>(s, a);
  }
}

}  // namespace

namespace {
// Time of the solve in four launches: few workgroups transform long lines
// where an axis is long and the others short.  A workgroup's transforms of
// nin inputs take 37 ns per input and round of its threads (the latency of
// a sum) or 9 per input and wavefront (the LDS of a CU; 12 where the outputs
// wanted are some of the transform's), whichever is longer; four launches.
double transforms_us(int lines, int nin, int m, int nout, int threads) {
  const bool full = nout == m;
  const int64_t sums = (int64_t)lines * (full ? m / (m % 4 == 0 ? 4 : m % 2 == 0 ? 2 : 1) : nout);
  const double rounds = (double)((sums + threads - 1) / threads), waves = (double)((sums + 63) / 64);
  return 1e-3 * nin * std::max(37.0 * rounds, (full ? 9.0 : 12.0) * waves);
}
double four_launches_us(const FieldPlan& p) {
  auto groups = [](int total, int each) { return (total + each - 1) / each; };
  auto turns = [](int workgroups) { return (workgroups + 255) / 256; };
  double planes = 0.0;
  for (int c = 0; c < p.n[2] && p.n[1] > 1; c += p.cols2)
    planes += transforms_us(std::min(p.cols2, p.n[2] - c), p.n[1], p.m[1], p.m[1], 512);
  for (int r = 0; r < p.m[1]; r += p.rows2) {
    const int rows = std::min(p.rows2, p.m[1] - r);
    planes += transforms_us(rows, p.n[2], p.m[2], p.m[2], 512) + transforms_us(rows, p.m[2], p.m[2], p.o[2], 512);
  }
  if (p.n[1] > 1) planes += transforms_us(p.o[2], p.m[1], p.m[1], p.o[1], 512);
  return turns(groups(p.n[1] * p.n[2], p.cols1)) * transforms_us(p.cols1, p.n[0], p.m[0], p.m[0], 256) +
         turns(p.m[0]) * planes +
         turns(groups(p.o[1] * p.o[2], p.cols3)) * transforms_us(p.cols3, p.m[0], p.m[0], p.o[0], 256) + 14.0;
}
// Time of the solve in a launch per axis, one thread per output: 150 ns per
// input, or 3 ps per product of the grid (1.3 where most of it is zero).
//   us, measured with the launches per axis / in four launches (and the moment):
// 64^2 69 / 27, 512^2 886 / 336, 4096 x 2 1312 / 1256, 4 x 3001 933 / 2284,
// 64^3 375 / 278, 90^3 1114 / 871, 4 x 90^2 129 / 225, 3 x 100 x 80 119 / 131,
// 8 x 8 x 256 99 / 78; isolated 64^3 1860 / 610, 128 x 8 x 8 178 / 38,
// 8 x 8 x 128 95 / 138.
double separate_launches_us(const FieldPlan& p) {
  const double all = (double)p.m[0] * p.m[1] * p.m[2];
  double t = 36.0;
  for (int l = 0; l < 3; ++l)
    if (p.m[l] > 1) t += 2e-3 * p.m[l] * std::max(150.0, (p.halo ? 1.3e-3 : 3e-3) * all);
  return t;
}
}  // namespace

// D axes of n cells each (periodic: transforms of n; isolated: of 2 n, with
// three halo cells of the potential on both sides).  ok == 0: the planes do
// not fit the LDS of a workgroup, or launches per axis are faster.
FieldPlan plan_field(int D, const int64_t* nx, const double* h, int order, bool isolated) {
  FieldPlan p{};
  p.D = D;
  p.order = order;
  p.halo = isolated ? 3 : 0;
  for (int l = 0; l < 3; ++l) p.n[l] = 1;
  p.n[0] = (int)nx[0];
  if (D == 2) p.n[2] = (int)nx[1];
  if (D == 3) {
    p.n[1] = (int)nx[1];
    p.n[2] = (int)nx[2];
  }
  int off = 0;
  for (int l = 0; l < 3; ++l) {
    p.m[l] = isolated ? 2 * p.n[l] : p.n[l];
    p.o[l] = p.n[l] + 2 * p.halo;
    // a doubled axis shorter than the potential with its halo wraps
    if (p.o[l] > p.m[l] && isolated) return FieldPlan{};
    p.tw[l] = 0;
  }
  // twiddles of the axes in the caller's order
  p.tw[0] = 0;
  off = p.m[0];
  if (D == 2) {
    p.tw[2] = off;
    p.tw[1] = 0;  // length 1: the first entry of any table
  } else if (D == 3) {
    p.tw[1] = off;
    p.tw[2] = off + p.m[1];
  }
  for (int l = 0; l < D; ++l) p.h[l] = h[l];
  const size_t most = 160 * 1024, few = 32 * 1024;
  auto cols_for = [&](size_t fixed, size_t each, int total) {
    int c = (int)std::max<size_t>(1, few > fixed ? (few - fixed) / each : 1);
    // enough workgroups to spread the columns over the GPU
    c = std::min(c, std::max(1, (total + 255) / 256));
    return std::max(1, c);
  };
  const size_t e1 = sizeof(double) * (p.n[0] | 1), e3 = sizeof(double2) * (p.m[0] | 1);
  const size_t f1 = sizeof(double2) * p.m[0];
  p.cols1 = cols_for(f1, e1, p.n[1] * p.n[2]);
  p.cols3 = cols_for(f1, e3, p.o[1] * p.o[2]);
  p.lds1 = f1 + p.cols1 * e1;
  p.lds3 = f1 + p.cols3 * e3;
  const size_t plane = sizeof(double2) * ((size_t)p.m[1] * (std::max(p.n[2], p.o[2]) | 1) + p.m[1] + p.m[2]);
  const size_t ec = sizeof(double2) * (p.n[1] | 1), er = sizeof(double2) * (p.m[2] | 1);
  if (plane + std::max(ec, er) > most || p.lds1 > most || p.lds3 > most) return FieldPlan{};
  // chunks: what is left of 64 KB, or of the whole LDS for large planes
  const size_t room = plane < 48 * 1024 ? 64 * 1024 - plane : most - plane;
  p.cols2 = (int)std::max<size_t>(1, std::min<size_t>(p.n[2], room / ec));
  p.rows2 = (int)std::max<size_t>(1, std::min<size_t>(p.m[1], room / er));
  p.lds2 = plane + std::max(p.cols2 * ec, p.rows2 * er);
  p.ok = four_launches_us(p) <= separate_launches_us(p) ? 1 : 0;
  return p;
}

namespace {
hipError_t allow_lds(const void* k, size_t lds) {
  return lds > 64 * 1024 ? hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)
                         : hipSuccess;
}
}  // namespace

hipError_t launch_field_forward(const FieldPlan& p, const double* part, bool pairs, int nsub,
                                double dvol, double* rho, double2* bufA, const double2* tw, hipStream_t s) {
  hipError_t e = allow_lds(reinterpret_cast<const void*>(field_forward_kernel), p.lds1);
  if (e != hipSuccess) return e;
  const int C1 = p.n[1] * p.n[2];
  hipLaunchKernelGGL(field_forward_kernel, dim3((C1 + p.cols1 - 1) / p.cols1), dim3(256), p.lds1, s, p,
                     part, pairs, nsub, dvol, rho, bufA, tw);
  return hipGetLastError();
}

// bufA, bufB: m1 n2 n3 and m1 o2 o3 complex values; phi_ext (isolated):
// o1 o2 o3 doubles, may be bufA.
hipError_t launch_field_rest(const FieldPlan& p, double* phi, double* accel, double2* bufA,
                             double2* bufB, double* phi_ext, const double2* tw, const double* green,
                             int dtype, int order, const FieldTables& tabs, hipStream_t s) {
  hipError_t e = allow_lds(reinterpret_cast<const void*>(field_planes_kernel), p.lds2);
  if (e == hipSuccess) e = allow_lds(reinterpret_cast<const void*>(field_inverse_kernel), p.lds3);
  if (e != hipSuccess) return e;
  const int C3 = p.o[1] * p.o[2];
  const int64_t nxs = (int64_t)p.n[0] * p.n[1] * p.n[2];
  double* ext = p.halo ? phi_ext : phi;
  hipLaunchKernelGGL(field_planes_kernel, dim3(p.m[0]), dim3(512), p.lds2, s, p, bufA, bufB, green, tw);
  const double scale = 1.0 / ((double)p.m[0] * p.m[1] * p.m[2]);
  hipLaunchKernelGGL(field_inverse_kernel, dim3((C3 + p.cols3 - 1) / p.cols3), dim3(256), p.lds3, s, p,
                     bufB, ext, scale, tw);
  const dim3 grid((unsigned)((nxs + 127) / 128), p.D);
  double* phi_out = p.halo ? phi : nullptr;
  auto force = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(128), 0, s, p, ext, phi_out, accel, tabs);
    return hipGetLastError();
  };
  if (dtype == SLMPP_F64)
    return order == 7 ? force(field_force_kernel<double, 7>) : force(field_force_kernel<double, 5>);
  return order == 7 ? force(field_force_kernel<float, 7>) : force(field_force_kernel<float, 5>);
}

// ---- one dimension --------------------------------------------------------
namespace {
constexpr int kConvLanes = 16;    // threads per output
constexpr int kConvThreads = 256;

// sum over the lanes of an output, in a fixed order
__device__ __forceinline__ void merge_lanes(KSum& v) {
#pragma unroll
  for (int off = 1; off < kConvLanes; off <<= 1) {
    const KSum o{__shfl_xor(v.s, off, kConvLanes), __shfl_xor(v.c, off, kConvLanes)};
    kadd(v, o.s);
    v.c += o.c;
  }
}

// phi = conv_phi * rho and a = conv_a * rho (circular), for 16 cells per
// workgroup, each workgroup with the whole density in LDS (from the row sums
// of an x_1 sweep: every workgroup adds them all, the first one stores rho).
// Only differences of the density enter (the kernels sum to zero), summed with
// compensation, so that no force of the density on itself builds up.  One launch
// in place of transforms, Green function, inverse, forces and tables: 256
// cells took 25 us in one workgroup and two launches for tables, now 6.8 us.
template <typename T, int ORDER>
__global__ void __launch_bounds__(kConvThreads) field_conv_kernel(
    int n, const double* __restrict__ part, bool pairs, int nsub, double dvol,
    double* __restrict__ rho, double* __restrict__ phi, double* __restrict__ accel, const double* __restrict__ conv,
    FieldTables tabs) {
  extern __shared__ __align__(16) unsigned char smem[];
  // the density and the kernels' first halves
  const int half = n / 2;
  double* x = reinterpret_cast<double*>(smem);
  double* kp = x + n;
  double* ka = kp + half + 1;
  const int tid = threadIdx.x;
  for (int i = tid; i <= half; i += kConvThreads) {
    kp[i] = conv[i];
    ka[i] = conv[n + i];
  }
  for (int i = tid; i < n; i += kConvThreads) {
    double r;
    if (part) {
      r = sum_rows(part, pairs, i, nsub, n, dvol);
      if (blockIdx.x == 0) rho[i] = r;
    } else {
      r = rho[i];
    }
    x[i] = r;
  }
  __syncthreads();
  const int lane = tid & (kConvLanes - 1);
  const int i = blockIdx.x * (kConvThreads / kConvLanes) + tid / kConvLanes;
  if (i >= n) return;
  // the kernels are even (phi) and odd (a) in the distance: pairs of cells at
  // the same distance on both sides, the odd one through their difference
  const double x0 = x[0];
  KSum sp{0.0, 0.0}, sa{0.0, 0.0};
  for (int d = lane; 2 * d <= n; d += kConvLanes) {
    int l = i - d, r = i + d;
    l += l < 0 ? n : 0;
    r -= r >= n ? n : 0;
    const double xl = x[l], xr = x[r];
    kadd(sp, kp[d] * (d == 0 || 2 * d == n ? xl - x0 : (xl - x0) + (xr - x0)));
    kadd(sa, ka[d] * (xl - xr));
  }
  merge_lanes(sp);
  merge_lanes(sa);
  const double phi_i = sp.s + sp.c, a_i = sa.s + sa.c;
  if (lane == 0) {
    phi[i] = phi_i;
    accel[i] = a_i;
    if (tabs.tab[0]) {
      SweepArgs s{};
      s.dt = tabs.dt;
      s.h = tabs.h[0];
      s.n = tabs.n[0];
      s.bc = tabs.bc;
      s.rk = tabs.rk;
      reinterpret_cast<PencilEntry<T>*>(tabs.tab[0])[i] = pencil_entry_of<T, ORDER>(s, a_i);
    }
  }
}

// The circular kernels of the periodic solve on n cells: the inverse
// transform of the Green function, conv[0..n), and of minus its FDA,
// conv[n..2n), whose symbol is i S(theta).  Only the first half of the roots
// of unity is used (those beyond pi carry the rounding of their angle), and
// the Green function through its sums over k and n - k, all that a real
// density sees of it.
__global__ void __launch_bounds__(kConvThreads) conv_setup_kernel(int n, double h, int order,
                                                         const double* __restrict__ green,
                                                         const double2* __restrict__ tw,
                                                         double* __restrict__ conv) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int half = n / 2;
  double* g = reinterpret_cast<double*>(smem);
  double* gs = g + half + 1;
  double* c = gs + half + 1;
  double* sn = c + n;
  for (int q = threadIdx.x; q < n; q += blockDim.x) {
    const double2 t = tw[q <= half ? q : n - q];
    c[q] = t.x;
    sn[q] = q <= half ? -t.y : t.y;
  }
  __syncthreads();
  for (int k = threadIdx.x; k <= half; k += blockDim.x) {
    const bool pair = k > 0 && 2 * k != n;
    g[k] = pair ? green[k] + green[n - k] : green[k];
    const double s1 = sn[k], s2 = sn[(2 * k) % n], s3 = sn[(3 * k) % n];
    const double sym = order == 2 ? s1 / h
                                  : (order == 4 ? (16.0 * s1 - 2.0 * s2) / (12.0 * h)
                                                : (90.0 * s1 - 18.0 * s2 + 2.0 * s3) / (60.0 * h));
    gs[k] = pair ? g[k] * sym : 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & (kConvLanes - 1);
  const int i = blockIdx.x * (kConvThreads / kConvLanes) + threadIdx.x / kConvLanes;
  if (i >= n) return;
  KSum p{0.0, 0.0}, a{0.0, 0.0};
  for (int k = lane; k <= half; k += kConvLanes) {
    const int q = (k * i) % n;
    kadd(p, g[k] * c[q]);
    kadd(a, gs[k] * sn[q]);
  }
  merge_lanes(p);
  merge_lanes(a);
  if (lane == 0) {
    conv[i] = (p.s + p.c) / n;
    conv[n + i] = (a.s + a.c) / n;
  }
}
}  // namespace

hipError_t launch_conv_setup(int n, double h, int order, const double* green, const double2* tw,
                             double* conv, hipStream_t s) {
  const size_t lds = sizeof(double) * (2 * (size_t)(n / 2 + 1) + 2 * (size_t)n);
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(conv_setup_kernel), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(conv_setup_kernel, dim3((n + kConvThreads / kConvLanes - 1) / (kConvThreads / kConvLanes)),
                     dim3(kConvThreads), lds, s, n, h, order, green, tw, conv);
  return hipGetLastError();
}

hipError_t launch_field_conv(int n, const double* part, bool pairs, int nsub, double dvol,
                             double* rho, double* phi, double* accel, const double* conv, int dtype, int order,
                             const FieldTables& tabs, hipStream_t s) {
  constexpr int per = kConvThreads / kConvLanes;
  const size_t lds = sizeof(double) * ((size_t)n + 2 * (size_t)(n / 2 + 1));
  auto go = [&](auto kern) {
    const hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((n + per - 1) / per), dim3(kConvThreads), lds, s, n, part, pairs, nsub, dvol, rho,
                       phi, accel, conv, tabs);
    return hipGetLastError();
  };
  if (dtype == SLMPP_F64)
    return order == 7 ? go(field_conv_kernel<double, 7>) : go(field_conv_kernel<double, 5>);
  return order == 7 ? go(field_conv_kernel<float, 7>) : go(field_conv_kernel<float, 5>);
}

}  // namespace slmpp
