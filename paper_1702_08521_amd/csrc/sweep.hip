// Fused SL-MPP sweep kernels for gfx950.
//
// One launch advances every pencil along one axis of f by one
// semi-Lagrangian step (Sec. 2.1.2, Eq. (SL)):
//   xi = c dt / h  ->  integer shift N = floor(xi + 1/2), zeta = xi - N
//   Phi_{i-1/2}    =  CSL5 / CSL7 polynomial in zeta (rows C_j / D_j)
//   Phibar         =  MP constraint (App. A) on the 5-point stencil
//   Phihat         =  PP flux limiter (Sec. 2.1.1)
//   f_i^{n+1}      =  f_{i-N} - zeta (Phihat_{i+1/2} - Phihat_{i-1/2})
// For zeta < 0 the shifted pencil is processed in reverse order, the
// mirror image of the c > 0 construction the paper writes out.
//
// Two kernels per sweep:
//  * pencil_table_kernel: one entry per distinct speed (a velocity cell
//    centre for x-sweeps, a spatial cell for v-sweeps) holding the integer
//    shift, direction, |zeta| and the CSL flux as FIR weights w_k(|zeta|),
//    all computed in FP64 (rounded once to the storage type).
//  * sweep_kernel: a workgroup owns a tile of W whole pencils.  It streams
//    the tile from HBM into LDS once (16-byte vectors, coalesced along the
//    contiguous axis whichever way the pencils run), adds ghost rows
//    (periodic images or zeros), advances every pencil from LDS with a
//    register sliding window (each interface flux computed once and used
//    by both neighbouring cells; each thread owns a segment of R cells),
//    writes the results back into the LDS tile and streams it out in place.
//    A sweep therefore reads and writes f exactly once; halos stay on chip.
//    sweep_fast_kernel is its persistent form with the next tile prefetched
//    into registers (several runs of one geometry per launch for batched
//    ensembles); batch_sweep_kernel walks a list of tiles of many runs.
//  * kick_plane_kernel: the sweeps along the last two velocity axes of a
//    kick in one pass over f, whole velocity planes in LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>

#include "slmpp_internal.hpp"
#include "sweep_device.hpp"
#include "sweep_launch.hpp"

namespace slmpp {
namespace {

size_t entry_bytes(int dtype) {
  return dtype == SLMPP_F64 ? sizeof(PencilEntry<double>) : sizeof(PencilEntry<float>);
}

}  // namespace

hipError_t launch_batch_tables(int dtype, const BatchSweep* sweeps, int nsweeps, int max_count,
                               hipStream_t s) {
  if (nsweeps <= 0 || max_count <= 0) return hipSuccess;
  return dtype == SLMPP_F64 ? SweepLaunch<double>::batch_tables(sweeps, nsweeps, max_count, s)
                            : SweepLaunch<float>::batch_tables(sweeps, nsweeps, max_count, s);
}

hipError_t prepare_batch_sweep(int dtype, size_t lds_bytes) {
  return dtype == SLMPP_F64 ? SweepLaunch<double>::prepare_batch(lds_bytes)
                            : SweepLaunch<float>::prepare_batch(lds_bytes);
}

int batch_sweep_blocks_per_cu(int dtype, size_t lds_bytes) {
  return dtype == SLMPP_F64 ? SweepLaunch<double>::batch_blocks_per_cu(lds_bytes)
                            : SweepLaunch<float>::batch_blocks_per_cu(lds_bytes);
}

hipError_t launch_batch_sweeps(int dtype, const BatchSweep* sweeps, const BatchItem* items,
                               int nitems, size_t lds_bytes, int grid, hipStream_t s) {
  if (nitems <= 0) return hipSuccess;
  return dtype == SLMPP_F64 ? SweepLaunch<double>::batch_sweeps(sweeps, items, nitems, lds_bytes, grid, s)
                            : SweepLaunch<float>::batch_sweeps(sweeps, items, nitems, lds_bytes, grid, s);
}

// Plan of a batch sweep: 256 threads, W pencils per tile (W * S = 256).
// A pencil length n = S * R with R in {8, 12, 16} takes the register
// variant (R); others the runtime segment length (R = 0), which also keeps
// its outputs in a second LDS tile.  lds_bytes == 0: the tile does not fit
// kBatchTileLdsMax.
SweepPlan plan_batch_sweep(int dtype, int order, int32_t n, int64_t npen, int64_t inner,
                           int32_t nfast, int W) {
  SweepPlan p{};
  const size_t es = dtype == SLMPP_F64 ? 8 : 4;
  const int gh = order == 7 ? 4 : 3;
  p.G = gh + nfast;
  const bool contiguous = inner == 1;
  int P = n + 2 * p.G;
  if ((P & 1) == 0) ++P;
  p.pitch = contiguous ? P : W;
  p.W = W;
  p.S = 256 / W;
  p.threads = 256;
  const int R = n % p.S == 0 ? n / p.S : 0;
  p.R = (R == 8 || R == 12 || R == 16) ? R : 0;
  const size_t elems = contiguous ? (size_t)W * P : (size_t)(n + 2 * p.G) * W;
  size_t b = (elems * es + 15) & ~(size_t)15;
  b += (size_t)W * entry_bytes(dtype);
  if (p.R == 0) b += elems * es;
  p.lds_bytes = b <= kBatchTileLdsMax ? b : 0;
  p.tiles = (npen + W - 1) / W;
  p.fast = 0;
  return p;
}


size_t pencil_table_bytes(int dtype, int64_t count) { return entry_bytes(dtype) * (size_t)count; }

SweepPlan plan_sweep(int dtype, int order, int limiter, int32_t n, int64_t npen, int64_t inner,
                     int32_t nfast, int W_override, int S_override, bool moment) {
  SweepPlan p{};
  const size_t es = dtype == SLMPP_F64 ? 8 : 4;
  const int gh = order == 7 ? 4 : 3;
  p.G = gh + nfast;
  const bool contiguous = inner == 1;
  auto pitch_of = [&](int W) {
    (void)W;
    int P = n + 2 * p.G;  // contiguous: pencil-major rows, odd pitch
    if ((P & 1) == 0) ++P;
    return contiguous ? P : W;
  };
  auto lds = [&](int W, bool regs) {
    const size_t elems = contiguous ? (size_t)W * pitch_of(W) : (size_t)(n + 2 * p.G) * W;
    size_t b = (elems * es + 15) & ~(size_t)15;
    b += (size_t)W * entry_bytes(dtype);
    if (!regs) b += elems * es;
    return b;
  };
  // W: pencils per tile.  Strided tiles should not straddle a block of
  // `inner` pencils, so W divides inner when a divisor in the list exists.
  // Wider tiles read longer contiguous runs of each row (128 pencils: 512 B
  // in FP32), which the strided x sweeps need; a width is taken only when
  // some compile-time segment length fits it.  Segments of 32 cells exist
  // only for strided 128-pencil tiles of 64-cell FP32 pencils, and not with
  // the row sums of the moment: with those, or in FP64, their registers
  // would halve the occupancy, and 64-pencil tiles of 16-cell segments are
  // faster.
  auto seg_ok = [&](int c, int Wc) {
    return n % c == 0 && Wc * (n / c) <= 256 &&
           (c != 32 || (Wc == 128 && n == 64 && !contiguous && !moment && es == 4));
  };
  auto has_r = [&](int Wc) {
    for (int c : {12, 16, 24, 32})
      if (seg_ok(c, Wc)) return true;
    return false;
  };
  int W = 0;
  if (W_override > 0) {
    W = W_override;
  } else if (contiguous) {
    W = 64;
  } else {
    for (int c : {128, 64, 48, 32, 16}) {
      if (inner % c == 0 && has_r(c)) {
        W = c;
        break;
      }
    }
    if (W == 0) {
      for (int c : {64, 48, 32, 16}) {
        if (inner % c == 0) {
          W = c;
          break;
        }
      }
    }
    if (W == 0) W = 64;
  }
  while (W > 1 && lds(W, false) > 96 * 1024) W /= 2;
  // 48-cell strided SL-MPP7 pencils take tiles of two 24-cell segments,
  // 256 pencils wide in FP32 (see sweep_fast_kernel) and 128 in FP64 (two
  // such workgroups fit a CU in registers and LDS, with 1 KiB per row)
  const bool wide = !contiguous && n == 48 && order == 7 && inner % (es == 4 ? 256 : 128) == 0 &&
                    W_override == 0 && S_override <= 0 && limiter == SLMPP_LIM_MPP;
  if (wide) W = es == 4 ? 256 : 128;
  // R: cells per thread; a compile-time length when it divides n
  int R = 0;
  if (S_override > 0) {
    const int S = S_override;
    R = (n % S == 0 && (n / S == 12 || n / S == 16 || n / S == 24)) ? n / S : 0;
    p.S = S;
  } else {
    for (int c : {12, 16, 24, 32}) {
      if (seg_ok(c, W)) {
        R = c;
        break;
      }
    }
    p.S = R ? n / R : std::max(1, std::min(256 / std::max(1, W), std::max(1, n / 8)));
  }
  p.S = std::max(1, std::min(p.S, 256 / std::max(1, W)));
  if (wide) {
    R = 24;
    p.S = 2;
  }
  if (R && p.S * R != n) R = 0;
  if (limiter != SLMPP_LIM_MPP) R = 0;  // compile-time segments exist for SL-MPP only
  p.R = R;
  p.W = W;
  p.threads = W * p.S;
  p.pitch = pitch_of(W);
  p.lds_bytes = lds(W, R > 0);
  p.tiles = (npen + W - 1) / W;
  // the persistent prefetching kernel (see sweep_fast_kernel)
  const int vn = dtype == SLMPP_F64 ? 2 : 4;
  const bool fits32 = npen < ((int64_t)1 << 31) && inner < ((int64_t)1 << 31) &&
                      (int64_t)n * W < ((int64_t)1 << 24);
  p.fast = R > 0 && R % vn == 0 && fits32 && W_override == 0 &&
           (contiguous ? (W == 64 && n % vn == 0) : (inner % W == 0 && inner % vn == 0 &&
                                                     (W == 256 || W == 128 || W == 64 || W == 48 || W == 32)));
  if (R == 32 && !p.fast) {  // 32-cell segments exist in the fast kernel only
    p.R = 0;
    p.lds_bytes = lds(W, false);
  }
  return p;
}

hipError_t resident_grid(const void* kernel, int threads, size_t lds_bytes, int64_t tiles, int max_per_cu,
                         int64_t* grid) {
  constexpr int kDevices = 64;
  static std::atomic<int> cus[kDevices];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  int n_cu = dev >= 0 && dev < kDevices ? cus[dev].load(std::memory_order_relaxed) : 0;
  if (n_cu == 0) {
    e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    n_cu = std::max(n_cu, 1);
    if (dev >= 0 && dev < kDevices) cus[dev].store(n_cu, std::memory_order_relaxed);
  }
  *grid = tiles;
  if (tiles <= n_cu) return hipSuccess;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, lds_bytes);
  if (e != hipSuccess) return e;
  per_cu = std::max(1, std::min(per_cu, max_per_cu));
  *grid = std::min<int64_t>(tiles, (int64_t)per_cu * n_cu);
  return hipSuccess;
}

hipError_t launch_tables(int dtype, int order, const TableJobs& jobs, hipStream_t s) {
  return dtype == SLMPP_F64 ? SweepLaunch<double>::tables(order, jobs, s)
                            : SweepLaunch<float>::tables(order, jobs, s);
}

hipError_t launch_sweep(int dtype, int order, int limiter, const SweepArgs& a, const SweepPlan& p,
                        const void* table, hipStream_t s) {
  return dtype == SLMPP_F64 ? SweepLaunch<double>::sweep(order, limiter, a, p, table, s)
                            : SweepLaunch<float>::sweep(order, limiter, a, p, table, s);
}

namespace {
// the host's copy of PlaneShape
template <typename T, int ORDER, int N, int PB>
void plane_shape(PlanePlan& p) {
  using Sh = PlaneShape<T, ORDER, N, PB>;
  p.N = N;
  p.PB = Sh::PB;
  p.G = Sh::G;
  p.pitch = Sh::P;
  p.plane_lds = Sh::PS;
}
template <typename T, int ORDER>
bool plane_shape_n(int N, int64_t vouter, PlanePlan& p) {
  const int pb = plane_count(sizeof(T) == 8, N, vouter);
  switch (N * 10 + pb) {
    case 244: plane_shape<T, ORDER, 24, 4>(p); return true;
    case 242: plane_shape<T, ORDER, 24, 2>(p); return true;
    case 322: plane_shape<T, ORDER, 32, 2>(p); return true;
    case 321: plane_shape<T, ORDER, 32, 1>(p); return true;
    case 481: plane_shape<T, ORDER, 48, 1>(p); return true;
    case 641: plane_shape<T, ORDER, 64, 1>(p); return true;
    default: return false;
  }
}
}  // namespace

PlanePlan plan_kick_plane(int dtype, int order, int32_t na, int32_t nb, int64_t planes,
                          int64_t vouter) {
  PlanePlan p{};
  if (na != nb || !(na == 24 || na == 32 || na == 48 || na == 64) || planes < 1 || vouter < 1)
    return p;
  const bool ok = dtype == SLMPP_F64
                      ? (order == 7 ? plane_shape_n<double, 7>(na, vouter, p) : plane_shape_n<double, 5>(na, vouter, p))
                      : (order == 7 ? plane_shape_n<float, 7>(na, vouter, p) : plane_shape_n<float, 5>(na, vouter, p));
  if (!ok) return PlanePlan{};
  p.planes = planes;
  p.vouter = vouter;
  p.tiles = (planes + p.PB - 1) / p.PB;
  // every tile's planes belong to one spatial cell: one pair of entries
  p.uni = vouter % p.PB == 0 ? 1 : 0;
  if (planes < ((int64_t)1 << 32) && vouter < ((int64_t)1 << 31)) p.vdiv = FastDiv32::of((uint32_t)vouter);
  const size_t es = dtype == SLMPP_F64 ? 8 : 4;
  const size_t lds = ((size_t)p.PB * p.plane_lds * es + 15) & ~(size_t)15;  // entries: registers
  p.lds_bytes = lds <= 80 * 1024 ? lds : 0;
  return p;
}

hipError_t launch_kick_plane(int dtype, int order, const SweepArgs& a, const PlanePlan& p,
                             const void* tabA, const void* tabB, hipStream_t s) {
  if (p.lds_bytes == 0) return hipErrorInvalidValue;
  return dtype == SLMPP_F64 ? SweepLaunch<double>::kick_plane(order, a, p, tabA, tabB, s)
                            : SweepLaunch<float>::kick_plane(order, a, p, tabA, tabB, s);
}

int32_t max_shift_velocity(double vlo, double dv, int32_t nvl, double dt, double h, int32_t n,
                           int32_t bc) {
  int64_t best = 0;
  for (int32_t j = 0; j < nvl; ++j) {
    double c, xi;
    {
#pragma clang fp contract(off)
      c = vlo + ((double)j + 0.5) * dv;
      xi = (c * dt) / h;
    }
    if (!(std::fabs(xi) < 4.0e18)) continue;
    int64_t N = (int64_t)std::floor(xi + 0.5);
    if (bc == SLMPP_BC_PERIODIC) {
      N %= n;
      if (N < 0) N += n;
      if (N > n / 2) N -= n;
    }
    const int64_t aN = N < 0 ? -N : N;
    best = std::max(best, aN);
  }
  return (int32_t)std::min<int64_t>(best, 64);
}

}  // namespace slmpp
