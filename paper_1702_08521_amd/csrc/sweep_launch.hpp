// Launches of the sweep kernels of one storage type (defined in
// sweep_kernels.hpp, instantiated in sweep_f32.hip and sweep_f64.hip), and the
// shapes of the two-axis pass.
#pragma once

#include <hip/hip_runtime.h>

#include "slmpp_internal.hpp"

namespace slmpp {

template <typename T>
struct SweepLaunch {
  static hipError_t tables(int order, const TableJobs& jobs, hipStream_t s);
  static hipError_t sweep(int order, int limiter, const SweepArgs& a, const SweepPlan& p,
                          const void* tab, hipStream_t s);
  static hipError_t kick_plane(int order, const SweepArgs& a, const PlanePlan& p, const void* tabA,
                               const void* tabB, hipStream_t s);
  static hipError_t batch_tables(const BatchSweep* sweeps, int nsweeps, int max_count, hipStream_t s);
  static hipError_t prepare_batch(size_t lds_bytes);
  static int batch_blocks_per_cu(size_t lds_bytes);
  static hipError_t batch_sweeps(const BatchSweep* sweeps, const BatchItem* items, int nitems,
                                 size_t lds_bytes, int grid, hipStream_t s);
};
extern template struct SweepLaunch<float>;
extern template struct SweepLaunch<double>;

constexpr int kPlaneFast = 4;  // integer shifts read directly in the plane kernel

// Planes per tile, for planes of which vouter in a row share their two pencil
// entries.  A tile within one such row reads the entries with scalar loads,
// and 24^2 planes in twos (fours) of four 6-cell segments fill whole
// wavefronts: at 24^3 x 20x24^2 the pass takes 307 us in FP32 with four planes
// (319 with two, 357 with three of 8-cell segments, whose last wavefront is
// 3/8 full) and 876 in FP64 with two (1062 with 8-cell segments); in 2D, where a
// tile's planes lie in different cells, a kick of 132^2 x 24^2 FP32 takes 78-81 us
// in twos against 93-99 in threes of 8-cell segments.  FP64 32^2 planes in twos
// keep one segment per wavefront: 595 against 608 us at 20^3 x 20x32^2 (530 with
// the kernel's compile-time data map), but 80 against 71 us at 132^2 x 32^2, where
// the planes of a tile would not share their entries.
constexpr int plane_count(bool f64, int N, int64_t vouter) {
  return N == 24 ? (!f64 && vouter % 4 == 0 ? 4 : 2) : N == 32 ? (!f64 || vouter % 2 == 0 ? 2 : 1) : 1;
}

template <typename T, int ORDER, int N, int PLANES>
struct PlaneShape {
  // cells per thread (FP32 64^2 planes: 512 threads of 8 cells, whose extra
  // waves outweigh the segment-boundary faces they add)
  static constexpr int R = N == 64 ? (sizeof(T) == 4 ? 8 : 16) : N == 48 ? 12 : N == 32 ? 8 : 6;
  static constexpr int S = N / R;                               // segments per pencil
  static constexpr int PB = PLANES;
  static constexpr int threads = PB * N * S;
  // ring width (shifts up to kPlaneFast cells read the ring directly)
  static constexpr int G = (ORDER == 7 ? 4 : 3) + kPlaneFast;
  // odd row pitch: the rows of one plane start on distinct banks
  static constexpr int P = (N + 2 * G) | 1;
  // plane stride: the plane's rows padded to N (mod 64) elements, so that
  // with PB N = 64 the two planes of a wavefront fall on disjoint banks
  static constexpr int rows = (N + 2 * G) * P;
  static constexpr int PS = PB == 1 ? rows : rows + (((N - rows) % 64) + 64) % 64;
};

}  // namespace slmpp
