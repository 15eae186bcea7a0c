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

template <typename T, int ORDER, int N>
struct PlaneShape {
  // cells per thread (FP32 64^2 planes: 512 threads of 8 cells, whose extra
  // waves outweigh the segment-boundary faces they add)
  static constexpr int R = N == 64 ? (sizeof(T) == 4 ? 8 : 16) : (N == 48 ? 12 : 8);
  static constexpr int S = N / R;                               // segments per pencil
  static constexpr int PB = sizeof(T) == 4 ? (N == 24 ? 3 : N == 32 ? 2 : 1) : (N == 24 ? 2 : 1);
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
