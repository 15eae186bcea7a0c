// Internal declarations shared by the HIP translation units of libslmpp.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>

#include "slmpp.h"

namespace slmpp {

// Validation of a grid description shared by single runs and ensembles.
slmpp_status check_grid_desc(const slmpp_grid_desc* d, std::string& msg);

// Speed of a pencil: from the velocity cell centre of the pencil (sweeps
// along x_l) or from an acceleration array indexed by the spatial cell
// (sweeps along v_l).
enum SpeedMode : int32_t { SPEED_FROM_VELOCITY = 0, SPEED_FROM_ACCEL = 1 };

// One sweep over an array viewed as [outer][n][inner]: pencil p = o*inner + j
// holds the elements o*n*inner + i*inner + j, i = 0..n-1.
struct SweepArgs {
  void* f;              // float* or double*
  const double* accel;  // SPEED_FROM_ACCEL: speed of the pencil = accel[(p/inner)/xdiv]
  int64_t npen;         // outer * inner
  int64_t inner;        // stride of the swept axis in elements
  int64_t vdiv;         // SPEED_FROM_VELOCITY: jv = ((p % inner) / vdiv) % nvl
  int64_t xdiv;
  double dt, h;         // time step and mesh spacing of the swept axis
  double vlo, dv;       // velocity axis of SPEED_FROM_VELOCITY
  double alpha;         // MP parameter
  int32_t n;            // pencil length
  int32_t nvl;
  int32_t bc;           // SLMPP_BC_*
  int32_t cmode;        // SpeedMode
  int32_t nfast;        // integer shifts |N| <= nfast read the LDS tile directly
  int32_t rk;           // 1: a TVD-RK stage (interface values at zero Courant
                        //    number, update with nu = c dt / h, no shift)
  double* mom;          // non-null: per-tile sums of the result over each tile row
                        // (strided tiles within one velocity block), mom[tile * n + i]
                        // (line_sweep_kernel: pairs, the sum and its error)
  // several runs of one geometry in one fast launch (batched ensembles):
  // tile t belongs to run t / tpr, whose f and pencil table are fmulti[r]
  // and tmulti[r] (null: the single run f, table)
  void* const* fmulti;
  const void* const* tmulti;
  int64_t tpr;
  // stages of the TVD-RK time integration (single runs, sweep_fast_kernel
  // and the tile kernels): the results go to fout (null: f, in place),
  // and with fblend non-null each result r becomes cb * fblend + cf * r at
  // the same element
  void* fout;
  const void* fblend;
  double cb, cf;
};

// Tiling of one sweep launch: W pencils per tile, S segments per pencil,
// W*S threads per workgroup, G ghost rows above and below the tile in LDS.
struct SweepPlan {
  int32_t W, S, R, threads, G, pitch;  // R: cells per thread (0: runtime length)
  int32_t fast;                        // use the persistent prefetching kernel
  size_t lds_bytes;
  int64_t tiles;
};

// Plans a sweep launch for the given sizes (dtype: SLMPP_F64/F32); moment:
// the sweep also leaves tile row sums (SweepArgs::mom) when its plan allows.
SweepPlan plan_sweep(int dtype, int order, int limiter, int32_t n, int64_t npen, int64_t inner,
                     int32_t nfast, int W_override = 0, int S_override = 0, bool moment = false);

// Pencil tables of up to six sweeps (count entries each, one per distinct
// speed; tab: device scratch of pencil_table_bytes()).
struct TableJobs {
  SweepArgs a[6];
  void* tab[6];
  int32_t count[6];
  int32_t n;
  void add(const SweepArgs& s, void* t, int64_t c) {
    a[n] = s;
    tab[n] = t;
    count[n++] = (int32_t)c;
  }
};
hipError_t launch_tables(int dtype, int order, const TableJobs& jobs, hipStream_t s);
// Workgroups of a persistent kernel for `tiles` tiles: as many as the device
// holds at once, at most max_per_cu on each CU.  The number of CUs is asked for
// once per device, and the occupancy only where there are more tiles than CUs.
hipError_t resident_grid(const void* kernel, int threads, size_t lds_bytes, int64_t tiles, int max_per_cu,
                         int64_t* grid);
hipError_t launch_sweep(int dtype, int order, int limiter, const SweepArgs& a,
                        const SweepPlan& p, const void* table, hipStream_t s);
size_t pencil_table_bytes(int dtype, int64_t count);

// n / d for 32-bit n by an invariant 32-bit divisor d >= 1 (Granlund and
// Montgomery, "Division by invariant integers using multiplication", 1994):
// t = mulhi(m, n), n / d = (t + ((n - t) >> s1)) >> s2 with
// l = ceil(log2 d), m = floor(2^32 (2^l - d) / d) + 1, s1 = min(l, 1),
// s2 = max(l - 1, 0).  m == 0 marks "not set up".
struct FastDiv32 {
  uint32_t m, s1, s2, pad;
  static FastDiv32 of(uint32_t d) {
    uint32_t l = 0;
    while (l < 32 && ((uint64_t)1 << l) < d) ++l;
    FastDiv32 f{};
    f.m = (uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << l) - d)) / d + 1);
    f.s1 = l < 1 ? l : 1;
    f.s2 = l > 1 ? l - 1 : 0;
    return f;
  }
  __host__ __device__ uint32_t div(uint32_t n) const {
    const uint32_t t = (uint32_t)(((uint64_t)m * n) >> 32);
    return (t + ((n - t) >> s1)) >> s2;
  }
};

// The last two velocity axes of one kick in one pass over f (outflow
// velocity boundaries, SL-MPP, square planes of N = 24, 32, 48 or 64
// cells): plane p = (x, v_1..v_{D-2}) is the contiguous block
// f[p * N^2 .. (p + 1) * N^2); its pencils along v_{D-1} take table entry
// tabA[p / vouter] and those along v_D tabB[p / vouter].  Several runs of
// one geometry in one launch: SweepArgs::fmulti / tmulti / tpr (tiles per
// run) with tmulti holding the v_{D-1} tables of the runs, then their v_D
// tables; planes and tiles as for one run, times the number of runs for
// tiles.
struct PlanePlan {
  int32_t N, PB;       // plane side, planes per tile
  int32_t G, pitch;    // ring of zero cells around each plane in LDS, LDS row
                       // pitch (fixed by order and N; shifts beyond the ring
                       // minus the stencil take bounds-checked reads)
  int32_t plane_lds;   // LDS elements from one plane to the next
  int32_t uni;         // the planes of a tile share one spatial cell (vouter % PB == 0)
  int64_t planes, vouter, tiles;
  FastDiv32 vdiv;      // plane -> spatial cell (plane / vouter) while planes < 2^32
  size_t lds_bytes;    // 0: the shape is not supported
};
// Tiling of a sweep by line_sweep_kernel: any limiter and stride, pencils of up
// to 2048 cells (1024 with TVD-RK, whose workgroups have half the threads) while
// a 16-byte vector of them fits the LDS.  A tile is W pencils of one block
// of `blen` consecutive pencils (rows of W elements, `inner` apart), or, when
// K > 0, K whole blocks of `inner` pencils each (contiguous in f).
struct LinePlan {
  int32_t W, K;        // pencils per row tile; blocks per tile (0: row tiles)
  int32_t pw;          // pencils per tile
  int32_t S, R;        // segments per pencil, cells per segment (at most 16)
  int32_t G;           // ghost cells on both sides of a pencil in LDS
  int32_t rs, bs;      // LDS elements between cells of a pencil, between blocks
  int32_t threads;     // pw * S rounded up to whole wavefronts
  int32_t lds_elems;
  int32_t tpb;         // row tiles per block
  int32_t blen;        // pencils of a block of row tiles
  int64_t blocks;      // number of blocks
  int64_t bstride;     // elements between blocks of row tiles
  int64_t tiles;
  int32_t reps;        // block tiles: sweeps of the tile one after the other
  int32_t stream;      // row tiles: nontemporal accesses
  FastDiv32 dtpb, dvdiv, dnvl, dxdiv;
  size_t lds_bytes;    // 0: the sweep is not one this kernel takes
};
// moment_block > 0: row tiles within velocity blocks of that many pencils,
// for the row sums of SweepArgs::mom (x_1 sweeps).
LinePlan plan_line(int dtype, int order, const SweepArgs& a, int64_t moment_block);
hipError_t launch_line_sweep(int dtype, int order, int limiter, const SweepArgs& a,
                             const LinePlan& p, const void* table, hipStream_t s);
PlanePlan plan_kick_plane(int dtype, int order, int32_t na, int32_t nb, int64_t planes,
                          int64_t vouter);
hipError_t launch_kick_plane(int dtype, int order, const SweepArgs& a, const PlanePlan& p,
                             const void* tabA, const void* tabB, hipStream_t s);

// The same pass for planes of any na x nb cells (kick_rect_kernel): one plane
// per tile, f[p na nb ..), tables as above.
struct RectPlan {
  int32_t na, nb;      // cells along v_{D-1}, v_D
  int32_t sa, ra, sb, rb;  // segments and cells per segment of the two sweeps
  int32_t G, pitch;    // ring of zero cells in LDS, LDS row pitch
  int32_t threads;
  int64_t planes;
  FastDiv32 vdiv;      // plane -> spatial cell
  size_t lds_bytes;    // 0: not a size the kernel takes
};
RectPlan plan_kick_rect(int dtype, int order, int64_t na, int64_t nb, int64_t planes, int64_t vouter);
hipError_t launch_kick_rect(int dtype, int order, const SweepArgs& a, const RectPlan& p,
                            const void* tabA, const void* tabB, hipStream_t s);

// The sweeps along x_3 and x_2 in one pass (pair_sweep_kernel): tiles of all
// nA x nB (x_2, x_3) of one x_1 and 128 bytes of consecutive velocities.
struct PairPlan {
  int32_t nA, nB;          // cells along x_2, x_3
  int32_t sA, rA, kA;      // x_2 sweep: segments, cells per segment, x_3 per round
  int32_t sB, rB, kB;      // x_3 sweep: segments, cells per segment, x_2 per round
  int32_t nvA, nvB;        // table entries of the two sweeps
  int32_t threads, tiles, nch;  // nch: tiles of one x_1
  int32_t inner32;
  int64_t inner;           // elements between rows: velocities of a spatial cell
  FastDiv32 dch, dvA, dvB, dnA, dnB;
  size_t lds_bytes;        // 0: not a grid the kernel takes
};
PairPlan plan_pair(int dtype, const SweepArgs& sA, const SweepArgs& sB, int64_t outer);
hipError_t launch_pair(int dtype, int order, const SweepArgs& a, const PairPlan& p, const void* tabA,
                       const void* tabB, hipStream_t s);

// Integer-shift bound of a sweep along x_l: max |N| over the velocity
// centres of axis l, with the same split as the kernels.
int32_t max_shift_velocity(double vlo, double dv, int32_t nvl, double dt, double h, int32_t n,
                           int32_t bc);

// ---- batched ensembles (many independent runs per launch) ----
// One sweep of one run inside a grouped launch.
struct BatchSweep {
  SweepArgs a;
  SweepPlan p;
  void* table;    // the run's pencil-table scratch
  int32_t order;  // 5 or 7
  int32_t count;  // table entries
};
// One work item of a grouped sweep launch: tile `tile` of sweep `sweep`.
struct BatchItem {
  int32_t sweep;
  int32_t pad;
  int64_t tile;
};
// Field data of one run.
struct BatchRun {
  const void* f;
  double* rho;
  double* phi;
  double* accel;
  int64_t nxs, nvs;
  int64_t nx[3];
  double h[3];
  double dvol;
  double kappa;
  int32_t D;
  int32_t poisson_order;
};
// rho of one run from the tile row sums of its x_1 sweep (fused moment):
// rho[i * ncol + c] = dvol * sum_{q < nsub} part[(c * nsub + q) * n + i]
struct BatchReduce {
  const double* part;
  double* rho;
  int64_t ncol, nsub;
  int32_t n, pad;
  double dvol;
};
hipError_t launch_batch_reduce(const BatchReduce* list, int nlist, int64_t max_cells,
                               hipStream_t s);
hipError_t launch_batch_tables(int dtype, const BatchSweep* sweeps, int nsweeps, int max_count,
                               hipStream_t s);
hipError_t launch_batch_sweeps(int dtype, const BatchSweep* sweeps, const BatchItem* items,
                               int nitems, size_t lds_bytes, int grid, hipStream_t s);
int batch_sweep_blocks_per_cu(int dtype, size_t lds_bytes);
SweepPlan plan_batch_sweep(int dtype, int order, int32_t n, int64_t npen, int64_t inner,
                           int32_t nfast, int W);
hipError_t launch_batch_moment(int dtype, const BatchRun* runs, const int2* items, int nitems,
                               hipStream_t s);
hipError_t launch_batch_poisson(const BatchRun* runs, int nruns, int max_nxs, hipStream_t s);
// Kernel attributes for the LDS sizes of a batch (outside any graph capture).
hipError_t prepare_batch_kernels(int dtype, size_t sweep_lds, int max_nxs);
constexpr int kBatchMaxSpace = 2048;  // spatial cells per run (one-workgroup Poisson)
// LDS of one batch tile: preferred budget (at least five 256-thread
// workgroups per CU) and hard limit
constexpr size_t kBatchTileLds = 32 * 1024;
constexpr size_t kBatchTileLdsMax = 96 * 1024;

// ---- field solve (poisson.hip) ----
// Sizes of the solve (D = 2 holds x_2 as the third axis): inputs n,
// transform lengths m (2 n for isolated boundaries), outputs o (n + 2 halo),
// twiddle offsets, columns and rows per workgroup or chunk, LDS bytes.
struct FieldPlan {
  int D, order, halo, ok;  // order: of the FDA; ok 0: not a size the kernels take
  int n[3], m[3], o[3], tw[3];
  int cols1, cols2, rows2, cols3;
  size_t lds1, lds2, lds3;
  double h[3];  // mesh spacing of component l
};
// Pencil tables of the velocity sweeps along v_l with the solved
// acceleration (tab[l] null: none).
struct FieldTables {
  void* tab[3];
  double h[3];
  int32_t n[3];
  int32_t bc, rk;
  double dt;
};
FieldPlan plan_field(int D, const int64_t* nx, const double* h, int order, bool isolated);
// Density (rho, or from row sums `part`, pairs or not: see field_forward_kernel)
// and its transform along x_1 into bufA; then the rest, phi and accel.
hipError_t launch_field_forward(const FieldPlan& p, const double* part, bool pairs, int nsub,
                                double dvol, double* rho, double2* bufA, const double2* tw, hipStream_t s);
hipError_t launch_field_rest(const FieldPlan& p, double* phi, double* accel, double2* bufA,
                             double2* bufB, double* phi_ext, const double2* tw, const double* green,
                             int dtype, int order, const FieldTables& tabs, hipStream_t s);
// D = 1: the whole solve as a convolution of the density with conv[0..n)
// (potential) and conv[n..2n) (acceleration).
hipError_t launch_conv_setup(int n, double h, int order, const double* green, const double2* tw,
                             double* conv, hipStream_t s);
hipError_t launch_field_conv(int n, const double* part, bool pairs, int nsub, double dvol,
                             double* rho, double* phi, double* accel, const double* conv, int dtype, int order,
                             const FieldTables& tabs, hipStream_t s);

// ---- field kernels (field.hip) ----
hipError_t launch_moment(int dtype, const void* f, int64_t nxs, int64_t nvs, double dvol,
                         double* rho, hipStream_t s);
// rho[i * ncol + c] = dvol * sum_{q < nsub} part[(c * nsub + q) * n + i] (pairs:
// sums with their errors): the velocity moment from the row sums of a fused x_1
// sweep (ncol spatial columns of x_2..x_D, nsub tiles per velocity block).
hipError_t launch_moment_reduce(const double* part, bool pairs, int n, int64_t ncol, int64_t nsub, double dvol,
                                double* rho, hipStream_t s);
hipError_t launch_poisson(const double* rho, double* phi, double* accel, double2* bufA,
                          double2* bufB, const double2* twiddles, const int64_t* tw_off,
                          const double* green, int D, const int64_t* nx, const double* h,
                          int order, hipStream_t s);
// isolated boundaries (D = 3): Fourier transform of the real-space Green
// function held in a (as complex, doubled grid of sizes m), real part to
// ghat; the solve itself with a, b as scratch of the doubled size
hipError_t launch_iso_green(double2* a, double2* b, const double2* tw, const int64_t* tw_off,
                            const int64_t* m, double* ghat, hipStream_t s);
hipError_t launch_poisson_isolated(const double* rho, double* phi, double* accel, double2* a,
                                   double2* b, const double2* tw, const int64_t* tw_off,
                                   const double* ghat, const int64_t* nx, const double* h,
                                   int order, hipStream_t s);
hipError_t launch_init_separable(int dtype, void* f, const double* s, const double* g1,
                                 const double* g2, const double* g3, int D, const int64_t* nv,
                                 int64_t nxs, int64_t nvs, hipStream_t st);
hipError_t launch_from_double(int dtype, void* f, const double* src, int64_t n, hipStream_t s);
hipError_t launch_to_double(int dtype, const void* f, double* dst, int64_t n, hipStream_t s);
// diagnostics of f (n values) and the acceleration: out[0..6] = sum of f,
// min, max, number of non-finite values, sum |a|^2, real and imaginary part
// of the first mode of a_1; partials: kDiagPartials doubles of scratch
hipError_t launch_diag(int dtype, const void* f, int64_t n, const double* accel, int D, int64_t nxs,
                       int64_t nx1, int64_t inner1, double* partials, double* out, hipStream_t s);
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s);
// velocity moments per spatial cell and the velocity distribution (double)
hipError_t launch_velocity_moments(int dtype, const void* f, int D, const int64_t* nv,
                                   const double* vlo, const double* dv, int64_t nxs,
                                   double* rho, double* mean, double* disp, double* scratch,
                                   int64_t scratch_doubles, hipStream_t s);
hipError_t launch_velocity_distribution(int dtype, const void* f, int64_t nxs, int64_t nvs,
                                        double xvol, double* F, double* scratch,
                                        int64_t scratch_doubles, hipStream_t s);
constexpr int kDiagBlocks = 2048;
constexpr int kDiagFieldBlocks = 64;
constexpr int64_t kDiagPartials = kDiagBlocks * 5 + kDiagFieldBlocks * 6;

}  // namespace slmpp
