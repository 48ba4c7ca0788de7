// Internal launch wrappers of libhydro (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hydro_device.h"

namespace gh {

// Group lattice and boundary conditions of one level (bc: x-, x+, y-, y+,
// z-, z+; 0 periodic, 1 outflow).
struct LevelGeom {
  int ngx, ngy, ngz;
  int bc[6];
};

// CFL outputs of a fused step (all optional): per-patch time-steps of the
// written state, an integer-minimum target for the level time-step (the bit
// pattern of a non-negative double), and a location the kernel resets to +inf.
struct CflOut {
  double* dt_patch;
  unsigned long long* dt_min;
  unsigned long long* reset;
  double c_cfl_dx;  // C_CFL * dx, formed on the host in double
  double gamma;
};

// Time of the fullest compute unit (256 of them) in a launch of `wgs` equal
// workgroups of which `slots` fit to a unit, in times of one workgroup alone:
// m of them together take 1 + share (m - 1) times as long (measured per
// kernel).
inline double fullest_unit(int64_t wgs, int slots, double share) {
  const int64_t n = (wgs + 255) / 256, rest = n % slots;
  return double(n / slots) * (1.0 + share * (slots - 1)) + (rest ? 1.0 + share * double(rest - 1) : 0.0);
}

// z segments per 16^3 group of a march over G groups.  A segment of n planes
// runs n + 2 iterations (it recomputes the states of one plane beyond each
// end).  The split with the least time on the fullest unit is taken,
// the fewest segments on ties.  PPM step, FP64 (share 0.36), by 1, 2, 4, 8, 16
// segments: 16 groups 169, 93, 55, 36, 29 us; 64 groups 173, 96, 61, 52, 75;
// 192 groups 175, 121, 132, 145, 208; 512 groups 230, 249, 292, 375, 538.
inline int march_segments(int64_t G, int slots, double share) {
  int best = 1;
  double cost = 0.0;
  for (int s = 1; s <= 16; s *= 2) {
    const double c = fullest_unit(G * s, slots, share) * (16 / s + 2);
    if (s == 1) cost = 0.9 * c;  // a split has to gain clearly
    else if (c < cost) {
      best = s;
      cost = c;
    }
  }
  return best;
}

// Segments per group of the default march and of the other PLM words' (FP64
// two workgroups to a compute unit, FP32 three).  whole_halves: per-patch
// time-steps are written, so no segment may hold part of a patch.  Padded
// step by 1, 2, 4, 8, 16 segments, us: FP64 8 groups 73, 46, 27, 17, 12; 64
// groups 74, 47, 28, 27, 36; 192 groups 75, 66, 62, 68, 86; 512 groups 113, 129,
// 142, 169, 213.  FP32 64 groups 59, 38, 23, 17, 22; 336 groups 71, 53, 57, 62,
// 78; 512 groups 72, 79, 76, 87, 115.
template <typename T>
int plm_segments(int64_t G, bool whole_halves) {
  const int s = sizeof(T) == 8 ? march_segments(G, 2, 0.5) : march_segments(G, 3, 0.22);
  return whole_halves && s > 2 ? 2 : s;
}

// split: groups may be shared by several workgroups (plm_segments); else
// exactly the shape `variant`.
template <typename T>
hipError_t launch_mhm_level(const T* level, T* level_out, const LevelGeom& geo, const Gas<T>& gas,
                            const double* dt_dev, double dx, int first_order, int ws, int* n_bad, const CflOut& cfl,
                            int variant, bool split, hipStream_t stream);

// The steps with every group shared by `segs` workgroups, one per z segment
// (mhm_seg.hip; levels of fewer than 2^32 elements).
template <typename T>
hipError_t launch_mhm_level_seg(const T* level, T* level_out, const LevelGeom& geo, const Gas<T>& gas,
                                const double* dt_dev, double dx, int first_order, int ws, int* n_bad,
                                const CflOut& cfl, int segs, hipStream_t stream);
template <typename T>
hipError_t launch_mhm_fwd_seg(const T* U_pad, T* U_out, int n_groups, int ghost, const Gas<T>& gas,
                              const double* dt_dev, double dx, int first_order, int ws, int* n_bad,
                              hipStream_t stream, T* face_flux, int segs);
template <typename T>
struct BatchArgs;
template <typename T>
hipError_t launch_mhm_batched_seg(const BatchArgs<T>& args, const Gas<T>& gas, int first_order, int ws, int* n_bad,
                                  int segs, hipStream_t stream);
struct ExtOpts;

// One level of a batched launch: input / output level storage, geometry,
// the level's dt/dx (or a device dt), and the index of its first work item.
template <typename T>
struct BatchLevel {
  const T* in;
  T* out;
  LevelGeom geo;
  long long g_begin;  // items [g_begin, next level's g_begin) are this level's groups
  T dtdx, half_dtdx;
  const double* dt_dev;
  double dt_scale;  // with dt_dev: dt = *dt_dev * dt_scale
  double dx;
  // CFL outputs of the level's written state (launches with the epilogue)
  double* dt_patch;              // [G][8] per-patch time-steps, or null
  unsigned long long* dt_min;    // minimum x fold_scale folded in (bits of a double), or null
  unsigned long long* reset;     // set to +inf at the start of the launch, or null
  double c_cfl_dx;               // C_CFL * dx
  double fold_scale;
};

constexpr int kMaxLevels = 8;

template <typename T>
struct BatchArgs {
  BatchLevel<T> lv[kMaxLevels];
  int n_levels;
  long long total;  // number of work items (groups over all levels)
  int cfl;          // some level requests CFL outputs (the launch runs the epilogue form)
  double gamma;     // adiabatic index in double (Eq. 2 signal speeds)
};

// work: kBatchWorkWords device uint32 (kQueues ticket counters and one
// departure counter), zero before the first launch; every launch leaves them
// zero.  grid: number of persistent workgroups.
template <typename T>
hipError_t launch_mhm_batched(const BatchArgs<T>& args, const Gas<T>& gas, int first_order, int ws, int* n_bad,
                              unsigned int* work, int variant, int grid, hipStream_t stream);

// The same launch with the work counters in the library's own per-device
// array (kBatchWorkWords words), cleared before the launch in stream order.
template <typename T>
hipError_t launch_mhm_batched_noalloc(const BatchArgs<T>& args, const Gas<T>& gas, int first_order, int ws,
                                      int* n_bad, int variant, int grid, hipStream_t stream);

// Adjoint of the step (mhm_adj.hip).  Workspace in elements of T:
// adjoint_workspace_elems(G, level).
size_t adjoint_workspace_elems(int64_t n_groups, bool level);

// split: the two-kernel form (face workspace) instead of the fused one.
template <typename T>
hipError_t launch_mhm_adjoint_padded(const T* U_pad, const T* g_out, T* g_pad, int64_t G, int ghost, const Gas<T>& gas,
                                     int first_order, int ws, T* work, bool split, hipStream_t stream);

template <typename T>
hipError_t launch_mhm_adjoint_level(const T* level, const T* g_out, T* g_in, const LevelGeom& geo, const Gas<T>& gas,
                                    const double* dt_dev, double dx, int first_order, int ws, T* work, bool split,
                                    hipStream_t stream);

// Adjoint of the ghost fill: g_level[cell] = sum of g_pad over every padded
// position that copies the cell (mhm_adj.hip).
template <typename T>
hipError_t launch_gather_ghost_adjoint(const T* g_pad, T* g_level, const LevelGeom& geo, int ghost,
                                       hipStream_t stream);

// Launch shapes of the level step (all give bit-identical results):
// bit 0 set = groups in plain order instead of XCD-blocked order,
// bit 1 set = lower occupancy target for the register allocator,
// bit 2 set = groups in column-tile order (tiles of group rows, marched up in z),
// bit 3 set = LDS tiles with padded rows,
// bit 4 set = two groups per 512-thread workgroup.
constexpr int kLevelVariants = 32;
// Batched kernel: ticket queues (one per XCD of MI355X), launch-shape variants
// (bit 0 item order, bit 1 occupancy target, bits 2-3 queue mode: one queue,
// per-XCD queues, static round-robin, per-XCD column-tile queues) and the
// uint32 words of its work buffer (kQueues tickets + 1 departure counter).
constexpr int kQueues = 8;
constexpr int kBatchedVariants = 16;
constexpr int kBatchWorkWords = 16;
static_assert(kQueues + 1 <= kBatchWorkWords, "work buffer too small");

template <typename T>
hipError_t launch_mhm_fwd(const T* U_pad, T* U_out, int64_t n_groups, int ghost, const Gas<T>& gas,
                          const double* dt_dev, double dx, int first_order, int ws, int* n_bad,
                          hipStream_t stream, T* face_flux = nullptr);

// The padded step for the other MHM + PLM words (ExtOpts with ctu, ppm and
// de all 0), in the fused per-group kernel.
struct ExtOpts;
template <typename T>
hipError_t launch_mhm_fwd_ext(const T* U_pad, T* U_out, int64_t n_groups, int ghost, const Gas<T>& gas,
                              const double* dt_dev, double dx, const ExtOpts& o, int* n_bad, hipStream_t stream,
                              T* face_flux);

// The padded step that also writes every group's branch record (FP64).
hipError_t launch_mhm_record(const double* U_pad, double* U_out, int64_t n_groups, int ghost, const Gas<double>& gas,
                             const double* dt_dev, double dx, int first_order, int ws, int* n_bad, unsigned* record,
                             hipStream_t stream);

// The other schemes of the scheme word (scheme_ext.hip): workspace size in
// elements of T for G groups of ghost width `ghost`, and the step.
struct ExtOpts;
int64_t ext_workspace_elems(int64_t n_groups, int ghost, const ExtOpts& o);
// Whether the step of G groups runs as the chain of kernels (else: the march).
bool ext_uses_chain(int64_t G, bool fp64, const ExtOpts& o);
// face_flux (optional): [G][9][5][256] fluxes on the patch-boundary faces.
template <typename T>
hipError_t launch_ext_step(const T* U_pad, T* U_out, int64_t G, int ghost, const Gas<T>& gas, const double* dt_dev,
                           double dx, const ExtOpts& o, int* n_bad, T* work, T* face_flux, hipStream_t stream);

// Steps (ii)-(iii) of the procedure for unphysical results on a level
// (fallback.hip); counts[3] device int32, added to: repaired unsplit,
// repaired split, still unphysical.
template <typename T>
hipError_t launch_repair(const T* level_in, T* level_out, const LevelGeom& geo, const Gas<T>& gas,
                         const double* dt_dev, double dx, const ExtOpts& o, int* counts, hipStream_t stream);
hipError_t launch_zero_ints(int* p, int n, hipStream_t stream);

// Coarse-fine coupling (amr.hip).  A level: group positions [G][3] and the
// dense map of its group lattice (n[2] x n[1] x n[0] entries, -1 if absent).
struct AmrLevelArgs {
  const int* pos;
  const int* map;
  int64_t G;
  int n[3];
};
struct AmrBc {
  int v[6];
};
// Group of the level's lattice at offset class t = (dz*3 + dy)*3 + dx (0, 1, 2:
// below, at, above) from position p, -1 if the level has none there or the
// domain ends (outflow).
__device__ __forceinline__ int amr_sibling(const AmrLevelArgs& F, const AmrBc& bc, int p0, int p1, int p2, int t) {
  auto along = [](int p, int n, int lo, int hi) {
    return p < 0 ? (lo != 0 ? -1 : p + n) : p >= n ? (hi != 0 ? -1 : p - n) : p;
  };
  const int x = along(p0 + t % 3 - 1, F.n[0], bc.v[0], bc.v[1]);
  const int y = along(p1 + (t / 3) % 3 - 1, F.n[1], bc.v[2], bc.v[3]);
  const int z = along(p2 + t / 9 - 1, F.n[2], bc.v[4], bc.v[5]);
  return (x < 0 || y < 0 || z < 0) ? -1 : F.map[(int64_t(z) * F.n[1] + y) * F.n[0] + x];
}
// Bits x-, x+, y-, y+, z-, z+: the group at p touches that face of the domain
// and it is an outflow face.
__device__ __forceinline__ unsigned amr_outflow_faces(const AmrLevelArgs& F, const AmrBc& bc, int p0, int p1, int p2) {
  return unsigned(bc.v[0] != 0 && p0 == 0) | unsigned(bc.v[1] != 0 && p0 == F.n[0] - 1) << 1 |
         unsigned(bc.v[2] != 0 && p1 == 0) << 2 | unsigned(bc.v[3] != 0 && p1 == F.n[1] - 1) << 3 |
         unsigned(bc.v[4] != 0 && p2 == 0) << 4 | unsigned(bc.v[5] != 0 && p2 == F.n[2] - 1) << 5;
}
// Scratch of the direct step, [G][5][kShellCells]: the cells two deep around a
// group (those inside are its own), of which only the ones that the step reads
// and no sibling holds are written.  The rims of planes -2 .. 17 (rows y = -2, -1,
// 16, 17, then x = -2, -1, 16, 17 of the others), then planes z = -2, -1, 16, 17
// over the group.  The padded block of 22^3 (3 ghosts) took 2.7 times as much, and
// with the second state buffer of the direct step 1.4 times what a padded step
// holds.
constexpr int kShellCells = 20 * 20 * 20 - 16 * 16 * 16;
__host__ __device__ __forceinline__ bool shell_in(int x, int y) { return x >= 0 && x <= 15 && y >= 0 && y <= 15; }
// place of a column in a plane, and offset of plane z
__host__ __device__ __forceinline__ unsigned shell_column(int x, int y) {
  if (shell_in(x, y)) return unsigned(y * 16 + x);
  return unsigned(y < 0 ? (y + 2) * 20 + (x + 2) : y > 15 ? (y - 14) * 20 + (x + 2) : 80 + y * 4 + (x < 0 ? x + 2 : x - 14));
}
__host__ __device__ __forceinline__ unsigned shell_plane(bool in, int z) {
  return unsigned(in ? 2880 + (z < 0 ? z + 2 : z - 14) * 256 : (z + 2) * 144);
}
__host__ __device__ __forceinline__ unsigned shell_cell(int x, int y, int z) {
  return shell_column(x, y) + shell_plane(shell_in(x, y), z);
}
template <typename T>
hipError_t launch_amr_fill_open(const AmrLevelArgs& F, const T* Cold, const T* Cnew, const AmrLevelArgs& C, double a,
                                const int bc[6], T* shell, hipStream_t stream);
// The default step of a level from its states and those cells (mhm_amr.hip),
// with the face fluxes that flux registers read (N: the next finer level, its map
// null if there is none).
template <typename T>
hipError_t launch_mhm_amr(const T* U, T* U_out, const AmrLevelArgs& F, const T* shell, const int bc[6],
                          const Gas<T>& gas, int first_order, int ws, int* n_bad, T* face_flux,
                          const AmrLevelArgs& N, hipStream_t stream);
template <typename T>
hipError_t launch_amr_fill(const T* Uf, const AmrLevelArgs& F, const T* Cold, const T* Cnew, const AmrLevelArgs& C,
                           double a, const int bc[6], int ghost, T* pad, hipStream_t stream);
template <typename T>
hipError_t launch_amr_accumulate(const AmrLevelArgs& F, const T* face_flux, double w, const int bc[6], T* R,
                                 hipStream_t stream);
template <typename T>
hipError_t launch_amr_restrict(const T* Uf, const AmrLevelArgs& F, T* Uc, const AmrLevelArgs& C, hipStream_t stream);
template <typename T>
hipError_t launch_amr_fixup(T* Uc, const AmrLevelArgs& C, const AmrLevelArgs& F, const T* cflux, const T* R,
                            double dtdx, const int bc[6], hipStream_t stream);

template <typename T>
hipError_t launch_fill_ghosts(const T* level, T* U_pad, int ngx, int ngy, int ngz, int ghost, const int bc[6],
                              hipStream_t stream);

template <typename T>
hipError_t launch_cfl_dt(const T* U_pad, int64_t n_groups, int ghost, double dx, double gamma, double c_cfl,
                         double* dt_patch, double* dt_min, hipStream_t stream);

}  // namespace gh
