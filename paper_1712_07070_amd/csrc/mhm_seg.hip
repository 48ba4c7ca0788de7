// The MHM step of few groups: every group's planes shared by several
// workgroups, each marching one z segment (ZPart, mhm_group.h).  One
// workgroup per group leaves the chip idle below 256 groups (one per compute
// unit), and a march of 18 iterations takes about 75 us (FP64) however few
// the groups; a segment of n planes runs n + 2.  Same arithmetic, same bits.
// Sources and outputs as in mhm_fwd.hip; the other words' segments are in
// mhm_fwd_ext.h.

#include "mhm_group.h"

namespace gh {

namespace {

// Waves per SIMD asked for: the low occupancy target in FP32 and the high one in
// FP64, as for the whole-group kernels.  FP64 gets two, FP32 three (144-165
// VGPRs), which plm_segments counts with.
constexpr int kSegWaves = 2;

template <typename T, bool kCfl>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kSegWaves))) void mhm_level_seg_kernel(
    const T* __restrict__ level, T* __restrict__ level_out, LevelGeom geo, Gas<T> gas,
    const double* __restrict__ dt_dev, double dx, int first_order, int ws, int* __restrict__ n_bad, CflOut cfl,
    int segs) {
  __shared__ Smem<T> sm;
  __shared__ double cfl_slots[kCfl ? 2 * kCflHalfStride : 1];
  set_dt(gas, dt_dev, dx);
  if (kCfl && cfl.reset != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *cfl.reset = 0x7ff0000000000000ull;
  const int g = int(blockIdx.x) / segs, n = 16 / segs, lo = (int(blockIdx.x) % segs) * n;
  const LevelSource<T, unsigned int> src{level, geo, g % geo.ngx, (g / geo.ngx) % geo.ngy, g / (geo.ngx * geo.ngy)};
  double* smax = nullptr;
  if (kCfl) {
    smax = cfl_slots + cfl_slot(threadIdx.x);
    smax[0] = 0.0;
    smax[kCflHalfStride] = 0.0;
  }
  const int bad = process_group<T, false>(src, level_out + int64_t(g) * 5 * 4096, gas, first_order, ws, sm, smax,
                                          cfl.gamma, threadIdx.x, (T*)nullptr, nullptr, DefaultScheme(),
                                          ZPart{lo, lo + n});
  if (n_bad != nullptr && bad != 0) atomicAdd(n_bad, bad);
  // a segment lies in one z half; the per-patch output is complete only when
  // it is that half (the launch asks for it with two segments at most)
  if (kCfl)
    cfl_epilogue(cfl_slots, cfl.c_cfl_dx, cfl.dt_patch != nullptr ? cfl.dt_patch + int64_t(g) * 8 : nullptr, cfl.dt_min,
                 1.0, threadIdx.x, lo >> 3);
}

// The groups of every level of a batched launch, one workgroup per segment
// (no queue: a launch this small has one round of workgroups).
template <typename T, bool kCfl>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kSegWaves))) void mhm_batched_seg_kernel(
    BatchArgs<T> args, Gas<T> gas, int first_order, int ws, int* __restrict__ n_bad, int segs) {
  __shared__ Smem<T> sm;
  __shared__ double cfl_slots[kCfl ? 2 * kCflHalfStride : 1];
  if (kCfl && blockIdx.x == 0 && threadIdx.x < unsigned(args.n_levels) && args.lv[threadIdx.x].reset != nullptr)
    *args.lv[threadIdx.x].reset = 0x7ff0000000000000ull;
  const int item = int(blockIdx.x) / segs, n = 16 / segs, lo = (int(blockIdx.x) % segs) * n;
  int l = 0;
  while (l + 1 < args.n_levels && item >= args.lv[l + 1].g_begin) ++l;
  const BatchLevel<T>& L = args.lv[l];
  const int g = item - int(L.g_begin);
  gas.dtdx = L.dtdx;
  gas.half_dtdx = L.half_dtdx;
  if (L.dt_dev != nullptr) {
    const double dt = *L.dt_dev * L.dt_scale;  // exact for a power-of-two scale
    gas.dtdx = T(dt / L.dx);
    gas.half_dtdx = T(0.5 * (dt / L.dx));
  }
  const LevelGeom& geo = L.geo;
  const LevelSource<T, unsigned int> src{L.in, geo, g % geo.ngx, (g / geo.ngx) % geo.ngy, g / (geo.ngx * geo.ngy)};
  double* smax = nullptr;
  if (kCfl && (L.dt_min != nullptr || L.dt_patch != nullptr)) {
    smax = cfl_slots + cfl_slot(threadIdx.x);
    smax[0] = 0.0;
    smax[kCflHalfStride] = 0.0;
  }
  const int bad = process_group<T, false>(src, L.out + int64_t(g) * 5 * 4096, gas, first_order, ws, sm, smax,
                                          args.gamma, threadIdx.x, (T*)nullptr, nullptr, DefaultScheme(),
                                          ZPart{lo, lo + n});
  if (n_bad != nullptr && bad != 0) atomicAdd(n_bad, bad);
  if (kCfl && smax != nullptr)
    cfl_epilogue(cfl_slots, L.c_cfl_dx, L.dt_patch != nullptr ? L.dt_patch + int64_t(g) * 8 : nullptr, L.dt_min,
                 L.fold_scale, threadIdx.x, lo >> 3);
}

template <typename T, bool kFlux>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kSegWaves))) void mhm_padded_seg_kernel(
    const T* __restrict__ Upad, T* __restrict__ Uout, int gh, Gas<T> gas, const double* __restrict__ dt_dev, double dx,
    int first_order, int ws, int* __restrict__ n_bad, T* __restrict__ face_flux, int segs) {
  __shared__ Smem<T> sm;
  __shared__ T stage[kFlux ? kFluxStage : 1];
  set_dt(gas, dt_dev, dx);
  const int g = int(blockIdx.x) / segs, n = 16 / segs, lo = (int(blockIdx.x) % segs) * n;
  const int P = 16 + 2 * gh;
  const PaddedSource<T> src{Upad + int64_t(g) * 5 * P * P * P, P, gh};
  T* ff = kFlux ? face_flux + int64_t(g) * 9 * 5 * 256 : nullptr;
  const int bad = process_group<T, false>(src, Uout + int64_t(g) * 5 * 4096, gas, first_order, ws, sm, nullptr, 0.0,
                                          threadIdx.x, ff, nullptr, DefaultScheme(), ZPart{lo, lo + n}, stage);
  if (n_bad != nullptr && bad != 0) atomicAdd(n_bad, bad);
}

}  // namespace

template <typename T>
hipError_t launch_mhm_level_seg(const T* level, T* level_out, const LevelGeom& geo, const Gas<T>& gas,
                                const double* dt_dev, double dx, int first_order, int ws, int* n_bad,
                                const CflOut& cfl, int segs, hipStream_t stream) {
  const dim3 grid(unsigned(geo.ngx * geo.ngy * geo.ngz * segs));
  if (cfl.dt_min != nullptr || cfl.dt_patch != nullptr || cfl.reset != nullptr)
    hipLaunchKernelGGL((mhm_level_seg_kernel<T, true>), grid, dim3(kThreads), 0, stream, level, level_out, geo, gas,
                       dt_dev, dx, first_order, ws, n_bad, cfl, segs);
  else
    hipLaunchKernelGGL((mhm_level_seg_kernel<T, false>), grid, dim3(kThreads), 0, stream, level, level_out, geo, gas,
                       dt_dev, dx, first_order, ws, n_bad, cfl, segs);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_mhm_batched_seg(const BatchArgs<T>& args, const Gas<T>& gas, int first_order, int ws, int* n_bad,
                                  int segs, hipStream_t stream) {
  const dim3 grid(unsigned(args.total * segs));
  if (args.cfl)
    hipLaunchKernelGGL((mhm_batched_seg_kernel<T, true>), grid, dim3(kThreads), 0, stream, args, gas, first_order, ws,
                       n_bad, segs);
  else
    hipLaunchKernelGGL((mhm_batched_seg_kernel<T, false>), grid, dim3(kThreads), 0, stream, args, gas, first_order, ws,
                       n_bad, segs);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_mhm_fwd_seg(const T* U_pad, T* U_out, int n_groups, int ghost, const Gas<T>& gas,
                              const double* dt_dev, double dx, int first_order, int ws, int* n_bad,
                              hipStream_t stream, T* face_flux, int segs) {
  const dim3 grid(unsigned(n_groups * segs));
  if (face_flux != nullptr)
    hipLaunchKernelGGL((mhm_padded_seg_kernel<T, true>), grid, dim3(kThreads), 0, stream, U_pad, U_out, ghost, gas,
                       dt_dev, dx, first_order, ws, n_bad, face_flux, segs);
  else
    hipLaunchKernelGGL((mhm_padded_seg_kernel<T, false>), grid, dim3(kThreads), 0, stream, U_pad, U_out, ghost, gas,
                       dt_dev, dx, first_order, ws, n_bad, face_flux, segs);
  return hipGetLastError();
}

#define GH_SEG_INST(T)                                                                                                \
  template hipError_t launch_mhm_level_seg<T>(const T*, T*, const LevelGeom&, const Gas<T>&, const double*, double,   \
                                              int, int, int*, const CflOut&, int, hipStream_t);                       \
  template hipError_t launch_mhm_batched_seg<T>(const BatchArgs<T>&, const Gas<T>&, int, int, int*, int, hipStream_t); \
  template hipError_t launch_mhm_fwd_seg<T>(const T*, T*, int, int, const Gas<T>&, const double*, double, int, int,   \
                                            int*, hipStream_t, T*, int);
GH_SEG_INST(double)
GH_SEG_INST(float)
#undef GH_SEG_INST

}  // namespace gh
