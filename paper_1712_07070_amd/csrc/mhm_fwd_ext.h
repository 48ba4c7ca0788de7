// The other MHM + PLM scheme words (limiters, characteristic variables,
// Roe / HLLE, wave speeds, first order) through the march of the default
// scheme (mhm_group.h) on padded input, one group per workgroup or, with few
// groups, several workgroups to a group (one z segment each, as in
// mhm_seg.hip).  The limiter (or first order, which has no slopes), the
// characteristic projection and the solver family (Roe, or HLLC / HLLE) are
// compile-time options of the kernel copies, the rest run time: one copy for
// every option carried the registers of all of them and spilled.
//
// Bound by VALU issue and latency at two waves per SIMD in FP64, three in
// FP32.  The limiter was a run-time branch for each variable of each slope
// vector first, then one for each vector, which made data with slopes
// everywhere 10% (FP64) and 19% (FP32) faster and data with few slopes up to
// 14% (a shear layer) and 22% (uniform) slower, as more was computed ahead of
// the skips.  Now, 2048 groups, average (worst) of 15 words against the first
// form: FP64 noise 0.74 (0.81), shear layer 0.82 (0.90), uniform 0.80 (0.87);
// FP32 0.75 (0.80), 0.93 (0.99), 0.92 (0.94).  With the limiter at run time and
// the same skips 0.90, 0.88, 0.82 and 1.00, 1.01, 0.94.
#pragma once

#include "mhm_group.h"

namespace gh {

namespace {

// kFlux: optional patch-boundary face fluxes as in mhm_padded_kernel.  Z: ZAll,
// or ZPart with `segs` workgroups to a group.
template <typename T, int kWaves, bool kFlux, int kChr, int kRoe, int kLim, class Z>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kWaves))) void mhm_padded_ext_kernel(
    const T* __restrict__ Upad, T* __restrict__ Uout, int gh, Gas<T> gas, const double* __restrict__ dt_dev, double dx,
    ExtOpts o, int* __restrict__ n_bad, T* __restrict__ face_flux, int segs) {
  __shared__ Smem<T> sm;
  __shared__ T stage[kFlux ? kFluxStage : 1];
  set_dt(gas, dt_dev, dx);
  const int P = 16 + 2 * gh;
  const int64_t P3 = int64_t(P) * P * P;
  Z zr;
  unsigned g = blockIdx.x;
  if constexpr (std::is_same<Z, ZPart>::value) {
    g = blockIdx.x / unsigned(segs);
    zr.lo = int(blockIdx.x % unsigned(segs)) * (16 / segs);
    zr.hi = zr.lo + 16 / segs;
  }
  PaddedSource<T> src{Upad + int64_t(g) * 5 * P3, P, gh};
  T* ff = kFlux ? face_flux + int64_t(g) * 9 * 5 * 256 : nullptr;
  const ExtSchemeT<kChr, kRoe, kLim> sch{o};
  const int bad = process_group<T, (kWaves >= 4)>(src, Uout + int64_t(g) * 5 * 4096, gas, kLim == kFirstOrder, o.ws,
                                                  sm, nullptr, 0.0, threadIdx.x, ff, nullptr, sch, zr, stage);
  if (n_bad != nullptr && bad != 0) atomicAdd(n_bad, bad);
}

// Occupancy target: FP32 at the low one (256 VGPRs instead of 128 with 16-41
// spilled: 256^3 steps 18-39% faster, measured), FP64 at the high one (the
// low one measured slower).
template <typename T, bool kFlux, int kChr, int kRoe, int kLim>
void launch_ext_copy(const T* U_pad, T* U_out, int64_t n, int segs, int ghost, const Gas<T>& gas, const double* dt_dev,
                     double dx, const ExtOpts& o, int* n_bad, hipStream_t stream, T* face_flux) {
  constexpr int kW = sizeof(T) == 4 ? MinWaves<T>::lo : MinWaves<T>::hi;
  if (segs > 1)
    hipLaunchKernelGGL((mhm_padded_ext_kernel<T, kW, kFlux, kChr, kRoe, kLim, ZPart>), dim3(unsigned(n * segs)),
                       dim3(kThreads), 0, stream, U_pad, U_out, ghost, gas, dt_dev, dx, o, n_bad, face_flux, segs);
  else
    hipLaunchKernelGGL((mhm_padded_ext_kernel<T, kW, kFlux, kChr, kRoe, kLim, ZAll>), dim3(unsigned(n)),
                       dim3(kThreads), 0, stream, U_pad, U_out, ghost, gas, dt_dev, dx, o, n_bad, face_flux, 1);
}

template <typename T, bool kFlux, int kLim>
void launch_ext(const T* U_pad, T* U_out, int64_t n, int segs, int ghost, const Gas<T>& gas, const double* dt_dev,
                double dx, const ExtOpts& o, int* n_bad, hipStream_t stream, T* face_flux) {
  const bool roe = o.solver == 1;
  if constexpr (kLim != kFirstOrder) {
    if (o.chr) {
      if (roe) launch_ext_copy<T, kFlux, 1, 1, kLim>(U_pad, U_out, n, segs, ghost, gas, dt_dev, dx, o, n_bad, stream, face_flux);
      else launch_ext_copy<T, kFlux, 1, 0, kLim>(U_pad, U_out, n, segs, ghost, gas, dt_dev, dx, o, n_bad, stream, face_flux);
      return;
    }
  }
  if (roe) launch_ext_copy<T, kFlux, 0, 1, kLim>(U_pad, U_out, n, segs, ghost, gas, dt_dev, dx, o, n_bad, stream, face_flux);
  else launch_ext_copy<T, kFlux, 0, 0, kLim>(U_pad, U_out, n, segs, ghost, gas, dt_dev, dx, o, n_bad, stream, face_flux);
}

}  // namespace

// The kernels of one limiter or of first order (mhm_ext_lim0.hip .. 3 and
// mhm_ext_first.hip).
template <typename T, int kLim>
hipError_t launch_mhm_ext_lim(const T* U_pad, T* U_out, int64_t n_groups, int ghost, const Gas<T>& gas,
                              const double* dt_dev, double dx, const ExtOpts& o, int* n_bad, hipStream_t stream,
                              T* face_flux) {
  const int segs = plm_segments<T>(n_groups, false);
  const int64_t chunk = int64_t(1) << 30;
  const int P = 16 + 2 * ghost;
  const int64_t P3 = int64_t(P) * P * P;
  for (int64_t g0 = 0; g0 < n_groups; g0 += chunk) {
    const int64_t n = n_groups - g0 < chunk ? n_groups - g0 : chunk;
    if (face_flux != nullptr)
      launch_ext<T, true, kLim>(U_pad + g0 * 5 * P3, U_out + g0 * 5 * 4096, n, segs, ghost, gas, dt_dev, dx, o, n_bad,
                                stream, face_flux + g0 * 9 * 5 * 256);
    else
      launch_ext<T, false, kLim>(U_pad + g0 * 5 * P3, U_out + g0 * 5 * 4096, n, segs, ghost, gas, dt_dev, dx, o, n_bad,
                                 stream, (T*)nullptr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

#define GH_EXT_LIM_INST(T, kLim)                                                                                     \
  template hipError_t launch_mhm_ext_lim<T, kLim>(const T*, T*, int64_t, int, const Gas<T>&, const double*, double,  \
                                                  const ExtOpts&, int*, hipStream_t, T*);

}  // namespace gh
