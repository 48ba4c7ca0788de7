// Launch of the other MHM + PLM scheme words (mhm_fwd_ext.h), by limiter (4:
// first order).

#include "ext_device.h"
#include "kernels.h"

namespace gh {

template <typename T, int kLim>
hipError_t launch_mhm_ext_lim(const T* U_pad, T* U_out, int64_t n_groups, int ghost, const Gas<T>& gas,
                              const double* dt_dev, double dx, const ExtOpts& o, int* n_bad, hipStream_t stream,
                              T* face_flux);

template <typename T>
hipError_t launch_mhm_fwd_ext(const T* U_pad, T* U_out, int64_t n_groups, int ghost, const Gas<T>& gas,
                              const double* dt_dev, double dx, const ExtOpts& o, int* n_bad, hipStream_t stream,
                              T* face_flux) {
  if (n_groups == 0) return hipSuccess;
  const auto go = [&](auto launch) {
    return launch(U_pad, U_out, n_groups, ghost, gas, dt_dev, dx, o, n_bad, stream, face_flux);
  };
  if (o.first_order) return go(launch_mhm_ext_lim<T, 4>);
  if (o.lim == 1) return go(launch_mhm_ext_lim<T, 1>);
  if (o.lim == 2) return go(launch_mhm_ext_lim<T, 2>);
  if (o.lim == 3) return go(launch_mhm_ext_lim<T, 3>);
  return go(launch_mhm_ext_lim<T, 0>);
}

template hipError_t launch_mhm_fwd_ext<double>(const double*, double*, int64_t, int, const Gas<double>&, const double*,
                                               double, const ExtOpts&, int*, hipStream_t, double*);
template hipError_t launch_mhm_fwd_ext<float>(const float*, float*, int64_t, int, const Gas<float>&, const double*,
                                              double, const ExtOpts&, int*, hipStream_t, float*);

}  // namespace gh
