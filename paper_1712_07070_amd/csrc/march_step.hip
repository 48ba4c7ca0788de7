// MHM steps with PPM, and with dual energy, through the march of ext_march.h.

#include "ext_march.h"

namespace gh {

template hipError_t launch_march_mode<double, 5, true, kStep>(const MarchArgs<double>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<float, 5, true, kStep>(const MarchArgs<float>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<double, 6, true, kStep>(const MarchArgs<double>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<float, 6, true, kStep>(const MarchArgs<float>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<double, 6, false, kStep>(const MarchArgs<double>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<float, 6, false, kStep>(const MarchArgs<float>&, int64_t, hipStream_t);

}  // namespace gh
