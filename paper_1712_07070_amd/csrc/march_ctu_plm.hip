// CTU with PLM (with and without dual energy) through the march of ext_march.h.

#include "ext_march.h"

namespace gh {

template hipError_t launch_march_mode<double, 5, false, kPredict>(const MarchArgs<double>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<float, 5, false, kPredict>(const MarchArgs<float>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<double, 5, false, kCorrect>(const MarchArgs<double>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<float, 5, false, kCorrect>(const MarchArgs<float>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<double, 6, false, kPredict>(const MarchArgs<double>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<float, 6, false, kPredict>(const MarchArgs<float>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<double, 6, false, kCorrect>(const MarchArgs<double>&, int64_t, hipStream_t);
template hipError_t launch_march_mode<float, 6, false, kCorrect>(const MarchArgs<float>&, int64_t, hipStream_t);

}  // namespace gh
