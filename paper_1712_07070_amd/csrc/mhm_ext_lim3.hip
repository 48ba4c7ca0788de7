// The other PLM words' kernels (mhm_fwd_ext.h) with the hybrid limiter.

#include "mhm_fwd_ext.h"

namespace gh {

GH_EXT_LIM_INST(double, 3)
GH_EXT_LIM_INST(float, 3)

}  // namespace gh
