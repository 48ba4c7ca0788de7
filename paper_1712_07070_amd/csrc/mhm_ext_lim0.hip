// The other PLM words' kernels (mhm_fwd_ext.h) with the generalized minmod limiter.

#include "mhm_fwd_ext.h"

namespace gh {

GH_EXT_LIM_INST(double, 0)
GH_EXT_LIM_INST(float, 0)

}  // namespace gh
