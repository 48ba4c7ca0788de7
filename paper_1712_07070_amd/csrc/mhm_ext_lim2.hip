// The other PLM words' kernels (mhm_fwd_ext.h) with the van Albada limiter.

#include "mhm_fwd_ext.h"

namespace gh {

GH_EXT_LIM_INST(double, 2)
GH_EXT_LIM_INST(float, 2)

}  // namespace gh
