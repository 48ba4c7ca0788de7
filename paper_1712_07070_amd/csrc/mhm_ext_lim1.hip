// The other PLM words' kernels (mhm_fwd_ext.h) with the van Leer limiter.

#include "mhm_fwd_ext.h"

namespace gh {

GH_EXT_LIM_INST(double, 1)
GH_EXT_LIM_INST(float, 1)

}  // namespace gh
