// The other PLM words' kernels (mhm_fwd_ext.h) of first order.

#include "mhm_fwd_ext.h"

namespace gh {

GH_EXT_LIM_INST(double, kFirstOrder)
GH_EXT_LIM_INST(float, kFirstOrder)

}  // namespace gh
