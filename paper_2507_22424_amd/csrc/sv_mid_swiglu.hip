#include "sv_products.h"

namespace sv {

SV_INSTANTIATE_MID(launch_mid_swiglu, EPI_SWIGLU, 3)

}  // namespace sv
