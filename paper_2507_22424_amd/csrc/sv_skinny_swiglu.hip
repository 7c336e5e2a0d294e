#include "sv_products.h"

namespace sv {

SV_INSTANTIATE_SKINNY(launch_skinny_swiglu, EPI_SWIGLU, 3)

}  // namespace sv
