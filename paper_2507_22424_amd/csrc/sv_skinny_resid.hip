#include "sv_products.h"

namespace sv {

SV_INSTANTIATE_SKINNY(launch_skinny_resid, EPI_RESID, 3)

}  // namespace sv
