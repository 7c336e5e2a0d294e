#include "sv_products.h"

namespace sv {

SV_INSTANTIATE_MID(launch_mid_resid, EPI_RESID, 3)

}  // namespace sv
