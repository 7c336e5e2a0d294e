#include "sv_products.h"

namespace sv {

SV_INSTANTIATE_MID(launch_mid_out, EPI_OUT, 1)

}  // namespace sv
