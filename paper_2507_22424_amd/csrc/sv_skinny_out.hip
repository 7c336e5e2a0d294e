#include "sv_products.h"

namespace sv {

SV_INSTANTIATE_SKINNY(launch_skinny_out, EPI_OUT, 1)

}  // namespace sv
