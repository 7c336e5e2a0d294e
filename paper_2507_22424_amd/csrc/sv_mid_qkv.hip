#include "sv_products.h"

namespace sv {

SV_INSTANTIATE_MID(launch_mid_qkv, EPI_QKV, 3)

}  // namespace sv
