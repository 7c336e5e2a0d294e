#include "sv_products.h"

namespace sv {

SV_INSTANTIATE_SKINNY(launch_skinny_qkv, EPI_QKV, 3)

}  // namespace sv
