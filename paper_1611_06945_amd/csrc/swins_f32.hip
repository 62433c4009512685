// Instantiations of the first-layer kernel on split products (fp32, 3 channels, 11x11 stride 4 and 7x7 stride 2).
#include "swins_kernel.h"

namespace convfwd {

void register_swins_f32(std::vector<Variant>& out)
{
    //                     S  ST TMB
    swins_register<SwinsCfg<11, 4, 3>>(out);
    swins_register<SwinsCfg<11, 4, 1>>(out);
    swins_register<SwinsCfg<7, 2, 2>>(out);
    swins_register<SwinsCfg<7, 2, 1>>(out);
}

}  // namespace convfwd
