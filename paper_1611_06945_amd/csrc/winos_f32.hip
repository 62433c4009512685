// Instantiations of the Winograd F(2x2, 3x3) kernel on split products (fp32, 3x3 stride-1 layers).
#include "winos_kernel.h"

namespace convfwd {

void register_winos_f32(std::vector<Variant>& out)
{
    //                     MB LBV RING
    winos_register<WinosCfg<1, 2, 2>>(out);
    winos_register<WinosCfg<1, 5, 2>>(out);
    winos_register<WinosCfg<2, 2, 4>>(out);
    winos_register<WinosCfg<2, 5, 4>>(out);
    winos_register<WinosCfg<3, 2, 3>>(out);
    winos_register<WinosCfg<3, 5, 3>>(out);
}

}  // namespace convfwd
