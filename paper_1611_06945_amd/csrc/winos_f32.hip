// Instantiations of the Winograd F(2x2, 3x3) kernel on split products (fp32, 3x3 stride-1 layers).
#include "winos_kernel.h"
#include "winow_kernel.h"

namespace convfwd {

void register_winos_f32(std::vector<Variant>& out)
{
    //                     MB LBV RING      call  own   chunk
    winos_register<WinosCfg<1, 2, 2>>(out, {7.62, 1.71, 0.865, 0});
    winos_register<WinosCfg<1, 5, 2>>(out, {5.27, 5.15, 1.206, 0});
    winos_register<WinosCfg<2, 2, 4>>(out, {5.95, 4.54, 1.179, 0});
    winos_register<WinosCfg<2, 5, 4>>(out, {8.12, 3.75, 1.418, 0});
    winos_register<WinosCfg<3, 2, 3>>(out, {5.28, 6.06, 1.465, 0});
    winos_register<WinosCfg<3, 5, 3>>(out, {7.93, 5.21, 1.753, 0});
    //                     PITCH    call own   chunk  halved round
    winow_register<WinowCfg<512>>(out, {9.9, 4.2, 2.35, 0.7});
    winow_register<WinowCfg<768>>(out, {9.9, 4.9, 2.37, 0.7});
}

}  // namespace convfwd
