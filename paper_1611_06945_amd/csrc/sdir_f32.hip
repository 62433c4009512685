// Instantiations of the direct window kernel on split products (fp32, 3x3 and 5x5, any stride up to 4).
#include "sdir_kernel.h"

namespace convfwd {

void register_sdir_f32(std::vector<Variant>& out)
{
    //                    R MBW NBW WN WK POS           call   own    chunk   grow
    sdir_register<SdirCfg<3, 2, 1, 4, 1, 768>>(out, {4.65f, 1.85f, 3.799f, 0.7f});
    sdir_register<SdirCfg<3, 1, 1, 4, 1, 768>>(out, {4.55f, 1.53f, 2.550f, 0.6f});
    sdir_register<SdirCfg<3, 2, 1, 2, 2, 384>>(out, {5.16f, 0.93f, 3.920f, 0.7f});
    sdir_register<SdirCfg<3, 1, 1, 2, 2, 384>>(out, {5.17f, 0.97f, 2.663f, 0.6f});
    sdir_register<SdirCfg<3, 1, 1, 1, 4, 384>>(out, {4.65f, 1.53f, 3.411f, 0.4f});
    sdir_register<SdirCfg<3, 1, 1, 1, 4, 192>>(out, {5.25f, 0.73f, 2.582f, 0.7f});
    sdir_register<SdirCfg<3, 1, 1, 1, 8, 192>>(out, {4.45f, 1.50f, 4.492f, 0.4f});
    sdir_register<SdirCfg<5, 2, 1, 4, 1, 768>>(out, {5.24f, 1.79f, 7.363f, 0.8f});
    sdir_register<SdirCfg<5, 1, 1, 4, 1, 768>>(out, {5.38f, 0.88f, 4.269f, 0.8f});
    sdir_register<SdirCfg<5, 2, 1, 2, 2, 384>>(out, {7.08f, -0.12f, 7.356f, 0.9f});
    sdir_register<SdirCfg<5, 1, 1, 2, 2, 384>>(out, {6.28f, 0.08f, 4.338f, 0.9f});
    sdir_register<SdirCfg<5, 1, 1, 1, 4, 384>>(out, {5.02f, 1.08f, 5.309f, 0.4f});
    sdir_register<SdirCfg<5, 1, 1, 1, 4, 192>>(out, {6.22f, -0.23f, 4.696f, 0.9f});
    sdir_register<SdirCfg<5, 1, 1, 1, 8, 192>>(out, {4.23f, 0.90f, 8.355f, 0.4f});
}

}  // namespace convfwd
