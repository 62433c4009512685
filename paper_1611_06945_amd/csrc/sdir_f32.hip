// Instantiations of the direct window kernel on split products (fp32, 3x3 and 5x5, any stride up to 4).
#include "sdir_kernel.h"

namespace convfwd {

// Layers (of 482 drawn 5x5 and 1994 drawn 3x3 ones, strides 1 and 2) on which a form is the fastest of all kernels, and the time without it there,
// mean and at most: 5x5 M32N128 106, 1.22 (2.29), M32N64 67, 1.11 (1.38), M32N32 in slabs of 384 54, 1.18 (1.52), with eight waves 48, 1.08
// (1.14), with four in slabs of 192 28, 1.01 (1.03), M64N128 31, 1.06 (1.14), M64N64 31, 1.04 (1.11); 3x3 in the same order 58, 1.07 (1.45), 65, 1.08 (1.25),
// 46, 1.08 (1.31), 68, 1.05 (1.15), 93, 1.04 (1.16), 47, 1.06 (1.24), 49, 1.05 (1.19).
// (A start of 0.0: the fit's was -0.1 and -0.2.  With 4.5e-6 for each filter value instead of 1.2e-6 every start comes out above zero and the fits are
// closer, 4 to 6 % at 5x5, but not the picks: 11 of 220 other layers more than 5 % slower than before this kernel, 10 with these constants.)
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
    sdir_register<SdirCfg<5, 2, 1, 2, 2, 384>>(out, {6.83f, 0.0f, 7.346f, 0.9f});
    sdir_register<SdirCfg<5, 1, 1, 2, 2, 384>>(out, {6.28f, 0.08f, 4.338f, 0.9f});
    sdir_register<SdirCfg<5, 1, 1, 1, 4, 384>>(out, {5.02f, 1.08f, 5.309f, 0.4f});
    sdir_register<SdirCfg<5, 1, 1, 1, 4, 192>>(out, {5.67f, 0.0f, 4.667f, 0.9f});
    sdir_register<SdirCfg<5, 1, 1, 1, 8, 192>>(out, {4.23f, 0.90f, 8.355f, 0.4f});
}

}  // namespace convfwd
