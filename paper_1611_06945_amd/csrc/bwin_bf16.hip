// bf16-storage instantiations of the many-pixel window kernel (stride-1 layers, filters in MFMA operand order).
#include "bwin_kernel.h"

namespace convfwd {

void register_bwin_bf16(std::vector<Variant>& out)
{
    //            DT        R  S WM WN TMB NBW AD LBT
    bwin_register<CONV_BF16, 3, 3, 1, 4, 2, 4, 3, 7, true>(out);   // M64  N512, 896 slab positions: the fewest operand bytes per MFMA
    bwin_register<CONV_BF16, 3, 3, 1, 4, 2, 3, 3, 8, true>(out);   // M64  N384, 1024 (rows of up to 128 pixels)
    bwin_register<CONV_BF16, 3, 3, 2, 2, 1, 4, 3, 5>(out);   // M64  N256, 640
    bwin_register<CONV_BF16, 3, 3, 2, 2, 1, 4, 3, 11>(out);  // M64  N256, 1408 (rows of up to 224 pixels)
    bwin_register<CONV_BF16, 3, 3, 1, 4, 2, 2, 9, 4, true>(out);   // M64  N256, 512: a whole chunk of filter look-ahead
    bwin_register<CONV_BF16, 3, 3, 2, 2, 2, 2, 9, 4, true>(out);   // M128 N128, 512
    bwin_register<CONV_BF16, 3, 3, 1, 4, 1, 4, 9, 7>(out);   // M32  N512, 896
    bwin_register<CONV_BF16, 3, 3, 1, 4, 1, 2, 9, 6>(out);   // M32  N256, 768
    bwin_register<CONV_BF16, 5, 5, 1, 4, 2, 2, 5, 6, true>(out);   // M64  N256, 768
    bwin_register<CONV_BF16, 5, 5, 2, 2, 2, 2, 5, 5, true>(out);   // M128 N128, 640
    bwin_register<CONV_BF16, 5, 5, 1, 4, 1, 2, 5, 6>(out);   // M32  N256, 768
}

}  // namespace convfwd
