// f16-storage instantiations of the pointwise kernel for many pixels.
#include "pwb_kernel.h"

namespace convfwd {

void register_pwb_f16(std::vector<Variant>& out) { pwb_register_all<CONV_F16>(out); }

}  // namespace convfwd
