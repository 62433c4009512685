// bf16-storage instantiations of the pointwise kernel for many pixels.
#include "pwb_kernel.h"

namespace convfwd {

void register_pwb_bf16(std::vector<Variant>& out) { pwb_register_all<CONV_BF16>(out); }

}  // namespace convfwd
