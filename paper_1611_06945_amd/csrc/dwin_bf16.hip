// bf16-storage instantiations of the one-launch window kernel.
#include "dwin_kernel.h"

namespace convfwd {

void register_dwin_bf16(std::vector<Variant>& out) { dwin_register_all<CONV_BF16>(out); }

}  // namespace convfwd
