// f16-storage instantiations of the one-launch window kernel.
#include "dwin_kernel.h"

namespace convfwd {

void register_dwin_f16(std::vector<Variant>& out) { dwin_register_all<CONV_F16>(out); }

}  // namespace convfwd
