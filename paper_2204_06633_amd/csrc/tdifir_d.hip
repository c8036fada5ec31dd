// TDI filters instantiated for tap counts 26, 28, 30, 32.
#include "tdi_fir.hpp"

namespace lr {
LR_INSTANTIATE_FIR(26)
LR_INSTANTIATE_FIR(28)
LR_INSTANTIATE_FIR(30)
LR_INSTANTIATE_FIR(32)
}  // namespace lr
