// TDI filters instantiated for tap counts 18, 20, 22, 24.
#include "tdi_fir.hpp"

namespace lr {
LR_INSTANTIATE_FIR(18)
LR_INSTANTIATE_FIR(20)
LR_INSTANTIATE_FIR(22)
LR_INSTANTIATE_FIR(24)
}  // namespace lr
