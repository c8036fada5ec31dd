// TDI filters instantiated for tap counts 10, 12, 14, 16.
#include "tdi_fir.hpp"

namespace lr {
LR_INSTANTIATE_FIR(10)
LR_INSTANTIATE_FIR(12)
LR_INSTANTIATE_FIR(14)
LR_INSTANTIATE_FIR(16)
}  // namespace lr
