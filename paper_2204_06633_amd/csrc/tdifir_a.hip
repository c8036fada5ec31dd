// TDI filters instantiated for tap counts 2, 4, 6, 8.
#include "tdi_fir.hpp"

namespace lr {
LR_INSTANTIATE_FIR(2)
LR_INSTANTIATE_FIR(4)
LR_INSTANTIATE_FIR(6)
LR_INSTANTIATE_FIR(8)
}  // namespace lr
