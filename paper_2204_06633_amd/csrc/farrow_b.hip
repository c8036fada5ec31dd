// Polynomial projection kernels instantiated for tap counts 10, 12, 14, 16.
#include "farrow_adjoint.hpp"
#include "farrow_forward.hpp"

namespace lr {
LR_INSTANTIATE_FARROW_ADJ(10)
LR_INSTANTIATE_FARROW_FWD(10)
LR_INSTANTIATE_FARROW_ADJ(12)
LR_INSTANTIATE_FARROW_FWD(12)
LR_INSTANTIATE_FARROW_ADJ(14)
LR_INSTANTIATE_FARROW_FWD(14)
LR_INSTANTIATE_FARROW_ADJ(16)
LR_INSTANTIATE_FARROW_FWD(16)
}  // namespace lr
