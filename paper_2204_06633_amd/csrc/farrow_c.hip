// Polynomial projection kernels instantiated for tap counts 18, 20, 22, 24.
#include "farrow_adjoint.hpp"
#include "farrow_forward.hpp"

namespace lr {
LR_INSTANTIATE_FARROW_ADJ(18)
LR_INSTANTIATE_FARROW_FWD(18)
LR_INSTANTIATE_FARROW_ADJ(20)
LR_INSTANTIATE_FARROW_FWD(20)
LR_INSTANTIATE_FARROW_ADJ(22)
LR_INSTANTIATE_FARROW_FWD(22)
LR_INSTANTIATE_FARROW_ADJ(24)
LR_INSTANTIATE_FARROW_FWD(24)
}  // namespace lr
