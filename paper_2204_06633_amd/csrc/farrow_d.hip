// Polynomial projection kernels instantiated for tap counts 26, 28, 30, 32.
#include "farrow_adjoint.hpp"
#include "farrow_forward.hpp"

namespace lr {
LR_INSTANTIATE_FARROW_ADJ(26)
LR_INSTANTIATE_FARROW_FWD(26)
LR_INSTANTIATE_FARROW_ADJ(28)
LR_INSTANTIATE_FARROW_FWD(28)
LR_INSTANTIATE_FARROW_ADJ(30)
LR_INSTANTIATE_FARROW_FWD(30)
LR_INSTANTIATE_FARROW_ADJ(32)
LR_INSTANTIATE_FARROW_FWD(32)
}  // namespace lr
