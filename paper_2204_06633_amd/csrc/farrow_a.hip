// Polynomial projection kernels instantiated for tap counts 2, 4, 6, 8.
#include "farrow_adjoint.hpp"
#include "farrow_forward.hpp"

namespace lr {
LR_INSTANTIATE_FARROW_ADJ(2)
LR_INSTANTIATE_FARROW_FWD(2)
LR_INSTANTIATE_FARROW_ADJ(4)
LR_INSTANTIATE_FARROW_FWD(4)
LR_INSTANTIATE_FARROW_ADJ(6)
LR_INSTANTIATE_FARROW_FWD(6)
LR_INSTANTIATE_FARROW_ADJ(8)
LR_INSTANTIATE_FARROW_FWD(8)
}  // namespace lr
