// Contraction kernels with tiles of 96 token rows.
#include "peqa_contract.h"

namespace peqa {
template struct GemmRows<6>;
}  // namespace peqa
