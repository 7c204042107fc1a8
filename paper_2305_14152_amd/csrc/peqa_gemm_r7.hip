// Contraction kernels with tiles of 112 token rows.
#include "peqa_contract.h"

namespace peqa {
template struct GemmRows<7>;
}  // namespace peqa
