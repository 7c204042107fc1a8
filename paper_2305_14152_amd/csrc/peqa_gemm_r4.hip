// Contraction kernels with tiles of 64 token rows.
#include "peqa_contract.h"

namespace peqa {
template struct GemmRows<4>;
}  // namespace peqa
