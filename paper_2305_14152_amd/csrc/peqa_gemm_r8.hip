// Contraction kernels with tiles of 128 token rows.
#include "peqa_contract.h"

namespace peqa {
template struct GemmRows<8>;
}  // namespace peqa
