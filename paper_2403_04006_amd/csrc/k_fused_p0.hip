// One-launch permanents of up to 14 columns.
#include "k_fused_impl.h"

namespace pq {
PQ_FINST(2)
PQ_FINST(4)
PQ_FINST(6)
PQ_FINST(8)
PQ_FINST(10)
PQ_FINST(12)
PQ_FINST(14)
}  // namespace pq
