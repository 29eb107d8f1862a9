// One-launch permanents of up to 24 columns.
#include "k_fused_impl.h"

namespace pq {
PQ_FINST(16)
PQ_FINST(18)
PQ_FINST(20)
PQ_FINST(22)
PQ_FINST(24)
}  // namespace pq
