// One-launch permanents of up to 32 columns.
#include "k_fused_impl.h"

namespace pq {
PQ_FINST(26)
PQ_FINST(28)
PQ_FINST(30)
PQ_FINST(32)
}  // namespace pq
