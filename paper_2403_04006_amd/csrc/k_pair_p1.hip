// Pair-sweep instances for 29 <= NC <= 32 columns.
#include "k_pair_impl.h"

namespace pq {
PQ_PINST(15)
PQ_PINST(16)
}  // namespace pq
