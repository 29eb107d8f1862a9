// Pair-sweep instances for 23 <= NC <= 28 columns.
#include "k_pair_impl.h"

namespace pq {
PQ_PINST(12)
PQ_PINST(13)
PQ_PINST(14)
}  // namespace pq
