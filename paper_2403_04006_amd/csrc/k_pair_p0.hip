// Pair-sweep instances for 25 <= NC <= 28 columns.
#include "k_pair_impl.h"

namespace pq {
PQ_PINST(13)
PQ_PINST(14)
}  // namespace pq
