// Instances of the extend-row sweep over the columns' signs, up to 16 rows.
#include "k_extcol_impl.h"
#include "many_kernels.h"

namespace pq {

PQ_XINST(4)
PQ_XINST(8)
PQ_XINST(12)
PQ_XINST(14)
PQ_XINST(16)

}  // namespace pq
