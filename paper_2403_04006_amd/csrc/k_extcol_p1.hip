// Instances of the extend-row sweep over the columns' signs, 18 to 24 rows.
#include "k_extcol_impl.h"
#include "many_kernels.h"

namespace pq {

PQ_XINST(18)
PQ_XINST(20)
PQ_XINST(22)
PQ_XINST(24)

}  // namespace pq
