// Work-queue kernel instances (forward/14, forward/18, forward/22).
#include "k_queue_inst.h"

namespace pq {

PQ_QINST(0, 14)
PQ_QINST(0, 18)
PQ_QINST(0, 22)

}  // namespace pq
