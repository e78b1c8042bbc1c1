// Whole-column walks, four columns to a lane: Retrace.
#include "rlcs_colvec.h"

namespace rlcs {

RLCS_COLVEC(RetraceOp)

}  // namespace rlcs
