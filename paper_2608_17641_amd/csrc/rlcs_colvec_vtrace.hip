// Whole-column walks, four columns to a lane: V-Trace.
#include "rlcs_colvec.h"

namespace rlcs {

RLCS_COLVEC(VtraceOp)

}  // namespace rlcs
