// Whole-column walks, four columns to a lane: GAE.
#include "rlcs_colvec.h"

namespace rlcs {

RLCS_COLVEC(GaeOp)

}  // namespace rlcs
