// Whole-column walks, four columns to a lane: TD(lambda) and discounted returns.
#include "rlcs_colvec.h"

namespace rlcs {

RLCS_COLVEC(TdLambdaOp)
RLCS_COLVEC(DiscountedOp)

}  // namespace rlcs
