// Whole-column walks, four columns to a lane: eligibility traces (scalar and vector) and prefix sums.
#include "rlcs_colvec.h"

namespace rlcs {

using Trace = ForwardOp<true, false>;
using PrefixEnds = ForwardOp<false, false>;
using PrefixStarts = ForwardOp<false, true>;
RLCS_COLVEC(Trace)
RLCS_COLVEC(PrefixEnds)
RLCS_COLVEC(PrefixStarts)

}  // namespace rlcs
