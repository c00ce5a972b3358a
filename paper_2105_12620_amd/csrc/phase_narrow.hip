// Energy change and decision of a colour phase on int8 deviations of the counts.
#include "phase_gram.h"

namespace bnlat {
BN_GRAM_FORM(FIELD_NARROW, narrow)
}  // namespace bnlat
