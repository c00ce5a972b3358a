// Energy change and decision of a colour phase on int8 deviations whose changes may exceed int8.
#include "phase_gram.h"

namespace bnlat {
BN_GRAM_FORM(FIELD_SPLIT, split)
}  // namespace bnlat
