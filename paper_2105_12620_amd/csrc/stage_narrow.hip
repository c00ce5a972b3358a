// Staged energy change on int8 deviations (stage_dev.h).
#include "stage_dev.h"

namespace bnlat {
BN_STAGE_FORM(FIELD_NARROW, narrow)
}  // namespace bnlat
