// Staged energy change on int8 deviations, changes beyond int8 (stage_dev.h).
#include "stage_dev.h"

namespace bnlat {
BN_STAGE_FORM(FIELD_SPLIT, split)
}  // namespace bnlat
