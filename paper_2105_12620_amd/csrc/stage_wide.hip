// Staged energy change on uint16 counts (stage_dev.h).
#include "stage_dev.h"

namespace bnlat {
BN_STAGE_FORM(FIELD_WIDE, wide)
}  // namespace bnlat
