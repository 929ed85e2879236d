// Splat instances of 1, 2, 3, 4, 5, 6 and 7 lines.
#include "k_splat.h"

namespace epr {
EPR_SPLAT_UNIT(1) EPR_SPLAT_UNIT(2) EPR_SPLAT_UNIT(3) EPR_SPLAT_UNIT(4)
EPR_SPLAT_UNIT(5) EPR_SPLAT_UNIT(6) EPR_SPLAT_UNIT(7)
}  // namespace epr
