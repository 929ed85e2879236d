// Splat instances of 8, 9 and 10 lines.
#include "k_splat.h"

namespace epr {
EPR_SPLAT_UNIT(8) EPR_SPLAT_UNIT(9) EPR_SPLAT_UNIT(10)
}  // namespace epr
