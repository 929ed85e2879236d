// Splat instances of 12 and 15 lines.
#include "k_splat.h"

namespace epr {
EPR_SPLAT_UNIT(12) EPR_SPLAT_UNIT(15)
}  // namespace epr
