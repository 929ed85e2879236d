// Splat instances of 11 and 16 lines.
#include "k_splat.h"

namespace epr {
EPR_SPLAT_UNIT(11) EPR_SPLAT_UNIT(16)
}  // namespace epr
