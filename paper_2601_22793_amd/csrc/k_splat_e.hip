// Splat instances of 13 and 14 lines.
#include "k_splat.h"

namespace epr {
EPR_SPLAT_UNIT(13) EPR_SPLAT_UNIT(14)
}  // namespace epr
