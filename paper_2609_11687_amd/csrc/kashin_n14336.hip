// Launch configuration for vectors of length 14336.
#include "kashin_pair_impl.h"

namespace kashin {
KASHIN_DEFINE_SIZE(14336, 512, 2, 32, 14, 32)
}  // namespace kashin
