// Launch configuration for vectors of length 16384.
#include "kashin_pair_impl.h"

namespace kashin {
KASHIN_DEFINE_SIZE(16384, 512, 2, 32, 16, 32)
}  // namespace kashin
