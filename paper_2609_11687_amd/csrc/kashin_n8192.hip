// Launch configuration for vectors of length 8192.
#include "kashin_pair_impl.h"

namespace kashin {
KASHIN_DEFINE_SIZE(8192, 256, 2, 32, 8, 32)
}  // namespace kashin
