// Launch configuration for vectors of length 6144.
#include "kashin_pair_impl.h"

namespace kashin {
KASHIN_DEFINE_SIZE(6144, 384, 4, 16, 24, 16)
}  // namespace kashin
