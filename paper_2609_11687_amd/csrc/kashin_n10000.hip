// Launch configuration for vectors of length 10000.
#include "kashin_pair_impl.h"

namespace kashin {
KASHIN_DEFINE_SIZE(10000, 512, 2, 20, 25, 20)
}  // namespace kashin
