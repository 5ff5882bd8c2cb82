// Launch configuration for vectors of length 13824.
#include "kashin_pair_impl.h"

namespace kashin {
KASHIN_DEFINE_SIZE(13824, 576, 3, 24, 24, 24)
}  // namespace kashin
