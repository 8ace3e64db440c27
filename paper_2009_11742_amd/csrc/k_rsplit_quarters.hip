// The resident row-split kernels with the row-split schedule's sums.
#include "k_rsplit.h"

namespace rom {
namespace rsplit {

const Tile kQuarterTiles[kQuarterCount] = {ROM_RT_kQuarters(1, 1, 1, 2.5f), ROM_RT_kQuarters(1, 2, 1, 3.5f),
                                           ROM_RT_kQuarters(1, 2, 2, 6.0f), ROM_RT_kQuarters(1, 4, 2, 9.0f),
                                           ROM_RT_LONG(kQuarters)};

}  // namespace rsplit
}  // namespace rom
