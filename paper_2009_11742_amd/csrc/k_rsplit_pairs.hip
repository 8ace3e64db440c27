// The resident row-split kernels with the column blocks' sums.
#include "k_rsplit.h"

namespace rom {
namespace rsplit {

const Tile kPairTiles[kPairCount] = {ROM_RT_kPairs(1, 1, 1, 2.5f), ROM_RT_kPairs(1, 2, 1, 3.5f), ROM_RT_LONG(kPairs)};

}  // namespace rsplit
}  // namespace rom
