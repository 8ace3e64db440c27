// The resident row-split kernels with the column blocks' sums.
#include "k_rsplit.h"

namespace rom {
namespace rsplit {

const Tile kPairTiles[kTiles] = ROM_RTILES(kPairs);

}  // namespace rsplit
}  // namespace rom
