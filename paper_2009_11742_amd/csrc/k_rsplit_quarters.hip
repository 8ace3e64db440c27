// The resident row-split kernels with the row-split schedule's sums.
#include "k_rsplit.h"

namespace rom {
namespace rsplit {

const Tile kQuarterTiles[kTiles] = ROM_RTILES(kQuarters);

}  // namespace rsplit
}  // namespace rom
