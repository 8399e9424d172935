// Instantiations of the particle-per-lane fused step: double storage, double arithmetic.
#include "dust_cells_kern.h"

namespace dust {

DUST_CELLS_ALL(, double, double)

}  // namespace dust
