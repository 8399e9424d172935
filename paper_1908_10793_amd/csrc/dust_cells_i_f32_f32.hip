// Instantiations of the particle-per-lane fused step: float storage, float arithmetic.
#include "dust_cells_kern.h"

namespace dust {

DUST_CELLS_ALL(, float, float)

}  // namespace dust
