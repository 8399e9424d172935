// Instantiations of the sums over sorted particles: float storage, double arithmetic.
#include "dust_sorted_kern.h"

namespace dust {

DUST_SORTED_INST(float, double, float, SORTED_DEPOSIT)
DUST_SORTED_INST(float, double, float, SORTED_SOURCE)
DUST_SORTED_INST(float, double, float, SORTED_MASS)
DUST_SORTED_STEP_INST(float, double)

}  // namespace dust
