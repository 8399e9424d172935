// Instantiations of the sums over sorted particles: float storage, float arithmetic.
#include "dust_sorted_kern.h"

namespace dust {

DUST_SORTED_INST(float, float, float, SORTED_DEPOSIT)
DUST_SORTED_INST(float, float, float, SORTED_SOURCE)
DUST_SORTED_INST(float, float, float, SORTED_MASS)

}  // namespace dust
