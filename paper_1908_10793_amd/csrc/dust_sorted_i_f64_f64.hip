// Instantiations of the sums over sorted particles: double storage, double arithmetic.
#include "dust_sorted_kern.h"

namespace dust {

DUST_SORTED_INST(double, double, double, SORTED_DEPOSIT)
DUST_SORTED_INST(double, double, double, SORTED_SOURCE)
DUST_SORTED_INST(double, double, double, SORTED_MASS)
DUST_SORTED_STEP_INST(double, double)

}  // namespace dust
