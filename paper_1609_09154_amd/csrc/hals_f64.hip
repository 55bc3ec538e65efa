// The HALS sweep for double factors.
#include "hals_sweep.h"

namespace nmfk {

template hipError_t hals_rows<double>(const double*, double*, Split<double>, const double*, int64_t, int, int,
                                     double*, double*, hipStream_t, const double*, FactorCopy);

}  // namespace nmfk
