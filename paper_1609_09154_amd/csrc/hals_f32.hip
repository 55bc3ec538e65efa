// The HALS sweep for float factors.
#include "hals_sweep.h"

namespace nmfk {

template hipError_t hals_rows<float>(const float*, float*, Split<float>, const float*, int64_t, int, int,
                                     float*, float*, hipStream_t, const float*, FactorCopy);

}  // namespace nmfk
