// The wide-tile grouped GEMMs for Q4_0 weights.
#include "wide.h"

namespace moecache {

template hipError_t wide_gateup<2>(bool, dim3, const GmParams &, hipStream_t, const Timing &);
template hipError_t wide_down<2>(bool, dim3, const GmParams &, hipStream_t, const Timing &);

}  // namespace moecache
