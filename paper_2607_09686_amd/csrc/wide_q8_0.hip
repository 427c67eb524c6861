// The wide-tile grouped GEMMs for Q8_0 weights.
#include "wide.h"

namespace moecache {

template hipError_t wide_gateup<8>(bool, dim3, const GmParams &, hipStream_t, const Timing &);
template hipError_t wide_down<8>(bool, dim3, const GmParams &, hipStream_t, const Timing &);

}  // namespace moecache
