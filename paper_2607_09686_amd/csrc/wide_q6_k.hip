// The wide-tile grouped GEMMs for Q6_K weights.
#include "wide.h"

namespace moecache {

template hipError_t wide_gateup<14>(bool, dim3, const GmParams &, hipStream_t, const Timing &);
template hipError_t wide_down<14>(bool, dim3, const GmParams &, hipStream_t, const Timing &);

}  // namespace moecache
