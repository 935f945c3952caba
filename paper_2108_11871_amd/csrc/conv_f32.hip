// Boundary convolution kernel, FP32 transforms of FP32 slot data (kernel: conv.h).
#include "conv.h"

namespace ips {

template hipError_t launch_cc_t<float, float, true>(const CcArgs &, int, hipStream_t);
template hipError_t launch_cc_t<float, float, false>(const CcArgs &, int, hipStream_t);

} // namespace ips
