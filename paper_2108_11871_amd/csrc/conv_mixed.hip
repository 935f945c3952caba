// Boundary convolution kernel, FP32 transforms of FP64 input (2D: rho itself) (kernel: conv.h).
#include "conv.h"

namespace ips {

template hipError_t launch_cc_t<float, double, true>(const CcArgs &, int, hipStream_t);
template hipError_t launch_cc_t<float, double, false>(const CcArgs &, int, hipStream_t);

} // namespace ips
