// Pencil transforms, FP64 input, FP32 transforms (kernels: pass.h).
#include "pass.h"

namespace ips {

template hipError_t launch_pass_t<float, double, float>(const PassArgs &, hipStream_t);
template hipError_t launch_pass_t<float, double, double>(const PassArgs &, hipStream_t);
template hipError_t launch_multi_t<float, double, float>(MultiPassArgs &, hipStream_t);

} // namespace ips
