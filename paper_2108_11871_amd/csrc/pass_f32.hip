// Pencil transforms, FP32 data and transforms (kernels: pass.h).
#include "pass.h"

namespace ips {

template hipError_t launch_pass_t<float, float, float>(const PassArgs &, hipStream_t);
template hipError_t launch_pass_t<float, float, double>(const PassArgs &, hipStream_t);
template hipError_t launch_multi_t<float, float, float>(MultiPassArgs &, hipStream_t);
template hipError_t launch_multi_t<float, float, double>(MultiPassArgs &, hipStream_t);

} // namespace ips
