// Pencil transforms in FP64, and the launchers (kernels: pass.h).
#include "pass.h"

namespace ips {

extern template hipError_t launch_pass_t<float, double, double>(const PassArgs &, hipStream_t);
extern template hipError_t launch_pass_t<float, float, float>(const PassArgs &, hipStream_t);
extern template hipError_t launch_pass_t<float, double, float>(const PassArgs &, hipStream_t);
extern template hipError_t launch_pass_t<float, float, double>(const PassArgs &, hipStream_t);
extern template hipError_t launch_multi_t<float, float, float>(MultiPassArgs &, hipStream_t);
extern template hipError_t launch_multi_t<float, double, float>(MultiPassArgs &, hipStream_t);
extern template hipError_t launch_multi_t<float, float, double>(MultiPassArgs &, hipStream_t);

hipError_t launch_pass_multi(const PassArgs *p, int n, bool in_f32, bool out_f32, hipStream_t st)
{
    if (n < 1 || n > kMultiPass) return hipErrorInvalidValue;
    MultiPassArgs m{};
    m.n = n;
    for (int i = 0; i < n; ++i) m.p[i] = p[i];
    if (!in_f32 && !out_f32) return launch_multi_t<double, double, double>(m, st);
    if (in_f32 && out_f32) return launch_multi_t<float, float, float>(m, st);
    if (!in_f32 && out_f32) return launch_multi_t<float, double, float>(m, st);
    return launch_multi_t<float, float, double>(m, st);
}

hipError_t launch_pass_f32t(const PassArgs &a, hipStream_t st)
{
    if (!pass_strides_ok(a)) return hipErrorInvalidValue;
    return launch_pass_t<float, double, double>(a, st);
}

hipError_t launch_pass(const PassArgs &a, bool in_f32, bool out_f32, hipStream_t st)
{
    if (!pass_strides_ok(a)) return hipErrorInvalidValue;
    if (!in_f32 && !out_f32) return launch_pass_t<double, double, double>(a, st);
    if (in_f32 && out_f32) return launch_pass_t<float, float, float>(a, st);
    if (!in_f32 && out_f32) return launch_pass_t<float, double, float>(a, st);
    return launch_pass_t<float, float, double>(a, st);
}

} // namespace ips
