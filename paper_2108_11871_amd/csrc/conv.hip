// Boundary convolution kernel, FP64 transforms, and the launcher (kernel: conv.h).
#include "conv.h"

namespace ips {

extern template hipError_t launch_cc_t<float, float, true>(const CcArgs &, int, hipStream_t);
extern template hipError_t launch_cc_t<float, float, false>(const CcArgs &, int, hipStream_t);
extern template hipError_t launch_cc_t<float, double, true>(const CcArgs &, int, hipStream_t);
extern template hipError_t launch_cc_t<float, double, false>(const CcArgs &, int, hipStream_t);

hipError_t launch_cc(const CcArgs &a, int nchunk, bool f32, bool in_f32, hipStream_t st)
{
    const int work = (a.W / 2) * a.fd.N;
    if (!big_fft(a.fd.N) && (work > 16 * NT || a.fd.N > 8 * NT)) return hipErrorInvalidValue;
    if (a.W < 2 || a.cols_per_chunk < 1) return hipErrorInvalidValue;
    if (!tile_strides_ok(a.nrows_in, a.irs, a.ncols, a.ics)) return hipErrorInvalidValue;
    const bool wb = a.Bout != nullptr;
    if (!f32) {
        if (in_f32) return hipErrorInvalidValue;
        return wb ? launch_cc_t<double, double, true>(a, nchunk, st)
                  : launch_cc_t<double, double, false>(a, nchunk, st);
    }
    if (in_f32) return wb ? launch_cc_t<float, float, true>(a, nchunk, st)
                          : launch_cc_t<float, float, false>(a, nchunk, st);
    return wb ? launch_cc_t<float, double, true>(a, nchunk, st)
              : launch_cc_t<float, double, false>(a, nchunk, st);
}

} // namespace ips
