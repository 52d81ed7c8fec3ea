// apply_nav_f64.hip -- kernels of the hot path for kernel family 2, FP64.
#include "volume_impl.hpp"

namespace bemfft {

template <>
int apply_prec<2, BEMFFT_FP64>(const ApplyArgs &a, hipStream_t st, hipEvent_t *ev) {
    return Launch<double, 2>::run(a, st, ev);
}
template <>
int apply_batch_prec<2, BEMFFT_FP64>(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
    return Launch<double, 2>::run_batch(dm, io, g, st);
}
template <>
int volume_prec<2, BEMFFT_FP64>(const ApplyArgs &a, double *out, hipStream_t st, hipEvent_t *ev) {
    return VolumeLaunch<double, 2>::run(a, out, st, ev);
}

}  // namespace bemfft
