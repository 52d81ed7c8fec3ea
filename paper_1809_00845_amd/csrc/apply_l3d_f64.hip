// apply_l3d_f64.hip -- kernels of the hot path for kernel family 1, FP64.
#include "volume_impl.hpp"

namespace bemfft {

template <>
int apply_prec<1, BEMFFT_FP64>(const ApplyArgs &a, hipStream_t st, hipEvent_t *ev) {
    return Launch<double, 1>::run(a, st, ev);
}
template <>
int apply_batch_prec<1, BEMFFT_FP64>(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
    return Launch<double, 1>::run_batch(dm, io, g, st);
}
template <>
int volume_prec<1, BEMFFT_FP64>(const ApplyArgs &a, double *out, hipStream_t st, hipEvent_t *ev) {
    return VolumeLaunch<double, 1>::run(a, out, st, ev);
}

}  // namespace bemfft
