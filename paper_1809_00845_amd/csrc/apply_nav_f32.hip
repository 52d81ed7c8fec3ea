// apply_nav_f32.hip -- kernels of the hot path for kernel family 2, FP32 and the 16-bit form.
#include "zpass16.hpp"

namespace bemfft {

template <>
int apply_prec<2, BEMFFT_FP32>(const ApplyArgs &a, hipStream_t st, hipEvent_t *ev) {
    return Launch<float, 2>::run(a, st, ev);
}
template <>
int apply_batch_prec<2, BEMFFT_FP32>(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
    return Launch<float, 2>::run_batch(dm, io, g, st);
}
template <>
int volume_prec<2, BEMFFT_FP32>(const ApplyArgs &a, double *out, hipStream_t st, hipEvent_t *ev) {
    return VolumeLaunch<float, 2>::run(a, out, st, ev);
}

template <>
int apply_prec<2, BEMFFT_BF16_MFMA>(const ApplyArgs &a, hipStream_t st, hipEvent_t *ev) {
    return Launch16<2>::run(a, st, ev);
}
template <>
int volume_prec<2, BEMFFT_BF16_MFMA>(const ApplyArgs &a, double *out, hipStream_t st, hipEvent_t *ev) {
    return VolumeLaunch16<2>::run(a, out, st, ev);
}

}  // namespace bemfft
