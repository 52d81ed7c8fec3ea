// apply_l3d_f32.hip -- kernels of the hot path for kernel family 1, FP32 and the 16-bit form.
#include "zpass16.hpp"

namespace bemfft {

template <>
int apply_prec<1, BEMFFT_FP32>(const ApplyArgs &a, hipStream_t st, hipEvent_t *ev) {
    return Launch<float, 1>::run(a, st, ev);
}
template <>
int apply_batch_prec<1, BEMFFT_FP32>(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
    return Launch<float, 1>::run_batch(dm, io, g, st);
}
template <>
int volume_prec<1, BEMFFT_FP32>(const ApplyArgs &a, double *out, hipStream_t st, hipEvent_t *ev) {
    return VolumeLaunch<float, 1>::run(a, out, st, ev);
}

template <>
int apply_prec<1, BEMFFT_BF16_MFMA>(const ApplyArgs &a, hipStream_t st, hipEvent_t *ev) {
    return Launch16<1>::run(a, st, ev);
}
template <>
int volume_prec<1, BEMFFT_BF16_MFMA>(const ApplyArgs &a, double *out, hipStream_t st, hipEvent_t *ev) {
    return VolumeLaunch16<1>::run(a, out, st, ev);
}

}  // namespace bemfft
