// apply_nav.hip -- hot path of kernel family 2: the choice of precision
// (kernels in apply_nav_f32.hip and apply_nav_f64.hip, compiled side by side).
#include "volume_impl.hpp"

namespace bemfft {

template <>
int apply_kind<2>(int precision, const ApplyArgs &a, hipStream_t st, hipEvent_t *ev) {
    if (precision == BEMFFT_BF16_MFMA) return apply_prec<2, BEMFFT_BF16_MFMA>(a, st, ev);
    if (precision == BEMFFT_FP32) return apply_prec<2, BEMFFT_FP32>(a, st, ev);
    return apply_prec<2, BEMFFT_FP64>(a, st, ev);
}

template <>
int apply_batch_kind<2>(int precision, const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
    if (precision == BEMFFT_BF16_MFMA) {
        set_error("batches of 16-bit plans are not supported");
        return BEMFFT_EINVAL;
    }
    if (precision == BEMFFT_FP32) return apply_batch_prec<2, BEMFFT_FP32>(dm, io, g, st);
    return apply_batch_prec<2, BEMFFT_FP64>(dm, io, g, st);
}

template <>
int volume_kind<2>(int precision, const ApplyArgs &a, double *out, hipStream_t st, hipEvent_t *ev) {
    if (precision == BEMFFT_BF16_MFMA) return volume_prec<2, BEMFFT_BF16_MFMA>(a, out, st, ev);
    if (precision == BEMFFT_FP32) return volume_prec<2, BEMFFT_FP32>(a, out, st, ev);
    return volume_prec<2, BEMFFT_FP64>(a, out, st, ev);
}

}  // namespace bemfft
