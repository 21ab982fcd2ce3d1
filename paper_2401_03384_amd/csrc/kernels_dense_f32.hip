// The dense convolution kernels in fp32 (32x32x2 MFMA, sums in two levels).
#include "dense_kernels.h"

namespace ce {

hipError_t dense_f32(const Launch& ln, const void* a, const void* b, void* c, void* d, hipStream_t s) {
    switch (ln.kind & 0xff) {
        case K_DCONV: return dense_conv<float>(ln, a, b, c, s);
        case K_DWGRAD: return dense_wgrad<float>(ln, a, b, d, s);
        case K_DPACK: return dense_pack<float>(ln, a, c, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace ce
