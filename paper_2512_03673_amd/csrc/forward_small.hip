// Launches of the one-launch forward (forward_small_kernel.h), but for 8-bit codes of g >= 256 (lanes8.hip).
#include "forward_small_kernel.h"

namespace convrot {

namespace {

template <int BITS>
hipError_t launch_group(const gemm::Operands &o, int group, void *Xq, float *x_scale)
{
    switch (group) {
        case 4: return launch_small_rows<BITS, 4>(o, Xq, x_scale);
        case 16: return launch_small_rows<BITS, 16>(o, Xq, x_scale);
        case 64: return launch_small_rows<BITS, 64>(o, Xq, x_scale);
        default: break;
    }
    if constexpr (BITS == 8) return forward_small_lanes8(o, group, Xq, x_scale);
    else if (group == 256) return launch_small_rows<BITS, 256>(o, Xq, x_scale);
    else if (group == 1024) return launch_small_rows<BITS, 1024>(o, Xq, x_scale);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_forward_small(const void *X, const void *Wq, const float *w_scale, const void *bias_bf16, int64_t M, int64_t N,
                                int64_t K, int group, int bits, void *Y_bf16, void *Xq, float *x_scale, hipStream_t stream)
{
    if (M == 0 || N == 0) return hipSuccess;
    const gemm::Operands o{X, nullptr, Wq, w_scale, bias_bf16, (int)M, (int)N, (int)K, Y_bf16, nullptr, stream};
    return bits == 4 ? launch_group<4>(o, group, Xq, x_scale) : launch_group<8>(o, group, Xq, x_scale);
}

}  // namespace convrot
