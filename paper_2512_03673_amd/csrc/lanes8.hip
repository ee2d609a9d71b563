// 8-bit codes at g >= 256, whose digits 3 and 4 go across lanes by DPP: rotate+quantise (rotquant_kernel.h) and the one-launch forward (forward_small_kernel.h), built
// without the SLP vectoriser (build.py).  It makes vectors of the pairs that these digits add; where there are no packed operations they are taken apart
// again, and the DPP operands no longer go into the instructions: 3 to 4 moves an element.  us, with / without:
//   rotate+quantise  [4608, 3072] g256 11.5 / 10.3, g1024 13.05 / 11.7, [4608, 6144] g1024 22.7 / 20.3, [4608, 12288] g256 35.0 / 31.2, g1024 42.3 / 36.4,
//                    [41771, 11264] g1024 312 / 271; over 124 inputs 0.93
//   forward          M17 x N230 x K1024 g1024 5.43 / 5.05, M3 x N128 x K4096 g1024 6.13 / 5.84, M5 x N5386 x K2048 g1024 6.17 / 6.01
// Kernels of smaller groups have no such digits.  Without it those of rotate+quantise were slower, the larger inputs above all ([4399, 6016] g64 15.9 / 17.7, [13789, 1472]
// g64 13.2 / 15.0, [16896, 12288] g16 103.6 / 113.6, [32362, 16160] g16 268 / 340; but [15500, 8832] g64 73.7 / 66.1; over 461 inputs 1.007); 4-bit ones are the same.
#include "forward_small_kernel.h"
#include "rotquant_kernel.h"

namespace convrot {

hipError_t rotquant_lanes8(const void *X, int64_t rows, int64_t K, int group, void *Xq, float *scale, hipStream_t stream)
{
    switch (group) {
        case 256: return launch_g<256, 8>(X, rows, (int)K, Xq, scale, stream);
        case 1024: return launch_g<1024, 8>(X, rows, (int)K, Xq, scale, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t forward_small_lanes8(const gemm::Operands &o, int group, void *Xq, float *x_scale)
{
    switch (group) {
        case 256: return launch_small_rows<8, 256>(o, Xq, x_scale);
        case 1024: return launch_small_rows<8, 1024>(o, Xq, x_scale);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace convrot
