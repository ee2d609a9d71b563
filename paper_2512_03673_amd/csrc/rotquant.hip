// Launches of the rotate+quantise kernel (rotquant_kernel.h), but for 8-bit codes of g >= 256 (lanes8.hip); and two diagnostics, the
// rotated rows' absmax and the codes as plain integers.
#include "rotquant_kernel.h"

namespace convrot {

namespace {

// Sylvester (Walsh) Hadamard matrix of order G on a unit: radix-2 butterflies (a, b) -> (a + b, a - b),
// in-group index bits 0-3 inside the lane's 16 elements, the higher ones across lanes.
template <int G>
__device__ __forceinline__ void sylvester_unit(float (&v)[kUnit], int lane)
{
    constexpr int kBitsInUnit = G >= 16 ? 4 : 2;
#pragma unroll
    for (int b = 0; b < kBitsInUnit; ++b)
#pragma unroll
        for (int e = 0; e < kUnit; ++e)
            if (!(e & (1 << b))) {
                const float lo = v[e], hi = v[e | (1 << b)];
                v[e] = lo + hi;
                v[e | (1 << b)] = lo - hi;
            }
    constexpr int kLaneBits = G == 64 ? 2 : G == 256 ? 4 : G == 1024 ? 6 : 0;
#pragma unroll
    for (int b = 0; b < kLaneBits; ++b) {
        const bool upper = (lane >> b) & 1;
#pragma unroll
        for (int e = 0; e < kUnit; ++e) {
            const float other = __shfl_xor(v[e], 1 << b, 64);
            v[e] = upper ? other - v[e] : v[e] + other;
        }
    }
}

}  // namespace

// Diagnostic (the paper's outlier-amplitude metric max |X H|, Sec. 4.2 and Table 5-1): per-row maximum of
// the rotated activations for KIND 0 = no rotation, 1 = the layer's regular Hadamard rotation, 2 = the
// Sylvester Hadamard matrix of the same order.  One wavefront per row, 1024 elements per pass.
template <int G, int KIND>
__global__ __launch_bounds__(256, 2) void rotated_absmax_kernel(const uint16_t *__restrict__ X, int64_t rows, int K,
                                                             float *__restrict__ out)
{
    __shared__ __attribute__((aligned(16))) uint8_t columns[KIND == 1 ? 4 * Item<G>::kBytes : 16];
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;                     // wavefront-uniform
    const int units = K / kUnit;
    const uint16_t *xrow = X + row * (int64_t)K;
    float amax = 0.0f;
    const Rotation<G> rot(lane);
    for (int base = 0; base < units; base += 64) {
        const int unit = base + (KIND == 1 ? Item<G>::unit(lane) : lane);
        const bool ok = unit < units;            // K % g == 0: a rotation group is all-valid or all-invalid
        float v[kUnit];
        if constexpr (KIND == 1) {
            // the layer's rotation, with the arithmetic of the rotate+quantise kernel (bit-identical maxima)
            u32x4 raw[2];
            Item<G>::load(xrow, base, units, lane, raw);
            Item<G>::rotate(rot, raw, columns + (threadIdx.x >> 6) * Item<G>::kBytes, lane, v);
        } else {
            const u32x4 *p = reinterpret_cast<const u32x4 *>(xrow + (int64_t)(ok ? unit : units - 1) * kUnit);
            const u32x4 lo = p[0], hi = p[1];
            const uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                v[2 * j] = __uint_as_float(w[j] << 16);
                v[2 * j + 1] = __uint_as_float(w[j] & 0xFFFF0000u);
            }
        }
        if constexpr (KIND == 2) sylvester_unit<G>(v, lane);
        float m = 0.0f;
#pragma unroll
        for (int e = 0; e < kUnit; ++e) m = fmaxf(m, fabsf(v[e]));
        amax = ok ? fmaxf(amax, m) : amax;
    }
    amax = max_of_lanes<32>(amax);
    if (lane == 0) out[row] = KIND == 0 ? amax : amax * group_norm<G>();
}

namespace {

template <int BITS>
hipError_t launch_bits(const void *X, int64_t rows, int64_t K, int group, void *Xq, float *scale, hipStream_t stream)
{
    switch (group) {
        case 4: return launch_g<4, BITS>(X, rows, (int)K, Xq, scale, stream);
        case 16: return launch_g<16, BITS>(X, rows, (int)K, Xq, scale, stream);
        case 64: return launch_g<64, BITS>(X, rows, (int)K, Xq, scale, stream);
        default: break;
    }
    if constexpr (BITS == 8) return rotquant_lanes8(X, rows, K, group, Xq, scale, stream);
    else if (group == 256) return launch_g<256, BITS>(X, rows, (int)K, Xq, scale, stream);
    else if (group == 1024) return launch_g<1024, BITS>(X, rows, (int)K, Xq, scale, stream);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_rotquant(const void *X, int64_t rows, int64_t K, int group, int bits, void *Xq, float *scale,
                           hipStream_t stream)
{
    if (rows == 0) return hipSuccess;
    if (bits == 4) return launch_bits<4>(X, rows, K, group, Xq, scale, stream);
    if (bits == 8) return launch_bits<8>(X, rows, K, group, Xq, scale, stream);
    return hipErrorInvalidValue;
}

namespace {

template <int G>
hipError_t launch_absmax_g(const void *X, int64_t rows, int K, int kind, float *out, hipStream_t stream)
{
    const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
    const uint16_t *x = (const uint16_t *)X;
    if (kind == 0) hipLaunchKernelGGL((rotated_absmax_kernel<G, 0>), grid, block, 0, stream, x, rows, K, out);
    else if (kind == 1) hipLaunchKernelGGL((rotated_absmax_kernel<G, 1>), grid, block, 0, stream, x, rows, K, out);
    else hipLaunchKernelGGL((rotated_absmax_kernel<G, 2>), grid, block, 0, stream, x, rows, K, out);
    return hipGetLastError();
}

}  // namespace

// ---- code matrix -> plain int8 codes (gate / debug export)
__global__ __launch_bounds__(256) void unpack_codes_kernel(const uint8_t *__restrict__ Xq, int64_t rows, int K,
                                                           int8_t *__restrict__ codes)
{
    // one thread per unit of 16 codes: its 12 bytes are the first or the last 12 of a 24-byte chunk
    const int units = K / kUnit;
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= rows * units) return;
    const int64_t row = id / units;
    const int unit = (int)(id - row * units);
    const uint8_t *blk = Xq + ((row / e2m3::kRows) * e2m3::stages(K) + unit / e2m3::kUnitsPerStage) * e2m3::kBlockBytes;
    const int r = (int)(row % e2m3::kRows), c = (unit % e2m3::kUnitsPerStage) >> 1;
    const uint32_t *pa = reinterpret_cast<const uint32_t *>(blk + e2m3::a_offset(r, c));
    const uint32_t *pb = reinterpret_cast<const uint32_t *>(blk + e2m3::b_offset(r, c));
    uint32_t w[3];
    if ((unit & 1) == 0) { w[0] = pa[0]; w[1] = pa[1]; w[2] = pa[2]; }
    else { w[0] = pa[3]; w[1] = pb[0]; w[2] = pb[1]; }
    int8_t out[kUnit];
#pragma unroll
    for (int e = 0; e < kUnit; ++e) {
        const int bit = 6 * (2 * (e % 8) + e / 8);
        uint32_t f = w[bit / 32] >> (bit % 32);
        if (bit % 32 > 26) f |= w[bit / 32 + 1] << (32 - bit % 32);
        const int ex = (f >> 3) & 3, mant = f & 7;
        const int mag = ex == 0 ? 0 : ((8 | mant) << ex) >> 4;   // E2M3, bias 1: (1 + mant / 8) * 2^(ex - 1)
        out[e] = (int8_t)((f & 32) ? -mag : mag);
    }
    int4 *dst = reinterpret_cast<int4 *>(codes + row * (int64_t)K + (int64_t)unit * kUnit);
    *dst = *reinterpret_cast<const int4 *>(out);
}

hipError_t launch_unpack_codes(const void *Xq, int64_t rows, int64_t K, int8_t *codes, hipStream_t stream)
{
    if (rows == 0) return hipSuccess;
    const int64_t n = rows * (K / kUnit);
    hipLaunchKernelGGL(unpack_codes_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, (const uint8_t *)Xq, rows,
                       (int)K, codes);
    return hipGetLastError();
}

hipError_t launch_rotated_absmax(const void *X, int64_t rows, int64_t K, int group, int kind, float *out,
                                 hipStream_t stream)
{
    if (rows == 0) return hipSuccess;
    if (kind < 0 || kind > 2) return hipErrorInvalidValue;
    switch (group) {
        case 4: return launch_absmax_g<4>(X, rows, (int)K, kind, out, stream);
        case 16: return launch_absmax_g<16>(X, rows, (int)K, kind, out, stream);
        case 64: return launch_absmax_g<64>(X, rows, (int)K, kind, out, stream);
        case 256: return launch_absmax_g<256>(X, rows, (int)K, kind, out, stream);
        case 1024: return launch_absmax_g<1024>(X, rows, (int)K, kind, out, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace convrot
