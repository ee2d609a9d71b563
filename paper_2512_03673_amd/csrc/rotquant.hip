// Kernel A of libconvrot: group-wise regular-Hadamard rotation + per-row absmax + 4-bit
// quantisation + packing of the codes, one pass over the bf16 input (ConvRot paper Sec. 4.2 Eq. 11-13,
// Eq. 1, Sec. 5.2).  Serves activations (rows = tokens) and weights (rows = output channels).
//
// Work split.  A "unit" is 16 consecutive elements of a row (32 B of bf16 in, 12 B of codes out)
// and belongs to one lane.  A row is spread over T = 64*Wv lanes (Wv wavefronts); lane t of the
// row owns units t, t+T, t+2T, ... (U of them), so the two load instructions of a wavefront for one
// such set of units cover a contiguous 2 KB span of the row.  The whole row stays in registers between the absmax
// reduction and the rounding, so X is read from HBM exactly once.
//
// The rotation and the quantiser themselves are rotate_quantise.h.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "convrot_internal.h"
#include "e2m3_layout.h"
#include "panel_layout.h"
#include "rotate_quantise.h"

namespace convrot {

namespace {

// Which unit of its row lane t holds as its i-th.  With g = 1024 and four units a lane these are of one group, 16 apart: digit 4
// runs over them and its radix-4 step is seven instructions on four values of one lane instead of three instructions and two wavefront
// shuffles an element ([4608, 15360]: 48.4 -> 42.7 us).  16 lanes still load 512 bytes of a row at a time.  (The same for digit 3
// of g = 256, where four lanes would load 128 bytes: no faster on large inputs, 15 % slower on 512 rows.)
template <int G, int U>
__device__ __forceinline__ int unit_of(int i, int t, int T)
{
    if constexpr (G == 1024 && U == 4) return ((t >> 4) << 6) + 16 * i + (t & 15);
    else return i * T + t;
}

// Digit 4 over a lane's four units, in the printed matrix's order.
__device__ __forceinline__ void rotate_registers(float (&v)[4][kUnit])
{
#pragma unroll
    for (int e = 0; e < kUnit; ++e) {
        const float x0 = v[0][e], x1 = v[1][e], x2 = v[2][e], x3 = v[3][e];
        const float s = (x0 + x1) + (x2 + x3);
        v[0][e] = fmaf(-2.0f, x3, s);
        v[1][e] = fmaf(-2.0f, x2, s);
        v[2][e] = fmaf(-2.0f, x1, s);
        v[3][e] = fmaf(-2.0f, x0, s);
    }
}

}  // namespace

// T = lanes per row.  Two ways of laying rows over wavefronts:
//   RPW = 1  a wavefront holds 64 lanes of one row (T = 64 * waves per row, BLOCK / T rows per block): any K, any g
//   RPW = 4  a wavefront holds 16 lanes of each of 4 consecutive rows (T = threads / 4, 4 rows per block): the cross-lane
//            digits stay inside 16 lanes; used for K <= 4096.  The four rows' pieces of an output block
//            are adjacent in memory, so a store instruction touches 256- and 128-byte runs instead of 64- and
//            32-byte ones: as few cache lines per instruction as a row-major stream would.
// grid.x = 8 * ceil(rows / (8 * group rows)) * group rows / rows per block (see the row mapping below).
// BITS = 4: codes in [-7, 7], stored as FP6 E2M3 (e2m3_layout.h); BITS = 8 (the W8A8 variant of the layer): one
// int8 per code, [-127, 127] (panel_layout.h).
// (At least two wavefronts per SIMD, i.e. at most 256 registers per lane: then the compiler keeps the MFMA results in
// ordinary registers instead of copying them out of the accumulation registers, one move per element.)
template <int G, int U, int BLOCK, int BITS, int RPW>
__global__ __launch_bounds__(BLOCK, BLOCK <= 256 ? 2 : 1) void rotquant_kernel(const uint16_t *__restrict__ X, int64_t rows, int K,
                                                         int T, uint8_t *__restrict__ Xq,
                                                         float *__restrict__ scale)
{
    constexpr bool kDigit4 = G == 1024 && U == 4;   // over a lane's units (unit_of)
    constexpr int kLaneG = kDigit4 ? 256 : G;       // the rest of the rotation: inside a unit and across lanes
    static_assert(RPW == 1 || (RPW == 4 && kLaneG <= 256), "four rows per wavefront need the rotation inside 16 lanes");
    __shared__ float s_part[BLOCK / 64 * RPW];

    const int tid = threadIdx.x;
    const int rib = RPW == 1 ? tid / T : (tid & 63) >> 4;                        // row inside the block
    const int t = RPW == 1 ? tid - rib * T : (tid >> 6) * 16 + (tid & 15);       // lane index inside the row
    const int rows_per_block = RPW == 1 ? BLOCK / T : RPW;
    // Blocks are dealt round-robin to the 8 XCDs, each with an L2 of its own.  The 16 rows of an output
    // panel go to consecutive blocks of one XCD, so that the 64-byte row pieces of a panel meet in one
    // L2 and leave it as whole lines.
    constexpr int kGroupRows = BITS == 4 ? e2m3::kRows : panel::kRows;   // rows that share an output block
    const int bpp = kGroupRows / rows_per_block;              // thread blocks per group of rows
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int64_t row = ((int64_t)(idx / bpp) * 8 + xcd) * kGroupRows + (idx % bpp) * rows_per_block + rib;
    const bool row_ok = row < rows;
    const int units = K / kUnit;

    // All loads are issued up front and unconditionally: a unit (or row) that does not exist is replaced
    // by the last unit of the last row, and its owner is masked out of the absmax and the stores.
    // K % g == 0 makes a rotation group all-valid or all-invalid, so such lanes never feed valid ones.
    // The units are fetched as operands of the rotation MFMAs (rotation_operand): for h = 0, 1 this lane
    // loads bytes 16 kb ... 16 kb + 15 (kb = lane / 32) of the units owned by lane (lane % 32) + 32 h.
    const int lane = tid & 63;
    const uint16_t *src[2];
    int t_src[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int otid = (tid & ~63) | (lane & 31) | (h << 5);                     // the owner
        const int orib = RPW == 1 ? rib : (otid & 63) >> 4;                        // (a wavefront lies inside one row if RPW == 1)
        t_src[h] = RPW == 1 ? otid - rib * T : (otid >> 6) * 16 + (otid & 15);
        const int64_t orow = row - rib + orib;
        src[h] = X + (orow < rows ? orow : rows - 1) * (int64_t)K + 8 * (lane >> 5);
    }
    u32x4 raw[U][2];
#pragma unroll
    for (int i = 0; i < U; ++i) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int unit = min(unit_of<G, U>(i, t_src[h], T), units - 1);
            raw[i][h] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src[h] + (int64_t)unit * kUnit));
        }
    }
    const v8bf rot0 = rotation_operand<G>(lane, 0), rot1 = rotation_operand<G>(lane, 1);

    float v[U][kUnit];
    float amax = 0.0f;
    if constexpr (kDigit4) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            rotate_units_mfma(rot0, rot1, raw[i][0], raw[i][1], v[i]);
            rotate_lanes<kLaneG>(v[i]);
        }
        rotate_registers(v);
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
        if constexpr (!kDigit4) {
            rotate_units_mfma(rot0, rot1, raw[i][0], raw[i][1], v[i]);
            rotate_lanes<kLaneG>(v[i]);
        }
        float m = 0.0f;
#pragma unroll
        for (int e = 0; e < kUnit; ++e) m = fmaxf(m, fabsf(v[i][e]));
        amax = (row_ok && unit_of<G, U>(i, t, T) < units) ? fmaxf(amax, m) : amax;
    }

    // row absmax: butterfly over the row's lanes of this wavefront, then across the row's wavefronts through LDS
    if constexpr (RPW == 1) {
        amax = max_of_64(amax);
        if (T > 64) {
            if ((tid & 63) == 0) s_part[tid >> 6] = amax;
            __syncthreads();
            const int w0 = (rib * T) >> 6;
            const int wv = T >> 6;
            float a = s_part[w0];
            for (int w = 1; w < wv; ++w) a = fmaxf(a, s_part[w0 + w]);
            amax = a;
        }
    } else {
        amax = max_of_16(amax);
        if ((tid & 15) == 0) s_part[(tid >> 6) * RPW + rib] = amax;
        __syncthreads();
        float a = s_part[rib];
#pragma unroll
        for (int w = 1; w < BLOCK / 64; ++w)
            a = !kDigit4 || w * 16 < T ? fmaxf(a, s_part[w * RPW + rib]) : a;
        amax = a;
    }

    const Quantiser q(amax, group_norm<G>(), BITS == 4 ? 7.0f : 127.0f);
    if (row_ok && t == 0) scale[row] = q.s;
    const int tf = t ^ lane_flip_mask<kLaneG>();

    if constexpr (BITS == 4) {
        const int padded_units = (units + e2m3::kUnitsPerStage - 1) / e2m3::kUnitsPerStage * e2m3::kUnitsPerStage;
        const int64_t stages = padded_units / e2m3::kUnitsPerStage;
        uint8_t *const row_block = Xq + (row / e2m3::kRows) * stages * e2m3::kBlockBytes;
        const int r32 = (int)(row % e2m3::kRows);
        auto store_unit = [&](int i, uint32_t w0, uint32_t w1, uint32_t w2) {
            // A 24-byte chunk (the 32 codes one MFMA lane consumes) is an even unit followed by the odd
            // unit next to it, which the neighbouring lane holds: its first 16 bytes go to the A plane of the
            // block, the other 8 to the B plane (e2m3_layout.h).  The even lane fetches the odd lane's first dword.
            const uint32_t nb0 = __builtin_amdgcn_update_dpp(0u, w0, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
            const int unit = unit_of<G, U>(i, tf, T);
            if (!(row_ok && unit < padded_units)) return;
            uint32_t nb = nb0;
            if (unit >= units) w0 = w1 = w2 = nb = 0;               // K padding: zero codes (units come in pairs: K % 32 == 0)
            uint8_t *blk = row_block + (int64_t)(unit / e2m3::kUnitsPerStage) * e2m3::kBlockBytes;
            const int c = (unit % e2m3::kUnitsPerStage) >> 1;       // chunk of the K128 stage
            if ((unit & 1) == 0) {
                *reinterpret_cast<u32x4 *>(blk + e2m3::a_offset(r32, c)) = u32x4{w0, w1, w2, nb};
            } else {
                *reinterpret_cast<u32x2 *>(blk + e2m3::b_offset(r32, c)) = u32x2{w1, w2};
            }
        };
#pragma unroll
        for (int i = 0; i < U; i += 2) {
            const bool pair = i + 1 < U;
            const v6u packed = codes4(q, pair, as_vector(v[i]), as_vector(v[pair ? i + 1 : i]));
            store_unit(i, packed[0], packed[1], packed[2]);
            if (pair) store_unit(i + 1, packed[3], packed[4], packed[5]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            u32x4 code = codes8(q, as_vector(v[i]));
            // Panel layout: 1 KB panels of 16 rows x 64 bytes, a unit is 16 bytes of its row; units past the
            // row's end inside its last K-panel are stored as zero codes.
            const int unit = unit_of<G, U>(i, tf, T);
            constexpr int kUnitsPerPanelRow = panel::kRowBytes / kUnit;
            const int padded_units = (units + kUnitsPerPanelRow - 1) / kUnitsPerPanelRow * kUnitsPerPanelRow;
            if (row_ok && unit < padded_units) {
                if (unit >= units) code = u32x4{0, 0, 0, 0};
                uint8_t *o = Xq + ((row >> 4) * (int64_t)(padded_units / kUnitsPerPanelRow) + unit / kUnitsPerPanelRow) * panel::kBytes +
                             (int)(row & 15) * panel::kRowBytes + (unit % kUnitsPerPanelRow) * kUnit;
                // plain (cacheable) stores: the pieces of a line are merged in L2
                *reinterpret_cast<u32x4 *>(o) = code;
            }
        }
    }
}

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
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;                     // wavefront-uniform
    const int units = K / kUnit;
    const uint16_t *xrow = X + row * (int64_t)K;
    float amax = 0.0f;
    v8bf rot0, rot1;
    if constexpr (KIND == 1) { rot0 = rotation_operand<G>(lane, 0); rot1 = rotation_operand<G>(lane, 1); }
    for (int base = 0; base < units; base += 64) {
        const int unit = base + lane;
        const bool ok = unit < units;            // K % g == 0: a rotation group is all-valid or all-invalid
        float v[kUnit];
        if constexpr (KIND == 1) {
            // the layer's rotation, with the arithmetic of the rotate+quantise kernel (bit-identical maxima)
            const int u0 = min(base + (lane & 31), units - 1), u1 = min(base + (lane & 31) + 32, units - 1);
            const uint16_t *half = xrow + 8 * (lane >> 5);
            const u32x4 b0 = *reinterpret_cast<const u32x4 *>(half + (int64_t)u0 * kUnit);
            const u32x4 b1 = *reinterpret_cast<const u32x4 *>(half + (int64_t)u1 * kUnit);
            rotate_units_mfma(rot0, rot1, b0, b1, v);
            rotate_lanes<G>(v);
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
    amax = max_of_64(amax);
    if (lane == 0) out[row] = KIND == 0 ? amax : amax * group_norm<G>();
}

namespace {

template <int G, int U, int BITS>
hipError_t launch_gu(const void *X, int64_t rows, int K, int waves_per_row, void *Xq, float *scale,
                     hipStream_t stream)
{
    const int T = 64 * waves_per_row;
    // grid: 8 XCDs x whole row groups per XCD x blocks per group (see the row mapping in the kernel)
    constexpr int kGroupRows = BITS == 4 ? e2m3::kRows : panel::kRows;
    auto grid_for = [&](int rpb) { return (unsigned)(((rows + 8 * kGroupRows - 1) / (8 * kGroupRows)) * 8 * (kGroupRows / rpb)); };
    if (T <= 256) {
        const int rpb = 256 / T;
        hipLaunchKernelGGL((rotquant_kernel<G, U, 256, BITS, 1>), dim3(grid_for(rpb)), dim3(256), 0, stream,
                           (const uint16_t *)X, rows, K, T, (uint8_t *)Xq, scale);
    } else if (T <= 512) {
        hipLaunchKernelGGL((rotquant_kernel<G, U, 512, BITS, 1>), dim3(grid_for(1)), dim3(512), 0, stream,
                           (const uint16_t *)X, rows, K, 512, (uint8_t *)Xq, scale);
    } else {
        hipLaunchKernelGGL((rotquant_kernel<G, U, 1024, BITS, 1>), dim3(grid_for(1)), dim3(1024), 0, stream,
                           (const uint16_t *)X, rows, K, 1024, (uint8_t *)Xq, scale);
    }
    return hipGetLastError();
}

// four rows per wavefront: 4 wavefronts of 16 lanes per row (blocks of 256 threads; with larger blocks, i.e.
// longer rows, the mapping loses more to the block-wide barrier than the stores gain: measured)
template <int G, int U, int BITS>
hipError_t launch_gu4(const void *X, int64_t rows, int K, void *Xq, float *scale, hipStream_t stream)
{
    constexpr int kGroupRows = BITS == 4 ? e2m3::kRows : panel::kRows;
    const unsigned grid = (unsigned)(((rows + 8 * kGroupRows - 1) / (8 * kGroupRows)) * 8 * (kGroupRows / 4));
    hipLaunchKernelGGL((rotquant_kernel<G, U, 256, BITS, 4>), dim3(grid), dim3(256), 0, stream, (const uint16_t *)X, rows, K,
                       64, (uint8_t *)Xq, scale);
    return hipGetLastError();
}

// g = 1024: four units a lane (digit 4 over them), as many wavefronts as the row needs; up to K = 4096 16 lanes of each of four
// rows a wavefront, for the stores' sake as above ([4608, 3072]: 13.4 us against 14.7 with one row a wavefront).  Rows of one
// or two groups have too few wavefronts that way ([1000, 1024]: 4.9 us against 4.2) and take digit 4 across lanes.
template <int BITS>
hipError_t launch_1024(const void *X, int64_t rows, int K, void *Xq, float *scale, hipStream_t stream)
{
    constexpr int kGroupRows = BITS == 4 ? e2m3::kRows : panel::kRows;
    auto go = [&](auto kernel, int rows_per_block, int threads, int T) {
        const unsigned grid = (unsigned)(((rows + 8 * kGroupRows - 1) / (8 * kGroupRows)) * 8 * (kGroupRows / rows_per_block));
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, stream, (const uint16_t *)X, rows, K, T, (uint8_t *)Xq, scale);
        return hipGetLastError();
    };
    const int groups = K / 1024;                             // 16 lanes each
    if (groups == 1) return launch_gu<1024, 1, BITS>(X, rows, K, 1, Xq, scale, stream);
    if (groups == 2) return launch_gu<1024, 2, BITS>(X, rows, K, 1, Xq, scale, stream);
    if (groups <= 4) return go(rotquant_kernel<1024, 4, 256, BITS, 4>, 4, 64 * groups, 16 * groups);
    const int T = (groups + 3) / 4 * 64;
    if (T <= 256) return go(rotquant_kernel<1024, 4, 256, BITS, 1>, 256 / T, 256 / T * T, T);
    if (T <= 512) return go(rotquant_kernel<1024, 4, 512, BITS, 1>, 1, T, T);
    return go(rotquant_kernel<1024, 4, 1024, BITS, 1>, 1, T, T);
}

template <int G, int BITS>
hipError_t launch_g(const void *X, int64_t rows, int K, void *Xq, float *scale, hipStream_t stream)
{
    // four rows per wavefront whenever 4 wavefronts x 16 lanes x 4 units hold a row (K <= 4096)
    const int spans = (K / kUnit + 15) / 16;   // 256-element spans per row
    if (spans <= 16) {
        switch ((spans + 3) / 4) {
            case 1: return launch_gu4<G, 1, BITS>(X, rows, K, Xq, scale, stream);
            case 2: return launch_gu4<G, 2, BITS>(X, rows, K, Xq, scale, stream);
            case 3: return launch_gu4<G, 3, BITS>(X, rows, K, Xq, scale, stream);
            default: return launch_gu4<G, 4, BITS>(X, rows, K, Xq, scale, stream);
        }
    }
    // Pick the wavefronts per row (1, 2, 4, 8 or 16) so that every lane holds at most 4 units,
    // preferring 3-4 units per lane (enough bytes in flight per wavefront, registers under 128).
    const int chunks = (K / kUnit + 63) / 64;  // 1024-element spans per row
    int wv = 1;
    while (wv < 16 && (chunks + wv - 1) / wv > 4) wv *= 2;
    const int u = (chunks + wv - 1) / wv;
    switch (u) {
        case 1: return launch_gu<G, 1, BITS>(X, rows, K, wv, Xq, scale, stream);
        case 2: return launch_gu<G, 2, BITS>(X, rows, K, wv, Xq, scale, stream);
        case 3: return launch_gu<G, 3, BITS>(X, rows, K, wv, Xq, scale, stream);
        default: return launch_gu<G, 4, BITS>(X, rows, K, wv, Xq, scale, stream);
    }
}

template <int BITS>
hipError_t launch_bits(const void *X, int64_t rows, int64_t K, int group, void *Xq, float *scale, hipStream_t stream)
{
    switch (group) {
        case 4: return launch_g<4, BITS>(X, rows, (int)K, Xq, scale, stream);
        case 16: return launch_g<16, BITS>(X, rows, (int)K, Xq, scale, stream);
        case 64: return launch_g<64, BITS>(X, rows, (int)K, Xq, scale, stream);
        case 256: return launch_g<256, BITS>(X, rows, (int)K, Xq, scale, stream);
        case 1024: return launch_1024<BITS>(X, rows, (int)K, Xq, scale, stream);
        default: return hipErrorInvalidValue;
    }
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
