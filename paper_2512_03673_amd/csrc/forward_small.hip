// The whole forward of a layer on a few rows in one launch: rotate, quantise, multiply, dequantise.
//
// With so few rows the rotate+quantise kernel is one launch's latency and nothing else, and the GEMM waits for it.  Here every
// block rotates and quantises all M rows for itself, into LDS, while the first stages of its share of W are on their way into
// registers, and goes on as gemm_small.h does, X fragments from LDS.  The rows' work is repeated by every block (about 170
// vector instructions for 1024 elements, shared by its eight wavefronts), which is what limits the sizes (forward_in_one).
// The first block also writes the codes and the scales to the workspace, where a caller may look for them.
#include "convrot_internal.h"
#include "gemm_small.h"
#include "rotate_quantise.h"

namespace convrot {

namespace {

constexpr int kWaves = 8;

// One item = up to 64 units (1024 elements) of one row, the work of one wavefront; a wavefront has at most I of them.
template <int BITS, int G, int WF, int I>
__global__ __launch_bounds__(64 * kWaves) void forward_small_kernel(const uint16_t *__restrict__ X, const uint8_t *__restrict__ Wq,
                                                                    const float *__restrict__ w_scale, const uint16_t *__restrict__ bias,
                                                                    int M, int N, int K, uint16_t *__restrict__ Y,
                                                                    uint8_t *__restrict__ Xq, float *__restrict__ x_scale, int per_xcd)
{
    using C = std::conditional_t<BITS == 4, gemm::Small4, gemm::Small8>;
    constexpr int S = kWaves, PD = BITS == 4 ? 4 : 6;
    constexpr int kStageUnits = BITS == 4 ? e2m3::kUnitsPerStage : panel::kRowBytes / kUnit;
    constexpr int kMaxRowStages = I * S * (64 / kStageUnits);            // rows x stages
    constexpr int kRowStageBytes = BITS == 4 ? e2m3::kARowBytes + e2m3::kBRowBytes : panel::kRowBytes;
    // Bytes between the stages of 8-bit codes.  Lanes of neighbouring columns write neighbouring stages, M * 64 bytes apart, which are the same
    // banks; an odd multiple of 16 bytes apart they are not (M2 x N750 x K6144 at g = 64 5.95 -> 5.81 us, M4 x N3072 x K2816 5.81 -> 5.63, M1 x N1000 x K12288 at
    // g = 256 8.71 -> 8.55).  With g <= 16 four lanes write a stage (1 % slower so), with 4 bits two (no difference).
    constexpr int kPad = BITS == 8 && G >= 64 ? 16 : 0;
    __shared__ __attribute__((aligned(16))) uint8_t codes[kMaxRowStages * (kRowStageBytes + kPad)];
    __shared__ __attribute__((aligned(16))) uint8_t part[S * WF * gemm::kTileBytes];
    __shared__ float item_max[I * S], row_scale[16];

    // as tile_of_block (gemm_plan.h): each XCD has one contiguous range of the tiles
    const int turn = (int)(blockIdx.x / gemm::kNumXcd), tn = (int)(blockIdx.x % gemm::kNumXcd) * per_xcd + turn, n0 = tn * 16 * WF;
    if (turn >= per_xcd || n0 >= N) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KS = C::stages(K), units = K / kUnit, spans = (units + 63) / 64, items = M * spans;

    // ---- X first, then W: the rotation must not wait for W
    using It = Item<G>;
    __shared__ __attribute__((aligned(16))) uint8_t columns[I * S * It::kBytes];
    u32x4 raw[I][2];
#pragma unroll
    for (int i = 0; i < I; ++i) {
        const int item = min(wave + S * i, items - 1), row = item / spans, span = item - row * spans;
        It::load(X + row * (int64_t)K, span * 64, units, lane, raw[i]);
    }
    C w[WF];
#pragma unroll
    for (int j = 0; j < WF; ++j) w[j].init(Wq, tn * WF + j, N, KS, lane);
    typename C::Frag fw[PD][WF];
    auto fetch = [&](int b, int s) {
#pragma unroll
        for (int j = 0; j < WF; ++j) fw[b][j] = w[j].load(s);
    };
#pragma unroll
    for (int p = 0; p < PD; ++p)
        if (wave + p * S < KS) fetch(p, wave + p * S);

    // ---- rotate; row maxima through LDS
    const Rotation<G> rot(lane);
    float v[I][kUnit];
    auto rotate = [&](int i) { It::rotate(rot, raw[i], columns + (wave + S * i) * It::kBytes, lane, v[i]); };
    auto maximum = [&](int i) {
        const int item = wave + S * i;
        float m = 0.0f;
#pragma unroll
        for (int e = 0; e < kUnit; ++e) m = fmaxf(m, fabsf(v[i][e]));
        m = item % spans * 64 + It::unit(lane) < units ? m : 0.0f;
        m = max_of_lanes<32>(m);
        if (lane == 0) item_max[item] = m;
    };
    // A wavefront with all its items: no branch between their chains of MFMAs (M4 x N3072 x K3072 at g = 256 and 8 bits, graph: 5.93 -> 5.65 us).
    // The others rotate what they have; chains of repeated items would cost M1 x N9216 x K3072 1 us of 6.4.
    if (I > 1 && wave + S * (I - 1) < items) {
#pragma unroll
        for (int i = 0; i < I; ++i) rotate(i);
#pragma unroll
        for (int i = 0; i < I; ++i) maximum(i);
    } else {
#pragma unroll
        for (int i = 0; i < I; ++i) {
            if (wave + S * i >= items) break;
            rotate(i);
            maximum(i);
        }
    }
    __syncthreads();

    // ---- codes: to LDS, [stage][row] with a row's quarters of a stage side by side (4 bits: the 16-byte parts of all
    // rows and stages, then the 8-byte parts), and from the first block to memory
    uint8_t *const bpart = codes + KS * M * e2m3::kARowBytes;
#pragma unroll
    for (int i = 0; i < I; ++i) {
        const int item = wave + S * i;
        if (item >= items) break;
        const int row = item / spans, span = item - row * spans;
        float amax = 0.0f;
        for (int j = 0; j < spans; ++j) amax = fmaxf(amax, item_max[row * spans + j]);
        const Quantiser q(amax, group_norm<G>(), BITS == 4 ? 7.0f : 127.0f);
        if (span == 0 && lane == 0) {
            row_scale[row] = q.s;
            if (tn == 0) x_scale[row] = q.s;
        }
        const int unit = span * 64 + It::out_unit(lane), s = unit / kStageUnits;
        if constexpr (BITS == 4) {
            const v6u packed = codes4(q, false, as_vector(v[i]), as_vector(v[i]));
            if (s >= KS) continue;
            const bool pad = unit >= units;                  // K padding: zero codes
            const uint32_t w0 = pad ? 0 : packed[0], w1 = pad ? 0 : packed[1], w2 = pad ? 0 : packed[2];
            const int c = unit % kStageUnits >> 1;
            auto store = [&](uint8_t *a, uint8_t *b) {
                if ((unit & 1) == 0) {
                    *reinterpret_cast<u32x2 *>(a) = u32x2{w0, w1};
                    *reinterpret_cast<uint32_t *>(a + 8) = w2;
                } else {
                    *reinterpret_cast<uint32_t *>(a + 12) = w0;
                    *reinterpret_cast<u32x2 *>(b) = u32x2{w1, w2};
                }
            };
            store(codes + (s * M + row) * e2m3::kARowBytes + c * 16, bpart + (s * M + row) * e2m3::kBRowBytes + c * 8);
            if (tn == 0) store(Xq + s * e2m3::kBlockBytes + e2m3::a_offset(row, c), Xq + s * e2m3::kBlockBytes + e2m3::b_offset(row, c));
        } else {
            u32x4 o = codes8(q, as_vector(v[i]));
            if (s >= KS) continue;
            if (unit >= units) o = u32x4{0, 0, 0, 0};        // K padding
            const int c = unit % kStageUnits;
            *reinterpret_cast<u32x4 *>(codes + (s * M + row) * panel::kRowBytes + s * kPad + c * 16) = o;
            if (tn == 0) *reinterpret_cast<u32x4 *>(Xq + s * panel::kBytes + row * panel::kRowBytes + c * 16) = o;
        }
    }
    __syncthreads();

    // ---- the product, as in gemm_small_kernel; lanes of rows past M repeat the last row, whose results nobody stores
    const int xrow = min(lane & 15, M - 1), quarter = lane >> 4;
    typename C::Acc acc[WF];
#pragma unroll
    for (int j = 0; j < WF; ++j) acc[j] = {0, 0, 0, 0};
    auto multiply = [&](int b, int s) {
        typename C::Frag x;
        if constexpr (BITS == 4) {
            x.a = *reinterpret_cast<const gemm::v4i *>(codes + (s * M + xrow) * e2m3::kARowBytes + quarter * 16);
            x.b = *reinterpret_cast<const gemm::v2i *>(bpart + (s * M + xrow) * e2m3::kBRowBytes + quarter * 8);
        } else {
            x.a = *reinterpret_cast<const gemm::v4i *>(codes + (s * M + xrow) * panel::kRowBytes + s * kPad + quarter * 16);
        }
#pragma unroll
        for (int j = 0; j < WF; ++j) C::mma(acc[j], fw[b][j], x);
    };
    for (int s = wave; s < KS; s += PD * S) {
#pragma unroll
        for (int p = 0; p < PD; ++p) {
            if (s + p * S < KS) {
                multiply(p, s + p * S);
                if (s + (p + PD) * S < KS) fetch(p, s + (p + PD) * S);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < WF; ++j)
        *reinterpret_cast<typename C::Acc *>(part + (wave * WF + j) * gemm::kTileBytes + (lane >> 4) * gemm::kSlabBytes + (lane & 15) * 16) = acc[j];
    __syncthreads();
    gemm::sum_and_store<C, false, 1, WF, S>(part, tid, 0, n0, M, N, [&](int m) { return row_scale[m]; }, w_scale, bias, Y, nullptr);
}

template <int BITS, int G>
hipError_t launch(const gemm::Operands &o, void *Xq, float *x_scale)
{
    const int items = (int)gemm::row_items(o.M, o.K);
    auto go = [&](auto kernel, int wf) {
        const int tiles_n = (o.N + 16 * wf - 1) / (16 * wf), per_xcd = (tiles_n + gemm::kNumXcd - 1) / gemm::kNumXcd;
        hipLaunchKernelGGL(kernel, dim3(per_xcd * gemm::kNumXcd), dim3(64 * kWaves), 0, o.stream, (const uint16_t *)o.Xq, (const uint8_t *)o.Wq, o.w_scale,
                           (const uint16_t *)o.bias, o.M, o.N, o.K, (uint16_t *)o.Y, (uint8_t *)Xq, x_scale, per_xcd);
        return hipGetLastError();
    };
    auto width = [&](auto WF) {
        constexpr int wf = decltype(WF)::value;
        return items <= kWaves ? go(forward_small_kernel<BITS, G, wf, 1>, wf) : go(forward_small_kernel<BITS, G, wf, 2>, wf);
    };
    if (items > 2 * kWaves || o.M > 16) return hipErrorInvalidValue;      // forward_in_one names no such shape
    switch (gemm::forward_in_one_columns(o.N)) {
        case 16: return width(std::integral_constant<int, 1>{});
        case 32: return width(std::integral_constant<int, 2>{});
        case 48: return width(std::integral_constant<int, 3>{});
        default: return width(std::integral_constant<int, 4>{});
    }
}

template <int BITS>
hipError_t launch_group(const gemm::Operands &o, int group, void *Xq, float *x_scale)
{
    switch (group) {
        case 4: return launch<BITS, 4>(o, Xq, x_scale);
        case 16: return launch<BITS, 16>(o, Xq, x_scale);
        case 64: return launch<BITS, 64>(o, Xq, x_scale);
        case 256: return launch<BITS, 256>(o, Xq, x_scale);
        case 1024: return launch<BITS, 1024>(o, Xq, x_scale);
        default: return hipErrorInvalidValue;
    }
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
