// The whole forward of a layer on a few rows in one launch: rotate, quantise, multiply, dequantise.
//
// With so few rows the rotate+quantise kernel is one launch's latency and nothing else, and the GEMM waits for it.  Here every
// block rotates and quantises all M rows for itself, into LDS, while the first stages of its share of W are on their way into
// registers, and goes on as gemm_small.h does, X fragments from LDS.  The rows' work is repeated by every block (about 170
// vector instructions for 1024 elements, shared by its eight wavefronts), which is what limits the sizes (forward_in_one).
// The first block also writes the codes and the scales to the workspace, where a caller may look for them.
//
// More rows go in tiles of up to sixteen, a stretch of 1024 elements for each of sixteen wavefronts (forward_in_row_tiles), which keeps the chain of one
// pass through load, rotation, codes and product; what bounds such a call is the launch and that chain: M256 x N1024 x K1024 5.5 us on the device as two
// launches and as one, 8.9 and 5.1 us as called.  The sixteen share K eight ways and the columns two ways, so that K = 1024 (eight stages) has work for
// all of them; the columns' and the partial tiles' LDS is one.  At 128 columns a wavefront requests two stages ahead: four do not fit 128 registers (389 x 437 x 1056 6.4 / 11.2 us).
#pragma once
#include "convrot_internal.h"
#include "gemm_small.h"
#include "rotate_quantise.h"

namespace convrot {

// The launches for 8-bit codes of g >= 256 (lanes8.hip).
hipError_t forward_small_lanes8(const gemm::Operands &o, int group, void *Xq, float *x_scale);

namespace {

constexpr int kWaves = 8;       // that share the stages of K

// One item = up to 64 units (1024 elements) of one row, the work of one wavefront; a wavefront has at most I of them.  CW = 1: one tile of all M
// rows; CW = 2: tiles of tile_rows rows, tiles_m of them side by side, and two groups of wavefronts that share a block's columns.
template <int BITS, int G, int WF, int I, int CW>
__global__ __launch_bounds__(64 * kWaves * CW) void forward_small_kernel(const uint16_t *__restrict__ X, const uint8_t *__restrict__ Wq,
                                                                    const float *__restrict__ w_scale, const uint16_t *__restrict__ bias,
                                                                    int M, int N, int K, uint16_t *__restrict__ Y,
                                                                    uint8_t *__restrict__ Xq, float *__restrict__ x_scale, int per_xcd,
                                                                    int tile_rows, int tiles_m, uint32_t by_tiles_m)
{
    using C = std::conditional_t<BITS == 4, gemm::Small4, gemm::Small8>;
    constexpr int S = kWaves, kAll = S * CW, PD = WF == 8 ? 2 : BITS == 4 ? 4 : 6;
    constexpr int WC = WF / CW;      // 16-column fragments of a wavefront
    constexpr int kStageUnits = BITS == 4 ? e2m3::kUnitsPerStage : panel::kRowBytes / kUnit;
    constexpr int kMaxRowStages = I * kAll * (64 / kStageUnits);            // rows x stages
    constexpr int kRowStageBytes = BITS == 4 ? e2m3::kARowBytes + e2m3::kBRowBytes : panel::kRowBytes;
    // Bytes between the stages of 8-bit codes.  Lanes of neighbouring columns write neighbouring stages, M * 64 bytes apart, which are the same
    // banks; an odd multiple of 16 bytes apart they are not (M2 x N750 x K6144 at g = 64 5.95 -> 5.81 us, M4 x N3072 x K2816 5.81 -> 5.63, M1 x N1000 x K12288 at
    // g = 256 8.71 -> 8.55).  With g <= 16 four lanes write a stage (1 % slower so), with 4 bits two (no difference).
    constexpr int kPad = BITS == 8 && G >= 64 ? 16 : 0;
    __shared__ __attribute__((aligned(16))) uint8_t codes[kMaxRowStages * (kRowStageBytes + kPad)];
    using It = Item<G>;
    // Columns on their way between lanes, and after the last barrier but one the partial tiles: in one place where they would not both fit.
    constexpr int kPart = S * WF * gemm::kTileBytes, kColumns = I * kAll * It::kBytes;
    __shared__ __attribute__((aligned(16))) uint8_t columns[CW == 1 || kColumns > kPart ? kColumns : kPart];
    __shared__ __attribute__((aligned(16))) uint8_t own_part[CW == 1 ? kPart : 16];
    uint8_t *const part = CW == 1 ? own_part : columns;
    __shared__ float item_max[I * kAll], row_scale[16];

    // as tile_of_block (gemm_plan.h): each XCD has one contiguous range of the tiles
    const int turn = (int)(blockIdx.x / gemm::kNumXcd), id = (int)(blockIdx.x % gemm::kNumXcd) * per_xcd + turn;
    const int tn = CW == 1 ? id : gemm::divide(id, tiles_m, by_tiles_m), n0 = tn * 16 * WF;      // (the row tiles of the same columns side by side)
    if (turn >= per_xcd || n0 >= N) return;
    const int m0 = CW == 1 ? 0 : (id - tn * tiles_m) * tile_rows, R = CW == 1 ? M : min(tile_rows, M - m0);       // the block's rows
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KS = C::stages(K), units = K / kUnit, spans = (units + 63) / 64, items = R * spans;
    const int ks = wave % S, c0 = wave / S * WC;         // first stage of K, first column fragment

    // ---- X first, then W: the rotation must not wait for W
    u32x4 raw[I][2];
#pragma unroll
    for (int i = 0; i < I; ++i) {
        const int item = min(wave + kAll * i, items - 1), row = item / spans, span = item - row * spans;
        It::load(X + (m0 + row) * (int64_t)K, span * 64, units, lane, raw[i]);
    }
    C w[WC];
#pragma unroll
    for (int j = 0; j < WC; ++j) w[j].init(Wq, tn * WF + c0 + j, N, KS, lane);
    typename C::Frag fw[PD][WC];
    auto fetch = [&](int b, int s) {
#pragma unroll
        for (int j = 0; j < WC; ++j) fw[b][j] = w[j].load(s);
    };
#pragma unroll
    for (int p = 0; p < PD; ++p)
        if (ks + p * S < KS) fetch(p, ks + p * S);

    // ---- rotate; row maxima through LDS
    const Rotation<G> rot(lane);
    float v[I][kUnit];
    auto rotate = [&](int i) { It::rotate(rot, raw[i], columns + (wave + kAll * i) * It::kBytes, lane, v[i]); };
    auto maximum = [&](int i) {
        const int item = wave + kAll * i;
        float m = 0.0f;
#pragma unroll
        for (int e = 0; e < kUnit; ++e) m = fmaxf(m, fabsf(v[i][e]));
        m = item % spans * 64 + It::unit(lane) < units ? m : 0.0f;
        m = max_of_lanes<32>(m);
        if (lane == 0) item_max[item] = m;
    };
    // A wavefront with all its items: no branch between their chains of MFMAs (M4 x N3072 x K3072 at g = 256 and 8 bits, graph: 5.93 -> 5.65 us).
    // The others rotate what they have; chains of repeated items would cost M1 x N9216 x K3072 1 us of 6.4.
    if (I > 1 && wave + kAll * (I - 1) < items) {
#pragma unroll
        for (int i = 0; i < I; ++i) rotate(i);
#pragma unroll
        for (int i = 0; i < I; ++i) maximum(i);
    } else {
#pragma unroll
        for (int i = 0; i < I; ++i) {
            if (wave + kAll * i >= items) break;
            rotate(i);
            maximum(i);
        }
    }
    __syncthreads();

    // ---- codes: to LDS, [stage][row] with a row's quarters of a stage side by side (4 bits: the 16-byte parts of all
    // rows and stages, then the 8-byte parts), and from the first block to memory
    uint8_t *const bpart = codes + KS * R * e2m3::kARowBytes;
#pragma unroll
    for (int i = 0; i < I; ++i) {
        const int item = wave + kAll * i;
        if (item >= items) break;
        const int row = item / spans, span = item - row * spans;
        float amax = 0.0f;
        for (int j = 0; j < spans; ++j) amax = fmaxf(amax, item_max[row * spans + j]);
        const Quantiser q(amax, group_norm<G>(), BITS == 4 ? 7.0f : 127.0f);
        if (span == 0 && lane == 0) {
            row_scale[row] = q.s;
            if (tn == 0) x_scale[m0 + row] = q.s;
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
            store(codes + (s * R + row) * e2m3::kARowBytes + c * 16, bpart + (s * R + row) * e2m3::kBRowBytes + c * 8);
            const int m = m0 + row;
            uint8_t *const block = Xq + ((int64_t)(m / e2m3::kRows) * KS + s) * e2m3::kBlockBytes;
            if (tn == 0) store(block + e2m3::a_offset(m % e2m3::kRows, c), block + e2m3::b_offset(m % e2m3::kRows, c));
        } else {
            u32x4 o = codes8(q, as_vector(v[i]));
            if (s >= KS) continue;
            if (unit >= units) o = u32x4{0, 0, 0, 0};        // K padding
            const int c = unit % kStageUnits;
            *reinterpret_cast<u32x4 *>(codes + (s * R + row) * panel::kRowBytes + s * kPad + c * 16) = o;
            const int m = m0 + row;
            if (tn == 0) *reinterpret_cast<u32x4 *>(Xq + ((int64_t)(m / panel::kRows) * KS + s) * panel::kBytes + m % panel::kRows * panel::kRowBytes + c * 16) = o;
        }
    }
    __syncthreads();

    // ---- the product, as in gemm_small_kernel; lanes of rows past the last repeat the last row, whose results nobody stores
    const int xrow = min(lane & 15, R - 1), quarter = lane >> 4;
    typename C::Acc acc[WC];
#pragma unroll
    for (int j = 0; j < WC; ++j) acc[j] = {0, 0, 0, 0};
    auto multiply = [&](int b, int s) {
        typename C::Frag x;
        if constexpr (BITS == 4) {
            x.a = *reinterpret_cast<const gemm::v4i *>(codes + (s * R + xrow) * e2m3::kARowBytes + quarter * 16);
            x.b = *reinterpret_cast<const gemm::v2i *>(bpart + (s * R + xrow) * e2m3::kBRowBytes + quarter * 8);
        } else {
            x.a = *reinterpret_cast<const gemm::v4i *>(codes + (s * R + xrow) * panel::kRowBytes + s * kPad + quarter * 16);
        }
#pragma unroll
        for (int j = 0; j < WC; ++j) C::mma(acc[j], fw[b][j], x);
    };
    for (int s = ks; s < KS; s += PD * S) {
#pragma unroll
        for (int p = 0; p < PD; ++p) {
            if (s + p * S < KS) {
                multiply(p, s + p * S);
                if (s + (p + PD) * S < KS) fetch(p, s + (p + PD) * S);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < WC; ++j)
        *reinterpret_cast<typename C::Acc *>(part + (ks * WF + c0 + j) * gemm::kTileBytes + (lane >> 4) * gemm::kSlabBytes + (lane & 15) * 16) = acc[j];
    __syncthreads();
    gemm::sum_and_store<C, false, 1, WF, S>(part, tid, m0, n0, m0 + R, N, [&](int m) { return row_scale[m - m0]; }, w_scale, bias, Y, nullptr);
}

template <int BITS, int G>
hipError_t launch_small_rows(const gemm::Operands &o, void *Xq, float *x_scale)
{
    auto go = [&](auto kernel, int wf, int threads, int rows) {
        const int tiles_m = (o.M + rows - 1) / rows, tiles = (o.N + 16 * wf - 1) / (16 * wf) * tiles_m, per_xcd = (tiles + gemm::kNumXcd - 1) / gemm::kNumXcd;
        hipLaunchKernelGGL(kernel, dim3(per_xcd * gemm::kNumXcd), dim3(threads), 0, o.stream, (const uint16_t *)o.Xq, (const uint8_t *)o.Wq, o.w_scale,
                           (const uint16_t *)o.bias, o.M, o.N, o.K, (uint16_t *)o.Y, (uint8_t *)Xq, x_scale, per_xcd, rows, tiles_m, gemm::reciprocal(tiles_m));
        return hipGetLastError();
    };
    if (gemm::forward_in_one(o.M, o.N, o.K)) {
        const int items = (int)gemm::row_items(o.M, o.K);
        auto width = [&](auto WF) {
            constexpr int wf = decltype(WF)::value;
            return items <= kWaves ? go(forward_small_kernel<BITS, G, wf, 1, 1>, wf, 64 * kWaves, o.M) : go(forward_small_kernel<BITS, G, wf, 2, 1>, wf, 64 * kWaves, o.M);
        };
        if (items > 2 * kWaves || o.M > 16) return hipErrorInvalidValue;      // forward_in_one names no such shape
        switch (gemm::forward_in_one_columns(o.N)) {
            case 16: return width(std::integral_constant<int, 1>{});
            case 32: return width(std::integral_constant<int, 2>{});
            case 48: return width(std::integral_constant<int, 3>{});
            default: return width(std::integral_constant<int, 4>{});
        }
    }
    const gemm::RowTiles t = gemm::forward_row_tiles(o.M, o.N, o.K);
    if (gemm::row_items(t.rows, o.K) > 2 * kWaves || t.rows > 16) return hipErrorInvalidValue;      // forward_in_row_tiles names no such shape
    auto width = [&](auto WF) {
        constexpr int wf = decltype(WF)::value;
        return go(forward_small_kernel<BITS, G, wf, 1, 2>, wf, 2 * 64 * kWaves, t.rows);
    };
    switch (t.columns) {
        case 32: return width(std::integral_constant<int, 2>{});
        case 64: return width(std::integral_constant<int, 4>{});
        default: return width(std::integral_constant<int, 8>{});
    }
}

}  // namespace

}  // namespace convrot
