// The GEMM of libconvrot for products that the tiles of gemm_tiled.h cannot fill the chip with: few tokens, narrow
// layers.  Same operands, same exact accumulation, same dequantisation.
//
// Such a product is bound by latency: the tiled kernel's blocks walk K one stage at a time (0.15-0.6 us each) and only a
// few of the 256 compute units have a block.  Here a block owns one small tile (16 XF x 16 WF) of the output and its
// S wavefronts split K between them: wavefront w takes stages w, w + S, ... of the whole tile, straight from memory
// into registers in the MFMA's operand shape (no LDS, no barrier, PD stages requested ahead), so that the tile's
// operand bytes are in flight at once and the serial chain is K / S long.  The S partial tiles meet in LDS once, at the
// end: sums of integers, exact in any order.  Measured against the 256 x 128 tile, us, 4 / 8 bits: M1 x N9216 x K3072
// 14.1 -> 4.9 / 19.3 -> 6.3; M256 x N1024 x K1024 8.2 -> 3.6 / 9.7 -> 4.0; M32 x N3072 x K15360 71 -> 10 / 124 -> 13.
// An operand byte is loaded once per tile that needs it and shared by nobody (18 TB/s over the chip, whatever the
// tile), so past a few tiles per compute unit the LDS-sharing tiles of gemm_tiled.h move less and win (gemm_plan.h).
//
// `C` (Small4 / Small8) says what a lane holds of 16 rows x one K stage: lane l has row l % 16 and quarter l / 16 of the
// stage, so that the lanes of a load cover whole contiguous lines; one MFMA per 16 x 16 tile and stage.
#pragma once
#include "e2m3_layout.h"
#include "gemm_common.h"
#include "gemm_plan.h"
#include "panel_layout.h"

namespace convrot {
namespace gemm {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v8i __attribute__((ext_vector_type(8)));

struct Small4 {   // stage of 128 codes: half of a 3 KB block (e2m3_layout.h); quarter = one chunk of 32 codes
    struct Frag { v4i a; v2i b; };
    typedef v4f Acc;
    static __device__ __forceinline__ int stages(int K) { return (K + e2m3::kStageCodes - 1) / e2m3::kStageCodes; }
    uint32_t a, b;
    const uint8_t *base;
    __device__ __forceinline__ void init(const uint8_t *m, int group, int rows, int KS, int lane)
    {
        const int g = min(group, (rows - 1) / 16), r = (g & 1) * 16 + (lane & 15), c = lane >> 4;
        base = m + (int64_t)(g >> 1) * KS * e2m3::kBlockBytes;
        a = e2m3::a_offset(r, c);
        b = e2m3::b_offset(r, c);
    }
    __device__ __forceinline__ Frag load(int s) const
    {
        const uint8_t *p = base + (uint32_t)s * e2m3::kBlockBytes;
        return {*reinterpret_cast<const v4i *>(p + a), *reinterpret_cast<const v2i *>(p + b)};
    }
    static __device__ __forceinline__ v8i op(const Frag &f)
    {
        const v4i b = {f.b.x, f.b.y, 0, 0};
        return __builtin_shufflevector(f.a, b, 0, 1, 2, 3, 4, 5, -1, -1);
    }
    static __device__ __forceinline__ void mma(Acc &c, const Frag &w, const Frag &x)
    {
        c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(op(w), op(x), c, 2, 2, 0, 0, 0, 0);
    }
};

struct Small8 {   // stage of 64 codes: one 1 KB panel of 16 rows (panel_layout.h); quarter = 16 codes
    struct Frag { v4i a; };
    typedef v4i Acc;
    static __device__ __forceinline__ int stages(int K) { return (K + panel::kRowBytes - 1) / panel::kRowBytes; }
    uint32_t a;
    const uint8_t *base;
    __device__ __forceinline__ void init(const uint8_t *m, int group, int rows, int KS, int lane)
    {
        base = m + (int64_t)min(group, (rows - 1) / 16) * KS * panel::kBytes;
        a = (lane & 15) * panel::kRowBytes + (lane >> 4) * 16;
    }
    __device__ __forceinline__ Frag load(int s) const { return {*reinterpret_cast<const v4i *>(base + (uint32_t)s * panel::kBytes + a)}; }
    static __device__ __forceinline__ void mma(Acc &c, const Frag &w, const Frag &x)
    {
        c = __builtin_amdgcn_mfma_i32_16x16x64_i8(w.a, x.a, c, 0, 0, 0);
    }
};

constexpr int kSlabBytes = 16 * 16 + 16;     // four consecutive n of 16 rows, padded so that a row's quads lie in different banks
constexpr int kTileBytes = 4 * kSlabBytes;   // one 16 x 16 partial tile

// The S partial tiles of the block's wavefronts, in LDS, to Y or to the raw accumulators; x_scale(m) is the scale of row m.
template <class C, bool RAW, int XF, int WF, int S, class Scale>
__device__ __forceinline__ void sum_and_store(const uint8_t *part, int tid, int m0, int n0, int M, int N, Scale x_scale,
                                              const float *__restrict__ w_scale, const uint16_t *__restrict__ bias,
                                              uint16_t *__restrict__ Y, int32_t *__restrict__ acc_out)
{
    constexpr int TM = 16 * XF, TN = 16 * WF, kThreads = 64 * S;
    constexpr int kQuads = TM * TN / 4;
#pragma unroll
    for (int it = 0; it < (kQuads + kThreads - 1) / kThreads; ++it) {
        const int u = it * kThreads + tid;
        if (u >= kQuads) break;
        const int ml = u / (TN / 4), q = u % (TN / 4);
        const int m = m0 + ml, n = n0 + 4 * q;
        if (m >= M || n >= N) continue;
        const uint8_t *p = part + ((ml / 16) * WF + q / 4) * kTileBytes + (q % 4) * kSlabBytes + (ml % 16) * 16;
        typename C::Acc v = *reinterpret_cast<const typename C::Acc *>(p);
#pragma unroll
        for (int s = 1; s < S; ++s) v += *reinterpret_cast<const typename C::Acc *>(p + s * (XF * WF * kTileBytes));
        if constexpr (RAW) {
            int32_t *dst = acc_out + (int64_t)m * N + n;
            if ((N & 3) == 0) {
                *reinterpret_cast<int4 *>(dst) = make_int4((int)v[0], (int)v[1], (int)v[2], (int)v[3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) dst[e] = (int)v[e];
            }
        } else {
            const float sx = x_scale(m);
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int nn = min(n + e, N - 1);
                const float t = (float)v[e] * sx;
                y[e] = bias ? fmaf(t, w_scale[nn], bf16_to_f32(bias[nn])) : t * w_scale[nn];
            }
            const uint32_t lo = pack_bf16x2(y[0], y[1]), hi = pack_bf16x2(y[2], y[3]);
            uint16_t *dst = Y + (int64_t)m * N + n;
            if (n + 4 <= N) {
                *reinterpret_cast<u32x2_row *>(dst) = u32x2_row{lo, hi};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) dst[e] = (uint16_t)((e < 2 ? lo : hi) >> (16 * (e & 1)));
            }
        }
    }
}

template <class C, bool RAW, int XF, int WF, int S, int PD>
__global__ __launch_bounds__(64 * S) void gemm_small_kernel(const uint8_t *__restrict__ Xq, const uint8_t *__restrict__ Wq, int M, int N, int K,
                                                            int per_xcd, int tiles_m, int rows, int span, uint32_t by_span, uint32_t by_rows,
                                                            uint32_t by_tail, const float *__restrict__ x_scale,
                                                            const float *__restrict__ w_scale, const uint16_t *__restrict__ bias,
                                                            uint16_t *__restrict__ Y, int32_t *__restrict__ acc_out)
{
    constexpr int TM = 16 * XF, TN = 16 * WF;
    __shared__ __attribute__((aligned(16))) uint8_t part[S * XF * WF * kTileBytes];

    int tm, tn;
    if (!tile_of_block({per_xcd, tiles_m, rows, span, by_span, by_rows, by_tail}, blockIdx.x, tm, tn) || !starts_inside(tn, TN, N)) return;
    const int m0 = tm * TM, n0 = tn * TN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KS = C::stages(K);

    C x[XF], w[WF];
#pragma unroll
    for (int i = 0; i < XF; ++i) x[i].init(Xq, tm * XF + i, M, KS, lane);
#pragma unroll
    for (int j = 0; j < WF; ++j) w[j].init(Wq, tn * WF + j, N, KS, lane);

    typename C::Acc acc[XF][WF];
#pragma unroll
    for (int i = 0; i < XF; ++i)
#pragma unroll
        for (int j = 0; j < WF; ++j) acc[i][j] = {0, 0, 0, 0};

    typename C::Frag fx[PD][XF], fw[PD][WF];
    auto fetch = [&](int b, int s) {
#pragma unroll
        for (int j = 0; j < WF; ++j) fw[b][j] = w[j].load(s);
#pragma unroll
        for (int i = 0; i < XF; ++i) fx[b][i] = x[i].load(s);
    };
    auto multiply = [&](int b) {
#pragma unroll
        for (int i = 0; i < XF; ++i)
#pragma unroll
            for (int j = 0; j < WF; ++j) C::mma(acc[i][j], fw[b][j], fx[b][i]);
    };
#pragma unroll
    for (int p = 0; p < PD; ++p)
        if (wave + p * S < KS) fetch(p, wave + p * S);
    for (int s = wave; s < KS; s += PD * S) {
#pragma unroll
        for (int p = 0; p < PD; ++p) {
            if (s + p * S < KS) {
                multiply(p);
                if (s + (p + PD) * S < KS) fetch(p, s + (p + PD) * S);
            }
        }
    }

    // ---- lane l, register r of a 16 x 16 tile: m = l % 16, n = 4 (l / 16) + r: a slab is four consecutive n of the 16 rows
#pragma unroll
    for (int i = 0; i < XF; ++i)
#pragma unroll
        for (int j = 0; j < WF; ++j)
            *reinterpret_cast<typename C::Acc *>(part + ((wave * XF + i) * WF + j) * kTileBytes + (lane >> 4) * kSlabBytes + (lane & 15) * 16) = acc[i][j];
    __syncthreads();
    sum_and_store<C, RAW, XF, WF, S>(part, tid, m0, n0, M, N, [&](int m) { return x_scale[m]; }, w_scale, bias, Y, acc_out);
}

template <class C, int XF, int WF, int S, int PD>
hipError_t launch_small(const Operands &o)
{
    const int tiles_m = (o.M + 16 * XF - 1) / (16 * XF), tiles_n = (o.N + 16 * WF - 1) / (16 * WF);
    if (!launchable((int64_t)tiles_m * tiles_n, 64 * S)) return hipErrorInvalidValue;
    const TileOrder t = tile_order(tiles_m, tiles_n, 8);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(t.per_xcd * kNumXcd), dim3(64 * S), 0, o.stream, (const uint8_t *)o.Xq, (const uint8_t *)o.Wq, o.M, o.N,
                           o.K, t.per_xcd, t.tiles_m, t.rows, t.span, t.by_span, t.by_rows, t.by_tail, o.x_scale, o.w_scale,
                           (const uint16_t *)o.bias, (uint16_t *)o.Y, o.acc);
        return hipGetLastError();
    };
    return o.acc ? go(gemm_small_kernel<C, true, XF, WF, S, PD>) : go(gemm_small_kernel<C, false, XF, WF, S, PD>);
}

}  // namespace gemm
}  // namespace convrot
