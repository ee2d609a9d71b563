// W8A8 variant of kernel B of libconvrot (the paper's W8A8 rows, Sec. 5, Tables 5-2 and 5-4): the same
// layer with 8-bit codes on both operands, int8 in [-127, 127], int32 accumulation, exact: |acc| <= 127^2 K < 2^31 for
// K <= 65536.
//
// A stage is 64 codes of K: the panel layout of the operands (panel_layout.h) keeps 16 rows of it in one contiguous
// kilobyte and pads the last one with zero codes.  A 16-byte fragment read from LDS is an operand of
// v_mfma_i32_16x16x64_i8 as it stands.  The kernel is gemm_tiled.h.
#include "gemm_plan.h"
#include "gemm_small.h"
#include "gemm_tiled.h"

#include "convrot_internal.h"
#include "panel_layout.h"

namespace convrot {

namespace {

using gemm::v4i;

struct Codes8 {
    typedef v4i Op;
    typedef v4i Acc;
    static constexpr int kRowBytes = panel::kRowBytes;
    static constexpr uint32_t kStageStride = panel::kBytes;

    static constexpr int kGroupRows = panel::kRows, kGroupPieces = 1;

    static __device__ __forceinline__ int stages(int K) { return (K + panel::kRowBytes - 1) / panel::kRowBytes; }

    template <int>
    static __device__ __forceinline__ uint32_t piece_place(int g, int) { return g * panel::kBytes; }
    // Lane l fills 16-byte slot l % 4 of row l / 4 of the panel in LDS, where the swizzle keeps piece slot ^ swz(row).
    static __device__ __forceinline__ uint32_t lane_offset(int lane) { return (lane / 4) * panel::kRowBytes + ((lane % 4) ^ gemm::swz(lane / 4)) * 16; }

    struct Reader {      // lane l holds piece piece_of(l / 16) of row row_of(l % 16, odd) of the pair's 32
        uint32_t a[2][2];     // as in gemm_w4a4.hip
        __device__ __forceinline__ Reader(int lane, int, int x_row, int w_row)
        {
            const int c = gemm::piece_of(lane >> 4);
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int odd = 0; odd < 2; ++odd) {
                    const int r = gemm::row_of(lane & 15, odd);
                    a[o][odd] = (r + (o ? w_row : x_row)) * panel::kRowBytes + ((c ^ gemm::swz(r & 15)) << 4);
                }
        }
        __device__ __forceinline__ void advance(uint32_t bytes)
        {
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int odd = 0; odd < 2; ++odd) {
                    a[o][odd] += bytes;
                    gemm::keep(a[o][odd]);
                }
        }
        template <int o, int f>
        __device__ __forceinline__ Op read(const uint8_t *lds) const
        {
            return *reinterpret_cast<const v4i *>(lds + a[o][f % 2] + f / 2 * 32 * panel::kRowBytes);
        }
    };
    static __device__ __forceinline__ void mma(Acc &c, const Op &x, const Op &w) { c = __builtin_amdgcn_mfma_i32_16x16x64_i8(x, w, c, 0, 0, 0); }
};

hipError_t launch_plan(gemm::Plan plan, const gemm::Operands &o)
{
    using gemm::Plan;
    using gemm::Tile;
    if (plan == Plan::kTile128x192 && gemm::deep_ring(gemm::tiles_of(o.M, o.N, 128, 192), panel::k_panels(o.K)))
        return gemm::launch_tiled<Codes8, Tile<2, 2, 2, 3, 4, 1, 8>>(o);
    if (gemm::rows_of_48<8>(plan, o.M, o.N, panel::k_panels(o.K))) return gemm::launch_small<gemm::Small8, 3, 2, 8, 2>(o);
    if (plan == Plan::kTile128x128 && gemm::four_wavefronts_8(gemm::tiles_of(o.M, o.N, 128, 128), panel::k_panels(o.K)))
        return gemm::launch_tiled<Codes8, Tile<2, 2, 2, 2, 4, 2, 8>>(o);
    switch (plan) {
        case Plan::kTile192x192: return gemm::launch_tiled<Codes8, Tile<2, 2, 3, 3, 3, 2, 8>>(o);
        case Plan::kTile256x128: return gemm::launch_tiled<Codes8, Tile<2, 2, 4, 2, 3, 2, 6>>(o);
        case Plan::kTile128x128: return gemm::launch_tiled<Codes8, Tile<4, 2, 1, 2, 4, 4, 8>>(o);
        case Plan::kTile64x64: return gemm::launch_tiled<Codes8, Tile<2, 2, 1, 1, 4, 4, 8>>(o);
        case Plan::kSplit32x64: return gemm::launch_small<gemm::Small8, 2, 4, 8, 2>(o);
        case Plan::kSplit32x32: return gemm::launch_small<gemm::Small8, 2, 2, 4, 3>(o);
        case Plan::kSplit16x32: return gemm::launch_small<gemm::Small8, 1, 2, 8, 4>(o);
        case Plan::kSplit16x16: return gemm::launch_small<gemm::Small8, 1, 1, 16, 4>(o);
        case Plan::kTile256x256: return gemm::launch_tiled<Codes8, Tile<2, 4, 4, 2, 3, 2, 0>>(o);
        case Plan::kTile128x192: return gemm::launch_tiled<Codes8, Tile<2, 2, 2, 3, 3, 2, 8>>(o);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_gemm_w8a8(const void *Xq, const float *x_scale, const void *Wq, const float *w_scale,
                            const void *bias_bf16, int64_t M, int64_t N, int64_t K, void *Y_bf16,
                            int32_t *acc_i32, hipStream_t stream)
{
    if (M == 0 || N == 0) return hipSuccess;
    const gemm::Plan plan = gemm::choose<8>(M, N, K);
    const gemm::Store store = gemm::store_kind<8>(plan, M, N, K, reinterpret_cast<uintptr_t>(Y_bf16));
    return launch_plan(plan, gemm::Operands{Xq, x_scale, Wq, w_scale, bias_bf16, (int)M, (int)N, (int)K, Y_bf16, acc_i32, stream, store});
}

}  // namespace convrot
