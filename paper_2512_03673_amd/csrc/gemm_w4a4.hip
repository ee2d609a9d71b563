// Kernel B of libconvrot: W4A4 GEMM on 4-bit codes with the dequantisation fused
// (ConvRot paper Sec. 4.3: 4-bit matrix multiplication, then dequantisation).
//
// gfx950 has no 4-bit integer MFMA, but every code in [-7, 7] is an FP6 (E2M3) number, and
// v_mfma_f32_16x16x128_f8f6f4 on FP6 operands runs at twice the rate of the int8 MFMA.  Products of two
// codes (|.| <= 49) and all their partial sums (|.| <= 49 K < 2^22 for K <= 65536) are integers that
// fp32 holds exactly, so the fp32 accumulators carry the exact integer result whatever the order of
// the additions.  The codes arrive from the rotate+quantise kernel already as FP6 (e2m3_layout.h), six
// bits each, in the register image the MFMA wants: nothing is unpacked or widened here.  (On this
// chip the int8 path is held back by power, not by issue: the int8 kernel that the 4-bit layer started with ran 98 us
// on all-zero codes and 113-135 us on real ones, and a register-only loop of 16 x 16 MFMAs sustains 4.2 POP/s of int8 against
// 8.6 POP/s of FP6 on workload-like data, of 32 x 32 ones 3.5 against 7.6, gemm_tiled.h.)
//
// The operands sit in HBM as 3 KB blocks of 32 rows x 128 codes (an A plane of 32 x 64 bytes and a B plane of
// 32 x 32 bytes, both XOR-swizzled for the fragment reads), so that a K128 stage of a tile is a list of contiguous
// kilobytes, copied as they are.  A fragment (16 rows x 128 codes, 24 bytes per lane) is one ds_read_b128 from the A
// plane and one ds_read_b64 from the B plane and is an MFMA operand as read.  The kernel is gemm_tiled.h.
#include "gemm_plan.h"
#include "gemm_small.h"
#include "gemm_tiled.h"

#include "convrot_internal.h"
#include "e2m3_layout.h"

namespace convrot {

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v8i __attribute__((ext_vector_type(8)));
using gemm::v4f;
using gemm::v4i;

struct Codes4 {
    typedef v8i Op;      // 6 dwords used
    typedef v4f Acc;
    static constexpr int kRowBytes = e2m3::kARowBytes + e2m3::kBRowBytes;     // of one row per stage
    static constexpr uint32_t kStageStride = e2m3::kBlockBytes;               // from a row's stage to its next one

    static constexpr int kGroupRows = e2m3::kRows, kGroupPieces = e2m3::kBlockBytes / 1024;

    static __host__ __device__ __forceinline__ int stages(int K) { return (K + e2m3::kStageCodes - 1) / e2m3::kStageCodes; }

    // Where kilobyte `part` of the block of the tile's 32-row group g goes: kilobytes 0, 1 are the A plane (rows 0-15, 16-31),
    // kilobyte 2 the B plane.  A stage buffer holds the A parts of all the tile's rows, then the B parts.
    template <int ROWS>
    static __device__ __forceinline__ uint32_t piece_place(int g, int part)
    {
        return part < 2 ? g * e2m3::kAPlaneBytes + part * 1024 : ROWS * e2m3::kARowBytes + g * e2m3::kBPlaneBytes;
    }
    static __device__ __forceinline__ uint32_t lane_offset(int lane) { return lane * 16; }

    struct Reader {      // lane l holds chunk piece_of(l / 16) of row row_of(l % 16, odd) of the pair's 32
        uint32_t a[2][2], b[2][2];     // [operand][odd fragment]: where the lane's A part and B part of the first pair's rows of X (0), W (1) are; others are constants further on
        __device__ __forceinline__ Reader(int lane, int rows, int x_row, int w_row)
        {
            const int c = gemm::piece_of(lane >> 4);
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int odd = 0; odd < 2; ++odd) {
                    const int r = gemm::row_of(lane & 15, odd), row = (o ? w_row : x_row) + r;
                    a[o][odd] = row * e2m3::kARowBytes + ((c ^ e2m3::swz_a(r)) << 4);
                    b[o][odd] = rows * e2m3::kARowBytes + row * e2m3::kBRowBytes + ((c ^ e2m3::swz_b(r)) << 3);
                }
        }
        __device__ __forceinline__ void advance(uint32_t bytes)      // to another stage buffer
        {
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int odd = 0; odd < 2; ++odd) {
                    a[o][odd] += bytes;
                    b[o][odd] += bytes;
                    gemm::keep(a[o][odd]);
                    gemm::keep(b[o][odd]);
                }
        }
        template <int o, int f>
        __device__ __forceinline__ Op read(const uint8_t *lds) const
        {
            const v4i a = *reinterpret_cast<const v4i *>(lds + this->a[o][f % 2] + f / 2 * e2m3::kAPlaneBytes);
            const v2i b = *reinterpret_cast<const v2i *>(lds + this->b[o][f % 2] + f / 2 * e2m3::kBPlaneBytes);
            Op v = __builtin_shufflevector(a, a, 0, 1, 2, 3, -1, -1, -1, -1);
            v[4] = b.x;
            v[5] = b.y;
            return v;
        }
    };
    static __device__ __forceinline__ void mma(Acc &c, const Op &x, const Op &w)
    {
        c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(x, w, c, 2, 2, 0, 0, 0, 0);
    }
};

hipError_t launch_256x256(const gemm::Operands &o)
{
    using gemm::Tile;
    typedef Tile<2, 4, 4, 2, 3, 2, 0> Whole;
    const int64_t per_xcd = ((int64_t)((o.M + 255) / 256) * ((o.N + 255) / 256) + 7) / 8;
    switch (gemm::parts_of_last_tiles(per_xcd)) {
        case 2: return gemm::launch_cut<Codes4, Whole, Tile<4, 2, 2, 2, 3, 2, 0>>(o, (int)(per_xcd % 32));
        case 4: return gemm::launch_cut<Codes4, Whole, Tile<4, 2, 1, 2, 4, 2, 0>>(o, (int)(per_xcd % 32));
        default: return gemm::launch_tiled<Codes4, Whole>(o);
    }
}

hipError_t launch_plan(gemm::Plan plan, const gemm::Operands &o)
{
    using gemm::Plan;
    using gemm::Tile;
    if (plan == Plan::kTile192x192 && gemm::deep_ring(gemm::tiles_of(o.M, o.N, 192, 192), e2m3::stages(o.K)))
        return gemm::launch_tiled<Codes4, Tile<2, 2, 3, 3, 4, 1, 8>>(o);
    if (plan == Plan::kTile64x64 && gemm::deep_ring(gemm::tiles_of(o.M, o.N, 64, 64), e2m3::stages(o.K)))
        return gemm::launch_tiled<Codes4, Tile<2, 2, 1, 1, 4, 3, 8>>(o);
    if (gemm::rows_of_48<4>(plan, o.M, o.N, e2m3::stages(o.K))) return gemm::launch_small<gemm::Small4, 3, 2, 8, 2>(o);
    if (plan == Plan::kTile128x128 && gemm::tiles_of(o.M, o.N, 128, 128) <= 256) return gemm::launch_tiled<Codes4, Tile<4, 2, 1, 2, 4, 2, 8>>(o);
    switch (plan) {
        case Plan::kTile192x192: return gemm::launch_tiled<Codes4, Tile<2, 2, 3, 3, 2, 2, 8>>(o);
        case Plan::kTile256x128: return gemm::launch_tiled<Codes4, Tile<2, 2, 4, 2, 2, 2, 6>>(o);
        case Plan::kTile256x128w8: return gemm::launch_tiled<Codes4, Tile<4, 2, 2, 2, 3, 2, 8>>(o);
        case Plan::kTile128x128: return gemm::launch_tiled<Codes4, Tile<4, 2, 1, 2, 3, 4, 8>>(o);
        case Plan::kTile64x64: return gemm::launch_tiled<Codes4, Tile<2, 2, 1, 1, 3, 4, 8>>(o);
        case Plan::kSplit32x64: return gemm::launch_small<gemm::Small4, 2, 4, 8, 2>(o);
        case Plan::kSplit32x32: return gemm::launch_small<gemm::Small4, 2, 2, 4, 3>(o);
        case Plan::kSplit16x32: return gemm::launch_small<gemm::Small4, 1, 2, 8, 4>(o);
        case Plan::kSplit16x16: return gemm::launch_small<gemm::Small4, 1, 1, 16, 4>(o);
        case Plan::kTile256x256: return launch_256x256(o);
        case Plan::kTile128x192: return gemm::launch_tiled<Codes4, Tile<2, 3, 2, 2, 4, 2, 8>>(o);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_gemm_w4a4(const void *Xq, const float *x_scale, const void *Wq, const float *w_scale,
                            const void *bias_bf16, int64_t M, int64_t N, int64_t K, void *Y_bf16,
                            int32_t *acc_i32, hipStream_t stream)
{
    if (M == 0 || N == 0) return hipSuccess;
    const gemm::Plan plan = gemm::choose<4>(M, N, K);
    const gemm::Store store = gemm::store_kind<4>(plan, M, N, K, reinterpret_cast<uintptr_t>(Y_bf16));
    return launch_plan(plan, gemm::Operands{Xq, x_scale, Wq, w_scale, bias_bf16, (int)M, (int)N, (int)K, Y_bf16, acc_i32, stream, store});
}

}  // namespace convrot
