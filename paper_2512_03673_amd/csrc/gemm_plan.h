// Which GEMM kernel a product takes.
//
// A launch's time is predicted for every compiled tile as
//
//   fixed + block b + max(latency c, rate K' b)        us, b = tiles of the busiest compute unit = ceil(tiles / 256),
//                                                      K' = stages of K, c = the stages one wavefront walks
//
// (`block`: prologue and epilogue of a tile; `latency`: a stage when its tile has the compute unit to itself; `rate`: a stage's
// share of a full compute unit) and the smallest prediction is taken.  The four constants of a tile are a robust fit
// to 320 launches on shapes drawn over M 1 ... 8000, N 32 ... 12288, K 64 ... 15360; on other shapes the tile taken
// costs 2 % more on average than the best of them would.
#pragma once
#include <stdint.h>

namespace convrot {
namespace gemm {

enum class Plan {
    kTile192x192,     // gemm_tiled.h
    kTile256x128,
    kTile256x128w8,   // the same tile on eight wavefronts, one block per compute unit (4-bit codes)
    kTile128x128,
    kTile64x64,
    kSplit32x64,      // gemm_small.h
    kSplit32x32,
    kSplit16x32,
    kSplit16x16,
    kCount
};

struct Cost {
    Plan plan;
    int tm, tn;
    int split;      // wavefronts that share the stages of K, or 1
    float fixed, block, latency, rate;
};

// The two large tiles.  Blocks are dealt to the 256 compute units as slots free up, so a launch lasts about as
// long as the busiest unit's share, ceil(tiles / 256) blocks of TM x TN products each; the square tile
// moves fewer operand bytes per product and takes the ties.
inline int large_tile_rows(int64_t M, int64_t N)
{
    auto work = [&](int64_t tm, int64_t tn) {
        const int64_t tiles = ((M + tm - 1) / tm) * ((N + tn - 1) / tn);
        return ((tiles + 255) / 256) * tm * tn;
    };
    return work(192, 192) <= work(256, 128) ? 192 : 256;
}

template <int BITS>
inline Plan choose(int64_t M, int64_t N, int64_t K)
{
    static_assert(BITS == 4 || BITS == 8, "code widths");
    static constexpr Cost k4[] = {
        {Plan::kTile192x192, 192, 192, 1, 3.23f, 3.28f, 0.451f, 0.3642f},
        {Plan::kTile256x128, 256, 128, 1, 3.06f, 3.15f, 0.426f, 0.3670f},
        {Plan::kTile256x128w8, 256, 128, 1, 0.0f, 5.25f, 0.377f, 0.4045f},
        {Plan::kTile128x128, 128, 128, 1, 2.69f, 2.13f, 0.266f, 0.2165f},
        {Plan::kTile64x64, 64, 64, 1, 2.47f, 0.58f, 0.153f, 0.1113f},
        {Plan::kSplit32x64, 32, 64, 8, 0.97f, 2.21f, 0.368f, 0.0958f},
        {Plan::kSplit32x32, 32, 32, 4, 2.41f, 0.43f, 0.250f, 0.0583f},
        {Plan::kSplit16x32, 16, 32, 8, 2.36f, 0.53f, 0.176f, 0.0440f},
        {Plan::kSplit16x16, 16, 16, 16, 1.90f, 0.98f, 0.445f, 0.0242f},
    };
    static constexpr Cost k8[] = {
        {Plan::kTile192x192, 192, 192, 1, 3.13f, 3.38f, 0.262f, 0.3407f},
        {Plan::kTile256x128, 256, 128, 1, 3.56f, 2.61f, 0.327f, 0.3270f},
        {Plan::kTile128x128, 128, 128, 1, 2.52f, 2.09f, 0.057f, 0.1869f},
        {Plan::kTile64x64, 64, 64, 1, 2.52f, 0.52f, 0.118f, 0.0849f},
        {Plan::kSplit32x64, 32, 64, 8, 2.06f, 1.07f, 0.246f, 0.0822f},
        {Plan::kSplit32x32, 32, 32, 4, 2.57f, 0.33f, 0.183f, 0.0539f},
        {Plan::kSplit16x32, 16, 32, 8, 2.29f, 0.42f, 0.321f, 0.0380f},
        {Plan::kSplit16x16, 16, 16, 16, 2.22f, 0.78f, 0.255f, 0.0243f},
    };
    const Plan other_large = large_tile_rows(M, N) == 192 ? Plan::kTile256x128 : Plan::kTile192x192;
    const float stages = (float)(BITS == 4 ? (K + 127) / 128 : (K + 63) / 64);
    Plan best = Plan::kCount;
    float least = 0.0f;
    auto consider = [&](const Cost &c) {
        if (c.plan == other_large) return;
        const int64_t tiles = ((M + c.tm - 1) / c.tm) * ((N + c.tn - 1) / c.tn);
        const float b = (float)((tiles + 255) / 256), chain = (float)(((int64_t)stages + c.split - 1) / c.split);
        const float alone = c.latency * chain, full = c.rate * stages * b;
        const float t = c.fixed + c.block * b + (alone > full ? alone : full);
        if (best == Plan::kCount || t < least) {
            best = c.plan;
            least = t;
        }
    };
    if constexpr (BITS == 4)
        for (const Cost &c : k4) consider(c);
    else
        for (const Cost &c : k8) consider(c);
    return best;
}

}  // namespace gemm
}  // namespace convrot
