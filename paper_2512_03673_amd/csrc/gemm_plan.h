// Which GEMM kernel a product takes.
//
// A launch's time is predicted for every compiled tile and the smallest prediction is taken.  b = tiles of the busiest
// compute unit = ceil(tiles / 256), K' = stages of K; us:
//
//   small tiles, many to a compute unit   fixed + block b + max(latency c, rate K' b), c = the stages one wavefront walks
//   tiles that share a unit two by two    fixed + block b + K' (pair floor(b / 2) + lone (b mod 2))
//   tiles that have a unit to themselves  fixed + b (block + rate K' (idle + (1 - idle) fill)), fill = share of the b rounds'
//                                         places that have a tile: the chip is limited by power, and a unit that has
//                                         no tile leaves its share to the others
//
// (`block`: prologue and epilogue of a tile; `latency`, `lone`: a stage of a tile that has the unit to itself; `rate`, `pair`: a
// stage of a full unit.)  The constants are robust fits: of the first kind to 320 launches on shapes drawn over M 1 ... 8000,
// N 32 ... 12288, K 64 ... 15360, of the other two to 230 over M 256 ... 16896, N 512 ... 12288, K 256 ... 15360 with at least
// 1.2e10 products, the large 4-bit tiles also to 120 such with operands that change from launch to launch (128 x 192: to 220
// with M 64 ... 8000 and 3e9 to 8e10 products).  On the larger shapes the tile taken costs 0.5 % more on average than the best of
// them would, on the others 1 to 2 %.  All fits but those of the large 4-bit tiles are thus of operands that the Infinity Cache holds.
// The fits are of kernels whose output went through the caches.  With every output past them the tiles' times fell together: over
// 150 shapes (4 bits) and 130 (8 bits) of 1e9 to 6.4e11 products with operands that change from launch to launch the
// tile taken costs 1.3 and 1.9 % more than the best, with constants fitted again to these 1.5 and 1.7 %.  (Tiles against each other;
// the stores themselves: store_kind.)
//
// No constant has been fitted again since the way to the first MFMA was halved (gemm_tiled.h), since deep_ring gives the 4-bit 64 x 64
// tile four stages, since the MFMAs are 16 x 16, or since 128 x 128 tiles are eight wavefronts and 4-bit 128 x 192 ones six; the 8-bit 128 x 192 tile is predicted with its three
// stages as well.  What that costs, every tile timed against the one taken, operands changing, kernels as of d223d18, over products of 5e9 to 2e11 (M 16 ... 16000, N 64 ... 12288,
// K 64 ... 15360): 4 bits, 250 of them, 0.9 % on average, 19 % at most (M2550 x N4544 x K896 15.4 / 13.15 with 256 x 128, M771 x N4800 x K1632 9.65 / 8.2 with 128 x 192,
// M10694 x N5683 x K352 47.9 / 43.0 with 128 x 128), 8 bits, 200, 1.8 and 24 % (M2427 x N12032 x K352 26.6 / 21.4 with 256 x 128, M13413 x N441 x K1632 22.5 / 19.0 with 128 x 128).
// At 4 bits it is 128 x 128, whose constants are of four wavefronts, in half of the products that lose 2 % and more; at 8 bits 64 x 64 where K split is better in a third of them.
#pragma once
#include <stdint.h>

namespace convrot {
namespace gemm {

constexpr int kNumXcd = 8;

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
    kTile256x256,     // gemm_tiled.h: eight wavefronts, one block per compute unit
    kTile128x192,     // gemm_tiled.h
    kCount
};

// Whether HIP can launch so many blocks: a grid has fewer than 2^32 threads.  (Blocks are dealt in eights: up to seven more.)
inline bool launchable(int64_t blocks, int threads) { return blocks + 7 < ((int64_t)1 << 32) / threads; }

// Stretches of up to 1024 elements in M rows, the unit of work of the one-launch forward (forward_small.hip).
inline int64_t row_items(int64_t M, int64_t K) { return M * ((K + 1023) / 1024); }

// Columns of a block of that forward: as few as leave every compute unit at most one block, which rotates all rows first (of up to 16384:
// forward_in_one).  us, 32 columns / this: M1 x N9216 x K3072 7.1 / 6.15 (64 columns 6.45), M2 x N9216 x K3072 at 8 bits 9.2 / 8.2,
// M1 x N12288 x K3072 7.5 / 7.1, M2 x N12010 x K1024 at 8 bits 6.55 / 5.6; over 110 drawn shapes 0.1 % slower than the best width.
inline int forward_in_one_columns(int64_t N) { return N <= 16 * 256 ? 16 : N <= 32 * 256 ? 32 : N <= 48 * 256 ? 48 : 64; }

// Whether a forward takes that one launch, in which every block repeats the rows' rotation, or two.  Two launches cost 1 us (short
// rows) to 4 us (long ones) more and the rotation 0.15 us an item for each block (of 16 or 32 columns) of a compute unit.  Over 110 drawn shapes
// (M 1-16, N 64-40000, K 64-15360) the line drawn here gives 0.5 to 5 us, us two / one: M1 x N9216 x K3072 10.8 / 7.3,
// M1 x N3072 x K12288 12.7 / 9.0, M4 x N3072 x K3072 8.7 / 6.1, M8 x N608 x K1024 6.3 / 5.2, M1 x N394 x K128 5.3 / 3.8; past it
// M12 x N9068 x K256 5.6 / 8.7, M14 x N1933 x K1088 6.0 / 7.0, M2 x N18018 x K192 5.8 / 6.9.  (All of blocks of 16 or 32 columns, and the line still counts
// these: it has not been drawn again for N of 8193 and more, whose blocks are fewer and wider now.)  What is past it is asked for by
// forward_in_row_tiles, whose sixteen wavefronts take these three in one launch too, 7.4 / 4.75, 7.4 / 5.1 and 7.4 / 4.7 as called, and
// M8 x N9216 x K1024, 7.4 / 4.95.
inline bool forward_in_one(int64_t M, int64_t N, int64_t K)
{
    const int64_t items = row_items(M, K), columns = N <= 4096 ? 16 : 32, blocks = (N + columns - 1) / columns;
    if (blocks > 512) return false;
    return items * (blocks > 256 ? blocks : 256) <= 8 * 256 || (M <= 4 && items <= 16 && blocks <= 256);
}

// The one-launch forward of more rows: tiles of as many rows as sixteen wavefronts rotate at once (a stretch of 1024 elements each), whose
// rotation every block of the same rows repeats, and as few columns as leave every compute unit at most one block.
struct RowTiles {
    int rows, columns;      // of a block
};
inline RowTiles forward_row_tiles(int64_t M, int64_t N, int64_t K)
{
    const int64_t most = 16 / row_items(1, K), tiles = (M + most - 1) / most, rows = (M + tiles - 1) / tiles;
    return {(int)rows, tiles * ((N + 31) / 32) <= 256 ? 32 : tiles * ((N + 63) / 64) <= 256 ? 64 : 128};
}

// Whether a forward that is called (not recorded into a graph) takes that.  The line is drawn by the time of such a call, which is
// the larger of what the calling thread and what the device needs: two launches take 7.4 us of the thread or more, one 4.5 to 5.
// us a call through the binding, two launches / one:
//   M256 x N1024 x K1024 g16 7.4 / 6.0, M389 x N437 x K1056 g4 7.4 / 7.2, M250 x N1000 x K1152 g16 7.5 / 7.0, M8 x N9216 x K1024 7.4 / 4.95,
//   M1 x N32768 x K1024 8.2 / 6.9, 8 bits M17 x N8192 x K1024 g64 7.5 / 5.2, M475 x N198 x K1024 g1024 7.5 / 7.5, M880 x N178 x K1024 g1024 7.5 / 7.8
// Over 793 shapes inside (all groups, 4 and 8 bits) one takes 0.74 of the time of two in the geometric mean and 1.04 at worst (the
// last one above; two more than 1.00).  Past the line (a block's columns times K) 0.92, and 12 of 64 are slower:
//   M389 x N437 x K1280 g4 7.4 / 7.4, M109 x N859 x K3232 g16 7.4 / 8.8, 8 bits M379 x N704 x K1024 g1024 7.8 / 8.4
// (Two stretches a wavefront would spill: M77 x N3072 x K3072 g64 at 8 bits 8.5 / 22.)
inline bool forward_in_row_tiles(int64_t M, int64_t N, int64_t K, int bits)
{
    if (M < 1 || M > 4096 || N > 32768 || K > 4096) return false;
    const RowTiles t = forward_row_tiles(M, N, K);
    return (M + t.rows - 1) / t.rows * ((N + t.columns - 1) / t.columns) <= 256 && K * t.columns * (bits / 4) <= 144 * 1024;
}

// Whether it takes that when it is recorded into a graph.  A replay costs what the device needs, and there the launch that is saved and
// the rotation that every block repeats come out about even: it pays for tiles of a few rows, and for long rows of a cheap
// rotation in not too many blocks.  us, replayed, two launches / one:
//   inside   M8 x N9216 x K1024 g16 5.9 / 4.8, M1 x N32768 x K1024 g16 8.1 / 6.9, M23 x N576 x K2048 g16 6.1 / 5.5, 8 bits M17 x N8192 x K1024 g64 6.1 / 5.2
//   outside  M256 x N1024 x K1024 g16 5.9 / 6.0, g256 5.8 / 6.1, M389 x N437 x K1056 g4 6.6 / 7.1, M250 x N1000 x K1152 g16 6.2 / 7.0,
//            M103 x N3648 x K128 g64 4.95 / 5.8, M596 x N448 x K256 g4 5.6 / 6.5, 8 bits M475 x N198 x K1024 g1024 6.4 / 7.5; M77 x N3072 x K1024 g16 6.4 / 5.7
// Over 793 shapes inside forward_in_row_tiles (all groups, 4 and 8 bits): the 241 inside here take 0.89 of the time of two launches in the
// geometric mean, 1.04 at worst (three more than 1.01); the others, which are recorded as two, would take 1.02 and 1.19, 312 more than 1.01.
inline bool row_tiles_in_graph(int64_t M, int64_t N, int64_t K, int group)
{
    const RowTiles t = forward_row_tiles(M, N, K);
    const int64_t blocks = (M + t.rows - 1) / t.rows * ((N + t.columns - 1) / t.columns);
    return t.rows <= 6 || row_items(t.rows, K) <= (t.columns <= 64 ? 10 : 8) || (K >= 1024 && group <= 256 && blocks <= 160);
}

inline int64_t tiles_of(int64_t M, int64_t N, int tm, int tn) { return ((M + tm - 1) / tm) * ((N + tn - 1) / tn); }

// Whether tiles that otherwise share a compute unit two by two take a ring of four stages: in a launch of one round each has its unit to
// itself, with LDS to spare, and what it waits for is operands (with a few stages there is nothing to run ahead with).  us, two / four
// stages: 4 bits, 192 x 192, M3000 x N3072 x K3072 25 / 16.3, geometric mean over 91 drawn shapes 1.35; three / four: 8 bits, 128 x 192, M300 x N12288 x
// K12288 80 / 65, over 69 shapes 1.11; 4 bits, 64 x 64, whose stages take 0.157 us so instead of 0.214, operands from the Infinity Cache: M700 x N1000 x K2048
// 5.7 / 5.1, M256 x N3072 x K3072 7.55 / 6.4, M1024 x N1024 x K4096 9.15 / 7.55 (six stages 5.55, 6.9, 8.0; of more than a round, where four blocks a unit
// become three, M512 x N3072 x K3072 8.2 / 8.45).  (No gain: 192 x 192 at 8 bits, 256 x 128 on eight wavefronts.)
inline bool deep_ring(int64_t tiles, int64_t stages) { return tiles <= 256 && stages >= 16; }

// Whether a small product goes in tiles of 48 x 32 instead of 32 x 64 or 16 x 32: where 32 x 32, which take less time in one round, would be more than a round and
// 48 x 32 are one.  What it takes then is its operand bytes, each loaded by every tile that needs it.  Tiles of 32 x 64 are mostly one round too, of two thirds as many blocks that
// load a fifth more rows each.  Tiles of 16 x 32 are two rounds and load W three times for twice in 48-row steps, but long chains of stages are what gains by it; in short ones, whose
// few blocks wait for a stage's latency, more of them are better.  us, plan's tile / 48 x 32, operands changing:
//   32 x 64  4 bits M40 x N5056 x K2336 4.75 / 4.4, M118 x N2620 x K9216 14.05 / 11.75, M48 x N4736 x K448 4.16 / 4.14; 8 bits M180 x N1664 x K15136
//            26.1 / 22.6; over 40 shapes each 0.92 and 0.93, none slower
//   16 x 32, inside   4 bits M104 x N2304 x K12864 17.7 / 14.7, M48 x N4920 x K8576 13.9 / 13.2; M142 x N1792 x K4320 7.2 / 5.9, over 43 shapes 0.93, none slower; 8 bits M77 x N3072 x K3072 6.3 / 5.9, N3200 x K5600 12.0 / 10.2, over 67 0.945, none slower
//            outside  4 bits, one row of tiles, M41 x N4416 x K3872 5.8 / 5.95 (6.3 / 6.9), M34 x N4181 x K4736 7.4 / 8.0, of 35 to 39 stages as many faster by 3 %; more rows M333 x N768 x K4032 5.8 / 5.95;
//            8 bits M76 x N2752 x K448 3.3 / 3.4, over 83 1.01, 49 slower
// (In place of 32 x 32 in one round 1.06 over 26, M233 x N741 x K2688 4.2 / 4.6.  80 x 16 to 80 x 32, the whole of M77 at once, 1.05 to 1.25.)
template <int BITS>
inline bool rows_of_48(Plan plan, int64_t M, int64_t N, int64_t stages)
{
    const bool gains = plan == Plan::kSplit32x64 || (plan == Plan::kSplit16x32 && stages >= (BITS == 8 ? 18 : M > 48 ? 34 : 40));
    return gains && tiles_of(M, N, 32, 32) > 256 && tiles_of(M, N, 48, 32) <= 256;
}

// 128 x 128 tiles are eight wavefronts of 32 x 64, two on each SIMD, which wait for their LDS-direct loads and fragments in turn; four of 64 x 64 read a
// third less from LDS, but alone on their SIMD every wait is the matrix pipe's (a stage 0.30 us, of which MFMAs take 0.11).  At 4 bits with a ring of four
// where every tile has its unit to itself, of three else, two blocks a unit.  us, four / eight wavefronts, operands changing: 4 bits, up to 256 tiles,
// M1619 x N1472 x K6432 16.6 / 15.3, M307 x N7296 x K5088 18.5 / 15.9, M336 x N5444 x K704 6.05 / 5.1, M424 x N6104 x K384 4.47 / 4.53; over 30 shapes 0.93,
// 1.01 at worst; more tiles, M7771 x N916 x K128 7.25 / 6.45, M2405 x N6769 x K64 11.2 / 10.5, M16544 x N640 x K832 13.2 / 13.4, over 16 shapes 0.96.  Sixteen wavefronts of 32 x 32: 1.02.  (Against
// four wavefronts on 32 x 32 MFMAs, 111 products of 257 to 600 tiles take 0.925, but M815 x N9344 x K768 9.5 / 9.75, M811 x N8256 x K544 8.1 / 8.3, M875 x N8448 x K512 8.15 / 8.35.)
// 8 bits, up to 256 tiles of up to 19 stages, M702 x N4580 x K384 6.5 / 5.5, M285 x N8951 x K1184 8.3 / 7.4, M522 x N4096 x K128 4.34 / 4.36, over 16 shapes 0.95; more tiles,
// M4990 x N1370 x K288 8.1 / 7.35, over 14 shapes 0.97; but longer products of up to 256 tiles M575 x N6336 x K1600 8.55 / 8.8, M1704 x N2304 x K2016 10.15 / 10.5,
// M638 x N4544 x K10816 49.1 / 48.8, over 12 shapes 1.01: these keep four.
inline bool four_wavefronts_8(int64_t tiles, int64_t stages) { return tiles <= 256 && stages >= 20; }

// Tile rows of a band of 256 x 256 tiles (tile_of_block), of which an XCD runs 32 at a time: 4 x 8 and 6 x 5.3 share
// operands about alike, and a last band of one to three rows shares little.  So four where they come out even or leave more rows over than
// six do, else six.  us, bands of 4 / 6: 66 tile rows, M16896 x N3072 x K12288, 268 / 256 (8: 277); 18, M4608 x N12288 x K3072, 78.8 / 76.7 (8: 77.6);
// 32, M8192 x N8192 x K4096, 107.8 / 110.2 (8: 112.2); 19, M4864 x N9152 x K12288, 199 / 217.  Over 23 shapes of 7, 19, 31, 43 and 55
// rows, where six would leave one over and four three, bands of four are 1 % faster on average and 2 % slower at most, over 142 others that are
// not even 0.4 % slower on average (22 rows, M5632 x N7680 x K12288, 198 / 209, the widest apart the other way).
constexpr int band_of_256(int tiles_m) { return tiles_m % 4 == 0 || tiles_m % 12 == 7 ? 4 : 6; }

// Tile order: blocks are dealt round-robin to the 8 XCDs by the hardware, each XCD has its own
// L2.  Give every XCD one contiguous range of logical tile ids, and walk that range in bands of
// `rows` tile rows (6 suits 256 x 128 tiles, 8 square ones, band_of_256 says for 256 x 256) so that tiles that run together share X and W
// panels.  Every block of a launch starts here, with nothing to hide it behind, so the host prepares the two divisions (two by run-time
// numbers take 60 scalar and vector instructions in a chain): quotient = high half of n times ceil(2^32 / d), one too many at most.
struct TileOrder {
    int per_xcd;        // tiles of an XCD's range
    int tiles_m, rows, span;      // span = tiles of a whole band
    uint32_t by_span, by_rows, by_tail;      // reciprocals of span, rows and the rows of the last band
};

constexpr uint32_t reciprocal(int d) { return d == 1 ? 0xFFFFFFFFu : (uint32_t)((((uint64_t)1 << 32) + (uint64_t)d - 1) / (uint64_t)d); }

// n / d for n < 2^31, d < 2^31, with m = reciprocal(d).  (m d is 2^32 plus less than d, so n m / 2^32 is n / d plus less than 1; d = 1 has one
// too little instead, for any n > 0.)
constexpr int divide(int n, int d, uint32_t m)
{
    int q = (int)(((uint64_t)(uint32_t)n * m) >> 32);
    const int rest = n - q * d;
    q -= rest < 0;
    return q + (rest >= d);
}

// (Of a launch that HIP takes: below 2^26 tiles.)
constexpr TileOrder tile_order(int tiles_m, int tiles_n, int rows)
{
    const int tail = tiles_m % rows ? tiles_m % rows : rows, span = rows * tiles_n;
    return {(tiles_m * tiles_n + kNumXcd - 1) / kNumXcd, tiles_m, rows, span, reciprocal(span), reciprocal(rows), reciprocal(tail)};
}

// The tile of block `bid`.  False where there is none; a block past an XCD's range or the last tile may also get a tile that lies
// outside Y (tn past the last column of tiles), for which its caller asks starts_inside.
constexpr bool tile_of_block(const TileOrder &o, uint32_t bid, int &tm, int &tn)
{
    const int turn = (int)(bid / kNumXcd), id = (int)(bid % kNumXcd) * o.per_xcd + turn;
    if (turn >= o.per_xcd) return false;
    const int band = divide(id, o.span, o.by_span), first = band * o.rows, left = o.tiles_m - first;
    if (left <= 0) return false;
    const int local = id - band * o.span;
    const bool tail = left < o.rows;
    const int rows = tail ? left : o.rows;
    tn = divide(local, rows, tail ? o.by_tail : o.by_rows);
    tm = first + local - tn * rows;
    return true;
}

// Whether a column of tiles of `width` columns starts inside N columns.  (Without signs: a tile outside starts up to seven widths past the
// last one, which is past 2^31 for the largest N.)
constexpr bool starts_inside(int tn, int width, int N) { return (uint32_t)tn * (uint32_t)width < (uint32_t)N; }

// How the tiled kernels store Y (gemm_tiled.h).
enum class Store {
    kCached,      // left to the caches
    kThrough,     // written through the L2: a line is on its way to memory at once, not when the next tiles' lines push it out or the kernel ends
    kPast,        // nontemporally, past the lines in use: operands that tiles and launches share stay in the L2 and the Infinity Cache
};

// Which of them a product takes; `y` = address of Y.
//   Rows of whole lines of 128 bytes: past the caches where a launch takes some 12 us or more, through otherwise, cached if Y is large.  A long product loses
//   more to the operands that its output pushes out than its stores cost, its own and those of the layers that follow; in a short one the
//   stores are the time and past the caches they run at the rate of the memory, and so they do written through when outputs, three of one activation
//   among them, no longer fit the Infinity Cache.
//   Lines that two rows share: never past the caches (two half lines, each written to memory by itself).  Through in short products while the L2s
//   hold all of Y, which would otherwise be written back when the kernel ends; cached beyond, where a line mostly gets its second half before
//   it leaves (8-bit 256 x 256 tiles, alone on their unit, end together with 128 KB each: no gain there in a short product).
// One activation that feeds three layers, three sets of operands in turn, through / past: M4608 x N3072 x K3072 91.1 / 88.8, M1891 x N6400 x K4224
// 106.3 / 100.0, M2824 x N7616 x K960 at 8 bits 109 / 91; over 36 shapes of 1.2e10 to 7e10 products past is 3 % faster there, the same in a GEMM alone
// or a forward (0.3 % slower) and 0.4 % faster with the next layer's rotate+quantise; of 1e9 to 1.5e10 products through is 0.2 % faster there and 4 % in the others.
// K below 512, GEMM alone / three layers of one activation, cached : through: Y of 31 MB, M6978 x N2240 x K64 10.8 : 9.6 / 35.7 : 31.7, of 60 MB, M9929 x N3008 x K448
// 19.2 : 18.9 / 66.6 : 67.2, of 117 MB, M7861 x N7424 x K64 at 8 bits 25.1 : 24.8 / 87.7 : 92.4, of 149 MB, M9753 x N7616 x K384 40.6 : 42.3 / 123 : 130, of 237 MB,
// M10684 x N11072 x K64 51.3 : 55.9 / 158 : 165 (past the caches 57.1 / 176).
// us, GEMM on three sets of buffers in turn, cached / through / past, 4 bits if not said:
//   M6398 x N11328 x K64 at 8 bits 32.3 / 32.5 / 35.6, M7023 x N4864 x K64 16.3 / 15.5 / 18.8, M4189 x N8768 x K1024 26.4 / 26.1 / 29.3, M423 x N8896 x K512
//   6.1 / 5.4 / 5.6; M4608 x N3072 x K3072 21.7 / 21.2 / 21.7, M4608 x N12288 x K3072 85.1 / 86.9 / 78.9 and at 8 bits 143 / 144 / 136, M4608 x N3072 x K12288
//   72.7 / 73.5 / 60.1, M16896 x N4096 x K3072 113 / 113 / 97; half lines: M13207 x N5816 x K64 46.5 / 90.4 / 86.8, M5644 x N3832 x K512 16.9 / 17.8 / 25.1,
//   M10772 x N672 x K512 8.3 / 6.6 / 6.9, M7622 x N10104 x K1024 74 / 110 / 97, M5082 x N6320 x K768 at 8 bits 37.6 / 33.5 / 47.1; long ones with Y of 17 to 25 MB,
//   M13752 x N856 x K5056 at 8 bits 71.9 / 74.0 / 69.0, M13111 x N888 x K14912 103.1 / 105.8 / 103.6, three layers of M3378 x N3640 x K8192 196 / 207 / 199
// The next layer, which reads Y from memory where it went past the caches, takes part of that back; GEMM and its rotate+quantise: M4608 x N12288 x K3072
// 106.5 / 108.7 / 106.9, at 8 bits 165 / 166 / 168, M4608 x N3072 x K12288 80.0 / 79.8 / 80.5, M16896 x N4096 x K3072 137 / 136 / 131.
// Over 336 shapes with whole lines and 264 without (4 and 8 bits, Y of 4 to 415 MB, K 64 ... 15360; mean of GEMM alone, into one output, with the
// next layer's rotate+quantise, whole forward) the rule, its line then at 6e10 products, was 5.2 and 4.3 % faster than cached stores (through where a
// block has its unit to itself) on average and 4 and 7 % slower at most; everything past the caches 2.6 % faster and 8 % slower, at most 18 and 120 % slower.
template <int BITS>
inline Store store_kind(Plan plan, int64_t M, int64_t N, int64_t K, uintptr_t y)
{
    const double outputs = (double)M * (double)N, products = outputs * (double)K * (BITS / 4);
    if (N % 64 == 0 && y % 128 == 0) {
        if (K >= 512 && products >= 1.5e10) return Store::kPast;
        return 2.0 * outputs <= 96e6 ? Store::kThrough : Store::kCached;
    }
    if (N % 8 != 0 || y % 16 != 0 || products >= 6e10) return Store::kCached;
    return 2.0 * outputs <= 8 * 4.0 * 1048576 || (BITS == 8 && plan == Plan::kTile256x256) ? Store::kThrough : Store::kCached;
}

struct Small {
    Plan plan;
    int tm, tn;
    int split;      // wavefronts that share the stages of K, or 1
    float fixed, block, latency, rate;
};

struct Paired {
    Plan plan;
    int tm, tn;
    float fixed, block, pair, lone;
};

struct Alone {
    int threads;
    float fixed, block, rate, idle;
};

struct Cut {        // a round of parts of 256 x 256 tiles
    float block, rate;
};

// A 256 x 256 tile of 4-bit codes has a compute unit to itself, so a last round that few of an XCD's 32 units have a tile of
// keeps the others waiting for a whole tile.  Such tiles are cut: into halves where they give every unit at most one, into
// quarters where those do (us, whole / cut: M4608 x N12288 x K3072, 12 left over, 87.6 / 85.4; M16896 x N3072 x K12288, 3 left over,
// 275.5 / 260.5; over 16 and 19 drawn shapes 6 and 14 % - more of them would take two rounds of parts and lose).  After
// many rounds the units no longer finish together and parts only cost (M16896 x N12288 x K3072, 12 rounds, 296 / 305).  8-bit
// products gain nothing there over 192 x 192 tiles.  (All with operands that change from launch to launch and outputs in the caches;
// with outputs past them M4608 x N12288 x K3072 takes 78.8 to 80 us in halves and 77.6 with 192 x 192 tiles.)  Parts a tile is cut
// into, 1 if none is; `per_xcd` = tiles of an XCD.
inline int parts_of_last_tiles(int64_t per_xcd)
{
    const int64_t rest = per_xcd % 32;
    return per_xcd < 32 || per_xcd >= 5 * 32 || rest == 0 || rest > 16 ? 1 : rest > 8 ? 2 : 4;
}

// Whether every other XCD begins with its parts instead of ending with them.  All units of a launch otherwise finish a round at once, and the rounds'
// outputs go to memory in bursts that the next tiles wait behind; half a tile apart, one half of the chip stores while the other multiplies.
// Outputs left to the caches make no such bursts.  Long products have little to gain, and lose the operands that XCDs ask for at the same time from the same cache, those of
// few columns of tiles, whose XCDs walk the same ones, before the others.  us, last / first on odd XCDs, operands changing:
//   inside   M4608 x N12288 x K3072 78.2 / 75.5, M4155 x N9216 x K1536 38.0 / 34.1, M16659 x N1088 x K1056 18.9 / 17.8, M12452 x N1728 x K2080 27.7 / 26.1,
//            M8854 x N2112 x K3168 31.1 / 31.2, M9469 x N3712 x K3104 54.5 / 55.3; over 84 shapes of K 1024 ... 3328 0.946, 1.015 at most
//   narrow and of more stages  M16078 x N1280 x K2912 32.7 / 39.0, M11872 x N1792 x K2720 32.6 / 34.5, M14049 x N1280 x K2624 27.2 / 27.0; over 9 shapes 1.075
//   rows that are not whole lines  M15579 x N2501 x K1984 57.6 / 64.5, M2230 x N10320 x K1152 26.7 / 31.2, M8087 x N2659 x K2368 44.3 / 38.0; over 95 shapes 1.010, 50 slower, 33 faster
//   longer   M7095 x N5248 x K4096 73.8 / 72.3, but M16525 x N1216 x K3584 40.9 / 42.9; over 34 shapes of K 3584 ... 12288 1.013
// With the four XCDs of one half of the chip first M4608 x N12288 x K3072 takes 80, with all of them 75.4; half a tile apart in products whose rounds come out
// even, by parts for whole tiles, 0 to 30 % slower.
constexpr int kPartsFirst = 1 << 8;      // (fewer than 5 * 32 tiles of an XCD are whole)
constexpr bool parts_first(Store store, int64_t N, int64_t stages) { return store == Store::kPast && stages <= (N > 7 * 256 ? 26 : 17); }

// The work of an XCD's `turn`-th block: a tile of its range, whole or one part of it.  `how`: the tiles that are whole, and kPartsFirst.
struct CutTurn {
    uint32_t tile, part;
    bool whole;
};
constexpr CutTurn cut_turn(uint32_t turn, uint32_t xcd, uint32_t per_xcd, uint32_t how, uint32_t parts)
{
    const uint32_t whole = how & (kPartsFirst - 1);
    if (xcd & how >> 8) {
        const uint32_t first = (per_xcd - whole) * parts;
        turn = turn < first ? whole + turn : turn - first;
    }
    if (turn < whole) return {turn, 0, true};
    return {whole + (turn - whole) / parts, (turn - whole) % parts, false};
}

template <int BITS>
inline Plan choose(int64_t M, int64_t N, int64_t K)
{
    static_assert(BITS == 4 || BITS == 8, "code widths");
    static constexpr Small small4[] = {
        {Plan::kTile64x64, 64, 64, 1, 2.47f, 0.58f, 0.153f, 0.1113f},
        {Plan::kSplit32x64, 32, 64, 8, 0.97f, 2.21f, 0.368f, 0.0958f},
        {Plan::kSplit32x32, 32, 32, 4, 2.41f, 0.43f, 0.250f, 0.0583f},
        {Plan::kSplit16x32, 16, 32, 8, 2.36f, 0.53f, 0.176f, 0.0440f},
        {Plan::kSplit16x16, 16, 16, 16, 1.90f, 0.98f, 0.445f, 0.0242f},
    };
    static constexpr Small small8[] = {
        {Plan::kTile64x64, 64, 64, 1, 2.52f, 0.52f, 0.118f, 0.0849f},
        {Plan::kSplit32x64, 32, 64, 8, 2.06f, 1.07f, 0.246f, 0.0822f},
        {Plan::kSplit32x32, 32, 32, 4, 2.57f, 0.33f, 0.183f, 0.0539f},
        {Plan::kSplit16x32, 16, 32, 8, 2.29f, 0.42f, 0.321f, 0.0380f},
        {Plan::kSplit16x16, 16, 16, 16, 2.22f, 0.78f, 0.255f, 0.0243f},
    };
    static constexpr Paired paired4[] = {
        {Plan::kTile192x192, 192, 192, 3.62f, 2.92f, 0.745f, 0.592f},
        {Plan::kTile256x128, 256, 128, 3.65f, 2.60f, 0.700f, 0.582f},
        {Plan::kTile128x128, 128, 128, 2.96f, 1.36f, 0.479f, 0.280f},
    };
    static constexpr Paired paired8[] = {
        {Plan::kTile192x192, 192, 192, 5.14f, 2.70f, 0.734f, 0.301f},
        {Plan::kTile256x128, 256, 128, 3.96f, 2.63f, 0.674f, 0.284f},
        {Plan::kTile128x128, 128, 128, 2.56f, 1.57f, 0.405f, 0.190f},
        {Plan::kTile128x192, 128, 192, 3.08f, 2.44f, 0.512f, 0.269f},
    };
    static constexpr Alone w8 = {512, 2.00f, 3.84f, 0.419f, 0.80f};                                                  // 256 x 128, 4 bits
    static constexpr Alone whole = BITS == 4 ? Alone{512, 1.10f, 5.83f, 0.606f, 0.69f} : Alone{512, 0.02f, 6.13f, 0.691f, 0.61f};     // 256 x 256

    // 128 x 192, 4 bits: one round of up to 256 tiles where 256 x 128 leaves units idle.  Six wavefronts of 64 x 64: an LDS-direct load takes longer to issue than a
    // 16 x 16 MFMA, and of four wavefronts, one on each SIMD, every load is the matrix pipe's wait.  us, operands changing, four / six: M801 x N5440 x K2432 10.5 / 9.7,
    // M2637 x N1728 x K4320 15.25 / 14.1, M512 x N12288 x K3072 16.3 / 15.8, M532 x N7752 x K4384 20.3 / 20.5; over 87 shapes 0.95, 1.01 at most.  (The fit is of four
    // wavefronts, times 1.05: a draw goes to the tiles that it is compared with, whose fits are of more shapes.)
    static constexpr Alone middle = {384, 1.70f, 4.55f, 0.347f, 0.98f};

    // 192 x 192, 4 bits, with a deep ring: between 128 x 192, of which such a product has more than a round, and 256 x 256, which leave units idle.
    static constexpr Alone square = {256, 1.99f, 4.53f, 0.493f, 0.532f};

    const float stages = (float)(BITS == 4 ? (K + 127) / 128 : (K + 63) / 64);
    Plan best = Plan::kCount;
    float least = 0.0f;
    bool best_fits = false;
    auto tiles = [&](int tm, int tn) { return tiles_of(M, N, tm, tn); };
    // (A launch of more tiles than HIP takes at once is no candidate while there is another: M1 x N2^30 x K32 in 64 x 64 tiles.)
    auto consider = [&](Plan plan, int64_t blocks, int threads, float t) {
        const bool fits = launchable(blocks, threads);
        if (best == Plan::kCount || (fits == best_fits ? t < least : fits)) {
            best = plan;
            least = t;
            best_fits = fits;
        }
    };
    auto paired = [&](const Paired &c) {
        const int64_t n = tiles(c.tm, c.tn), b = (n + 255) / 256;
        const int threads = c.plan == Plan::kTile128x128 ? 512 : 256;
        consider(c.plan, n, threads, c.fixed + c.block * (float)b + stages * (c.pair * (float)(b / 2) + c.lone * (float)(b % 2)));
    };
    auto small = [&](const Small &c) {
        const int64_t n = tiles(c.tm, c.tn);
        const float b = (float)((n + 255) / 256), chain = (float)(((int64_t)stages + c.split - 1) / c.split);
        const float alone = c.latency * chain, full = c.rate * stages * b;
        consider(c.plan, n, c.split == 1 ? 256 : 64 * c.split, c.fixed + c.block * b + (alone > full ? alone : full));
    };
    auto alone = [&](Plan plan, int tm, int tn, const Alone &c) {
        const int64_t n = tiles(tm, tn), b = (n + 255) / 256;
        const float fill = (float)n / (256.0f * (float)b);
        consider(plan, n, c.threads, c.fixed + (float)b * (c.block + c.rate * stages * (c.idle + (1.0f - c.idle) * fill)));
    };

    if constexpr (BITS == 4) {
        const bool deep = deep_ring(tiles(192, 192), (int64_t)stages);
        for (const Paired &c : paired4)
            if (!(deep && c.plan == Plan::kTile192x192)) paired(c);
        if (deep) alone(Plan::kTile192x192, 192, 192, square);
        for (const Small &c : small4) small(c);
        alone(Plan::kTile256x128w8, 256, 128, w8);
        alone(Plan::kTile128x192, 128, 192, middle);
    } else {
        for (const Paired &c : paired8) paired(c);
        for (const Small &c : small8) small(c);
    }
    // With only a few stages a block that is alone on its unit cannot hide its first loads and its stores behind another one
    // (M7557 x N3773 x K640: 24.6 us against 22.9 with 256 x 128 tiles), which the prediction knows nothing of.
    if (stages >= 8.0f) {
        const int64_t per_xcd = (tiles(256, 256) + 7) / 8;
        const int parts = BITS == 4 ? parts_of_last_tiles(per_xcd) : 1;
        if (parts == 1) {
            alone(Plan::kTile256x256, 256, 256, whole);
        } else {      // full rounds and one of parts
            const Cut c = parts == 2 ? Cut{3.90f, 0.340f} : Cut{3.30f, 0.240f};
            consider(Plan::kTile256x256, 4 * 8 * per_xcd, whole.threads, whole.fixed + (float)(per_xcd / 32) * (whole.block + whole.rate * stages) + c.block + c.rate * stages);
        }
    }
    return best;
}

}  // namespace gemm
}  // namespace convrot
