// Kernel A of libconvrot: group-wise regular-Hadamard rotation + per-row absmax + 4-bit
// quantisation + packing of the codes, one pass over the bf16 input (ConvRot paper Sec. 4.2 Eq. 11-13,
// Eq. 1, Sec. 5.2).  Serves activations (rows = tokens) and weights (rows = output channels).
//
// Work split.  A column is 64 consecutive elements of a row: 128 bytes of bf16 in, two chunks of 32 codes (four units) out.  A
// chunk is what one lane feeds one MFMA of the GEMM; a wavefront rotates 16 or 32 columns at a time (a set) and a lane ends up
// with a unit or with a whole chunk.  The whole row stays in registers between the absmax
// reduction and the rounding, so X is read from HBM exactly once.
//
// What bounds it: memory, 2.75 bytes an element (a large copy runs at 6.1 TB/s), on rows of 3072 elements and more; the launch and one
// pass of every wavefront through load, arithmetic and store on smaller inputs.  Vector instructions, 7.5 to 9 an element
// (g <= 64; 9.7 counted on [4608, 3072] at g = 16, where lanes hold single units) to 13.4 (g = 1024), would take two thirds of that time and overlap with it.  With digit 2 on the vector ALU, a bracketing
// second product for every code and a unit's 12 bytes stored in two places by pairs of lanes they were 10.9 to 18.
//
// The rotation and the quantiser themselves are rotate_quantise.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "convrot_internal.h"
#include "e2m3_layout.h"
#include "gemm_common.h"
#include "panel_layout.h"
#include "rotate_quantise.h"

namespace convrot {

// The launches for 8-bit codes of g >= 256 (lanes8.hip).
hipError_t rotquant_lanes8(const void *X, int64_t rows, int64_t K, int group, void *Xq, float *scale, hipStream_t stream);

namespace {

// All but the last N * n of this wavefront's loads have landed (n is known where the call is inlined).
template <int N>
__device__ __forceinline__ void wait_loads(int n)
{
    if (n == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (n == 1) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
    else if (n == 2) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * N) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(3 * N) : "memory");
}

// Codes to memory, left to the L2 or written through it.  (The wait state: see gemm::store_row.)
template <bool THROUGH>
__device__ __forceinline__ void store16(void *out, u32x4 v)
{
    if constexpr (THROUGH) asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(out), "v"(v) : "memory");
    else *reinterpret_cast<u32x4 *>(out) = v;
}
template <bool THROUGH>
__device__ __forceinline__ void store8(void *out, u32x2 v)
{
    if constexpr (THROUGH) asm volatile("global_store_dwordx2 %0, %1, off sc1" :: "v"(out), "v"(v) : "memory");
    else *reinterpret_cast<u32x2 *>(out) = v;
}

}  // namespace

// A set is what a wavefront rotates at a time: 16 U columns, U units a lane, 16 U / RPW columns of each of RPW consecutive rows.
// A wavefront holds S sets of its rows and WPR wavefronts side by side, one block, hold the whole rows.
//   U = 2  lanes n and n + 32 hold the even and the odd chunk of column n and store them whole
//   U = 1  lanes n, n + 16, n + 32, n + 48 hold the units of column n: twice the wavefronts, for short rows
// BITS = 4: codes in [-7, 7], stored as FP6 E2M3 (e2m3_layout.h); BITS = 8 (the W8A8 variant of the layer): one
// int8 per code, [-127, 127] (panel_layout.h).
template <int U, int RPW, int WPR, int S>
struct Split {
    static constexpr int kThreads = 64 * WPR;
    // (At least two wavefronts per SIMD, i.e. at most 256 registers per lane: then the compiler keeps the MFMA results in
    // ordinary registers instead of copying them out of the accumulation registers, one move per element.)
    static constexpr int kOccupancy = WPR <= 4 ? 2 : 1;
    static constexpr int kColumns = 16 * U / RPW;             // of a row, in one set
    static constexpr int kSetBytes = 2048 * U;
    static_assert((U == 1 || U == 2) && WPR <= 16 && S <= 4, "split");
};

// Whether codes are written through the L2: where a store instruction holds two rows' pieces side by side (128 bytes of an output block's A
// plane or of two panel rows).  Left to the L2 they go to memory when the kernel ends, all at once and with nothing to do meanwhile: of the 83 000 lines of
// [4608, 3072] 82 800 are written back then, written through 144, and the writes to memory are the same (TCC_ALL_TC_OP_WB_WRITEBACK,
// TCC_EA0_WRREQ).  us, left / written through:
//   [4608, 3072] g256 9.8 / 8.7, [12288, 3072] g256 21.4 / 19.4, 8 bits [9000, 2048] g256 14.1 / 12.4; over 63 shapes of 3000 to 30000
//   rows of 1280 to 4096 elements 4.4 % less; with the GEMM that reads them M4608 x N12288 x K3072 at 8 bits 159.9 / 158.7
//   4 bits, g <= 16, where there is less arithmetic to do meanwhile: [12501, 1280] g16 10.9 / 10.05, [9864, 2048] g16 11.3 / 11.4, [6576, 3072]
//   g16 11.3 / 11.6, over 24 inputs of 2048 and 3072 elements 0.9 % more, eleven whole forwards 0.4 % less
// Not the pieces of single rows, which then go to memory by themselves ([8000, 1024] 5.9 / 6.5, [16896, 12288] 92 / 136), nor, at g <= 16 and
// 4 bits, rows of four wavefronts of U = 1 ([3000, 4096] 7.4 / 7.6).
template <int G, int BITS, int U, int RPW, int WPR>
constexpr bool kThrough = RPW >= 2 && WPR >= 2 && (BITS == 8 || G >= 64 || U == 2 || WPR <= 3);

// Wavefronts that a SIMD has at most, by registers set aside: eight by their number, six where memory takes no more of them at once well.  8-bit codes of g >= 256, built
// without the SLP vectoriser (lanes8.hip), need 60 registers instead of 73, and rows of 4097 to 8192 elements, a block of three or four wavefronts each, are slower with the
// eight that then fit.  us, eight / six: [4608, 5120] g256 19.7 / 17.3, g1024 21.1 / 19.9, [3126, 7168] g256 18.1 / 16.7, over 44 inputs 0.986, 1.01 at most.  Five
// wavefronts and more (six of [4608, 12288] g1024 36.4 / 38.9) and two rows a block ([4608, 3072] g256 10.3 / 10.7, g1024 11.7 / 11.9) keep eight.
template <int G, int BITS, int U, int RPW, int WPR>
constexpr int kMostWaves = BITS == 8 && G >= 256 && U == 2 && RPW == 1 && WPR <= 4 ? 6 : 8;

template <int G, int BITS, int U, int RPW, int WPR, int S>
__global__ __launch_bounds__((Split<U, RPW, WPR, S>::kThreads))
__attribute__((amdgpu_waves_per_eu((Split<U, RPW, WPR, S>::kOccupancy), (kMostWaves<G, BITS, U, RPW, WPR>)))) void rotquant_kernel(
    const uint16_t *__restrict__ X, int64_t rows, int K, uint8_t *__restrict__ Xq, float *__restrict__ scale)
{
    using Sp = Split<U, RPW, WPR, S>;
    constexpr int C = Sp::kColumns;
    constexpr bool kThru = kThrough<G, BITS, U, RPW, WPR>;
    static_assert(G <= 64 || G / 64 <= C, "the lanes of a rotation group lie in one row");
    __shared__ float part[WPR * RPW];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Blocks are dealt round-robin to the 8 XCDs, each with an L2 of its own.  The rows of an output
    // block go to consecutive thread blocks of one XCD, so that their pieces of a line meet in one
    // L2 and leave it as whole lines.
    constexpr int kGroupRows = BITS == 4 ? e2m3::kRows : panel::kRows;   // rows that share an output block
    constexpr int kBlocks = kGroupRows / RPW;                            // thread blocks per group of rows
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int64_t row0 = ((int64_t)(idx / kBlocks) * 8 + xcd) * kGroupRows + idx % kBlocks * RPW;
    if (row0 >= rows) return;
    const int left = (int)min((int64_t)RPW, rows - row0) - 1;            // the last of its rows that exists
    const int rib = (lane & (16 * U - 1)) / C;                           // row of the block
    const bool row_ok = rib <= left;
    const int h = lane >> 5, odd16 = (lane >> 4) & 1, chunks = K / 32;
    const int column0 = wave * C + (lane & (C - 1));                     // this lane's column of the first set

    // The columns come through LDS: lanes n and n + 32 need the 16-byte halves of the four units of column n, 32 lines of 32 bytes
    // for a load straight into registers; copied there (LDS-direct, a kilobyte of consecutive columns at a time) the
    // lines are read whole.  Slot p of column n holds piece p ^ (n & 7), so that eight lanes read different banks.
    // All loads are issued up front and unconditionally: a column (or row) that does not exist is replaced
    // by the last one of the row (of the last row), and its owner is masked out of the absmax and the stores.
    // K % g == 0 makes a rotation group all-valid or all-invalid, so such lanes never feed valid ones.
    __shared__ __attribute__((aligned(1024))) uint8_t lds[WPR * S * Sp::kSetBytes];
    uint8_t *const mine = lds + wave * (S * Sp::kSetBytes);
    {
        const uint8_t *const x = reinterpret_cast<const uint8_t *>(X + row0 * K);
        const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)mine;
        const int n0 = lane >> 3, p = (lane & 7) ^ n0;       // column of the first kilobyte, its piece
#pragma unroll
        for (int i = 0; i < S; ++i)
#pragma unroll
            for (int j = 0; j < 2 * U; ++j) {
                const int n = 8 * j + n0;
                const int piece = min(8 * ((wave + i * WPR) * C + (n & (C - 1))) + p, 4 * chunks - 1);
                gemm::lds_dma16<true>(x, (uint32_t)min(n / C, left) * (uint32_t)K * 2 + 16 * piece, base + (i * 2 * U + j) * 1024);
            }
    }
    const Rotation<G> rot(lane);

    float v[S][U][kUnit];
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < S; ++i) {
        float m = 0.0f;
        wait_loads<2 * U>(S - 1 - i);
        auto piece = [&](int c) { return *reinterpret_cast<const u32x4 *>(mine + i * Sp::kSetBytes + (lane & (16 * U - 1)) * 128 + (((2 * c + h) ^ (lane & 7)) << 4)); };
        if constexpr (U == 2) {
            u32x4 raw[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) raw[c] = piece(c);
#pragma unroll
            for (int odd = 0; odd < 2; ++odd) rot.apply([&](int c) { return raw[c ^ odd]; }, v[i][odd]);
        } else {
            rot.apply([&](int c) { return piece(c ^ odd16); }, v[i][0]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) rotate_lanes<G>(v[i][u]);
#pragma unroll
        for (int e = 0; e < U * kUnit; ++e) m = fmaxf(m, fabsf(v[i][e / kUnit][e % kUnit]));
        amax = 2 * (column0 + i * WPR * C) + h < chunks ? fmaxf(amax, m) : amax;
    }

    // row absmax: the row's lanes of this wavefront, then the row's wavefronts through LDS
    amax = max_of_lanes<C, 16 * U>(amax);
    if constexpr (WPR > 1) {
        if ((lane & (C - 1)) == 0 && h == 0 && (U == 2 || odd16 == 0)) part[wave * RPW + rib] = amax;
        __syncthreads();
        amax = part[rib];
#pragma unroll
        for (int w = 1; w < WPR; ++w) amax = fmaxf(amax, part[w * RPW + rib]);
    }

    const Quantiser q(amax, group_norm<G>(), BITS == 4 ? 7.0f : 127.0f);
    if (row_ok && column0 + h + (U == 2 ? 0 : odd16) == 0) scale[row0 + rib] = q.s;

    const int out0 = column0 ^ column_flip<G>();             // (sets are apart by multiples of the flipped columns)
    const int r = (int)(row0 % kGroupRows) + rib;
    if constexpr (BITS == 4) {
        const int stages = (K + e2m3::kStageCodes - 1) / e2m3::kStageCodes;
        uint8_t *const out = Xq + row0 / e2m3::kRows * stages * e2m3::kBlockBytes;
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const v6u packed = codes4(q, U == 2, as_vector(v[i][0]), as_vector(v[i][U - 1]));
            const int chunk = 2 * (out0 + i * WPR * C) + h;
            const bool pad = chunk >= chunks;                // K padding: zero codes
            uint8_t *const block = out + (uint32_t)(chunk >> 2) * (uint32_t)e2m3::kBlockBytes;
            if constexpr (U == 2) {
                if (!(row_ok && chunk < 4 * stages)) continue;
                store16<kThru>(block + e2m3::a_offset(r, chunk & 3), pad ? u32x4{0, 0, 0, 0} : u32x4{packed[0], packed[1], packed[2], packed[3]});
                store8<kThru>(block + e2m3::b_offset(r, chunk & 3), pad ? u32x2{0, 0} : u32x2{packed[4], packed[5]});
            } else {        // lanes 16 further on hold the chunk's odd units
                const uint32_t next = __builtin_amdgcn_permlane16_swap(packed[0], packed[0], false, false)[1];
                if (!(row_ok && chunk < 4 * stages)) continue;
                if (odd16 == 0)
                    store16<kThru>(block + e2m3::a_offset(r, chunk & 3), pad ? u32x4{0, 0, 0, 0} : u32x4{packed[0], packed[1], packed[2], next});
                else
                    store8<kThru>(block + e2m3::b_offset(r, chunk & 3), pad ? u32x2{0, 0} : u32x2{packed[1], packed[2]});
            }
        }
    } else {
        // a column is a panel's 64 bytes of its row, four units
        const int panels = (K + panel::kRowBytes - 1) / panel::kRowBytes;
        const bool odd = (out0 & 1) != 0;
        uint8_t *const out = Xq + row0 / panel::kRows * panels * panel::kBytes + (uint32_t)(r * panel::kRowBytes + 32 * h);
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const int column = out0 + i * WPR * C;
            u32x4 a = codes8(q, as_vector(v[i][0]));
            u32x4 *const o = reinterpret_cast<u32x4 *>(out + (uint32_t)column * (uint32_t)panel::kBytes);
            const bool ok = row_ok && column < panels, pad = 2 * column + h >= chunks;      // K padding: zero codes
            if constexpr (U == 1) {
                if (ok) store16<kThru>(o + odd16, pad ? u32x4{0, 0, 0, 0} : a);
            } else {
                // Neighbouring lanes exchange one unit each, so that a store instruction writes whole columns, the even ones first.
                u32x4 b = codes8(q, as_vector(v[i][1]));
                if (pad) a = b = u32x4{0, 0, 0, 0};
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const uint32_t other = __builtin_amdgcn_update_dpp(0u, odd ? a[w] : b[w], 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
                    a[w] = odd ? other : a[w];
                    b[w] = odd ? b[w] : other;
                }
                const int even = column & ~1;
                u32x4 *const oe = reinterpret_cast<u32x4 *>(out + (odd ? 16 : 0) + (uint32_t)even * (uint32_t)panel::kBytes);
                if (row_ok && even < panels) store16<kThru>(oe, a);
                if (row_ok && even + 1 < panels) store16<kThru>(oe + panel::kBytes / 16, b);
            }
        }
    }
}

namespace {      // (not exported: a weak definition could be taken over by another library of the process)

template <int G, int BITS, int U, int RPW, int WPR, int S>
hipError_t launch_rows(const void *X, int64_t rows, int K, void *Xq, float *scale, hipStream_t stream)
{
    constexpr int kThreads = Split<U, RPW, WPR, S>::kThreads, kGroupRows = BITS == 4 ? e2m3::kRows : panel::kRows;
    constexpr int64_t kStep = 8 * kGroupRows;                // a row group for each XCD (see the row mapping in the kernel)
    constexpr int64_t kMost = ((int64_t)1 << 32) / kThreads * RPW / kStep * kStep - kStep;      // HIP launches fewer than 2^32 threads
    for (int64_t r = 0; r < rows; r += kMost) {
        const int64_t n = rows - r < kMost ? rows - r : kMost;
        const unsigned grid = (unsigned)((n + kStep - 1) / kStep * kStep / RPW);
        const int64_t bytes = BITS == 4 ? e2m3::matrix_bytes(r, K) : panel::matrix_bytes(r, K);
        hipLaunchKernelGGL((rotquant_kernel<G, BITS, U, RPW, WPR, S>), dim3(grid), dim3(kThreads), 0, stream,
                           (const uint16_t *)X + r * K, n, K, (uint8_t *)Xq + bytes, scale + r);
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Wavefronts of `rows` rows, 1024 elements each.
inline int64_t row_waves(int64_t rows, int64_t K) { return rows * ((K + 1023) / 1024); }

// From how many elements on lanes hold whole chunks instead of units (4 bits, rows of 1025 to 4096 elements).  us, units / whole chunks:
//   g256                 [3906, 3072] 8.3 / 8.7, [6510, 3072] 12.4 / 12.2, [5859, 4096] 14.0 / 13.5, [9765, 4096] 21.1 / 19.8
//   g16                  [3906, 3072] 7.95 / 8.3, [6510, 3072] 11.7 / 11.6, [9765, 2048] 11.7 / 11.6, [17090, 2048] 17.0 / 16.8
//   g16, half-full sets  [15782, 1280] 11.5 / 12.0, [21876, 1280] 14.35 / 14.7, [26563, 1280] 16.7 / 16.8
//   g16, four wavefronts [4932, 4096] 10.9 / 11.4, [6836, 4096] 14.0 / 14.4, [8301, 4096] 16.5 / 16.5, [9765, 4096] 18.9 / 18.7
template <int G>
constexpr int64_t whole_chunks_from(int K) { return G <= 16 && (K <= 1536 || K > 3072) ? 34000000 : 20000000; }

// The split of a row, by its length and the number of rows.
//
// A few rows (up to 12 wavefronts a compute unit, rows of 1025 to 12288 elements) are one pass of each wavefront through load, arithmetic
// and store: a row a block, 1024 elements a wavefront.  (Five, seven and nine to eleven stretches take 6, 8 and 12 wavefronts.)  us, as more rows are
// split / so: [77, 3072] g16 3.1 / 2.8, [512, 2048] g256 3.75 / 3.5, [256, 12288] g256 4.7 / 3.9, [1000, 3072] 3.7 / 3.45.  Over 264
// inputs of 6 to 18 wavefronts a unit 8 % less on average, up to the line 9 % (1 % more at most), past it, at 14 and 18, 7 % (2 % more at most); far past it
// [1000, 12288], 47 a unit, 7.6 / 8.9.
//
// For more rows, enough wavefronts first: with U = 1 twice as many that do half the work each, and one or two sets of each; rows side by side
// in a wavefront as long as their digits across lanes fit (g / 64 columns), so that a store instruction finds more of an output block's 64- and
// 32-byte row pieces adjacent; from some 2e7 elements on lanes that store whole chunks (whole_chunks_from).  Past 4096 elements a block is one
// row of whole chunks, as few wavefronts as hold it once.  us, cold, against a kernel of 16 consecutive elements a lane with digit 2 by DPP:
//   [8000, 256] g64 5.2 -> 3.9, [8000, 512] g64 5.6 -> 4.2, [12288, 1024] g256 9.6 -> 9.0, [4608, 3072] g16 8.9 -> 8.5, g256 11.2 -> 9.8,
//   [12288, 3072] g256 23.0 -> 22.1 (now 18.8), [4608, 4096] g64 13.5 -> 10.5, [4608, 12288] g16 28.4 -> 27.9, [4608, 15360] g1024 43.8 -> 40.5,
//   8 bits [16896, 12288] g16 121 -> 103
// and the other splits at those sizes: U = 2 [8000, 512] 5.0, [4608, 1024] g256 5.7 against 5.0; one row a wavefront [4608, 3072] g16 8.9;
// two rows a block [4608, 12288] 28.2 to 30.5, four rows 36.3; half the wavefronts with two sets each 28.1.
template <int G, int BITS>
hipError_t launch_g(const void *X, int64_t rows, int K, void *Xq, float *scale, hipStream_t stream)
{
#define CONVROT_ROWS(U, RPW, WPR, S) launch_rows<G, BITS, U, RPW, WPR, S>(X, rows, K, Xq, scale, stream)
    if constexpr (G <= 256) {
        if (K <= 256) return CONVROT_ROWS(1, 4, 1, 1);
        if (K <= 512) return CONVROT_ROWS(1, 2, 1, 1);
    }
    if (K <= 1024) return CONVROT_ROWS(1, 1, 1, 1);
    if (K <= 12288 && row_waves(rows, K) <= 12 * 256) {
        switch ((K + 1023) / 1024) {
            case 2: return CONVROT_ROWS(1, 1, 2, 1);
            case 3: return CONVROT_ROWS(1, 1, 3, 1);
            case 4: return CONVROT_ROWS(1, 1, 4, 1);
            case 5: case 6: return CONVROT_ROWS(1, 1, 6, 1);
            case 7: case 8: return CONVROT_ROWS(1, 1, 8, 1);
            default: return CONVROT_ROWS(1, 1, 12, 1);
        }
    }
    if constexpr (BITS == 4) {
        if (K <= 4096 && rows * K >= whole_chunks_from<G>(K)) {
            if (K <= 2048) return CONVROT_ROWS(2, 2, 2, 1);
            if (K <= 3072) return CONVROT_ROWS(2, 2, 3, 1);
            return CONVROT_ROWS(2, 2, 4, 1);
        }
    }
    if constexpr (G <= 256) {
        if (K <= 2048) return CONVROT_ROWS(1, 2, 2, 2);
        if (K <= 3072) return CONVROT_ROWS(1, 2, 3, 2);
        if (K <= 4096) return CONVROT_ROWS(1, 2, 4, 2);
    } else {
        if (K <= 2048) return CONVROT_ROWS(2, 2, 2, 1);
        if (K <= 3072) return CONVROT_ROWS(2, 2, 3, 1);
        if (K <= 4096) return CONVROT_ROWS(2, 2, 4, 1);
    }
    switch ((K + 2047) / 2048) {
        case 3: return CONVROT_ROWS(2, 1, 3, 1);
        case 4: return CONVROT_ROWS(2, 1, 4, 1);
        case 5: return CONVROT_ROWS(2, 1, 5, 1);
        case 6: return CONVROT_ROWS(2, 1, 6, 1);
        case 7: return CONVROT_ROWS(2, 1, 7, 1);
        case 8: return CONVROT_ROWS(2, 1, 8, 1);
        default: return K <= 32768 ? CONVROT_ROWS(2, 1, 8, 2) : CONVROT_ROWS(2, 1, 8, 4);
    }
#undef CONVROT_ROWS
}

}  // namespace

}  // namespace convrot
