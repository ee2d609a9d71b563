// Shared pieces of the GEMM kernels of libconvrot, 4-bit and 8-bit (LDS swizzle, LDS-direct loads, which the
// rotate+quantise kernel uses too, stores of Y).  gemm_tiled.h and gemm_small.h describe the method, gemm_plan.h the tile order.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "fragment_rows.h"
#include "gemm_plan.h"

namespace convrot {
namespace gemm {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

// Which of the four 16-byte slots of its LDS row a piece of row 0 ... 15 of a panel lands in: slot = piece ^ swz(row) (fragment_rows.h).
__device__ __forceinline__ int swz(int row) { return ((row >> 1) ^ (row >> 3)) & 3; }

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    // gfx9 encoding: vmcnt = {imm[15:14], imm[3:0]}, expcnt = imm[6:4], lgkmcnt = imm[11:8]
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// The same, and every LDS (and scalar memory) operation of the wavefront returned as well.
template <int N>
__device__ __forceinline__ void wait_vmcnt_lgkm0()
{
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0x0 << 8));
}

// global_load_lds_dwordx4: lane l copies 16 bytes from its global address to LDS address M0 + 16 l.
// M0 is written here and not named as a clobber.  This relies on a property of the AMDGPU backend, not on a
// documented contract: M0 is a reserved register that the register allocator never assigns a value to; every
// instruction the backend itself emits that reads M0 (LDS-direct loads from the builtin, s_movrel, GWS, s_sendmsg)
// is preceded by its own write in the same block.  Naming a reserved register in a clobber list is rejected with
// a warning ("may not be preserved ... may lead to undefined behaviour") and changes nothing in the generated code,
// so it would only look like a guarantee.  None of the instructions above occurs in the GEMM kernels besides this
// one (the build prints the hipcc version it ran with, and the bit-exact GEMM tests are the check that a new
// toolchain still behaves so: a stale M0 sends a kilobyte of operands to the wrong place in the ring).
// (STREAM: data that is read once and should not push other lines out of the caches.)
template <bool STREAM = false>
__device__ __forceinline__ void lds_dma16(const uint8_t *base, uint32_t lane_off, uint32_t lds_addr)
{
    if constexpr (STREAM)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" :: "v"(lane_off), "s"(base), "s"(lds_addr) : "memory");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(lane_off), "s"(base), "s"(lds_addr) : "memory");
}
// A sum that is to stay one: constants added to it later become offsets of the memory instructions, where the compiler would
// rather hold base + constant of each of them in a register through a loop and add to it every time (fragment reads: 4 additions
// a step instead of 12, M512 x N12288 x K3072 13.7 -> 13.1 us, M2000 x N3072 x K3072 13.8 -> 13.1).
__device__ __forceinline__ void keep(uint32_t &v) { asm("" : "+v"(v)); }

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b)
{
    v2bf r = __builtin_convertvector((v2f){a, b}, v2bf);   // v_cvt_pk_bf16_f32: round to nearest even
    return *reinterpret_cast<uint32_t *>(&r);
}

// Eight (four) bf16 of a row of Y.  A row starts at any multiple of two bytes when N is odd; the memory path takes
// such addresses in one store, and the compiler is told no more than that.
typedef uint32_t u32x4_row __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x2_row __attribute__((ext_vector_type(2), aligned(2)));
typedef int32_t i32x2_row __attribute__((ext_vector_type(2), aligned(4)));      // two accumulators of a row

// Eight bf16 of a row of Y; but for kCached `out` is a multiple of 16 bytes.  (The wait state is the one that a store of more than 64 bits
// needs before its data registers are written again, which the compiler cannot see in the asm.)
template <Store KIND>
__device__ __forceinline__ void store_row(uint16_t *out, const v4i &v)
{
    if constexpr (KIND == Store::kPast) __builtin_nontemporal_store(v, reinterpret_cast<v4i *>(out));
    else if constexpr (KIND == Store::kThrough) asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(out), "v"(v) : "memory");
    else *reinterpret_cast<u32x4_row *>(out) = __builtin_bit_cast(u32x4_row, v);
}

// One product, as the launchers pass it on: the arguments of launch_gemm_w4a4 / launch_gemm_w8a8.
struct Operands {
    const void *Xq;
    const float *x_scale;
    const void *Wq;
    const float *w_scale;
    const void *bias;
    int M, N, K;
    void *Y;          // bf16 output, or
    int32_t *acc;     // raw accumulators
    hipStream_t stream;
    Store store = Store::kCached;     // of Y, where a tiled kernel writes it
};

}  // namespace gemm

}  // namespace convrot
