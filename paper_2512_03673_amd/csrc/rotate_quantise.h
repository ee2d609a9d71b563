// The rotation and the quantiser of the rotate+quantise kernels, on units of 16 consecutive elements of a row that
// belong to one lane each.
//
// Rotation.  H_g = H_4 (x) ... (x) H_4 (Thm 3.3) is separable: one radix-4 step per base-4 digit
// of the in-group index.  With the printed H_4 (all ones, -1 on the anti-diagonal) a step is
//     y_j = (x_0 + x_1 + x_2 + x_3) - 2 x_{3-j}.
// Digits 0 and 1 live inside a lane's 16 elements: a 16 x 16 matrix of +-1 (H_4 (x) H_4) applied to
// every unit, which is what the otherwise idle matrix pipe does for 64 units at a time, the bf16 -> fp32
// widening and the hand-over of each unit to its lane included (rotation_operand below): the vector ALU,
// which bounds this kernel on small inputs, sees none of it.
// Digits 2, 3 (g = 64, 256) run across lanes with DPP adds and digit 4 (g = 1024) over a lane's four units or, in
// short rows, with lane swaps; across lanes the step is taken as y_j = s - 2 x_j (the matrix J - 2I, which is
// the printed matrix with its columns reversed) and the flip is applied once, for free, to the
// lane's output address.  The 1/sqrt(g) = 2^-k normalisation is folded into the scale.
//
// Quantiser.  a = 2^-k max|z| (exact), s = a / 7 (IEEE division), r = 2^-k / s (IEEE division),
// q = rne(z / (2^k s)) decided exactly from two bracketing multiply-adds, with an exact-residual
// fallback for the few wavefronts that hold a (near-)tie (see the comment at the code).
// |z| / (2^k s) <= 7 (1 + 2^-22), so no clamp is needed.
//
// Output.  The codes leave in the layouts the GEMMs load from (e2m3_layout.h for 4-bit codes,
// panel_layout.h for 8-bit ones).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace convrot {
namespace {

constexpr int kUnit = 16;  // elements per unit

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int v6u __attribute__((ext_vector_type(6)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

// s - 2 x with s the sum over the four lanes that differ in one base-4 digit of the lane id.
template <int CTRL_A, int CTRL_B>
__device__ __forceinline__ float radix4_lanes_dpp(float x)
{
    float t = x + dpp_f32<CTRL_A>(x);
    float s = t + dpp_f32<CTRL_B>(t);
    return fmaf(-2.0f, x, s);
}

// The values of lanes l and l ^ 16 (l ^ 32), in the same order on both: v_permlane16_swap / v_permlane32_swap of a register with
// its copy.  A vector instruction where a wavefront shuffle is a trip through LDS.
__device__ __forceinline__ float radix4_lanes_16_32(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const float t = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return fmaf(-2.0f, x, __uint_as_float(q[0]) + __uint_as_float(q[1]));
}

// Maximum over the lane's row of 16 lanes, and over the whole wavefront, of values that are neither negative nor NaN: their bits
// order as they do, and integers need no canonicalising moves.  (A butterfly of wavefront shuffles waits for LDS four to six times,
// and a rotate+quantise block can do nothing else meanwhile: [12288, 3072] at g = 256 21.7 -> 21.0 us, [8000, 1024] 6.6 -> 6.3.)
template <int CTRL>
__device__ __forceinline__ uint32_t max_dpp(uint32_t x)
{
    return max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float max_of_16(float x)
{
    uint32_t u = max_dpp<0xB1>(__float_as_uint(x));      // quad_perm [1,0,3,2]
    u = max_dpp<0x4E>(u);                                // quad_perm [2,3,0,1]
    return __uint_as_float(max_dpp<0x128>(max_dpp<0x124>(u)));   // row_ror:4, row_ror:8
}
__device__ __forceinline__ float max_of_64(float x)
{
    const uint32_t u = __float_as_uint(max_of_16(x));
    const auto p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const uint32_t m = max((uint32_t)p[0], (uint32_t)p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(m, m, false, false);
    return __uint_as_float(max((uint32_t)q[0], (uint32_t)q[1]));
}

// The digits that live across lanes (in-group index digits 2 and up), on a unit whose digits 0 and 1 are done.
template <int G>
__device__ __forceinline__ void rotate_lanes(float (&v)[kUnit])
{
    if constexpr (G >= 64) {  // lanes l ^ 1, l ^ 2: quad_perm [1,0,3,2] then [2,3,0,1]
#pragma unroll
        for (int e = 0; e < kUnit; ++e) v[e] = radix4_lanes_dpp<0xB1, 0x4E>(v[e]);
    }
    if constexpr (G >= 256) {  // lanes l ^ 8, l ^ 4 inside a row of 16: row_ror:8 then row_ror:4
#pragma unroll
        for (int e = 0; e < kUnit; ++e) v[e] = radix4_lanes_dpp<0x128, 0x124>(v[e]);
    }
    if constexpr (G >= 1024) {
#pragma unroll
        for (int e = 0; e < kUnit; ++e) v[e] = radix4_lanes_16_32(v[e]);
    }
}

// The digits inside a unit on the matrix pipe.  v_mfma_f32_32x32x16_bf16 computes D = A B with B a 16 x 32
// matrix of bf16 whose column n is spread over lanes n (rows 0-7) and n + 32 (rows 8-15), eight consecutive
// rows = 16 contiguous bytes each, and leaves column n of D in lanes n (rows 8 b + r) and n + 32 (rows
// 8 b + 4 + r), register 4 b + r.  With the 32 units of lanes 0-31 as the columns of B and the 16 rows of
// R = H_4 (x) H_4 (I_4 (x) H_4 for g = 4; both symmetric) put at the rows 8 b + r of A, zeros elsewhere, lane n
// receives its whole rotated unit in element order, as fp32; a second MFMA with the rows of R at 8 b + 4 + r and
// the units of lanes 32-63 as B accumulates the other half of the wavefront on top.  Products with +-1 are
// exact and the sums are taken in fp32, as the register butterflies take them; the bf16 -> fp32 widening
// comes with it.  The price is that a lane fetches halves of two other lanes' units instead of its own.
// Returns this lane's eight entries of A for the MFMA that serves lanes 32 * half ... 32 * half + 31.
template <int G>
__device__ __forceinline__ v8bf rotation_operand(int lane, int half)
{
    const int i = lane & 31, kb = lane >> 5;
    const int o = 4 * (i >> 3) + (i & 3);             // element of the unit that accumulator row i holds
    const bool mine = ((i >> 2) & 1) == half;
    union { v8bf v; uint16_t u[8]; } a;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        const int k = 8 * kb + x;
        const bool neg = ((o & 3) + (k & 3) == 3) != (G >= 16 && (o >> 2) + (k >> 2) == 3);
        const bool zero = !mine || (G < 16 && (o >> 2) != (k >> 2));
        a.u[x] = zero ? (uint16_t)0 : (neg ? (uint16_t)0xBF80 : (uint16_t)0x3F80);    // bf16 0, -1, +1
    }
    return a.v;
}

// Digits 0 and 1 of 64 units, one per lane: b0 / b1 = bytes 16 (lane / 32) ... + 15 of the units owned by lanes
// lane % 32 and lane % 32 + 32; v = this lane's unit.
__device__ __forceinline__ void rotate_units_mfma(const v8bf &rot0, const v8bf &rot1, const u32x4 &b0, const u32x4 &b1,
                                                  float (&v)[kUnit])
{
    v16f d = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rot0, __builtin_bit_cast(v8bf, b0), d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rot1, __builtin_bit_cast(v8bf, b1), d, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < kUnit; ++e) v[e] = d[e];
}

template <int G>      // of the digits across lanes
constexpr int lane_flip_mask() { return G >= 1024 ? 63 : (G >= 256 ? 15 : (G >= 64 ? 3 : 0)); }

template <int G>
constexpr float group_norm() { return G == 4 ? 0.5f : G == 16 ? 0.25f : G == 64 ? 0.125f : G == 256 ? 0.0625f : 0.03125f; }

// Codes.  a = 2^-k max|z| (exact), s = a / qmax, q = rne(z / su) with su = s / norm, decided exactly although the lane only
// multiplies.  r approximates 1 / su to 2^-24, so z / su lies strictly between z * r_lo and z * r_hi
// (r_lo, r_hi = r (1 -+ 2^-21)); rounding to an integer is monotonic, hence when both products
// round to the same integer so does the exact quotient.  One fused multiply-add against
// 1.5 * 2^23 (+ an offset) rounds a product to nearest, ties to even, and leaves the integer in
// the low mantissa bits.  A wavefront in which any pair disagrees (a few in a thousand on random
// data; every exact tie, which bf16-grid inputs do produce when the scale is a short dyadic
// number) redoes its codes through the exact residual e = z - q su (one rounding of a quantity
// that is representable whenever q is the nearest or a neighbouring integer), which decides the
// rounding, ties to even, without a division.
struct Quantiser {
    float s, r, su, r_lo, r_hi, half_su;
    __device__ __forceinline__ Quantiser(float amax, float norm, float qmax)
    {
        const float a = amax * norm;                  // exact: power-of-two scaling
        s = (a == 0.0f) ? 1.0f : a / qmax;            // IEEE division
        r = norm / s;                                 // IEEE division
        su = s / norm;                                // scale in un-normalised units (exact)
        r_lo = r * (1.0f - 0x1p-21f);
        r_hi = r * (1.0f + 0x1p-21f);
        half_su = 0.5f * su;
    }
    __device__ __forceinline__ float exact(float z) const   // rne(z / su) as a float, from the exact residual
    {
        float q = rintf(z * r);
        const float res = fmaf(-q, su, z);
        const bool odd = ((int)q & 1) != 0;
        const bool up = res > half_su || (res == half_su && odd);
        const bool dn = res < -half_su || (res == -half_su && odd);
        return q + ((up ? 1.0f : 0.0f) - (dn ? 1.0f : 0.0f));
    }
};

// A unit as a value: handed over as an array it would hold six registers more, which cost [4608, 3072] 3 % of its time.
__device__ __forceinline__ v16f as_vector(const float (&v)[kUnit])
{
    v16f r;
#pragma unroll
    for (int e = 0; e < kUnit; ++e) r[e] = v[e];
    return r;
}

// 4-bit codes leave as FP6 (E2M3) numbers, the operand format of the GEMM's MFMA: every integer in
// [-7, 7] is one.  v_cvt_scalef32_2xpk16_fp6_f32 packs 2 x 16 floats into 6 dwords, interleaving
// its two sources (a0 b0 a1 b1 ...): fed (unit[0..7], next unit[0..7]) and (unit[8..15], next
// unit[8..15]) it returns this unit's 16 codes in dwords 0-2 and the next unit's in dwords 3-5.
// The order of the codes inside a unit does not matter to the GEMM as long as it is the same for
// activations and weights, which it is.
// (`pair` is known where the call is inlined; without it v1 is not looked at.)
__device__ __forceinline__ v6u codes4(const Quantiser &q, bool pair, v16f v0, v16f v1)
{
    constexpr float kMagic = 12582912.0f;                       // 1.5 * 2^23
    // the two brackets agree on every code exactly when the sum of |difference of their bit patterns|
    // is zero (the patterns share their upper halves, so the 16-bit SAD sees the whole difference)
    uint32_t disagree = 0;
    v16f qa, qb;    // conversion sources; the halves of a missing second unit stay unset (their output is not used)
#pragma unroll
    for (int e = 0; e < kUnit; ++e) {
        const float lo0 = fmaf(v0[e], q.r_lo, kMagic), hi0 = fmaf(v0[e], q.r_hi, kMagic);
        disagree = __builtin_amdgcn_sad_u16(__float_as_uint(lo0), __float_as_uint(hi0), disagree);
        if (e < 8) qa[e] = lo0 - kMagic;
        else qb[e - 8] = lo0 - kMagic;
        if (pair) {
            const float lo1 = fmaf(v1[e], q.r_lo, kMagic), hi1 = fmaf(v1[e], q.r_hi, kMagic);
            disagree = __builtin_amdgcn_sad_u16(__float_as_uint(lo1), __float_as_uint(hi1), disagree);
            if (e < 8) qa[8 + e] = lo1 - kMagic;
            else qb[e] = lo1 - kMagic;
        }
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(disagree != 0) != 0, 0)) {   // wavefront-uniform, rare
#pragma unroll
        for (int e = 0; e < kUnit; ++e) {
            const float q0 = q.exact(v0[e]);
            if (e < 8) qa[e] = q0;
            else qb[e - 8] = q0;
            if (pair) {
                const float q1 = q.exact(v1[e]);
                if (e < 8) qa[8 + e] = q1;
                else qb[e] = q1;
            }
        }
    }
    return __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(qa, qb, 1.0f);
}

// 8-bit codes: q + 128 in the low byte of the rounded sum, four codes per dword by a Horner sum over
// the raw float bits, sum_e (C + u_e) 2^(8 e) mod 2^32 with C the magic's bits (the same sum over the
// other bracket: digits differ by at most one, so the two sums are equal exactly when every pair of
// codes is).
__device__ __forceinline__ u32x4 codes8(const Quantiser &q, v16f v)
{
    constexpr uint32_t kOff = 128u;                            // offset that keeps every digit positive
    constexpr float kMagic = 12582912.0f + (float)kOff;
    constexpr uint32_t kC = 0x4B400000u;                       // bits of 1.5 * 2^23
    constexpr uint32_t kFlip = 0x80808080u;                    // offset-binary digits -> two's complement
    constexpr uint32_t kBias = kC + (kC << 8);                 // sum_e C 2^(8 e) mod 2^32: only the first terms survive
    uint32_t disagree = 0;
    u32x4 code;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        uint32_t acc = 0, acc_hi = 0;
#pragma unroll
        for (int e = 3; e >= 0; --e) {
            const float z = v[4 * w + e];
            acc = (acc << 8) + __float_as_uint(fmaf(z, q.r_lo, kMagic));
            acc_hi = (acc_hi << 8) + __float_as_uint(fmaf(z, q.r_hi, kMagic));
        }
        disagree |= acc ^ acc_hi;
        code[w] = (acc - kBias) ^ kFlip;
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(disagree != 0) != 0, 0)) {   // wavefront-uniform, rare
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            uint32_t d = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) d |= ((uint32_t)(int)q.exact(v[4 * w + e]) & 0xFFu) << (8 * e);
            code[w] = d;
        }
    }
    return code;
}

}  // namespace
}  // namespace convrot
