// The rotation and the quantiser of the rotate+quantise kernels, on units of 16 consecutive elements of a row; four units
// are a column of 64.
//
// Rotation.  H_g = H_4 (x) ... (x) H_4 (Thm 3.3) is separable: one radix-4 step per base-4 digit
// of the in-group index.  With the printed H_4 (all ones, -1 on the anti-diagonal) a step is
//     y_j = (x_0 + x_1 + x_2 + x_3) - 2 x_{3-j}.
// Digits 0 and 1 live inside a unit and digit 2 inside a column: a matrix of +-1 (H_4 (x) H_4 (x) H_4) applied to every column,
// which is what the otherwise idle matrix pipe does, the bf16 -> fp32 widening and the hand-over of each unit to its lane
// included (Rotation below): the vector ALU, which bounds these kernels as much as memory does, sees none of it.
// Digits 3 and 4 (g = 256, 1024) run across lanes with DPP adds; there the step is taken as y_j = s - 2 x_j (the matrix
// J - 2I, which is the printed matrix with its columns reversed) and the flip is applied once, for free, to the
// lane's output address.  The 1/sqrt(g) = 2^-k normalisation is folded into the scale.
//
// Quantiser.  a = 2^-k max|z| (exact), s = a / 7 (IEEE division), r = 2^-k / s (IEEE division),
// q = rne(z / (2^k s)) decided exactly from a multiplication and its residual, with an exact
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

// s - 2 x with s the sum over the four lanes that differ in one base-4 digit of the lane id: the neighbour's value minus the lane's
// own, plus the sum of the other two.  (Three roundings of sums of at most two, two and four values; s first and then s - 2 x as a
// fused multiply-add takes three instructions too and rounds one more time.)
template <int CTRL_A, int CTRL_B>
__device__ __forceinline__ float radix4_lanes_dpp(float x)
{
    const float y = dpp_f32<CTRL_A>(x);
    return (y - x) + dpp_f32<CTRL_B>(x + y);
}

// Maximum over the lane's C consecutive lanes and those P, 2 P, ... further on (C = 4 ... 32, P = 16 or 32), of values that are neither negative nor NaN: their bits
// order as they do, and integers need no canonicalising moves.  (A butterfly of wavefront shuffles waits for LDS four to six times,
// and a rotate+quantise block can do nothing else meanwhile: [12288, 3072] at g = 256 21.7 -> 21.0 us, [8000, 1024] 6.6 -> 6.3.)
template <int CTRL>
__device__ __forceinline__ uint32_t max_dpp(uint32_t x)
{
    return max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false));
}
template <int C, int P = 32>
__device__ __forceinline__ float max_of_lanes(float x)
{
    static_assert((C == 4 || C == 8 || C == 16 || C == 32) && (P == 16 || P == 32) && C <= P, "lanes");
    uint32_t u = max_dpp<0xB1>(__float_as_uint(x));      // quad_perm [1,0,3,2]
    u = max_dpp<0x4E>(u);                                // quad_perm [2,3,0,1]
    if constexpr (C >= 8) u = max_dpp<0x141>(u);         // row_half_mirror: the other quad of eight lanes
    if constexpr (C >= 16) u = max_dpp<0x128>(u);        // row_ror:8
    if constexpr (C == 32 || P == 16) {
        const auto p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        u = max((uint32_t)p[0], (uint32_t)p[1]);
    }
    const auto q = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(max((uint32_t)q[0], (uint32_t)q[1]));
}

// The digits that live across lanes (in-group index digits 3 and up), on a unit whose digits 0 to 2 are done; neighbouring
// lanes hold neighbouring columns.
template <int G>
__device__ __forceinline__ void rotate_lanes(float (&v)[kUnit])
{
    if constexpr (G >= 256) {  // lanes l ^ 1, l ^ 2: quad_perm [1,0,3,2] then [2,3,0,1]
#pragma unroll
        for (int e = 0; e < kUnit; ++e) v[e] = radix4_lanes_dpp<0xB1, 0x4E>(v[e]);
    }
    if constexpr (G >= 1024) {  // lanes l ^ 8, l ^ 4 inside a row of 16: row_ror:8 then row_ror:4
#pragma unroll
        for (int e = 0; e < kUnit; ++e) v[e] = radix4_lanes_dpp<0x128, 0x124>(v[e]);
    }
}

// Where the result of lane l's column belongs: column number ^ flip.
template <int G>
constexpr int column_flip() { return G >= 1024 ? 15 : (G >= 256 ? 3 : 0); }

// The digits inside a column on the matrix pipe.  v_mfma_f32_32x32x16_bf16 computes D = A B + C with B a 16 x 32
// matrix of bf16 whose column n is spread over lanes n (rows 0-7) and n + 32 (rows 8-15), eight consecutive
// rows = 16 contiguous bytes each, and leaves column n of D in lanes n (rows 8 b + r) and n + 32 (rows
// 8 b + 4 + r), register 4 b + r.  B is unit c of 32 columns; a lane's sixteen rows of D are one unit in element order,
// as fp32.  With R = H_4 (x) H_4 (both halves of A's rows may hold it, with a sign each; I_4 (x) H_4 for g = 4):
//   g <= 16   lane n gets R x_c of one unit, lane n + 32 of another: two MFMAs, each with zeros in the other's rows of A
//   g >= 64   out_u = R (x_0 + x_1 + x_2 + x_3 - 2 x_{3-u}): four MFMAs with the signs of rows u of H_4 (lanes n) and
//             u + 2 (lanes n + 32) accumulate the whole 64-term sum, 0.125 cycles an element on a pipe that has nothing else
//             to do, where a radix-4 step across lanes took three vector instructions an element
// The odd units (1 and 3) are the even ones' sums with x_c and x_{c^1} exchanged, so that A is the same and a lane may as well
// be given either kind.  Products with +-1 are exact, sums are fp32; the bf16 -> fp32 widening
// comes with it.  The price is that a lane fetches parts of the columns' units instead of its own.  What one column holds never
// meets another (0 x infinity), and a column lies in one row.
template <int G>
struct Rotation {
    v8bf a[G >= 64 ? 3 : 2];

    __device__ __forceinline__ explicit Rotation(int lane)
    {
        // Row i of A: element o = 4 (i / 8) + i % 4 of the unit of lanes n (i / 4 even) or n + 32; this lane's entries are rows
        // k = 8 (lane / 32) + x of R's column o, -1 where the digits (o, k) sum to 3 in one of their two places.
        const int kb = lane >> 5, o1 = (lane >> 3) & 3;
        const bool upper = (lane & 4) != 0;
        const uint64_t minus = (uint64_t)0x8000 << (16 * (3 - (lane & 3)));     // digit 0: four entries of two bytes
        const uint32_t m[2] = {(uint32_t)minus, (uint32_t)(minus >> 32)};
        uint32_t base[4];
#pragma unroll
        for (int x1 = 0; x1 < 2; ++x1) {
            const int k1 = 2 * kb + x1;
#pragma unroll
            for (int w = 0; w < 2; ++w)
                base[2 * x1 + w] = G < 16 ? (o1 == k1 ? 0x3F803F80u ^ m[w] : 0u) : (o1 + k1 == 3 ? 0xBF80BF80u : 0x3F803F80u) ^ m[w];
        }
        u32x4 r[3];
        const uint32_t u = upper ? 0xFFFFFFFFu : 0u;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if constexpr (G >= 64) {
                r[0][w] = base[w];
                r[1][w] = base[w] ^ (u & 0x80008000u);       // minus in the rows of lanes n + 32
                r[2][w] = base[w] ^ (~u & 0x80008000u);      // minus in the rows of lanes n
            } else {
                r[0][w] = base[w] & ~u;
                r[1][w] = base[w] & u;
            }
        }
#pragma unroll
        for (int i = 0; i < (G >= 64 ? 3 : 2); ++i) a[i] = __builtin_bit_cast(v8bf, r[i]);
    }

    // This lane's unit: of an even pair (unit 0, in lanes n + 32 unit 2) from the bytes b(c) of unit c, of an odd pair (1, 3)
    // from those of unit c ^ 1.  b(c) = 16 (lane / 32) ... + 15 of the unit's 32 bytes; g <= 16 asks for c = 0 and 2 only.
    template <class B>
    __device__ __forceinline__ void apply(B b, float (&v)[kUnit]) const
    {
        v16f d = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (G >= 64) {      // rows 0 and 2 of H_4: + + + -, + - + +
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], __builtin_bit_cast(v8bf, b(0)), d, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], __builtin_bit_cast(v8bf, b(1)), d, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], __builtin_bit_cast(v8bf, b(2)), d, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], __builtin_bit_cast(v8bf, b(3)), d, 0, 0, 0);
        } else {
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], __builtin_bit_cast(v8bf, b(0)), d, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], __builtin_bit_cast(v8bf, b(2)), d, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < kUnit; ++e) v[e] = d[e];
    }
};

// 1024 elements of a row (64 units from unit `base` on, 16 columns) that a wavefront rotates at a time, a unit a lane, loaded a
// kilobyte an instruction: every block of a launch asks for the same few lines, and an instruction that takes halves of them asks twice.
// With g >= 64 they are loaded as they lie and change lanes in kBytes of LDS that are the wavefront's own: lanes n and n + 32 need the
// halves of column n's units (one-launch forwards, us, through LDS / units n in 64-byte pieces straight to their lanes, with the
// pairs that two lanes need loaded twice / loaded once and exchanged between rows of 16 lanes: M2 x N1536 x K3072 at g = 64 and 8 bits 4.39 / 5.07 / 4.72,
// M4 x N3072 x K3072 at 4 bits 5.04 / 6.34 / 5.58).  Piece p of column n lies in slot p ^ (n & 7), so that eight lanes read and write different banks.
// With g <= 16 no digit needs a column: lanes n and n + 32 load the halves of unit n, then of unit n + 32, which is where the MFMAs want them
// (through LDS / so: M4 x N3072 x K3072 at g = 4 and 8 bits 6.54 / 6.35, M2 x N750 x K6144 6.23 / 6.07, M8 x N1024 x K1024 at 4 bits 4.05 / 3.92).
template <int G>
struct Item {
    static constexpr bool kColumns = G >= 64;
    static constexpr int kBytes = kColumns ? 2048 : 16;
    static __device__ __forceinline__ int unit(int lane) { return kColumns ? 4 * (lane & 15) + ((lane >> 4) & 1) + 2 * (lane >> 5) : lane; }
    static __device__ __forceinline__ int out_unit(int lane) { return unit(lane ^ column_flip<G>()); }
    static __device__ __forceinline__ void load(const uint16_t *row, int base, int units, int lane, u32x4 (&raw)[2])
    {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int at = kColumns ? min(base * 32 + j * 1024 + lane * 16, units * 32 - 16)      // past the row's end its last 16 bytes again
                                    : min(base + j * 32 + (lane & 31), units - 1) * 32 + (lane >> 5) * 16;      // ... its last unit
            raw[j] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const uint8_t *>(row) + at);
        }
    }
    static __device__ __forceinline__ void rotate(const Rotation<G> &rot, const u32x4 (&raw)[2], uint8_t *lds, int lane, float (&v)[kUnit])
    {
        if constexpr (kColumns) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
                *reinterpret_cast<u32x4 *>(lds + j * 1024 + (lane >> 3) * 128 + (((lane & 7) ^ (lane >> 3)) << 4)) = raw[j];
            asm volatile("" ::: "memory");       // (other lanes' pieces; a wavefront's LDS operations stay in order)
            const int odd = (lane >> 4) & 1, h = lane >> 5;
            rot.apply([&](int c) { return *reinterpret_cast<const u32x4 *>(lds + (lane & 15) * 128 + (((2 * (c ^ odd) + h) ^ (lane & 7)) << 4)); }, v);
            asm volatile("" ::: "memory");
            rotate_lanes<G>(v);
        } else {
            rot.apply([&](int c) { return raw[c / 2]; }, v);
        }
    }
};

template <int G>
constexpr float group_norm() { return G == 4 ? 0.5f : G == 16 ? 0.25f : G == 64 ? 0.125f : G == 256 ? 0.0625f : 0.03125f; }

// Codes.  a = 2^-k max|z| (exact), s = a / qmax, q = rne(z / su) with su = s / norm, decided exactly although the lane only
// multiplies.  One fused multiply-add against 1.5 * 2^23 (+ an offset) rounds a product to nearest, ties to even, and leaves the
// integer in the low mantissa bits.  Whether the exact quotient rounds to the same integer is known from
//   4 bits   the residual z r - q: r approximates 1 / su to 2^-24, so it is within 7 * 2^-24 + 2^-26 < 2^-20 of z / su - q, and a
//            residual of at most 1/2 - 2^-20 says that q is the nearest integer
//   8 bits   a second product: z / su lies strictly between z * r_lo and z * r_hi (r_lo, r_hi = r (1 -+ 2^-21)), rounding is
//            monotonic, hence when both round to the same integer so does the exact quotient
// A wavefront in which any code is not known so (a few in a thousand on random
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
    float worst = 0.0f;                                         // largest residual
    v16f qa, qb;    // conversion sources; the halves of a missing second unit stay unset (their output is not used)
#pragma unroll
    for (int e = 0; e < kUnit; ++e) {
        const float q0 = fmaf(v0[e], q.r, kMagic) - kMagic;
        worst = fmaxf(worst, fabsf(fmaf(v0[e], q.r, -q0)));
        if (e < 8) qa[e] = q0;
        else qb[e - 8] = q0;
        if (pair) {
            const float q1 = fmaf(v1[e], q.r, kMagic) - kMagic;
            worst = fmaxf(worst, fabsf(fmaf(v1[e], q.r, -q1)));
            if (e < 8) qa[8 + e] = q1;
            else qb[e] = q1;
        }
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(worst > 0.5f - 0x1p-20f) != 0, 0)) {   // wavefront-uniform, rare
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
