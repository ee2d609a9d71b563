// The tiled GEMM kernel of libconvrot, shared by the 4-bit and the 8-bit layer (gemm_w4a4.hip, gemm_w8a8.hip).
//
//   acc[m,n] = sum_k q_x[m,k] q_w[n,k]        exact
//   Y[m,n]   = bf16( float(acc) * s_x[m] * s_w[n] + bias[n] )
//
// `C` (Codes4 / Codes8) says what a stage of the operands looks like in memory and how a fragment is read from LDS and
// multiplied; `T` (Tile) is the block's share of the output.
//
// Data movement.  A block of WGM x WGN wavefronts owns a TM x TN tile of the output.  A K stage of the tile's operand
// rows is kPieces contiguous kilobytes in memory, copied by LDS-direct loads (dealt evenly to the wavefronts)
// into a ring of NS stage buffers.  A fragment is 16 rows of a whole stage and one operand of an MFMA.  A stage is two steps, in which a wavefront
// multiplies the first and the second half of its X fragments by all of its W fragments; it holds one stage's fragments and reads each of the next one's
// in the slots behind the last use of the one whose registers it takes, so that no MFMA waits for LDS.
//
// The block meets once per stage, between its two steps: by then every wavefront has read the whole of stage s into
// registers, so the buffer can take stage s + NS, and everybody's share of stage s + 1 has landed.  With NS = 2 the
// refill has to be issued at once, in the second step of stage s; with more stages half of it waits for the first
// step of stage s + 1, so that the load path has work in both halves of the stage (it would otherwise idle in one and
// hold up the MFMAs in the other: 256 x 128 tiles, eight wavefronts, M512 x N12288 x K3072, 17.2 -> 16.4 us).
//
// A block's first MFMA waits for the arguments, the tile's place, addresses and the first stage's way from memory, with nothing to hide them
// behind but, in products of a few rounds, another block.  So arguments come in registers, in the order they are needed, the place without divisions,
// a wavefront loads whole groups of rows (one address for three pieces), the first stage is issued before anything else is asked for, and
// the last buffer's stage not before the first MFMAs.  By the device's clock from a block's start, 256 x 256 tiles at 4 bits with a bias: first
// operands there after 1.4 us, where five dependent loads of arguments, two divisions and a bias that was widened (hence waited for) first
// took 3.1; M2000 x N3072 x K3072 13.7 -> 13.25 us, M500 x N4096 x K2048 at 8 bits 9.1 -> 8.5, M300 x N2000 x K512 (gemm_small.h) 3.6 -> 3.35, a product of three
// rounds, where the power that is saved in a pause is spent after it, 0.5 to 3 %.
//
// A wavefront issues in order, so every memory instruction gets an MFMA slot of its own (scheduling barriers pin the
// order) instead of queueing up in a burst.
//
// MFMAs are 16 x 16, 128 codes deep at 4 bits and 64 at 8, with the X fragment as the row operand: of the forms that the chip runs at one rate this
// takes the least power, and the clock falls with power.  A register-only loop on codes like a layer's, POP/s, 32 x 32 with W / X as the row
// operand : 16 x 16 with W / X: 4 bits, X of g = 16 (one code in seven not zero) 7.6 / 7.2 : 8.1 / 8.6, g = 64 6.7 / 6.6 : 7.4 / 7.5, g = 1024 6.4 / 6.4 : 7.2 / 7.2; 8 bits
// 3.5 : 4.2; zeros 9.7 : 9.6 and 4.9 : 4.8.  The GEMM alone, us, 32 x 32 with W / 16 x 16 with X, operands changing: 4 bits M4608 x N12288 x K3072 77.3 / 74.7,
// M16896 x N3072 x K12288 254 / 233, 8 bits M4608 x N12288 x K3072 136.3 / 127.4.  A lane of the result has four rows of one column; pairs of fragments share
// their rows so that it has two neighbouring columns of each (fragment_rows.h), and the epilogue scales, rounds to bf16, transposes through LDS and
// writes 16 bytes per lane, whole contiguous rows of the wavefront's tile, in or past the caches (store_kind).
//
// What bounds the large tiles is power, by the clock, and waits: M4608 x N12288 x K3072 at 4 bits takes 81 to 84 us on a layer's codes and 66 on zeros, and of the former's cycles
// the matrix pipe is busy for 47 %, at N3072 x K12288 for 53 %, at 8 bits for 68 %.  Operand bytes cost both.  So the tile that moves the fewest bytes a product wins where its rounds are not too uneven: 256 x 256
// on eight wavefronts with a ring of three stages (150 KB, the compute unit to itself) against two 192 x 192 or 256 x 128 blocks
// a unit, us: 4 bits M4608 x N3072 x K12288 73.1 / 71.1 -> 60.8, K3072 23.9 / 23.2 -> 20.2, N9216 70.2 / 69.7 -> 66.1; 8 bits
// M4608 x N3072 x K12288 137.5 / 132.9 -> 126.  (A ring of two: 68.6 -> 80.6.  A 288 x 192 tile fills 256 units exactly at M4608 x N3072,
// where 256 x 256 leaves 40 idle, and is slower, 72.5 against 68.6: idle units leave their power to the others.)
//
// Products of one round or less are bound by a lone tile's walk along K, 0.3 to 0.4 us a stage.  Tiles that otherwise share a unit two by
// two wait for operands there and take a ring of four stages, which their lone unit has the LDS for (deep_ring); for 256 x 128 on
// eight wavefronts and 192 x 192 at 8 bits a fourth stage made no difference, nor did fragments read a whole stage ahead instead of a step on any tile.
// What is left is to spread such a product over the most units: 128 x 192, us: 4 bits M512 x N12288 x K3072 14.9 -> 13.8, M578 x N9408 x K9600 34.2 -> 31.0; 8 bits
// M854 x N6464 x K1024 11.0 -> 10.1, M1803 x N5056 x K4992 49.2 -> 46.2.
#pragma once
#include "gemm_common.h"
#include "gemm_plan.h"

namespace convrot {
namespace gemm {

// WGM x WGN wavefronts of XF x WF 32 x 32 shares of the output each (2 XF x 2 WF accumulator tiles), NS stage buffers, OCC wavefronts per SIMD that the
// registers have to leave room for, BAND tile rows per band of the XCD-aware tile order.
template <int WGM_, int WGN_, int XF_, int WF_, int NS_, int OCC_, int BAND_>
struct Tile {
    static constexpr int WGM = WGM_, WGN = WGN_, XF = XF_, WF = WF_, NS = NS_, OCC = OCC_, kBandRows = BAND_;
    static constexpr int NW = WGM * WGN, kThreads = 64 * NW;
    static constexpr int WM = XF * 32, WN = WF * 32;          // wavefront tile
    static constexpr int TM = WGM * WM, TN = WGN * WN, kRows = TM + TN;
    static constexpr int kXs = 2 * XF, kWs = 2 * WF;          // fragments (16 rows) of a stage per wavefront
    static constexpr int kMfmas = XF * kWs;                   // slots of a step: half of the X fragments with every W fragment
    // Two MFMAs a step take less time than a read: all of the next stage's fragments are read behind the meeting, with one wait for them.  (64 x 64 tiles alone on
    // their unit, us, one of them read in the next step / so: M256 x N3072 x K3072 6.6 / 6.35, M804 x N1216 x K9216 13.85 / 13.15.)
    static constexpr bool kAtOnce = kMfmas == 2;
    static constexpr bool kSpare = kXs * kWs < 32;            // registers to spare: the last stage apart, the epilogue's addresses early
    static constexpr int kEpiBytes = NW * 32 * WN * 2;        // 32 rows of every wavefront's tile in bf16
};

template <class C, class T>
struct Stage {
    static constexpr int kBytes = T::kRows * C::kRowBytes;    // a K stage of the tile's operand rows, X rows first
    static constexpr int kPieces = kBytes / 1024;
    static constexpr int kLoads = kPieces / T::NW;            // loads per wavefront and stage ...
    static constexpr int kExtra = kPieces % T::NW;            // ... and one more for this many wavefronts
    static constexpr int kMaxLoads = kLoads + (kExtra != 0);
    static constexpr int kRing = T::NS * kBytes;
    static constexpr int kScales = kRing > T::kEpiBytes ? kRing : T::kEpiBytes;     // scales and bias, past the ring
    static constexpr int kLds = kScales + (T::TM + 2 * T::TN) * 4;
    static_assert(kPieces * 1024 == kBytes && T::NW % 2 == 0, "stage must split into kilobytes");
    static_assert(T::NS >= 2 && T::NS <= 4 && T::kRows % 64 == 0, "ring");
    static_assert(kLds * (T::OCC * 4 / T::NW) <= 160 * 1024, "blocks per compute unit");
};

// f(0), f(1), ... f(N - 1), each with its number as a constant.
template <class F, int... I>
__device__ __forceinline__ void each_of(const F &f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void each(const F &f)
{
    each_of(f, std::make_integer_sequence<int, N>{});
}

enum class Refill { kNone, kShare, kAll };      // the loads of a stage that a step issues: its share of them, or all

struct Product {      // what every block of a launch is told
    const uint8_t *Xq;
    const float *x_scale;
    const uint8_t *Wq;
    const float *w_scale;
    const uint16_t *bias;
    int M, N, K;
    uint16_t *Y;
    int32_t *acc_out;
    Store store;
};

// The tile of the output from row m0 and column n0 on; `lds` holds Stage<C, T>::kLds bytes.
template <class C, bool RAW, class T>
__device__ __forceinline__ void tile_product(const Product &p, int m0, int n0, uint8_t *lds)
{
    using St = Stage<C, T>;
    constexpr int TM = T::TM, TN = T::TN, WM = T::WM, WN = T::WN, XF = T::XF, kXs = T::kXs, kWs = T::kWs, NW = T::NW, NS = T::NS;
    constexpr int kMfmas = T::kMfmas, kLoads = St::kLoads, kMaxLoads = St::kMaxLoads;
    constexpr bool kUneven = St::kExtra != 0;
    const uint8_t *const Xq = p.Xq, *const Wq = p.Wq;
    const float *const x_scale = p.x_scale, *const w_scale = p.w_scale;
    const uint16_t *const bias = p.bias;
    const int M = p.M, N = p.N, K = p.K;
    uint16_t *const Y = p.Y;
    int32_t *const acc_out = p.acc_out;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave % T::WGM) * WM, wn0 = (wave / T::WGM) * WN;
    const int KS = C::stages(K);   // the last one is zero-padded

    // ---- global -> LDS (direct).  A stage of kGroupRows rows is kGroupPieces consecutive kilobytes.  Wavefront w loads groups w, w + NW, ... of the
    // tile's (X rows first) whole and a share of the pieces of those that are left.  Rows past the
    // operand's last block (edge tiles) re-read that block, whose results are never stored.
    constexpr int kGroups = T::kRows / C::kGroupRows, kXGroups = TM / C::kGroupRows, kOwn = kGroups / NW, kP = C::kGroupPieces;
    constexpr int kOwnLoads = kOwn * kP, kRest = (kGroups - kOwn * NW) * kP;
    static_assert(kGroups * kP == St::kPieces && kXGroups * C::kGroupRows == TM, "groups of a stage");
    const uint8_t *src[kMaxLoads];   // stage 0 source of each of this wavefront's loads (wavefront-uniform)
    uint32_t dst[kMaxLoads];         // its place in a stage buffer
    const uint32_t group_bytes = (uint32_t)KS * C::kStageStride;
    auto group_source = [&](int g) {
        const bool is_x = g < kXGroups;
        const int at = is_x ? min(m0 / C::kGroupRows + g, (M - 1) / C::kGroupRows) : min(n0 / C::kGroupRows + g - kXGroups, (N - 1) / C::kGroupRows);
        return (is_x ? Xq : Wq) + (uint64_t)(uint32_t)at * group_bytes;
    };
#pragma unroll
    for (int i = 0; i < kMaxLoads; ++i) {
        const int j = wave + NW * (i - kOwnLoads);            // past the wavefront's own groups
        const int rest = kUneven ? min(j, kRest - 1) : j;
        const int g = i < kOwnLoads ? wave + NW * (i / kP) : kOwn * NW + rest / kP, part = i < kOwnLoads ? i % kP : rest % kP;
        src[i] = group_source(g) + part * 1024;
        dst[i] = C::template piece_place<T::kRows>(g, part);
    }
    const bool extra = kUneven && wave < St::kExtra;    // this wavefront has kMaxLoads loads
    // LDS-direct loads are issued from inline assembly so that the compiler does not serialise every
    // later LDS read behind them; completion is tracked by hand with vmcnt.
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;
    const uint32_t lane_off = C::lane_offset(lane);
    auto load_piece = [&](auto IC, int s, uint32_t buf) {   // load i of this wavefront's share of stage s
        constexpr int i = decltype(IC)::value;
        if constexpr (i < kMaxLoads)
            if (i < kLoads || extra) lds_dma16(src[i], lane_off + (uint32_t)s * C::kStageStride, lds_base + buf + dst[i]);
    };
    auto load_stage = [&](int s, uint32_t buf) {
#define CONVROT_L(i) load_piece(std::integral_constant<int, i>{}, s, buf);
        CONVROT_L(0) CONVROT_L(1) CONVROT_L(2) CONVROT_L(3) CONVROT_L(4) CONVROT_L(5) CONVROT_L(6) CONVROT_L(7) CONVROT_L(8)
#undef CONVROT_L
        static_assert(kMaxLoads <= 9, "loads of a stage");
    };
    // all of this wavefront's loads but those of the `n` youngest stages have landed; its LDS reads have returned
    auto wait_loads = [&](auto NI) {
        constexpr int n = decltype(NI)::value;
        if constexpr (kUneven) {
            if (extra) wait_vmcnt_lgkm0<n * kMaxLoads>();
            else wait_vmcnt_lgkm0<n * kLoads>();
        } else {
            wait_vmcnt_lgkm0<n * kLoads>();
        }
    };
    auto wait_loads_upto = [&](int n) {      // the same for a count known at run time (the last stages)
        if (NS > 3 && n >= 3) wait_loads(std::integral_constant<int, 3>{});
        else if (NS > 2 && n == 2) wait_loads(std::integral_constant<int, 2>{});
        else if (n == 1) wait_loads(std::integral_constant<int, 1>{});
        else wait_loads(std::integral_constant<int, 0>{});
    };

    // ---- LDS -> registers
    typename C::Reader reader(lane, T::kRows, wm0, TM + wn0);
    typename C::Op xop[kXs], wop[kWs];      // of the stage; fragments f and f + 1, f even, share 32 rows (fragment_rows.h)
    auto read_x = [&](auto F) { xop[decltype(F)::value] = reader.template read<0, decltype(F)::value>(lds); };
    auto read_w = [&](auto F) { wop[decltype(F)::value] = reader.template read<1, decltype(F)::value>(lds); };

    typename C::Acc acc[kXs][kWs];
#pragma unroll
    for (int i = 0; i < kXs; ++i)
#pragma unroll
        for (int j = 0; j < kWs; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0;

    // Step ks of a stage, slot by slot, in issue order: X fragments XF ks ... XF ks + XF - 1 with W fragment 0, then with 1, ... (there and back, so that
    // one operand stays from every MFMA to the next).  Slot m: MFMA; with REFILL this slot's share of the LDS-direct loads of stage rs into
    // buffer rbuf; a fragment.  The second step reads what the next stage starts with: the first half of its X, whose registers the first step
    // has left, and W fragment j as soon as it is done with the present one; the first step reads the last W fragment and the other half of X.  Spread over
    // the step, behind their MFMAs: 96 stages on all-zero codes, where only cycles count, 61.1 us with the reads in the first slots, 57.4 so.
    auto slot = [&](auto MI, auto KSI, auto REFILL, auto READS, int rs, uint32_t rbuf) {
        constexpr int m = decltype(MI)::value, ks = decltype(KSI)::value, j = m / XF;
        constexpr int i = ks * XF + (j % 2 ? XF - 1 - m % XF : m % XF);
        C::mma(acc[i][j], xop[i], wop[j]);
        if constexpr (decltype(REFILL)::value != Refill::kNone) {
            // NS = 2: everything in the second step; otherwise its second half in the first step of the next stage
            constexpr bool all = decltype(REFILL)::value == Refill::kAll;
            constexpr int half = all ? 0 : NS > 2 ? kMaxLoads / 2 : kMaxLoads;
            constexpr int first = ks == 1 ? 0 : half, count = ks == 1 ? half : kMaxLoads - half;
            constexpr int l0 = first + m * count / kMfmas, l1 = first + (m + 1) * count / kMfmas;
            static_assert(l1 - l0 <= 3, "loads per slot");
            if constexpr (l0 < l1) load_piece(std::integral_constant<int, l0>{}, rs, rbuf);
            if constexpr (l0 + 1 < l1) load_piece(std::integral_constant<int, l0 + 1>{}, rs, rbuf);
            if constexpr (l0 + 2 < l1) load_piece(std::integral_constant<int, l0 + 2>{}, rs, rbuf);
        }
        __builtin_amdgcn_sched_barrier(0);
        constexpr int gap = XF > 1 ? XF - 1 : 1;
        if constexpr (!decltype(READS)::value) {
        } else if constexpr (T::kAtOnce) {
            if constexpr (ks == 1) {
                if constexpr (m == 0) read_x(std::integral_constant<int, 0>{});
                read_w(MI);
                if constexpr (m == kMfmas - 1) read_x(std::integral_constant<int, 1>{});
            }
        } else if constexpr (ks == 1) {
            if constexpr (m % gap == 0 && m / gap < XF) read_x(std::integral_constant<int, m / gap>{});
            if constexpr (m > 0 && m % XF == 0) read_w(std::integral_constant<int, j - 1>{});
        } else {
            if constexpr (m == 0) read_w(std::integral_constant<int, kWs - 1>{});
            if constexpr (m > 0 && (m - 1) % gap == 0 && (m - 1) / gap < XF) read_x(std::integral_constant<int, XF + (m - 1) / gap>{});
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto step = [&](auto KSI, auto REFILL, auto READS, int rs, uint32_t rbuf) {
        __builtin_amdgcn_sched_barrier(0);
        each<kMfmas>([&](auto MI) { slot(MI, KSI, REFILL, READS, rs, rbuf); });
    };

    // ---- pipeline
    using K0 = std::integral_constant<int, 0>;
    using K1 = std::integral_constant<int, 1>;
    using No = std::integral_constant<Refill, Refill::kNone>;
    using Yes = std::integral_constant<Refill, Refill::kShare>;
    using All = std::integral_constant<Refill, Refill::kAll>;
    load_stage(0, 0);
    // Dequantisation scales of the tile's rows and columns: thread t fetches x_scale[m0 + t] and
    // w_scale[n0 + t] now, so that the latency hides under the main loop, and parks them in LDS (past
    // the ring) once the loop is over.  Behind the first stage and with nothing done to them, so that no operand waits for them (vmcnt counts in order;
    // with the bias widened here the whole block waited for it first); past an operand's end the last one again.
    static_assert(TM <= T::kThreads && TN <= T::kThreads, "one scale per thread");
    float my_sx = 0.0f, my_sw = 0.0f;
    uint16_t my_b = 0;
    if constexpr (!RAW) {
        __builtin_amdgcn_sched_barrier(0);
        my_sx = x_scale[min((uint32_t)m0 + tid, (uint32_t)M - 1)];
        const uint32_t n = min((uint32_t)n0 + tid, (uint32_t)N - 1);
        my_sw = w_scale[n];
        if (bias) my_b = bias[n];
        __builtin_amdgcn_sched_barrier(0);
    }
    // (The last buffer's stage can wait for the first MFMAs, unless the product is shorter than the ring.)
    const bool late = NS > 2 && KS > NS;
#pragma unroll
    for (int p = 1; p < NS; ++p)
        if (p < KS && !(p == NS - 1 && late)) load_stage(p, p * St::kBytes);
    wait_loads_upto((late ? NS - 1 : min(KS, NS)) - 1);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    each<T::kAtOnce ? kXs : XF>(read_x);
    each<T::kAtOnce ? kWs : kWs - 1>(read_w);

    int s = 0;
    uint32_t buf = 0;      // stage s's buffer
    auto stage = [&](auto REST, auto REFILL, auto WAIT) {
        const uint32_t next = buf + St::kBytes == St::kRing ? 0 : buf + St::kBytes;
        const uint32_t prev = buf == 0 ? St::kRing - St::kBytes : buf - St::kBytes;
        step(K0{}, REST, std::true_type{}, s - 1 + NS, prev);      // fetches the other fragments of the stage
        __builtin_amdgcn_sched_barrier(0);
        reader.advance(next - buf);               // (here and not behind the barrier, where every wavefront would wait for it)
        __builtin_amdgcn_sched_barrier(0);
        WAIT();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        step(K1{}, REFILL, std::true_type{}, s + NS, buf);         // fetches the first fragments of stage s + 1
        buf = next;
        ++s;
    };
    auto steady = [&]() { wait_loads(std::integral_constant<int, NS - 2>{}); };
    auto drain = [&]() { wait_loads_upto(max(min(KS - 2 - s, NS - 2), 0)); };
    if constexpr (NS == 2) {
        while (s < KS - NS) stage(No{}, Yes{}, steady);
    } else if (KS > NS) {
        stage(All{}, Yes{}, steady);
        while (s < KS - NS) stage(Yes{}, Yes{}, steady);
        // (Of raw accumulators, where registers are short, in a loop of one trip, which keeps every accumulator in its registers: the straight copy of the stage spills eight
        // there.  Outputs of 256 x 256 tiles are no faster so, and tiles alone on their unit slower.)
        int once = 1;
        if constexpr (RAW && !T::kSpare && T::OCC == 2) asm volatile("" : "+s"(once));
        do stage(Yes{}, No{}, steady);
        while (--once > 0);
    }
    while (s < KS - T::kSpare) stage(No{}, No{}, drain);          // (what the very last step fetches is unused)

    // The scales, parked so that a lane finds those of its four rows of an X fragment side by side, and a W fragment's columns in lane order.
    float *const sx_lds = reinterpret_cast<float *>(lds + St::kScales), *const sw_lds = sx_lds + TM;
    auto park = [&](int t) {
        const int c = (t & 31) >> 1, half = (t & 1) ^ crossed(c);
        if (t < TM) sx_lds[(t & ~31) + (c >> 2) * 8 + half * 4 + (c & 3)] = my_sx;
        if (t < TN) {
            sw_lds[(t & ~31) + half * 16 + c] = my_sw;
            sw_lds[TN + (t & ~31) + half * 16 + c] = bf16_to_f32(my_b);
        }
    };
    if constexpr (T::kSpare) {
        // The last stage, of which nothing is read ahead.  Between its steps all loads and LDS reads of the block are over, so that is the last meeting: the ring may
        // be written from there on, and scales that were parked before be read (with the meeting after it M5000 x N4000 x K256 13.25 us, so 13.0; where
        // registers are short the compiler's copy of the stage spills).  The scales are plain stores, which the fences of __syncthreads keep on their side of the
        // meeting; what the loop's meetings hand over has been loaded by inline assembly, which they wait for by hand.
        step(K0{}, No{}, std::true_type{}, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        wait_loads(std::integral_constant<int, 0>{});
        if constexpr (!RAW) park(tid);
        __syncthreads();
        step(K1{}, No{}, std::false_type{}, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- epilogue.  Lane l, register r of accumulator tile (i, j): row 32 (i / 2) + row_of(4 (l / 16) + r, i % 2), column 32 (j / 2) +
    // row_of(l % 16, j % 2) of the wavefront's.
    uint32_t late_tid = threadIdx.x;      // (what follows from it is computed here, not held in registers through the loop)
    if constexpr (!T::kSpare) keep(late_tid);
    const int tid2 = late_tid, lane2 = tid2 & 63, quad = lane2 >> 4, col16 = lane2 & 15;
    if constexpr (RAW) {
        // A lane's two neighbouring columns at once, eight bytes at any multiple of four, so that sixteen lanes write 128 bytes in a row.  us, four bytes at a time (and, the
        // first, eight registers spilled) / so: 4 bits M9559 x N2845 x K2208 53.7 / 48.0, M2153 x N10560 x K128 19.6 / 16.3, 8 bits M2927 x N10368 x K768 41.2 / 37.2.
        const int32_t n = n0 + wn0 + 2 * col16, swap = crossed(col16);
#pragma unroll
        for (int i = 0; i < kXs; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm0 + i / 2 * 32 + row_of(quad * 4 + r, i % 2);
                if (m >= M) continue;
                int32_t *const row = acc_out + (int64_t)m * N + n;
#pragma unroll
                for (int j = 0; j < kWs; j += 2) {
                    const int32_t a = (int32_t)acc[i][j][r], b = (int32_t)acc[i][j + 1][r];   // exact: a float holds an integer below 2^24
                    const i32x2_row two = {swap ? b : a, swap ? a : b};
                    if (n + j * 16 + 1 < N) *reinterpret_cast<i32x2_row *>(row + j * 16) = two;
                    else if (n + j * 16 < N) row[j * 16] = two.x;
                }
            }
    } else {
        if constexpr (!T::kSpare) {
            park(tid2);
            __syncthreads();     // every wavefront has finished reading the ring; the scales are visible
        }
        uint8_t *stage_lds = lds + wave * (32 * WN * 2);      // this wavefront's 32 x WN bf16 staging tile
        // A lane has two neighbouring columns of a row in two accumulators, four bytes (the halves exchanged where the columns are crossed).  Rows of
        // the staging tile need no pad: the rows that a store's two halves write lie an odd number apart, and what is read back is one straight kilobyte a pass.
        const uint32_t crossed16 = crossed(col16) * 16;
        uint8_t *const stage_row[2] = {stage_lds + row_of(quad * 4, 0) * (WN * 2) + col16 * 4, stage_lds + row_of(quad * 4, 1) * (WN * 2) + col16 * 4};
        // read-back: the 32 rows of WN bf16 are 32 * WN / 8 pieces of 16 bytes, dealt to the 64 lanes in order
        // (piece p = 64 pass + lane: row p / (WN / 8), columns 8 (p % (WN / 8)) ...), so every pass has all
        // lanes at work and stores whole rows of the wavefront tile back to back
        constexpr int kRowPieces = WN / 8, kRbPasses = 32 * kRowPieces / 64;
        static_assert(kRbPasses * 64 == 32 * kRowPieces, "read-back passes");
        const int rb_row0 = lane2 / kRowPieces, rb_piece0 = lane2 % kRowPieces;   // pass 0; 64 more pieces per pass
        // the column scales and biases of the lane's accumulator registers, fetched once for all rows
        float swv[kWs];
#pragma unroll
        for (int j = 0; j < kWs; ++j) swv[j] = sw_lds[wn0 + j * 16 + col16];
        auto body = [&](auto EDGE, auto BIAS, auto KIND) {
            float bv[kWs];
#pragma unroll
            for (int j = 0; j < kWs; ++j) bv[j] = decltype(BIAS)::value ? sw_lds[TN + wn0 + j * 16 + col16] : 0.0f;
#pragma unroll
            for (int i = 0; i < XF; ++i) {
                const int mrow = m0 + wm0 + i * 32;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const v4f sx = *reinterpret_cast<const v4f *>(sx_lds + wm0 + i * 32 + quad * 8 + h * 4);
#pragma unroll
                    for (int j = 0; j < kWs; j += 2)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float t[2] = {(float)acc[2 * i + h][j][r] * sx[r], (float)acc[2 * i + h][j + 1][r] * sx[r]};
                            float y[2];
#pragma unroll
                            for (int e = 0; e < 2; ++e)      // explicitly fused, so that every tile shape rounds alike
                                y[e] = decltype(BIAS)::value ? fmaf(t[e], swv[j + e], bv[j + e]) : t[e] * swv[j + e];
                            const uint32_t two = pack_bf16x2(y[0], y[1]);
                            *reinterpret_cast<uint32_t *>(stage_row[h] + r * 2 * (WN * 2) + j * 32) = __builtin_amdgcn_alignbit(two, two, crossed16);
                        }
                }
                // the same wavefront reads back row-contiguous
#pragma unroll
                for (int it = 0; it < kRbPasses; ++it) {
                    int piece = rb_piece0 + (it * 64) % kRowPieces, r = rb_row0 + (it * 64) / kRowPieces;
                    if ((it * 64) % kRowPieces != 0 && piece >= kRowPieces) { piece -= kRowPieces; ++r; }
                    const v4i v = *reinterpret_cast<const v4i *>(stage_lds + (it * 64 + lane2) * 16);
                    const int mo = mrow + r, ncol = n0 + wn0 + piece * 8;
                    uint16_t *out = Y + (int64_t)mo * N + ncol;
                    if constexpr (decltype(EDGE)::value == 0) {
                        store_row<decltype(KIND)::value>(out, v);
                    } else if constexpr (decltype(EDGE)::value == 1) {
                        if (mo < M && ncol < N) store_row<decltype(KIND)::value>(out, v);
                    } else {
                        if (mo < M && ncol + 8 <= N) {
                            store_row<decltype(KIND)::value>(out, v);
                        } else if (mo < M) {
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                if (ncol + e < N) out[e] = (uint16_t)((uint32_t)v[e >> 1] >> (16 * (e & 1)));
                        }
                    }
                }
            }
        };
        // Bounds checks only where the tile crosses the edge of Y, and element stores only where it ends inside a
        // 16-byte piece (uniform over the block; the edge bodies add a bias of zero where there is none).
        using Edge0 = std::integral_constant<int, 0>;
        using Edge1 = std::integral_constant<int, 1>;
        using Edge2 = std::integral_constant<int, 2>;
        using Cached = std::integral_constant<Store, Store::kCached>;
        const bool inside = m0 + TM <= M && n0 + TN <= N;
        auto rows = [&](auto KIND) {
            if (!inside) body(Edge1{}, std::true_type{}, KIND);
            else if (bias) body(Edge0{}, std::true_type{}, KIND);
            else body(Edge0{}, std::false_type{}, KIND);
        };
        if (!inside && (N & 7) != 0) body(Edge2{}, std::true_type{}, Cached{});
        else if (p.store == Store::kPast) rows(std::integral_constant<Store, Store::kPast>{});
        else if (p.store == Store::kThrough) rows(std::integral_constant<Store, Store::kThrough>{});
        else rows(Cached{});
    }
}

// Statically sized LDS: above 64 KB a dynamic allocation would need a per-device function attribute set from the host
// before the first launch, i.e. hidden library state; a static one needs nothing.
// (Arguments in the order they are needed: the first fourteen words of them come in registers.)
#define CONVROT_TILED_FIRST const uint8_t *__restrict__ Xq, const uint8_t *__restrict__ Wq, int M, int N, int K, int per_xcd, int tiles_m
#define CONVROT_TILED_LAST                                                                                                          \
    int span, uint32_t by_span, uint32_t by_rows, uint32_t by_tail, const float *__restrict__ x_scale, const float *__restrict__ w_scale, \
        const uint16_t *__restrict__ bias, uint16_t *__restrict__ Y, int32_t *__restrict__ acc_out, Store store
template <class C, bool RAW, class T>
__global__ __launch_bounds__(T::kThreads, T::OCC) void gemm_tiled_kernel(CONVROT_TILED_FIRST, int rows, CONVROT_TILED_LAST)
{
    __shared__ __attribute__((aligned(1024))) uint8_t lds[Stage<C, T>::kLds];
    int tm, tn;
    if (!tile_of_block({per_xcd, tiles_m, rows, span, by_span, by_rows, by_tail}, blockIdx.x, tm, tn) || !starts_inside(tn, T::TN, N)) return;
    tile_product<C, RAW, T>(Product{Xq, x_scale, Wq, w_scale, bias, M, N, K, Y, acc_out, store}, tm * T::TM, tn * T::TN, lds);
}

// Tiles of T, of which each XCD's last ones (from its `whole`-th on) are cut into `parts` of shape P: a block of T takes a
// compute unit to itself, so a last round that few tiles share would keep most of the chip waiting for a whole tile.
// `rows_whole`: rows of a band, and << 8 what cut_turn is told.
template <class C, bool RAW, class T, class P>
__global__ __launch_bounds__(T::kThreads, T::OCC) void gemm_cut_kernel(CONVROT_TILED_FIRST, int rows_whole, CONVROT_TILED_LAST)
{
    constexpr uint32_t kM = T::TM / P::TM, kN = T::TN / P::TN, kParts = kM * kN;
    static_assert(T::kThreads == P::kThreads && kM * P::TM == T::TM && kN * P::TN == T::TN, "parts of a tile");
    constexpr int kLds = Stage<C, T>::kLds > Stage<C, P>::kLds ? Stage<C, T>::kLds : Stage<C, P>::kLds;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kLds];
    const Product p{Xq, x_scale, Wq, w_scale, bias, M, N, K, Y, acc_out, store};
    const TileOrder order{per_xcd, tiles_m, rows_whole & 0xFF, span, by_span, by_rows, by_tail};
    const uint32_t xcd = blockIdx.x % kNumXcd;
    const CutTurn at = cut_turn(blockIdx.x / kNumXcd, xcd, (uint32_t)per_xcd, (uint32_t)rows_whole >> 8, kParts);
    int tm, tn;
    if (!tile_of_block(order, at.tile * kNumXcd + xcd, tm, tn) || !starts_inside(tn, T::TN, N)) return;
    const int m0 = tm * T::TM + (int)(at.part % kM) * P::TM, n0 = tn * T::TN + (int)(at.part / kM) * P::TN;
    if (m0 >= M || n0 >= N) return;
    if (at.whole) tile_product<C, RAW, T>(p, m0, n0, lds);
    else tile_product<C, RAW, P>(p, m0, n0, lds);
}
#undef CONVROT_TILED_FIRST
#undef CONVROT_TILED_LAST

template <class T>
int band_rows(int tiles_m) { return T::kBandRows != 0 ? T::kBandRows : band_of_256(tiles_m); }

// `rows`: of a band of tiles, and for the cut kernel more.
template <class Kernel>
hipError_t launch_order(Kernel kernel, const Operands &o, const TileOrder &t, int rows, int grid, int threads)
{
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, o.stream, (const uint8_t *)o.Xq, (const uint8_t *)o.Wq, o.M, o.N, o.K, t.per_xcd,
                       t.tiles_m, rows, t.span, t.by_span, t.by_rows, t.by_tail, o.x_scale, o.w_scale, (const uint16_t *)o.bias, (uint16_t *)o.Y,
                       o.acc, o.store);
    return hipGetLastError();
}

template <class C, class T>
hipError_t launch_tiled(const Operands &o)
{
    const int tiles_m = (o.M + T::TM - 1) / T::TM, tiles_n = (o.N + T::TN - 1) / T::TN;
    if (!launchable((int64_t)tiles_m * tiles_n, T::kThreads)) return hipErrorInvalidValue;
    const TileOrder t = tile_order(tiles_m, tiles_n, band_rows<T>(tiles_m));
    auto go = [&](auto kernel) { return launch_order(kernel, o, t, t.rows, t.per_xcd * kNumXcd, T::kThreads); };
    return o.acc ? go(gemm_tiled_kernel<C, true, T>) : go(gemm_tiled_kernel<C, false, T>);
}

// `cut` tiles of every XCD's share of T's go as parts of shape P.
template <class C, class T, class P>
hipError_t launch_cut(const Operands &o, int cut)
{
    const int tiles_m = (o.M + T::TM - 1) / T::TM, tiles_n = (o.N + T::TN - 1) / T::TN;
    if (!launchable((int64_t)tiles_m * tiles_n * (T::TM / P::TM) * (T::TN / P::TN), T::kThreads)) return hipErrorInvalidValue;
    const TileOrder t = tile_order(tiles_m, tiles_n, band_rows<T>(tiles_m));
    const int whole = t.per_xcd - cut, grid = (whole + cut * (T::TM / P::TM) * (T::TN / P::TN)) * kNumXcd;
    const int first = parts_first(o.store, o.N, C::stages(o.K)) ? kPartsFirst : 0;
    auto go = [&](auto kernel) { return launch_order(kernel, o, t, t.rows | (whole | first) << 8, grid, T::kThreads); };
    return o.acc ? go(gemm_cut_kernel<C, true, T, P>) : go(gemm_cut_kernel<C, false, T, P>);
}

}  // namespace gemm
}  // namespace convrot
