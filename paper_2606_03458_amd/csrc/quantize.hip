// KVarN tile quantizer for gfx950: Hadamard rotation (Sec. 2.2, App. A), VarN (App. H,
// Algorithm 1), asymmetric RTN (Sec. 2.1, Eq. 1) and bit-packing with the dual-scale aux of
// App. D.  One 256-thread workgroup quantizes one 128-token x 128-channel tile held entirely
// in registers: thread (tr, tc) owns tokens 8*tr..8*tr+7 and channels 8*tc..8*tc+7, with
// tc the channel block of lane % 16 (a DPP row of 16 lanes spans all 128 channels of a token)
// and tr = 4*wave + lane / 16.  Row (per-token) reductions stay inside a 16-lane row; column
// (per-channel) reductions cross the four 16-lane groups of a wave and then the four waves
// through LDS, in a fixed order so that every thread sees bit-identical results.
//
// Bound by the vector ALU, whose instructions are not equal on gfx950 (measured per SIMD with four
// waves): a plain fp32 add, multiply or multiply-add issues every 2.4 cycles, a max, min, byte permute,
// conversion or any lane move every 4.3, a row swap or a transcendental every 8.2.  Half of a VarN
// iteration is its 384 multiply-adds; so sums go as reduce-scatters, statistics are kept by the one lane
// that owns a row or column, and lane moves are folded into the arithmetic.  32768 key tiles from bf16
// at 2 bits: 1443 us (every lane all sums, rotation stages through the LDS crossbar, IEEE divisions) ->
// 1207 us, 872 -> 1043 GB/s; 4099 value tiles from fp32 at 4 bits, compact aux, 238 -> 191 us.
#include <type_traits>

#include "common.hpp"

namespace kvarn {
namespace {

constexpr int kThreads = 256;

struct QuantSmem {
    alignas(16) float red[2][4][kD];  // column partials [buffer][wave][channel]
    alignas(16) float tot[kD];        // column totals
    float stat[4][4];                 // per-wave partials of the row maximum and minimum, or of the tile shift
    alignas(16) uint8_t codes[kG * kD];  // keys: [token][channel]; values: [channel][token] (swizzled)
};

// Lane tc of a DPP row holds channel block cb, channels 8 cb .. 8 cb + 7, such that the lanes whose
// blocks differ in bit 0, 1, 2 or 3 alone are tc ^ 15 (the row mirror), tc ^ 7 (the half-row mirror),
// tc ^ 2 and tc ^ 1.  Every stage of the rotation is then one lane move, and the stages of scatter_rows
// add neighbouring blocks, then neighbouring pairs, quads and halves: a sum's terms are grouped by their
// channels, so the statistics, and with them the stored tiles, do not change with the order of the lanes.
struct Lane {
    int tid, lane, wave, tc, tr, G, cb;
    __device__ Lane() {
        tid = threadIdx.x;
        asm volatile("" : "+v"(tid));  // formed anew for each tile of a flush, not held in registers across them
        lane = tid & 63;
        wave = tid >> 6;
        tc = lane & 15;
        G = lane >> 4;
        tr = wave * 4 + G;
        const int b2 = (tc >> 2) & 1, b3 = tc >> 3;
        cb = b3 | (b3 ^ b2) << 1 | (((tc >> 1) & 1) ^ b2) << 2 | ((tc & 1) ^ b2) << 3;
    }
};

// ---- lane moves folded into arithmetic -------------------------------------------------------
// x[j] += move(x[j]) * B, and x[j] = min or max(x[j], move(x[j])), for eight values, the lane move folded
// into the instruction (the compiler emits moves of their own here, with wait states between).  An
// instruction may read a register through a lane move no sooner than two after it was written: the
// s_nop covers what came before, the eight values each other.
#define KVARN_EACH8(OP, TAIL)                                                                          \
    "s_nop 1\n\t" OP " %0, %0, " TAIL(0) "\n\t" OP " %1, %1, " TAIL(1) "\n\t" OP " %2, %2, " TAIL(2) "\n\t" OP \
    " %3, %3, " TAIL(3) "\n\t" OP " %4, %4, " TAIL(4) "\n\t" OP " %5, %5, " TAIL(5) "\n\t" OP " %6, %6, " TAIL(6) \
    "\n\t" OP " %7, %7, " TAIL(7)
#define KVARN_REGS8 "+&v"(x[0]), "+&v"(x[1]), "+&v"(x[2]), "+&v"(x[3]), "+&v"(x[4]), "+&v"(x[5]), "+&v"(x[6]), "+&v"(x[7])
#define KVARN_ALL " row_mask:0xf bank_mask:0xf"
template <int M>
__device__ __forceinline__ void butterfly8(float (&x)[8], float B) {
#define TAIL1(k) "%8 row_mirror" KVARN_ALL
#define TAIL2(k) "%8 row_half_mirror" KVARN_ALL
#define TAIL4(k) "%8 quad_perm:[2,3,0,1]" KVARN_ALL
#define TAIL8(k) "%8 quad_perm:[1,0,3,2]" KVARN_ALL
    if constexpr (M == 1) asm(KVARN_EACH8("v_fmac_f32_dpp", TAIL1) : KVARN_REGS8 : "v"(B));
    else if constexpr (M == 2) asm(KVARN_EACH8("v_fmac_f32_dpp", TAIL2) : KVARN_REGS8 : "v"(B));
    else if constexpr (M == 4) asm(KVARN_EACH8("v_fmac_f32_dpp", TAIL4) : KVARN_REGS8 : "v"(B));
    else asm(KVARN_EACH8("v_fmac_f32_dpp", TAIL8) : KVARN_REGS8 : "v"(B));
#undef TAIL1
#undef TAIL2
#undef TAIL4
#undef TAIL8
}
// Minimum and maximum over the 16 lanes of a row, in every lane.
#define TAILA(k) "%" #k " quad_perm:[1,0,3,2]" KVARN_ALL
#define TAILB(k) "%" #k " quad_perm:[2,3,0,1]" KVARN_ALL
#define TAILC(k) "%" #k " row_half_mirror" KVARN_ALL
#define TAILD(k) "%" #k " row_mirror" KVARN_ALL
__device__ __forceinline__ void rows_min8(float (&x)[8]) {
    asm(KVARN_EACH8("v_min_f32_dpp", TAILA) "\n\t" KVARN_EACH8("v_min_f32_dpp", TAILB) "\n\t" KVARN_EACH8("v_min_f32_dpp", TAILC)
        "\n\t" KVARN_EACH8("v_min_f32_dpp", TAILD) "\n\ts_nop 1" : KVARN_REGS8);
}
__device__ __forceinline__ void rows_max8(float (&x)[8]) {
    asm(KVARN_EACH8("v_max_f32_dpp", TAILA) "\n\t" KVARN_EACH8("v_max_f32_dpp", TAILB) "\n\t" KVARN_EACH8("v_max_f32_dpp", TAILC)
        "\n\t" KVARN_EACH8("v_max_f32_dpp", TAILD) "\n\ts_nop 1" : KVARN_REGS8);
}
#undef TAILA
#undef TAILB
#undef TAILC
#undef TAILD
#undef KVARN_EACH8
#undef KVARN_REGS8
#undef KVARN_ALL

// ---- reductions ---------------------------------------------------------------------------
struct OpSum {
    __device__ static float f(float a, float b) { return a + b; }
};
// Max and min in the NaN-propagating forms: fmaxf / fminf would first quiet every operand that comes
// from another lane or from LDS (one more instruction each).
__device__ __forceinline__ float fmax_any(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float fmin_any(float a, float b) { return __builtin_elementwise_minimum(a, b); }
struct OpMax {
    __device__ static float f(float a, float b) { return fmax_any(a, b); }
};
struct OpMin {
    __device__ static float f(float a, float b) { return fmin_any(a, b); }
};

template <int CTRL>
__device__ __forceinline__ float dppf(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}

// Op over the 16 lanes of a DPP row: quad partners ^1 and ^2, then the other quad of the half
// (mirror within 8 lanes) and the other half (mirror within 16).  Each step combines two
// equal partial results, so every lane of the row ends with the same value.
template <class Op>
__device__ __forceinline__ float row16(float v) {
    v = Op::f(v, dppf<0xB1>(v));
    v = Op::f(v, dppf<0x4E>(v));
    v = Op::f(v, dppf<0x141>(v));
    return Op::f(v, dppf<0x140>(v));
}

// Op over lanes l, l ^ 16, l ^ 32, l ^ 48 (the four rows of a wave).  With both operands equal,
// a row-pair swap returns (value of the even row, value of the odd row) in every lane of the
// pair, so all four lanes end with the same value.
template <class Op>
__device__ __forceinline__ float across_rows(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = Op::f(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return Op::f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Maximum of mx and minimum of mn over the wave, left in lane 63 (a NaN, the variance of a row or column with
// a NaN or an infinite value, counts for nothing): quad, half-row and row exchanges, then row 0 into row 1
// and row 2 into row 3, then row 1 into rows 2 and 3.  Moves and comparisons in one instruction each, at
// half the rate of an add; a row-pair swap costs twice that.  (Two wait states between an instruction and a
// lane move of its result: the other chain's instruction and the s_nop.)
__device__ __forceinline__ void wave_max_min(float& mx, float& mn) {
    asm("s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_max_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_max_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_max_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "v_min_f32_dpp %1, %1, %1 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "s_nop 1"
        : "+&v"(mx), "+&v"(mn));
}
__device__ __forceinline__ float lane63(float v) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Column reductions, across the 16 threads that share a channel block (all token blocks): the four
// rows of the wave here, then the four waves through LDS.  The rows go as a reduce-scatter:
// permlane16_swap of two different values leaves, in every lane, the even-row and odd-row partials
// of one of them (rows 0, 2: the first, rows 1, 3: the second), and permlane32_swap of two such words
// the two half sums, so no lane computes results it then discards.  Row G of a wave ends with columns
// G and 4 + G of the block's eight, which it writes to red[buf][wave] side by side (column k of the
// block at 8 tc + 2 (k % 4) + k / 4): consecutive lanes write and read consecutive words.
template <class Op>
__device__ __forceinline__ void scatter_cols(const float (&s)[8], QuantSmem& sm, int buf, const Lane& L) {
    float t[4], rr[2];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(s[2 * p]), __float_as_uint(s[2 * p + 1]), false, false);
        t[p] = Op::f(__uint_as_float(x[0]), __uint_as_float(x[1]));
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(t[2 * k]), __float_as_uint(t[2 * k + 1]), false, false);
        rr[k] = Op::f(__uint_as_float(y[0]), __uint_as_float(y[1]));
    }
    *reinterpret_cast<float2*>(&sm.red[buf][L.wave][8 * L.tc + 2 * L.G]) = make_float2(rr[0], rr[1]);
}
// Each column's four wave partials, combined once (by the first two waves), times scale;
// every thread of the channel block then reads its eight.  Between scatter_cols and the end two
// barriers, so the buffer and tot can be written again by the next call.
template <class Op>
__device__ __forceinline__ void total_cols(float (&s)[8], float scale, QuantSmem& sm, int buf, const Lane& L) {
    if (L.tid < kD) {
        const int c = L.tid;
        const float v = Op::f(Op::f(Op::f(sm.red[buf][0][c], sm.red[buf][1][c]), sm.red[buf][2][c]), sm.red[buf][3][c]);
        sm.tot[c] = v * scale;
    }
    __syncthreads();
    const float4 lo = *reinterpret_cast<const float4*>(&sm.tot[8 * L.tc]);
    const float4 hi = *reinterpret_cast<const float4*>(&sm.tot[8 * L.tc + 4]);
    s[0] = lo.x; s[4] = lo.y; s[1] = lo.z; s[5] = lo.w;
    s[2] = hi.x; s[6] = hi.y; s[3] = hi.z; s[7] = hi.w;
}

// Sum over the 16 lanes of a DPP row of s[tc / 2], as a reduce-scatter (16 instructions against 32
// for the eight sums in every lane).  Two stages of adds that write part of the row only: the row
// mirror leaves s[0..3] in lanes 0-7 and s[4..7] in lanes 8-15, the half mirror two of those in
// the lower and upper quad of each half; then one select and exchange inside the quad.  The
// instructions read a register through DPP no sooner than two after it was written, inside the
// block by their order, at its ends by the s_nop.
__device__ __forceinline__ float scatter_rows(float (&s)[8], const Lane& L) {
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %0, %4, %4 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %1, %1 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %1, %5, %5 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %2, %2 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %2, %6, %6 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %3, %3, %3 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %3, %7, %7 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %1, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "s_nop 1"
        : "+&v"(s[0]), "+&v"(s[1]), "+&v"(s[2]), "+&v"(s[3])
        : "v"(s[4]), "v"(s[5]), "v"(s[6]), "v"(s[7]));
    const bool odd = (L.tc & 2) != 0;
    float v = odd ? s[1] : s[0];
    v += dppf<0x4E>(odd ? s[0] : s[1]);
    return v + dppf<0xB1>(v);
}
// The value of token i in every lane of the row, from the lanes 2 i that own it.
__device__ __forceinline__ void gather_rows(float own, float (&out)[8]) {
    out[0] = dppf<0x150>(own); out[1] = dppf<0x152>(own); out[2] = dppf<0x154>(own); out[3] = dppf<0x156>(own);
    out[4] = dppf<0x158>(own); out[5] = dppf<0x15A>(own); out[6] = dppf<0x15C>(own); out[7] = dppf<0x15E>(own);
}

// Variance over tokens of the columns of T*w (two-pass, ddof = 1) that this lane owns, columns
// G and 4 + G of its eight.  The means go to every lane; the first LDS round also reduces the wave's
// (rmax, rmin) of the row variances, in lane 63, to the workgroup's.
__device__ __forceinline__ void column_var(const float (&x)[8][8], const float (&w)[8], float (&var)[2],
                                           QuantSmem& sm, const Lane& L, float& rmax, float& rmin) {
    // (explicit fmas: each pass forms x * w inside its own fma)
    float s[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc = fmaf(x[i][j], w[i], acc);
        s[j] = acc;
    }
    scatter_cols<OpSum>(s, sm, 0, L);
    if (L.lane == 63) *reinterpret_cast<float2*>(sm.stat[L.wave]) = make_float2(rmax, rmin);
    __syncthreads();
    rmax = fmax_any(fmax_any(sm.stat[0][0], sm.stat[1][0]), fmax_any(sm.stat[2][0], sm.stat[3][0]));
    rmin = fmin_any(fmin_any(sm.stat[0][1], sm.stat[1][1]), fmin_any(sm.stat[2][1], sm.stat[3][1]));
    float mean[8];
    total_cols<OpSum>(mean, 1.0f / kG, sm, 0, L);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float d = fmaf(x[i][j], w[i], -mean[j]);
            acc = fmaf(d, d, acc);
        }
        s[j] = acc;
    }
    scatter_cols<OpSum>(s, sm, 1, L);
    __syncthreads();
    // (no second round: the owners read the four wave partials of their two columns themselves)
    float2 p[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) p[k] = *reinterpret_cast<const float2*>(&sm.red[1][k][8 * L.tc + 2 * L.G]);
    var[0] = (((p[0].x + p[1].x) + p[2].x) + p[3].x) * (1.0f / (kG - 1));
    var[1] = (((p[0].y + p[1].y) + p[2].y) + p[3].y) * (1.0f / (kG - 1));
}

// Variance over channels of the row of T*u that this lane owns, token tc / 2 of its eight (two-pass,
// ddof = 1); mean_out: its mean.
__device__ __forceinline__ float row_var(const float (&x)[8][8], const float (&u)[8], const Lane& L, float* mean_out = nullptr) {
    float s[8], mean[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float acc = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc = fmaf(x[i][j], u[j], acc);
        s[i] = acc;
    }
    const float own = scatter_rows(s, L) * (1.0f / kD);
    if (mean_out) *mean_out = own;
    gather_rows(own, mean);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float acc = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float d = fmaf(x[i][j], u[j], -mean[i]);
            acc = fmaf(d, d, acc);
        }
        s[i] = acc;
    }
    return scatter_rows(s, L) * (1.0f / (kD - 1));
}

// Imb of Algorithm 1 from the row variances (one token per lane) and the column variances (two
// channels per lane), in two parts: the wave's max / min of the row variances (reduced over the
// workgroup by column_var's first LDS round), then the value.
__device__ __forceinline__ float imbalance(float rmax, float rmin, const float (&vc)[2]) {
    // all 128 channels live in the wave
    float cmax, cmin;
    asm("v_max_f32 %0, %1, %2" : "=v"(cmax) : "v"(vc[0]), "v"(vc[1]));  // (fmaxf would quiet both first)
    asm("v_min_f32 %0, %1, %2" : "=v"(cmin) : "v"(vc[0]), "v"(vc[1]));
    wave_max_min(cmax, cmin);
    // (hardware reciprocal, ~1 ulp: Imb only ranks iterations, and values that close are ties)
    return rmax * __builtin_amdgcn_rcpf(fmaxf(rmin, 1e-8f)) + lane63(cmax) * __builtin_amdgcn_rcpf(fmaxf(lane63(cmin), 1e-8f));
}

__device__ __forceinline__ float clampf(float v, float lo, float hi) { return fminf(fmaxf(v, lo), hi); }

// Natural log and exp on the hardware log2 / exp2.  Their arguments stay far from the denormal
// range (variances clamped to [var_min, var_max] >= 1e-30, log-scales to [log_lo, log_hi]
// within +-40), so no range fix-up is needed.
__device__ __forceinline__ float ln_hw(float v) { return __builtin_amdgcn_logf(v) * 0.6931471805599453f; }
__device__ __forceinline__ float exp_hw(float v) { return __builtin_amdgcn_exp2f(v * kLog2e); }

constexpr float kMaxF32 = 3.402823466e38f;

// x / d, correctly rounded, from r = the rounded 1 / d: the product, corrected once by its exact
// remainder (Markstein).  The remainder is formed as q d - x, so that a zero keeps the sign that the
// division gives it (the offset of a group is stored with its sign).  The product x r must be finite (an
// infinite one would make the correction inf - inf).
__device__ __forceinline__ float corrected_quotient(float x, float d, float q, float r) {
    return fmaf(-fmaf(q, d, -x), r, q);
}

// ---- shared log-scale updates ----------------------------------------------------------------
// Every column and token is updated by the lanes that own it: of the four lanes of a wave that hold
// the same eight columns (lanes l, l^16, l^32, l^48) each updates columns G and 4 + G of them
// (G = lane / 16); of the sixteen lanes of a DPP row, which hold the same eight tokens, lane tc
// updates token tc / 2.  The results are gathered back into every lane: with equal operands a
// 16-lane-row swap returns the (even row, odd row) values of a row pair and a half swap the (lower
// half, upper half) values; a DPP row broadcast returns one lane of the row.
__device__ __forceinline__ void gather_cols(const float (&own)[2], float (&out)[8]) {
    const auto a0 = __builtin_amdgcn_permlane16_swap(__float_as_uint(own[0]), __float_as_uint(own[0]), false, false);
    const auto a1 = __builtin_amdgcn_permlane16_swap(__float_as_uint(own[1]), __float_as_uint(own[1]), false, false);
    // row pair P holds (own of row 2P, own of row 2P + 1); the half swap then gives pairs 0 and 1
    const auto b0 = __builtin_amdgcn_permlane32_swap(a0[0], a0[0], false, false);  // columns 0, 2
    const auto b1 = __builtin_amdgcn_permlane32_swap(a0[1], a0[1], false, false);  // columns 1, 3
    const auto b2 = __builtin_amdgcn_permlane32_swap(a1[0], a1[0], false, false);  // columns 4, 6
    const auto b3 = __builtin_amdgcn_permlane32_swap(a1[1], a1[1], false, false);  // columns 5, 7
    out[0] = __uint_as_float(b0[0]); out[2] = __uint_as_float(b0[1]);
    out[1] = __uint_as_float(b1[0]); out[3] = __uint_as_float(b1[1]);
    out[4] = __uint_as_float(b2[0]); out[6] = __uint_as_float(b2[1]);
    out[5] = __uint_as_float(b3[0]); out[7] = __uint_as_float(b3[1]);
}

// ---- narrow formats of the compact aux (App. D: 8-bit float scales, 16-bit float offset) ----
// OCP E4M3: 4-bit exponent with bias 7, 3-bit mantissa, subnormals m * 2^-9, largest 448.
// Grid value of x > 0 on the E4M3 grid of its binade (spacing 2^(e-3), 2^-9 below 2^-6),
// nearest with ties to even or upward, saturating at 448.  Scaling by powers of two is exact.
__device__ __forceinline__ float e4m3_round(float x, bool up) {
    if (x >= 448.f) return 448.f;
    int ex;
    frexpf(x, &ex);  // x in [2^(ex-1), 2^ex)
    const int E = max(ex - 1, -6);
    const float q = x * ldexpf(1.f, 3 - E);
    return (up ? ceilf(q) : rintf(q)) * ldexpf(1.f, E - 3);
}
// Byte of a value on the E4M3 grid (0 <= v <= 448).
__device__ __forceinline__ uint32_t e4m3_bits(float v) {
    if (v < 0.015625f) return (uint32_t)(v * 512.f);  // subnormal: m * 2^-9
    const uint32_t u = __float_as_uint(v);
    return ((((u >> 23) & 255u) - 120u) << 3) | ((u >> 20) & 7u);  // exponent - 127 + 7
}
// Nearest binary16 (ties to even), saturating at +-65504; returns the value and its bits.
__device__ __forceinline__ float fp16_round(float x, uint32_t& bits) {
    const _Float16 h = (_Float16)fminf(fmaxf(x, -65504.f), 65504.f);
    bits = __builtin_bit_cast(uint16_t, h);
    return (float)h;
}

// Byte of a code in QuantSmem::codes: rows of 128 bytes, their 16-byte (keys) or 8-byte (values) blocks
// permuted by the row, and every other eight tokens' rows swapped in pairs, so that neither the writes
// (8 bytes per lane, a row or a column of blocks at once) nor the gathers of the packing meet a bank
// more often than their width needs (unswizzled, two thirds of the LDS cycles were conflicts).
__device__ __forceinline__ int key_code_at(int t, int c) {
    return (t ^ ((t >> 3) & 1)) * kD + 16 * ((c >> 4) ^ (t & 7)) + (c & 15);
}
__device__ __forceinline__ int value_code_at(int c, int t) {
    return (c ^ ((t >> 3) & 1)) * kG + 8 * ((t >> 3) ^ (c >> 3) ^ ((c & 7) << 1)) + (t & 7);
}

// Quantize one tile.  src: token t at src + t*tstride elements, channels contiguous (16-byte
// aligned rows).  dst: the packed tile (16-byte aligned).
template <bool COMPACT, bool EXACT>
__device__ void quantize_tile(const void* src, bool bf16, int64_t tstride, int kind, const QParams& P, uint8_t* dst,
                              int32_t* best_out, QuantSmem& sm) {
    const Lane L;
    float x[8][8];

    // ---- a1: load -------------------------------------------------------------------------
    // One branch on the type, so that all eight rows are in flight before the first is used: a branch per
    // row waited for each, eight memory round trips in turn (12 prompts of up to 4k tokens 101.5 -> 97.7 us,
    // a call of few tiles 22.5 -> 21.4, 32768 tiles 1228 -> 1207).
    const int64_t at = 8 * L.tr * tstride + 8 * L.cb;
    if (bf16) {
        const uint16_t* p = static_cast<const uint16_t*>(src) + at;
        uint4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const uint4*>(p + i * tstride);
        __builtin_amdgcn_sched_barrier(0);  // (the first conversion is otherwise put before the other loads)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                x[i][2 * k] = __uint_as_float(w[k] << 16);
                x[i][2 * k + 1] = __uint_as_float(w[k] & 0xFFFF0000u);
            }
        }
    } else {
        const float* p = static_cast<const float*>(src) + at;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float4 a = *reinterpret_cast<const float4*>(p + i * tstride);
            const float4 b = *reinterpret_cast<const float4*>(p + i * tstride + 4);
            x[i][0] = a.x; x[i][1] = a.y; x[i][2] = a.z; x[i][3] = a.w;
            x[i][4] = b.x; x[i][5] = b.y; x[i][6] = b.z; x[i][7] = b.w;
        }
    }

    // ---- a2: Hadamard along channels, butterflies of stride 1, 2, ..., 64 (not in the ablations
    // without rotation) ----------------------------------------------------------------------
    if (P.rotate) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
#pragma unroll
            for (int h = 1; h < 8; h <<= 1) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (!(j & h)) {
                        const float a = x[i][j], b = x[i][j + h];
                        x[i][j] = a + b;
                        x[i][j + h] = a - b;
                    }
                }
            }
        }
        // Cross-lane stages as one multiply-add each, x + p * B with B = +1 in the lower lane of
        // a pair and -1 in the upper one: the upper lane then holds -(a - b) instead of a - b.
        // Partners always hold values of the same sign, so the signs stay consistent and every
        // value is exactly +- the butterfly's (round to nearest is symmetric); after the four
        // stages block cb's lane holds (-1)^popcount(cb) times it, which the final scaling removes.
        // (channel stride 8 m lives in the lane of block cb ^ m)
#pragma unroll
        for (int i = 0; i < 8; ++i) butterfly8<1>(x[i], L.cb & 1 ? -1.f : 1.f);
#pragma unroll
        for (int i = 0; i < 8; ++i) butterfly8<2>(x[i], L.cb & 2 ? -1.f : 1.f);
#pragma unroll
        for (int i = 0; i < 8; ++i) butterfly8<4>(x[i], L.cb & 4 ? -1.f : 1.f);
#pragma unroll
        for (int i = 0; i < 8; ++i) butterfly8<8>(x[i], L.cb & 8 ? -1.f : 1.f);
        const float scale = (__builtin_popcount(L.cb) & 1) ? -kInvSqrt128 : kInvSqrt128;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
#pragma unroll
            for (int j = 0; j < 8; ++j) x[i][j] *= scale;
        }
    }

    // ---- a3/a4: VarN (Algorithm 1), Cur = T * u[c] * w[t] with u = exp(-L_c), w = exp(-L_r) -
    // Each lane keeps the log-scales it updates (columns G, 4 + G and token tc / 2 of its eight,
    // current and best) and all eight scale factors u, w (gathered).
    float Lc2[2] = {0.f, 0.f}, bLc2[2] = {0.f, 0.f};
    float Lr1 = 0.f, bLr1 = 0.f, wo = 1.f;
    float u[8], w[8], vc[2];
#pragma unroll
    for (int k = 0; k < 8; ++k) u[k] = w[k] = 1.f;
    float rmax, rmin, row_mean;
    rmax = rmin = row_var(x, u, L, &row_mean);  // variance over channels of T's rows
    // Whether a value of the wave's rows may pass 1.2e30 (a value is within 12 deviations of its row's
    // mean), so that a quotient by a stored scale, 2^-6 or more, may pass the fp32 range.
    const bool huge_x = COMPACT && __any(!(fabsf(row_mean) < 1e30f && rmax < 1e30f));
    wave_max_min(rmax, rmin);
    column_var(x, w, vc, sm, L, rmax, rmin);  // variance over tokens of T's columns
    float I_best = imbalance(rmax, rmin, vc);
    int best = 0;
    for (int k = 1; k <= P.iters; ++k) {
        // column update from the current column variances u^2 * var_t(T w)
        float uo[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            Lc2[q] = clampf(Lc2[q] + 0.5f * ln_hw(clampf(vc[q], P.var_min, P.var_max)), P.log_lo, P.log_hi);
            uo[q] = exp_hw(-Lc2[q]);
        }
        gather_cols(uo, u);
        // row update from the row variances w^2 * var_c(T u)
        const float rv = row_var(x, u, L);
        Lr1 = clampf(Lr1 + 0.5f * ln_hw(clampf(wo * wo * rv, P.var_min, P.var_max)), P.log_lo, P.log_hi);
        wo = exp_hw(-Lr1);
        gather_rows(wo, w);
        // imbalance of the new Cur; its column variances seed the next column update
        rmax = rmin = wo * wo * rv;
        wave_max_min(rmax, rmin);
        column_var(x, w, vc, sm, L, rmax, rmin);
        vc[0] *= uo[0] * uo[0];
        vc[1] *= uo[1] * uo[1];
        const float I = imbalance(rmax, rmin, vc);
        if (I <= I_best) {  // later iteration wins ties
            I_best = I;
            best = k;
            bLc2[0] = Lc2[0];
            bLc2[1] = Lc2[1];
            bLr1 = Lr1;
        }
    }

    // ---- a5: balanced tile B = T / S_c* / S_r* ---------------------------------------------
    float Sc[8], Sr[8];
    {
        const float sc[2] = {exp_hw(bLc2[0]), exp_hw(bLc2[1])}, ui[2] = {exp_hw(-bLc2[0]), exp_hw(-bLc2[1])};
        gather_cols(sc, Sc);
        gather_cols(ui, u);
        gather_rows(exp_hw(bLr1), Sr);
        gather_rows(exp_hw(-bLr1), w);
    }
    float s2q[8];  // compact aux: the stored (E4M3) other-axis scale of this thread's rows/columns
    if constexpr (COMPACT) {
        // the other-axis scale is rounded first and the group RTN sees z = T / s2 (stored
        // value); the group-axis scale is absorbed exactly (RTN of a group ignores a common
        // factor)
#pragma unroll
        for (int m = 0; m < 8; ++m)
            s2q[m] = e4m3_round(clampf(kind == KVARN_KEYS ? Sr[m] : Sc[m], 0.015625f, 448.f), false);
        // T / s2, a division each being four times as long.  Huge values are divided at a 2^16-th of their
        // size and scaled up again, so that a quotient beyond the fp32 range is the infinity that the
        // division gives (a step of that size is stored as the largest scale).  An infinite value is divided
        // as 2^121, which passes the range for every divisor when it is scaled up.
        if (huge_x) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
#pragma unroll
                for (int j = 0; j < 8; ++j) x[i][j] = fabsf(x[i][j]) > kMaxF32 ? copysignf(0x1p121f, x[i][j]) : 0x1p-16f * x[i][j];
            }
        }
        float inv[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) inv[m] = 1.0f / s2q[m];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float d = kind == KVARN_KEYS ? s2q[i] : s2q[j], r = kind == KVARN_KEYS ? inv[i] : inv[j];
                x[i][j] = corrected_quotient(x[i][j], d, x[i][j] * r, r);
            }
        }
        if (huge_x) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
#pragma unroll
                for (int j = 0; j < 8; ++j) x[i][j] *= 0x1p16f;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
#pragma unroll
            for (int j = 0; j < 8; ++j) x[i][j] = x[i][j] * u[j] * w[i];
        }
    }

    // ---- a6: RTN along the group axis (keys: per channel, values: per token) ----------------
    const float qmax = (float)((1 << P.bits) - 1), inv_qmax = P.bits == 2 ? 1.0f / 3.0f : 1.0f / 15.0f;
    auto over_qmax = [&](float v) { return corrected_quotient(v, qmax, fminf(v * inv_qmax, kMaxF32), inv_qmax); };
    float mn[8], mx[8];
    if (kind == KVARN_KEYS) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            mn[j] = mx[j] = x[0][j];
#pragma unroll
            for (int i = 1; i < 8; ++i) {
                mn[j] = fminf(mn[j], x[i][j]);
                mx[j] = fmaxf(mx[j], x[i][j]);
            }
        }
        scatter_cols<OpMin>(mn, sm, 0, L);
        __syncthreads();  // (also: every owner is done with red[1] of the last column variances)
        scatter_cols<OpMax>(mx, sm, 1, L);
        total_cols<OpMin>(mn, 1.f, sm, 0, L);
        __syncthreads();  // tot is read
        total_cols<OpMax>(mx, 1.f, sm, 1, L);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            mn[i] = mx[i] = x[i][0];
#pragma unroll
            for (int j = 1; j < 8; ++j) {
                mn[i] = fminf(mn[i], x[i][j]);
                mx[i] = fmaxf(mx[i], x[i][j]);
            }
        }
        // A lane whose eight values are all NaN makes its row's range one; the folded lane moves would pass
        // over it.  (0 unless a minimum is a NaN or infinite)
        float odd = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) odd = fmaf(mn[i], 0.f, odd);
        if (__any(odd != 0.f)) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                mn[i] = row16<OpMin>(mn[i]);
                mx[i] = row16<OpMax>(mx[i]);
            }
        }
        rows_min8(mn);
        rows_max8(mx);
    }
    if constexpr (COMPACT) {
        // Both stored scales are E4M3 (at most 448) while their product is fixed by the data:
        // when the largest group step of the tile exceeds 448, a tile-wide 2^e moves from the
        // group scale into s2 (z / 2^e and s2 * 2^e leave every dequantized value unchanged,
        // and both products are exact), for the smallest such e >= 0 and no further than the
        // largest other-axis scale times 2^e stays within 448.  The shift needs every
        // other-axis scale at least 2^-6 (true unless log_lo is set below -4.1), so that s2 was
        // not clamped and scaling the stored s2 by 2^e equals storing 2^e times the scale.
        float st[3] = {0.f, 0.f, -__builtin_inff()};  // largest step, largest and -smallest other-axis scale
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const float so = kind == KVARN_KEYS ? Sr[m] : Sc[m];
            st[0] = fmaxf(st[0], over_qmax(mx[m] - mn[m]));
            st[1] = fmaxf(st[1], so);
            st[2] = fmaxf(st[2], -so);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) st[k] = across_rows<OpMax>(row16<OpMax>(st[k]));
        if (L.lane == 0) {
#pragma unroll
            for (int k = 0; k < 3; ++k) sm.stat[L.wave][k] = st[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 3; ++k)
            st[k] = fmax_any(fmax_any(sm.stat[0][k], sm.stat[1][k]), fmax_any(sm.stat[2][k], sm.stat[3][k]));
        int e = 0;
        if (-st[2] >= 0.015625f)
            while (e < 64 && ldexpf(st[0], -e) > 448.f && ldexpf(st[1], e + 1) <= 448.f) ++e;
        if (e > 0) {
            const float down = ldexpf(1.f, -e), up = ldexpf(1.f, e);
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                mn[m] *= down;
                mx[m] *= down;
                s2q[m] *= up;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
#pragma unroll
                for (int j = 0; j < 8; ++j) x[i][j] *= down;
            }
        }
    }
    // step and offset of each group: fp32 aux keeps them; the compact aux stores the step
    // rounded upward to E4M3 (the stored range covers the group) and the nearest binary16 of
    // the minimum, and the codes are chosen for those stored values
    float s[8], inv_s[8], off[8];
    uint32_t abits[8], bbits[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const float step = over_qmax(mx[m] - mn[m]);
        if constexpr (COMPACT) {
            s[m] = step == 0.f ? 1.f : e4m3_round(step, true);
            off[m] = fp16_round(mn[m], bbits[m]);
            abits[m] = e4m3_bits(s[m]);
        } else {
            s[m] = step == 0.f ? 1.f : step;
            off[m] = mn[m];
        }
        const float r = __builtin_amdgcn_rcpf(s[m]);  // one Newton step: the division's result, over every mantissa
        inv_s[m] = fmaf(fmaf(-s[m], r, 1.f), r, r);
    }
    // (steps near the ends of the fp32 range, where the reciprocal or the step is subnormal)
    float s_lo = s[0], s_hi = s[0];
#pragma unroll
    for (int m = 1; m < 8; ++m) {
        s_lo = fminf(s_lo, s[m]);
        s_hi = fmaxf(s_hi, s[m]);
    }
    if (!(s_lo > 1e-36f && s_hi < 1e36f)) {
#pragma unroll
        for (int m = 0; m < 8; ++m) inv_s[m] = 1.0f / s[m];
    }
    // codes -> LDS (keys [t][c], values [c][t]), 8 bytes per thread per token / channel.
    // EXACT (unrotated and unbalanced tiles, the KIVI-style ablation, fp32 aux): the tile holds
    // the inputs themselves and a bf16 value can lie exactly halfway between two levels; the
    // quotient is then formed as qmax (x - mn) / (mx - mn) with one correctly rounded division,
    // which keeps such a value an exact half-integer, rounded half to even.  Otherwise the
    // reciprocal step is used.
    auto write_codes = [&](auto exact) {
        constexpr bool kExact = decltype(exact)::value;
        float den[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) den[m] = mx[m] > mn[m] ? mx[m] - mn[m] : 1.f;
        // With fp32 aux the offset is the group minimum itself, so v - off >= 0 exactly, and at
        // the group maximum the quotient is qmax within a few ulps (correctly rounded step and
        // reciprocal, or division): rounding lands in [0, qmax] without a clamp.  The compact
        // aux rounds the offset to binary16 and the step up to E4M3, so its codes are clamped.
        // The code in the low byte of a word: u + 1.5 * 2^23 rounds u (0 <= u <= 15) to the
        // nearest integer, ties to even as rintf, into the low mantissa bits.
        auto code = [&](float v, int m) -> uint32_t {
            float u = kExact ? ((v - off[m]) * qmax) / den[m] : (v - off[m]) * inv_s[m];
            if constexpr (COMPACT) u = clampf(u, 0.f, qmax);  // (before rounding: the same codes)
            return __float_as_uint(u + 12582912.f);
        };
        // four such words -> their low bytes in order, by two byte permutes
        auto pack4 = [](uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
            return __builtin_amdgcn_perm(__builtin_amdgcn_perm(d, c, 0x0c0c0400u), __builtin_amdgcn_perm(b, a, 0x0c0c0400u),
                                         0x05040100u);
        };
        if (kind == KVARN_KEYS) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                uint32_t q[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) q[j] = code(x[i][j], j);
                *reinterpret_cast<uint2*>(&sm.codes[key_code_at(8 * L.tr + i, 8 * L.cb)]) =
                    make_uint2(pack4(q[0], q[1], q[2], q[3]), pack4(q[4], q[5], q[6], q[7]));
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                uint32_t q[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) q[i] = code(x[i][j], i);
                *reinterpret_cast<uint2*>(&sm.codes[value_code_at(8 * L.cb + j, 8 * L.tr)]) =
                    make_uint2(pack4(q[0], q[1], q[2], q[3]), pack4(q[4], q[5], q[6], q[7]));
            }
        }
    };
    write_codes(std::integral_constant<bool, EXACT>{});

    // ---- a7: aux (absorbed scales) --------------------------------------------------------
    float* aux = reinterpret_cast<float*>(dst + code_bytes(P.bits));
    uint8_t* caux = dst + code_bytes(P.bits);  // compact: b16[128] | a8[128] | s2_8[128]
    // group-axis values of 8 groups g0 .. g0 + 7 (a as E4M3 bytes, b as binary16), and the
    // other-axis s2 of 8 indices o0 .. o0 + 7
    auto put_group = [&](int g0) {
        *reinterpret_cast<uint4*>(caux + 2 * g0) =
            make_uint4(bbits[0] | bbits[1] << 16, bbits[2] | bbits[3] << 16, bbits[4] | bbits[5] << 16,
                       bbits[6] | bbits[7] << 16);
        *reinterpret_cast<uint2*>(caux + 256 + g0) =
            make_uint2(abits[0] | abits[1] << 8 | abits[2] << 16 | abits[3] << 24,
                       abits[4] | abits[5] << 8 | abits[6] << 16 | abits[7] << 24);
    };
    auto put_s2 = [&](int o0) {
        uint32_t sb[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) sb[m] = e4m3_bits(s2q[m]);
        *reinterpret_cast<uint2*>(caux + 384 + o0) =
            make_uint2(sb[0] | sb[1] << 8 | sb[2] << 16 | sb[3] << 24, sb[4] | sb[5] << 8 | sb[6] << 16 | sb[7] << 24);
    };
    if constexpr (COMPACT) {
        if (kind == KVARN_KEYS) {
            if (L.tr == 0) put_group(8 * L.cb);  // per channel
            if (L.tc == 0) put_s2(8 * L.tr);     // per token
        } else {
            if (L.tc == 0) put_group(8 * L.tr);  // per token
            if (L.tr == 0) put_s2(8 * L.cb);     // per channel
        }
    } else {
      if (kind == KVARN_KEYS) {
        if (L.tr == 0) {  // per channel: a = s * S_c*, b = mn * S_c*
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                aux[8 * L.cb + j] = s[j] * Sc[j];
                aux[kD + 8 * L.cb + j] = mn[j] * Sc[j];
            }
        }
        if (L.tc == 0) {  // s2 per token
#pragma unroll
            for (int i = 0; i < 8; ++i) aux[2 * kD + 8 * L.tr + i] = Sr[i];
        }
    } else {
        if (L.tc == 0) {  // per token: a = s * S_r*, b = mn * S_r*
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                aux[8 * L.tr + i] = s[i] * Sr[i];
                aux[kD + 8 * L.tr + i] = mn[i] * Sr[i];
            }
        }
        if (L.tr == 0) {  // s2 per channel
#pragma unroll
            for (int j = 0; j < 8; ++j) aux[2 * kD + 8 * L.cb + j] = Sc[j];
        }
      }
    }
    if (best_out && L.tid == 0) *best_out = best;
    __syncthreads();

    // ---- a7: pack ------------------------------------------------------------------------------
    // Unit (sigma, lane L, w): its 16 codes e = 4s + q come from four 4-byte LDS reads d_s (byte
    // q = code e); code e goes to bit 8q + bits*(s % p) of word s / p, p = 8 / bits, so a word
    // is the OR of d_s shifted by bits*(s % p).  A 16-byte piece holds p units of one lane:
    // piece k of lane L in half sigma is stored at piece index 128*(bits/2)*sigma + 64*k + L, so
    // thread tid writes piece tid (and tid + 256 at 4 bits) and every store is contiguous.
    auto gather = [&](int sigma, int lanep, int wsel, uint32_t (&d)[4]) {
        const int m = lanep & 15, G4 = lanep >> 4;
        if (kind == KVARN_KEYS) {
            const int t = 64 * sigma + 16 * (wsel >> 1) + m;
            const int c0 = 64 * (wsel & 1) + 16 * G4;
            const uint4 v = *reinterpret_cast<const uint4*>(&sm.codes[key_code_at(t, c0)]);
            d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
        } else {
            const int c = 16 * wsel + m;
#pragma unroll
            for (int ss = 0; ss < 4; ++ss)
                d[ss] = *reinterpret_cast<const uint32_t*>(&sm.codes[value_code_at(c, 64 * sigma + 16 * ss + 4 * G4)]);
        }
    };
    if (P.bits == 2) {
        const int sigma = L.tid >> 7, k = (L.tid >> 6) & 1, lanep = L.tid & 63;
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t d[4];
            gather(sigma, lanep, 4 * k + i, d);
            w[i] = d[0] | (d[1] << 2) | (d[2] << 4) | (d[3] << 6);
        }
        reinterpret_cast<uint4*>(dst)[L.tid] = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
#pragma unroll
        for (int pi = 0; pi < 2; ++pi) {
            const int pc = L.tid + 256 * pi;
            const int sigma = pc >> 8, k = (pc >> 6) & 3, lanep = pc & 63;
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                uint32_t d[4];
                gather(sigma, lanep, 2 * k + i, d);
                w[2 * i] = d[0] | (d[1] << 4);
                w[2 * i + 1] = d[2] | (d[3] << 4);
            }
            reinterpret_cast<uint4*>(dst)[pc] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
}

// Body tile blk of (sequence b, kv head kh) in the cache's tiles: dense [batch][n_kv][max_blocks],
// or paged (tile kh of pool block block_table[b][blk]).  -1 (and bit 1 of err_word) for a pool
// id outside [0, n_phys).
__device__ __forceinline__ int64_t body_tile(const kvarn_cache& c, int b, int kh, int blk) {
    if (!c.block_table) return ((int64_t)b * c.n_kv + kh) * c.max_blocks + blk;
    const int id = c.block_table[(size_t)b * c.max_blocks + blk];
    if (id < 0 || id >= c.n_phys) {
        if (threadIdx.x == 0 && c.err_word)
            __hip_atomic_fetch_or(c.err_word, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return -1;
    }
    return (int64_t)id * c.n_kv + kh;
}

struct TileArgs {
    QParams P;
    int kind;
    int x_bf16;
    const void* x;
    int64_t tile0, n_inner, x_outer, x_inner, x_token;
    uint8_t* out;
    int64_t out_outer, out_inner;
    int32_t* best_iter;
};

// Grids of many tiles: 4 waves per SIMD (128 VGPRs; the compact and exact variants keep 5 to 7 values in
// scratch, the others none, one in the flush) hide the barrier and LDS latency of the reductions better
// than 3 (measured 11 % faster).  So does the flush, whose grids are one tile per stream and
// K/V: 1024 tiles fit the card at once (56 us against 67 at 3).
template <bool COMPACT, bool EXACT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_quantize_tiles(TileArgs a) {
    __shared__ QuantSmem sm;
    const int64_t tile = a.tile0 + blockIdx.x;
    const int64_t i = tile / a.n_inner, j = tile % a.n_inner;
    const size_t esz = a.x_bf16 ? 2 : 4;
    const char* src = static_cast<const char*>(a.x) + (size_t)(i * a.x_outer + j * a.x_inner) * esz;
    uint8_t* dst = a.out + (size_t)(i * a.out_outer + j * a.out_inner) * tile_bytes(a.P.bits, COMPACT);
    quantize_tile<COMPACT, EXACT>(src, a.x_bf16 != 0, a.x_token, a.kind, a.P, dst, a.best_iter ? a.best_iter + tile : nullptr,
                           sm);
}

struct FlushArgs {
    QParams P;
    kvarn_cache c;
    int n_sink;
};

// Runs after the append kernel has incremented seq_len: the tile (sequence, kv head, K|V) of a
// sequence whose residual just reached 128 tokens is quantized into body tile
// (len - n_sink)/128 - 1; nothing else is written.  Workgroup w owns tiles w, w + gridDim.x,
// ...: with one workgroup per tile (a flush known to be due for every sequence) that is one
// tile, and with a grid of resident size (due tiles unknown on the host) its 256 threads check
// up to 256 of its tiles at once and the workgroup quantizes the due ones, so that a call with
// few or no due tiles costs one round of short workgroups.
template <bool COMPACT, bool EXACT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_flush(FlushArgs a) {
    __shared__ QuantSmem sm;
    __shared__ uint64_t due_mask[kThreads / 64];
    // tile indices fit 32 bits: the host bounds batch * n_kv
    const int n = a.c.batch * a.c.n_kv * 2;
    const int step = (int)gridDim.x;
    // the body tile a due tile goes to, or -1 when it is not due (or the append refused it)
    auto target_block = [&](int t) -> int {
        const int b = (t >> 1) / a.c.n_kv;
        const int len = a.c.seq_len[b];
        if (len <= a.n_sink || (len - a.n_sink) % kG != 0) return -1;
        const int nb = (len - a.n_sink) / kG - 1;
        return nb < a.c.max_blocks ? nb : -1;
    };
    for (int base = (int)blockIdx.x; base < n; base += step * kThreads) {
        const int mine = base + (int)threadIdx.x * step;
        const bool due = mine < n && target_block(mine) >= 0;
        const uint64_t m = __ballot(due);
        __syncthreads();  // the previous round is done with due_mask and the tile state in sm
        if ((threadIdx.x & 63) == 0) due_mask[threadIdx.x >> 6] = m;
        __syncthreads();
        bool first = true;
        for (int w = 0; w < kThreads / 64; ++w) {
            // uniform across the workgroup: kept in scalar registers
            const uint64_t dm = due_mask[w];
            uint64_t mm = (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)dm) |
                          (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(dm >> 32)) << 32;
            for (; mm; mm &= mm - 1) {
                const int t = base + (64 * w + __builtin_ctzll(mm)) * step;
                const int kind = t & 1;
                const int stream = t >> 1;
                const int b = stream / a.c.n_kv;
                const int64_t ti = body_tile(a.c, b, stream % a.c.n_kv, target_block(t));
                if (ti < 0) continue;
                if (!first) __syncthreads();  // every thread is done with the previous tile's LDS
                first = false;
                const uint16_t* src =
                    static_cast<const uint16_t*>(kind ? a.c.v_resid : a.c.k_resid) + (size_t)stream * kG * kD;
                uint8_t* dst =
                    static_cast<uint8_t*>(kind ? a.c.v_body : a.c.k_body) + (size_t)ti * tile_bytes(a.P.bits, COMPACT);
                quantize_tile<COMPACT, EXACT>(src, true, kD, kind, a.P, dst, nullptr, sm);
            }
        }
    }
}

struct PrefillArgs {
    QParams P;
    kvarn_cache c;
    int n_sink;
    const void* k;
    const void* v;
    int x_bf16;
    const int32_t* cu;  // [batch + 1] prompt offsets (rows of k, v)
    int max_len;
    int groups;         // body tiles per (sequence, kv head) the grid covers
    int64_t tile_blocks;  // workgroups of tiles; the rest copy bf16 rows
};

// Prompt length of sequence b, or -1 when it cannot be written (longer than the launch bound or
// than the body).
__device__ __forceinline__ int prefill_len(const PrefillArgs& a, int b) {
    const int L = a.cu[b + 1] - a.cu[b];
    const int nb = L > a.n_sink ? (L - a.n_sink) / kG : 0;
    return (L < 0 || L > a.max_len || nb > a.c.max_blocks) ? -1 : L;
}

// Sink and residual rows of one (sequence, kv head, K|V) as bf16, and the sequence's length.  Bound by
// latency: 8 channels per lane and four rows in flight (2-byte accesses in a launch of their own took
// 48 us for 12 prompts of up to 4k tokens, 8 kv heads, with a 128-token sink; beside the tiles, 0).
__device__ __forceinline__ void prefill_copy(const PrefillArgs& a, int64_t stream, int kind) {
    const int b = (int)(stream / a.c.n_kv), kh = (int)(stream % a.c.n_kv);
    const int L = prefill_len(a, b);
    if (threadIdx.x == 0 && kh == 0 && kind == 0) {
        a.c.seq_len[b] = L < 0 ? 0 : L;
        if (L < 0 && a.c.err_word)
            __hip_atomic_fetch_or(a.c.err_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (L < 0) return;
    const int ns = min(L, a.n_sink);
    const int nr = L > a.n_sink ? (L - a.n_sink) % kG : 0;
    const int r0 = L - nr;  // first residual row of the prompt
    const void* src = kind ? a.v : a.k;
    uint16_t* sink = static_cast<uint16_t*>(kind ? a.c.v_sink : a.c.k_sink) + (size_t)stream * a.n_sink * kD;
    uint16_t* resid = static_cast<uint16_t*>(kind ? a.c.v_resid : a.c.k_resid) + (size_t)stream * kG * kD;
    constexpr int U = 4, P = kD / 8;  // pieces of 8 channels
    const int n = (ns + nr) * P;
    for (int i0 = threadIdx.x; i0 < n; i0 += U * kThreads) {
        uint4 w[U];
        if (a.x_bf16) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = min(i0 + u * kThreads, n - 1), t = i / P;
                const size_t row = (size_t)(a.cu[b] + (t < ns ? t : r0 + (t - ns))) * a.c.n_kv + kh;
                w[u] = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(src) + row * kD + 8 * (i % P));
            }
        } else {
            float4 lo[U], hi[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = min(i0 + u * kThreads, n - 1), t = i / P;
                const size_t row = (size_t)(a.cu[b] + (t < ns ? t : r0 + (t - ns))) * a.c.n_kv + kh;
                const float4* p = reinterpret_cast<const float4*>(static_cast<const float*>(src) + row * kD + 8 * (i % P));
                lo[u] = p[0];
                hi[u] = p[1];
            }
            auto pair = [](float x, float y) { return (uint32_t)f32_to_bf16(x) | ((uint32_t)f32_to_bf16(y) << 16); };
#pragma unroll
            for (int u = 0; u < U; ++u)
                w[u] = make_uint4(pair(lo[u].x, lo[u].y), pair(lo[u].z, lo[u].w), pair(hi[u].x, hi[u].y), pair(hi[u].z, hi[u].w));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kThreads, t = i / P;
            if (i >= n) break;
            uint16_t* dst = t < ns ? sink + (size_t)t * kD : resid + (size_t)(t - ns) * kD;
            *reinterpret_cast<uint4*>(dst + 8 * (i % P)) = w[u];
        }
    }
}

// One workgroup per (sequence, kv head, K|V, body tile), which quantizes the prompt's tile straight
// from the packed rows (token stride n_kv * 128 elements), then one per (sequence, kv head, K|V) for
// the rows that stay bf16: these fill the tail of the tiles' last round.
template <bool COMPACT, bool EXACT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_prefill(PrefillArgs a) {
    __shared__ QuantSmem sm;
    if ((int64_t)blockIdx.x >= a.tile_blocks) {
        const int64_t c = (int64_t)blockIdx.x - a.tile_blocks;
        prefill_copy(a, c >> 1, (int)(c & 1));
        return;
    }
    const int blk = (int)(blockIdx.x % a.groups);
    const int64_t rest = blockIdx.x / a.groups;
    const int kind = (int)(rest & 1);
    const int64_t stream = rest >> 1;
    const int b = (int)(stream / a.c.n_kv), kh = (int)(stream % a.c.n_kv);
    const int L = prefill_len(a, b);
    if (L < 0 || blk >= (L > a.n_sink ? (L - a.n_sink) / kG : 0)) return;
    const int64_t ti = body_tile(a.c, b, kh, blk);
    if (ti < 0) return;
    const size_t esz = a.x_bf16 ? 2 : 4;
    const int64_t row = (int64_t)a.cu[b] + a.n_sink + (int64_t)blk * kG;
    const char* src = static_cast<const char*>(kind ? a.v : a.k) + (size_t)((row * a.c.n_kv + kh) * kD) * esz;
    uint8_t* dst = static_cast<uint8_t*>(kind ? a.c.v_body : a.c.k_body) + (size_t)ti * tile_bytes(a.P.bits, COMPACT);
    quantize_tile<COMPACT, EXACT>(src, a.x_bf16 != 0, (int64_t)a.c.n_kv * kD, kind, a.P, dst, nullptr, sm);
}

}  // namespace

// Unrotated, unbalanced tiles with fp32 aux (the KIVI-style ablation) take the quantizer variant
// whose RTN quotient keeps exact ties exact.
bool exact_quotient(const QParams& qp) { return !qp.compact && qp.iters == 0 && !qp.rotate; }

hipError_t launch_quantize_tiles(const QParams& qp, int kind, const void* x, bool x_bf16, int64_t n_outer,
                                 int64_t n_inner, int64_t x_outer, int64_t x_inner, int64_t x_token, void* out,
                                 int64_t out_outer, int64_t out_inner, int32_t* best_iter, hipStream_t stream) {
    const bool exact = exact_quotient(qp);
    const int64_t total = n_outer * n_inner;
    const int64_t kMaxGrid = 1 << 30;
    for (int64_t t0 = 0; t0 < total; t0 += kMaxGrid) {
        const int64_t n = total - t0 < kMaxGrid ? total - t0 : kMaxGrid;
        TileArgs a{qp, kind, x_bf16 ? 1 : 0, x, t0, n_inner, x_outer, x_inner, x_token,
                   static_cast<uint8_t*>(out), out_outer, out_inner, best_iter};
        if (qp.compact)
            hipLaunchKernelGGL((k_quantize_tiles<true, false>), dim3((unsigned)n), dim3(kThreads), 0, stream, a);
        else if (exact)
            hipLaunchKernelGGL((k_quantize_tiles<false, true>), dim3((unsigned)n), dim3(kThreads), 0, stream, a);
        else
            hipLaunchKernelGGL((k_quantize_tiles<false, false>), dim3((unsigned)n), dim3(kThreads), 0, stream, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_prefill(const QParams& qp, const kvarn_cache& c, int n_sink, const void* k, const void* v,
                          bool x_bf16, const int32_t* cu_seqlens, int max_len, hipStream_t stream) {
    const bool exact = exact_quotient(qp);
    int groups = max_len > n_sink ? (max_len - n_sink) / kG : 0;
    if (groups > c.max_blocks) groups = c.max_blocks;
    const int64_t streams = (int64_t)c.batch * c.n_kv, tiles = streams * 2 * groups, copies = streams * 2;
    if (tiles >= (int64_t)1 << 31) return hipErrorInvalidValue;
    PrefillArgs a{qp, c, n_sink, k, v, x_bf16 ? 1 : 0, cu_seqlens, max_len, groups, tiles};
    auto launch = [&](int64_t n) {
        if (qp.compact)
            hipLaunchKernelGGL((k_prefill<true, false>), dim3((unsigned)n), dim3(kThreads), 0, stream, a);
        else if (exact)
            hipLaunchKernelGGL((k_prefill<false, true>), dim3((unsigned)n), dim3(kThreads), 0, stream, a);
        else
            hipLaunchKernelGGL((k_prefill<false, false>), dim3((unsigned)n), dim3(kThreads), 0, stream, a);
        return hipGetLastError();
    };
    // A launch has at most 2^32 - 1 threads: where the tiles alone fit and the copies no longer do, they
    // go in a launch of their own.
    if (tiles > 0 && tiles + copies > 0xFFFFFFFFll / kThreads) {
        const hipError_t e = launch(tiles);
        if (e != hipSuccess) return e;
        a.tile_blocks = 0;
        return launch(copies);
    }
    return launch(tiles + copies);
}

hipError_t launch_flush(const QParams& qp, const kvarn_cache& c, int n_sink, bool all_due, hipStream_t stream) {
    const bool exact = exact_quotient(qp);
    FlushArgs a{qp, c, n_sink};
    // resident grid: three workgroups of 256 threads on each of 256 CUs (a CU holds four)
    constexpr int64_t kResidentGrid = 768;
    const int64_t n = (int64_t)c.batch * c.n_kv * 2;
    const unsigned grid = (unsigned)(all_due ? n : (n < kResidentGrid ? n : kResidentGrid));
    if (qp.compact)
        hipLaunchKernelGGL((k_flush<true, false>), dim3(grid), dim3(kThreads), 0, stream, a);
    else if (exact)
        hipLaunchKernelGGL((k_flush<false, true>), dim3(grid), dim3(kThreads), 0, stream, a);
    else
        hipLaunchKernelGGL((k_flush<false, false>), dim3(grid), dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

}  // namespace kvarn
