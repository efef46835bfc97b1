// KVarN decode attention for gfx950 (App. D three-region cache, App. I fused second scale,
// App. A rotation layout).
//
// Body tiles are attended in the rotated domain.  With q_rot = H q and a tile's aux
//   logit[t]  = s2K[t] * (sum_c q~[c] code[t][c] + beta),   q~ = q_rot * a_K, beta = q_rot . b_K
//   o_rot[c] += s2V[c] * (sum_t p~[t] code[t][c] + gamma),  p~ = p * a_V,   gamma = p . b_V
// so both dual-scale products are fused into one pass over the codes (App. I).
//
// The two sums over codes are matrix products on the int8 matrix cores
// (v_mfma_i32_16x16x64_i8).  The codes are exact int8 operands taken straight from the packed
// words (the tile format stores them in the MFMA register order).  The real-valued side is
// written as a fixed-point integer split into signed base-256 digits, recombined exactly in
// int32.  Integer accumulation is exact, so the only rounding in the code terms is that of q~
// and p~ to their fixed-point grids.
//
// The digits of a head are rows of one MFMA operand (three digits for both q~ and p~: 22 bits
// at 2-bit codes, 20 at 4-bit), and beta, gamma are plain fp32 dot products of the unrounded
// q_rot and p with the offsets.  A wave takes up to eight query heads of a kv head's group (one
// or two head groups of four, or four plus a fifth carried in the empty digit slots); larger
// groups are taken in chunks of at most eight heads, one wave per chunk.
//
// Sink and residual tokens (bf16, unrotated) use the bf16 matrix cores for q . k (q as a bf16
// pair hi + lo when it is fp32) and plain FMAs for p . v, in chunks of 32 tokens.  The waves of
// one workgroup share a (sequence, kv head, head chunk): its body tiles and its sink and residual
// chunks are dealt out as evenly as they go, by the sequence's own length, and the waves' parts
// are combined by log-sum-exp through LDS, each wave finishing some of the heads.  A workgroup
// has as many waves as leave every CU full (plan_decode): with one wave per SIMD a wave's chain
// of loads, LDS exchanges and products is exposed (one tile takes 1.45 us alone, 0.25 us per CU with
// twelve waves), and a few waves over a long sequence of a ragged batch last longer than the rest
// of the card.  Against at most four waves, fixed spans of tiles and one wave finishing alone: one
// layer of 32 sequences at 32k tokens, compact aux, 131 -> 102 us; 48 sequences of 1k to 16k
// tokens 84 -> 50 us; a step of 64 sequences at 1k tokens 19.5 -> 15.0 us.  Streams with too few
// workgroups to fill the card take several, whose partials the merge kernel combines (a step of
// one sequence at 8k tokens 13.9 -> 10.7 us: 17 partials per head instead of 37).
//
// A lock-step decode step can append its token in the same launch (Fig. 4): the new row is the
// residual's last, read from the token input by the wave that attends that chunk, which also
// stores it into the residual; the step's length comes from the host.
#include "common.hpp"

namespace kvarn {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

constexpr int kPart = 260;  // floats per partial: m, l, 2 pad, o_rot[128], o_plain[128]

// A fixed-point grid is only formed for a maximum above this; below it the values are taken
// as zero.  For p~ this drops a tile whose probabilities are all below 1e-30 relative to the
// running maximum (whose own probability, 1, is already in l): far below fp32 resolution of
// the sums.  It keeps grid scale = bound / max finite (a denormal or tiny max would make it
// inf, and 0 * inf a NaN).
constexpr float kTinyMax = 1e-30f;

struct DecodeArgs {
    // asked for at once at the start of the kernel (see there)
    const uint8_t* k_body;
    const uint8_t* v_body;
    const void* q;
    int32_t* seq_len;   // read, and written only by a fused append
    // Fused append of a lock-step step: step_len > 0 is the common length of the sequences with the
    // token of k_new / v_new ([batch][n_kv][kD], bf16 or fp32) appended as their last residual row;
    // 0: lengths from seq_len and no append.
    const void* k_new;
    const void* v_new;
    float* ws;         // [batch][n_q][n_wg][kPart] when n_wg > 1
    void* out;
    int step_len;
    int n_wg, group;   // workgroups per (stream, head chunk), waves per workgroup
    float inv_waves;   // 1 / (n_wg * group)
    int n_streams;     // batch * n_kv
    int n_chunk, g_chunk;  // head chunks per stream and heads per chunk
    int order;         // 1: longest sequences first (batch at most kOrderBatch)
    int n_kv, n_q, g, max_blocks, n_sink;
    int q_bf16, out_bf16;
    int rotate;        // 1: body tiles hold the Hadamard-rotated domain; 0: unrotated (ablations)
    float scale_log2;  // sm_scale * log2(e): logits are kept in log2 units
    int new_f32;
    int n_rows;        // batch * n_q
    // the rest
    uint16_t* k_resid;  // written only by a fused append
    uint16_t* v_resid;
    const uint16_t* k_sink;
    const uint16_t* v_sink;
    const int32_t* block_table;  // paged body: [batch][max_blocks] pool block ids, or null (dense)
    uint32_t* err_word;
    int n_phys;                  // pool size in blocks (paged)
};

__device__ __forceinline__ v4i mfma_i8(v4i a, v4i b, v4i c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma_bf16(v8bf a, v8bf b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// v_perm_b32: byte selector 0-3 picks from `lo`, 4-7 from `hi`, 0x0c gives zero.
__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
    return __builtin_amdgcn_perm(hi, lo, sel);
}

// The 16 codes of one unit as an int8 MFMA operand: byte q of dword s is code 4*s + q.
template <int BITS>
__device__ __forceinline__ v4i unit_i8(const uint32_t* w) {
    if constexpr (BITS == 2) {
        const uint32_t x = w[0], M = 0x03030303u;
        return v4i{(int)(x & M), (int)((x >> 2) & M), (int)((x >> 4) & M), (int)((x >> 6) & M)};
    } else {
        const uint32_t M = 0x0F0F0F0Fu;
        return v4i{(int)(w[0] & M), (int)((w[0] >> 4) & M), (int)(w[1] & M), (int)((w[1] >> 4) & M)};
    }
}

// Max in the NaN-propagating form: no operand of the reductions here is a NaN, and fmaxf would
// first quiet every operand that comes from another lane (one more instruction per step).
__device__ __forceinline__ float fmax_any(float x, float y) { return __builtin_elementwise_maximum(x, y); }

// Four values y0..y3, each a fixed-point integer plus 0x808080, to one dword per digit k whose
// byte i is the signed digit k of value i ((byte k of y_i) ^ 0x80).
__device__ __forceinline__ void digits4(uint32_t y0, uint32_t y1, uint32_t y2, uint32_t y3, uint32_t& d0,
                                        uint32_t& d1, uint32_t& d2) {
    const uint32_t t01 = perm(y1, y0, 0x05010400u), t23 = perm(y3, y2, 0x05010400u);
    d0 = perm(t23, t01, 0x05040100u) ^ 0x80808080u;
    d1 = perm(t23, t01, 0x07060302u) ^ 0x80808080u;
    const uint32_t u01 = perm(y1, y0, 0x0c0c0602u), u23 = perm(y3, y2, 0x0c0c0602u);
    d2 = perm(u23, u01, 0x05040100u) ^ 0x80808080u;
}

// Body tiles are read once per decode step: non-temporal 16-byte loads stream them from HBM
// faster than ordinary loads and leave the caches to reused data.
__device__ __forceinline__ uint4 load_stream(const uint8_t* p) {
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const v4u*>(p)));
}

// Body tile addressing.  Dense bodies: tile blk of a stream at stream * max_blocks + blk.
// Paged bodies: tile kvh of pool block block_table[b][blk].  block_id_t gives the block index
// (dense) or the pool block id (paged) of the stream's body tile blk.
template <int PG>
__device__ __forceinline__ int block_id_t(const DecodeArgs& a, int b, int blk) {
    if constexpr (PG) return a.block_table[(size_t)b * a.max_blocks + blk];
    else return blk;
}
// Paged bodies: the wave checks the pool ids of its tiles [blk0, blk1) once; an id outside the
// pool sets bit 1 of err_word and the caller skips the body (nothing outside the pool is read).
__device__ __forceinline__ bool body_ids_ok(const DecodeArgs& a, int b, int blk0, int blk1, int l) {
    if (!a.block_table) return true;
    bool bad = false;
    for (int i = blk0 + l; i < blk1; i += 64) {
        const int id = a.block_table[(size_t)b * a.max_blocks + i];
        bad |= id < 0 || id >= a.n_phys;
    }
    if (!__any(bad)) return true;
    if (l == 0 && a.err_word) __hip_atomic_fetch_or(a.err_word, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
}

// The aux of one K tile and one V tile as loaded for the row-digit kernels: lane l holds entries
// 2l and 2l + 1 of each row (a, b, s2 of the K tile's channels, of the V tile's tokens).  fp32:
// three 8-byte loads per tile; compact: the two binary16 offsets (4 bytes) and the two E4M3
// values of each scale row (2 bytes each).
template <int CMP>
struct HalfAux {
    uint2 a, b, s;
};
template <>
struct HalfAux<1> {
    uint32_t b, a, s;
};
__device__ __forceinline__ uint2 load_stream2(const uint8_t* p) {
    return __builtin_bit_cast(uint2, __builtin_nontemporal_load(reinterpret_cast<const v2u*>(p)));
}
template <int CMP>
__device__ __forceinline__ void load_half_aux(HalfAux<CMP>& r, const uint8_t* t, size_t cb, int l) {
    // (lane offsets as unsigned 32-bit values: the loads then take the uniform tile address as
    // their scalar base, with no 64-bit address arithmetic per lane)
    const uint8_t* x = t + cb;
    const uint32_t u = (uint32_t)l;
    if constexpr (CMP) {
        r.b = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(x + 4u * u));
        r.a = __builtin_nontemporal_load(reinterpret_cast<const uint16_t*>(x + (256u + 2u * u)));
        r.s = __builtin_nontemporal_load(reinterpret_cast<const uint16_t*>(x + (384u + 2u * u)));
    } else {
        r.a = load_stream2(x + 8u * u);
        r.b = load_stream2(x + (512u + 8u * u));
        r.s = load_stream2(x + (1024u + 8u * u));
    }
}
// -> fp32 rows a, b, s2 (rows r0, r0 + 1, r0 + 2 of aux), entries 2l and 2l + 1; both compact
// conversions are exact
template <int CMP>
__device__ __forceinline__ void stage_half_aux(float (&aux)[6][kD], int r0, const HalfAux<CMP>& r, int l) {
    float a0, a1, b0, b1, s0, s1;
    if constexpr (CMP) {
        const auto ap = __builtin_amdgcn_cvt_pk_f32_fp8((int)r.a, false);
        const auto sp = __builtin_amdgcn_cvt_pk_f32_fp8((int)r.s, false);
        a0 = ap[0];
        a1 = ap[1];
        s0 = sp[0];
        s1 = sp[1];
        b0 = (float)__builtin_bit_cast(_Float16, (uint16_t)(r.b & 0xFFFFu));
        b1 = (float)__builtin_bit_cast(_Float16, (uint16_t)(r.b >> 16));
    } else {
        a0 = __uint_as_float(r.a.x);
        a1 = __uint_as_float(r.a.y);
        b0 = __uint_as_float(r.b.x);
        b1 = __uint_as_float(r.b.y);
        s0 = __uint_as_float(r.s.x);
        s1 = __uint_as_float(r.s.y);
    }
    *reinterpret_cast<float2*>(&aux[r0][2 * l]) = make_float2(a0, a1);
    *reinterpret_cast<float2*>(&aux[r0 + 1][2 * l]) = make_float2(b0, b1);
    *reinterpret_cast<float2*>(&aux[r0 + 2][2 * l]) = make_float2(s0, s1);
}

// Orders this wave's accesses to its own LDS: a wave's LDS operations execute in issue order,
// so no wait is needed, only a point that the compiler does not move memory operations across.
// (Each wave of a decode workgroup has an LDS block of its own.)
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// NB runs of 8 consecutive query values, run r starting at element idx[r] (a multiple of 8), with
// one branch on the dtype.
template <int NB>
__device__ __forceinline__ void load_q_runs(const DecodeArgs& a, const size_t (&idx)[NB], float (&v)[NB][8]) {
    if (a.q_bf16) {
        const uint32_t* q2 = static_cast<const uint32_t*>(a.q);
#pragma unroll
        for (int r = 0; r < NB; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t w = q2[idx[r] / 2 + e];
                v[r][2 * e] = __uint_as_float(w << 16);
                v[r][2 * e + 1] = __uint_as_float(w & 0xFFFF0000u);
            }
    } else {
        const float* q1 = static_cast<const float*>(a.q);
#pragma unroll
        for (int r = 0; r < NB; ++r)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[r][e] = q1[idx[r] + e];
    }
}

// ---- group size <= 4: digit planes in the MFMA rows ----------------------------------------
// Both products take the real-valued side (q~ or p~, as base-256 digit planes) as the A operand
// and the codes as B.  Row 4*h + j of A is digit j of head h (j = 3 is zero).  The A and B
// register layouts of the 16x16x64 product are mirror images, so the code operands are the same
// registers as with codes in A.  Output lane (G, n) then receives, in its four accumulator
// registers, the digit partial sums of head G for column n (a token in QK, a channel in PV) and
// recombines them in-lane with two shifted adds.  One MFMA serves all three digits, and each
// lane finishes exactly one useful value per product.
//
// Between the products the probabilities move from the QK output layout (lane (G, n) = head G,
// token n of each 16) to the PV A layout (lane (G, 4h + j) = digit j of head h, tokens 4G..4G+3
// of each 16): a byte transpose inside each quad, then one lane permutation (ds_bpermute).

__device__ __forceinline__ int dpp_x1(int v) { return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true); }
__device__ __forceinline__ int dpp_x2(int v) { return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true); }
__device__ __forceinline__ int dpp_half_mirror(int v) { return __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true); }
__device__ __forceinline__ int dpp_mirror(int v) { return __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true); }
__device__ __forceinline__ float fdpp_x1(float v) { return __int_as_float(dpp_x1(__float_as_int(v))); }
__device__ __forceinline__ float fdpp_x2(float v) { return __int_as_float(dpp_x2(__float_as_int(v))); }
__device__ __forceinline__ float fdpp_half_mirror(float v) { return __int_as_float(dpp_half_mirror(__float_as_int(v))); }
__device__ __forceinline__ float fdpp_mirror(float v) { return __int_as_float(dpp_mirror(__float_as_int(v))); }
// The 128-point butterflies (unnormalized) over a wave's lanes, lane l holding channels 2l, 2l + 1:
// stride 1 in the lane, then lane partners l ^ 1, 2, 4, ..., 32, all by lane moves (partner ^4 is
// the half-row mirror of the quad-reversed value, ^8 a rotation of the row by 8).
template <int M>
__device__ __forceinline__ float lane_xor(float v, int l) {
    if constexpr (M == 1) return fdpp_x1(v);
    else if constexpr (M == 2) return fdpp_x2(v);
    else if constexpr (M == 4) return fdpp_half_mirror(__int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x1B, 0xF, 0xF, true)));
    else if constexpr (M == 8) return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xF, 0xF, true));
    else if constexpr (M == 16) {
        const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        return __uint_as_float(((l >> 4) & 1) ? x[0] : x[1]);
    } else {
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        return __uint_as_float(l < 32 ? x[1] : x[0]);
    }
}
template <int M>
__device__ __forceinline__ void fwht_stage(float (&x)[2], int l) {
    const bool upper = (l & M) != 0;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float p = lane_xor<M>(x[e], l);
        x[e] = upper ? p - x[e] : x[e] + p;
    }
}
__device__ __forceinline__ void fwht128(float (&x)[2], int l) {
    const float t = x[0];
    x[0] = t + x[1];
    x[1] = t - x[1];
    fwht_stage<1>(x, l);
    fwht_stage<2>(x, l);
    fwht_stage<4>(x, l);
    fwht_stage<8>(x, l);
    fwht_stage<16>(x, l);
    fwht_stage<32>(x, l);
}

// Query rows qrow .. qrow + g - 1 (lane l holds channels 2l, 2l + 1), rotated and normalized or as
// given, into LDS rows 0 .. NR - 1 (rows >= g zero).  One branch on the dtype, so every load is in
// flight before the first is used (q is only 4-byte aligned).  The rotation runs in registers: its
// seven stages through LDS cost a wave's set-up seven LDS round trips.
template <int NR>
__device__ __forceinline__ void q_to_lds(float (&q)[NR][kD], const DecodeArgs& a, size_t qrow, int g, int l) {
    float v0[NR], v1[NR];
    if (a.q_bf16) {
        const uint32_t* q2 = static_cast<const uint32_t*>(a.q);
#pragma unroll
        for (int h = 0; h < NR; ++h) {
            const uint32_t w = q2[(qrow + min(h, g - 1)) * (kD / 2) + l];
            v0[h] = __uint_as_float(w << 16);
            v1[h] = __uint_as_float(w & 0xFFFF0000u);
        }
    } else {
        const float* q1 = static_cast<const float*>(a.q);
#pragma unroll
        for (int h = 0; h < NR; ++h) {
            const size_t i = (qrow + min(h, g - 1)) * kD + 2 * l;
            v0[h] = q1[i];
            v1[h] = q1[i + 1];
        }
    }
    const float qs = a.rotate ? kInvSqrt128 : 1.f;
#pragma unroll
    for (int h = 0; h < NR; ++h) {
        float x[2] = {v0[h], v1[h]};
        if (a.rotate) fwht128(x, l);
        *reinterpret_cast<float2*>(&q[h][2 * l]) = h < g ? make_float2(x[0] * qs, x[1] * qs) : make_float2(0.f, 0.f);
    }
}

// max / sum over the 16 lanes of a row (lanes 16G .. 16G + 15): the quad (partners ^1, ^2), then
// the other quad of the half (mirror within 8), then the other half (mirror within 16).  Every
// step combines two equal-shaped partial results, so all 16 lanes end with identical values.
__device__ __forceinline__ float row_max(float v) {
    v = fmax_any(v, fdpp_x1(v));
    v = fmax_any(v, fdpp_x2(v));
    v = fmax_any(v, fdpp_half_mirror(v));
    return fmax_any(v, fdpp_mirror(v));
}
// The same for values >= 0: their bit patterns order as signed integers, so the steps run as
// integer max instructions with the lane move folded in.
__device__ __forceinline__ float row_max_nonneg(float v) {
    int b = __float_as_int(v);
    b = max(b, dpp_x1(b));
    b = max(b, dpp_x2(b));
    b = max(b, dpp_half_mirror(b));
    return __int_as_float(max(b, dpp_mirror(b)));
}
__device__ __forceinline__ float row_sum(float v) {
    v += fdpp_x1(v);
    v += fdpp_x2(v);
    v += fdpp_half_mirror(v);
    return v + fdpp_mirror(v);
}

// The digit-weighted sum of one output lane: register i holds the partial sum of digit i.  The
// true sum fits int32, so the wrapping arithmetic below is exact.  Horner form, two
// shift-and-add instructions (v_lshl_add_u32); the empty asm statement keeps the compiler from
// distributing the outer shift over the inner sum, which costs a third instruction.
__device__ __forceinline__ int digit_sum(v4i c) {
    uint32_t t = ((uint32_t)c[2] << 8) + (uint32_t)c[1];
    asm("" : "+v"(t));
    return (int)((t << 8) + (uint32_t)c[0]);
}

// Lane j of a quad holds y (row j of a 4 x 4 byte matrix); returns column j: byte i of the
// result is byte j of lane i's y.  Two exchanges (partners j ^ 2, then j ^ 1), each a DPP move
// and a byte permute.
__device__ __forceinline__ uint32_t quad_transpose_bytes(uint32_t y, int j) {
    const uint32_t selA = j < 2 ? 0x05040100u : 0x03020706u;
    const uint32_t selB = (j & 1) ? 0x03070105u : 0x06020400u;
    const uint32_t t = perm((uint32_t)dpp_x2((int)y), y, selA);
    return perm((uint32_t)dpp_x1((int)t), t, selB);
}

// The codes of one unit as the B operand of the row-digit kernel.  At 2 bits one shift gives
// all four byte planes: dwords 0 and 2 carry the codes, dwords 1 and 3 four times the codes;
// the A operand compensates with elements kPlaneMul times larger in dwords 0 and 2.
template <int BITS>
__device__ __forceinline__ v4i unit_planes(const uint32_t* w) {
    if constexpr (BITS == 2) {
        const uint32_t x = w[0], x4 = x >> 4, M = 0x03030303u;
        return v4i{(int)(x & M), (int)(x & (M << 2)), (int)(x4 & M), (int)(x4 & (M << 2))};
    } else {
        return unit_i8<BITS>(w);
    }
}
template <int BITS>
constexpr float kPlaneMul = BITS == 2 ? 4.f : 1.f;

// Query heads are taken in groups of four (NH groups, g <= 4 * NH): every group repeats the
// per-head work on the same code operands, which are extracted once per tile.
template <int NH, int X1>
struct Smem4 {
    float q[4 * NH + X1][kD];       // rotated q (rows >= g zero); reused for the inverse rotation of the output
    float aux[6][kD];               // a_K b_K s2_K a_V b_V s2_V of the current tile
    uint4 qp[NH][4][2][16];         // q~ digit planes [group][digit slot][kappa][qslot(slot, G, head)]; slot 3 stays zero
    uint4 qp4[X1 ? 4 : 1][2][4];    // X1: the extra head's q~ digit planes [digit slot][kappa][G]; slot 3 zero
    float hv[4 * NH + X1][4];       // per head: beta, q~ step, alpha, l
    float p[4 * NH + X1][kRC];      // probabilities of a bf16 chunk (sink / residual)
};

// Position of the 16-byte piece (K group G, head h) in a digit slot's row of the q~ planes.  The
// QK operand read has lane (G, 4h + j) fetch piece (G, h) of slot j; the slot-dependent swizzle
// gives the 16 lanes of a row 16 different bank groups (unswizzled, the four slots of one (G, h)
// share a bank group).
__device__ __forceinline__ int qslot(int slot, int G, int h) { return (4 * G + h) ^ (4 * slot); }

// Max and sum over the whole wave (the four DPP rows, then row pairs): every lane ends with
// the same value.
template <class F>
__device__ __forceinline__ float across_rows4(float v, F f) {
    const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = f(__uint_as_float(x[0]), __uint_as_float(x[1]));
    const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return f(__uint_as_float(y[0]), __uint_as_float(y[1]));
}
__device__ __forceinline__ float wave_max(float v) {
    return across_rows4(row_max(v), [](float x, float y) { return fmax_any(x, y); });
}
__device__ __forceinline__ float wave_max_nonneg(float v) {
    return across_rows4(row_max_nonneg(v), [](float x, float y) {
        return __int_as_float(max(__float_as_int(x), __float_as_int(y)));
    });
}
__device__ __forceinline__ float wave_sum(float v) {
    return across_rows4(row_sum(v), [](float x, float y) { return x + y; });
}

// Digit-weighted sum over the four row groups of a wave (lanes n, 16 + n, 32 + n, 48 + n),
// scattered: row group G receives the sum over r of x_G(row group r) * 256^r.
// permlane32_swap(a, b) returns {a's rows 0-1, b's rows 0-1} and {a's rows 2-3, b's rows 2-3}, so
// after the first two swaps a lane of row group R holds x(R mod 2) and x(R mod 2 + 2) of x0, x1
// (rows 0-1) or x2, x3 (rows 2-3); their weights differ by 256^2, so the lane adds the second
// times 2^16 and keeps the common factor 256^(R mod 2) for later.  permlane16_swap(a, b) returns
// {a's even rows in even rows, b's even rows in odd rows} and {a's odd rows in even rows, b's odd
// rows in odd rows}: the even-row partial (factor 1) plus 2^8 times the odd-row partial (factor
// 256) completes each row group's sum.  Integer arithmetic wraps exactly.
__device__ __forceinline__ uint32_t rows_digit_reduce_scatter4(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3) {
    const auto a = __builtin_amdgcn_permlane32_swap(x0, x2, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(x1, x3, false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0] + (a[1] << 16), b[0] + (b[1] << 16), false, false);
    return c[0] + (c[1] << 8);
}

// The sequence with the given rank by length, the longest first (equal ones in order of index).
// Every wave ranks the whole batch, two sequences per lane; where all are equally long, rank is index.
__device__ __forceinline__ int sequence_of_rank(const int32_t* seq_len, int batch, int rank, int l) {
    const int i0 = min(l, batch - 1), i1 = min(64 + l, batch - 1);
    const int len0 = seq_len[i0], len1 = seq_len[i1];
    const int first = __builtin_amdgcn_readfirstlane(len0);
    if (!__any(len0 != first || len1 != first)) return rank;
    // unique keys: the length (capped, an order is all that is asked), then the smaller index
    const uint32_t k0 = (uint32_t)min(max(len0, 0), 0xFFFFFF) << 7 | (uint32_t)(kOrderBatch - 1 - i0);
    const uint32_t k1 = (uint32_t)min(max(len1, 0), 0xFFFFFF) << 7 | (uint32_t)(kOrderBatch - 1 - i1);
    int r0 = 0, r1 = 0;
    for (int i = 0; i < min(batch, 64); ++i) {
        const uint32_t k = __builtin_amdgcn_readlane(k0, i);
        r0 += k > k0;
        r1 += k > k1;
    }
    for (int i = 64; i < batch; ++i) {
        const uint32_t k = __builtin_amdgcn_readlane(k1, i - 64);
        r0 += k > k0;
        r1 += k > k1;
    }
    // (clamped lanes repeat the last sequence; the first lane that holds the rank is taken)
    const uint64_t m0 = __ballot(r0 == rank), m1 = __ballot(r1 == rank);
    return min(m0 ? __builtin_ctzll(m0) : 64 + __builtin_ctzll(m1), batch - 1);
}

// X1 = 1 (group size 5, with NH = 1): a fifth query head spread over the whole wave instead of a
// second head group of four slots, carried by the head group's own products in the digit slot
// the group leaves empty: q~ and p~ have three digits, so A row 4 h + 3 (slot 3 of head h) is
// zero, and rows 3, 7 and 11 take the extra head's digits 0, 1 and 2.  Accumulator 3 of lane
// (G, n) then holds its digit-G partial sum for column n (a token in QK, a channel in PV; row
// group 3 gets zero from row 15), and a reduce-scatter over the row groups combines the digits
// so that lane (G, n) holds the head's logits for tokens 64 sg + 16 G + n and its outputs for
// channels 16 (4 q + G) + n (sg, q = 0, 1): two values per lane, no padded head slots and no
// MFMA of its own.
// NEW32 = 1: the fused step's token is fp32.  (Kernels of their own, for dense bodies: as a branch of
// the others its code costs a short bf16 step 1 to 10 %.)
template <int BITS, int NH, int CMP, int PG, int X1, int NEW32>
__global__ __launch_bounds__(64 * (BITS == 2 && NH == 1 && !X1 ? kMaxGroup3 : kMaxGroup2))
__attribute__((amdgpu_waves_per_eu(BITS == 2 && NH == 1 && !X1 ? 3 : 2, 8)))
void k_decode4(DecodeArgs a) {
    static_assert(X1 == 0 || NH == 1, "the extra head is only for one head group");
    // one LDS block per wave (dynamic: a.group waves per workgroup)
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Smem4<NH, X1>& sm = reinterpret_cast<Smem4<NH, X1>*>(dyn_lds)[wave];
    constexpr int WPU = BITS / 2;
    constexpr int NHD = 4 * NH;   // head slots of the head groups
    constexpr int NHX = NHD + X1;  // all head slots
    // Fixed point: q~ and p~ in even dwords of the A operand are scaled by MUL (the code planes
    // there are not shifted up), so every product term carries weight MUL.  The exact sum is
    // bounded by MUL * (2^BITS - 1) * 128 * QMAX < 2^31 and MUL * QMAX < 2^22 keeps the
    // rounding below exact.
    constexpr float MUL = kPlaneMul<BITS>;
    constexpr int QMAX = 1048575;
    constexpr float MAGIC = 12582912.f;  // 1.5 * 2^23: x + MAGIC rounds x to an integer
    constexpr uint32_t MAGIC_BITS = 0x4B400000u;
    // output role: head 4*hg + G, column n; A-operand role: row 4*h + j (digit j of head 4*hg + h)
    const int l = threadIdx.x & 63, G = l >> 4, n = l & 15, h = (l >> 2) & 3, j = l & 3;
    // workgroup = (head chunk, stream, part of the stream), the chunk slowest: the chunks of a
    // stream read the same tiles, n_streams * n_wg workgroups apart, which keeps them on one XCD
    // when that distance is a multiple of 8.
    // Every argument of the set-up is asked for here, in one round of scalar loads: fetched where it is
    // first used, each line of them costs the wave a miss of its own (the steps of one sequence at 8k
    // tokens 11.65 -> 11.2 us, of 64 at 1k 15.9 -> 15.3).
    asm volatile("" ::"s"(a.k_body), "s"(a.v_body), "s"(a.q), "s"(a.seq_len), "s"(a.k_new), "s"(a.v_new), "s"(a.ws), "s"(a.out),
                 "s"(a.step_len), "s"(a.n_wg), "s"(a.group), "s"(a.inv_waves), "s"(a.n_streams), "s"(a.n_chunk), "s"(a.g_chunk),
                 "s"(a.order), "s"(a.n_kv), "s"(a.n_q), "s"(a.g), "s"(a.max_blocks), "s"(a.n_sink), "s"(a.q_bf16),
                 "s"(a.out_bf16), "s"(a.rotate), "s"(a.scale_log2), "s"(a.new_f32));
    const uint32_t cs = a.n_wg > 1 ? blockIdx.x / (uint32_t)a.n_wg : blockIdx.x;
    const int wgi = (int)(blockIdx.x - cs * (uint32_t)a.n_wg);
    const int chunk = a.n_chunk > 1 ? (int)(cs / (uint32_t)a.n_streams) : 0;
    int stream = (int)(cs - (uint32_t)chunk * (uint32_t)a.n_streams);
    const int g = min(a.g_chunk, a.g - chunk * a.g_chunk);  // query heads of this wave
    int b = (int)((uint32_t)stream / (uint32_t)a.n_kv);
    const int kvh = stream - b * a.n_kv;
    if (a.order) {
        b = sequence_of_rank(a.seq_len, a.n_streams / a.n_kv, b, l);
        stream = b * a.n_kv + kvh;
    }
    // A fused append takes the step's length from the host (the stored one is read later, off the
    // wave's path, and only checked).
    int len = a.step_len;
    if (a.step_len == 0) len = max(a.seq_len[b], 0);
    const int ns = min(len, a.n_sink);
    const int nbody = min(len > a.n_sink ? (len - a.n_sink) / kG : 0, a.max_blocks);
    const int nr = len > a.n_sink ? (len - a.n_sink) % kG : 0;
    // The stream's work in units, its body tiles, then the 32-token chunks of its sink and of its
    // residual: wave i of the stream's n_waves takes an even share of consecutive units (the first
    // waves one more where it does not divide), by the sequence's own length, so that the waves
    // of a short sequence of a ragged batch share its tiles too.
    const int nsc = (ns + kRC - 1) / kRC, nch = nsc + (nr + kRC - 1) / kRC;
    const int n_waves = a.n_wg * a.group, wi = wgi * a.group + wave;
    int blk0 = 0, blk1 = nbody, c0 = 0, c1 = nch;
    if (n_waves > 1) {
        const int nu = nbody + nch;
        int base = (int)((float)nu * a.inv_waves), rem = nu - base * n_waves;  // nu / n_waves, or one off
        if (rem < 0) {
            --base;
            rem += n_waves;
        } else if (rem >= n_waves) {
            ++base;
            rem -= n_waves;
        }
        const int u0 = wi * base + min(wi, rem), u1 = u0 + base + (wi < rem ? 1 : 0);
        blk0 = min(u0, nbody);
        blk1 = min(u1, nbody);
        c0 = max(u0 - nbody, 0);
        c1 = max(u1 - nbody, 0);
    }
    if (PG && blk0 < blk1 && !body_ids_ok(a, b, blk0, blk1, l)) blk1 = blk0;
    const size_t qrow = (size_t)b * a.n_q + (size_t)kvh * a.g + (size_t)chunk * a.g_chunk;
    const size_t tb = tile_bytes(BITS, CMP), cb = code_bytes(BITS);

    float m_run[NH], l_run[NH];  // head 4*hg + G; l_run is this lane's partial sum
    float orot[NH][8];           // head 4*hg + G, channel 16*mt + n (rotated domain)
    // X1: the extra head's running max, this lane's partial sum, and its output channels
    // 16 (4 q + G) + n, q = 0, 1
    float m4 = -INFINITY, l4 = 0.f, orot4[2] = {0.f, 0.f};
#pragma unroll
    for (int hg = 0; hg < NH; ++hg) {
        m_run[hg] = -INFINITY;
        l_run[hg] = 0.f;
#pragma unroll
        for (int mt = 0; mt < 8; ++mt) orot[hg][mt] = 0.f;
    }

    // online softmax of group hg over this lane's logits (log2 units; -inf = absent) -> p,
    // returns alpha
    auto softmax_update = [](auto& lg, bool maybe_absent, float& m, float& lsum) -> float {
        constexpr int N = sizeof(lg) / sizeof(lg[0]);
        float mx = lg[0];
#pragma unroll
        for (int k = 1; k < N; ++k) mx = fmaxf(mx, lg[k]);
        mx = row_max(mx);
        const float m_new = fmaxf(m, mx);
        const float alpha = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - m_new);
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            float p = __builtin_amdgcn_exp2f(lg[k] - m_new);
            if (maybe_absent) p = lg[k] == -INFINITY ? 0.f : p;
            lg[k] = p;
            s += p;
        }
        lsum = lsum * alpha + s;
        m = m_new;
        return alpha;
    };

    // the same for the extra head, whose 128 logits are spread over the wave (two per lane)
    auto softmax_wave = [](float (&lg)[2], bool maybe_absent, float& m, float& lsum) -> float {
        const float mx = wave_max(fmaxf(lg[0], lg[1]));
        const float m_new = fmaxf(m, mx);
        const float alpha = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - m_new);
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            float p = __builtin_amdgcn_exp2f(lg[k] - m_new);
            if (maybe_absent) p = lg[k] == -INFINITY ? 0.f : p;
            lg[k] = p;
            s += p;
        }
        lsum = lsum * alpha + s;
        m = m_new;
        return alpha;
    };

    if (blk0 < blk1) {
        // Two register buffers, one tile each, alternate between tiles.  While a tile is
        // consumed from one, the next tile's parts go into the other: its aux right after the
        // current aux is staged in LDS, its key codes after the QK products, its value codes
        // after the PV products.  The first tile's loads go out before the query set-up.  No
        // load sits behind a branch (the prefetch past the last tile re-reads that tile), so
        // each wait counts exactly the loads it needs.
        struct TileRegs {
            uint4 k[2][2 * WPU], v[2][2 * WPU];
            HalfAux<CMP> ak, av;
        };
        TileRegs ra, rb;
        // tiles by block_id (pool id when paged); the id of the next tile is read a tile ahead
        auto tile_of = [&](int id) { return PG ? (size_t)id * a.n_kv + kvh : (size_t)stream * a.max_blocks + id; };
        auto tile_k = [&](int id) { return a.k_body + tile_of(id) * tb; };
        auto tile_v = [&](int id) { return a.v_body + tile_of(id) * tb; };
        auto load_aux = [&](TileRegs& r, int id) {
            load_half_aux<CMP>(r.ak, tile_k(id), cb, l);
            load_half_aux<CMP>(r.av, tile_v(id), cb, l);
        };
        auto load_codes = [&](const uint8_t* t, uint4 (&c)[2][2 * WPU]) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int k = 0; k < 2 * WPU; ++k) c[s][k] = load_stream(t + 16u * (unsigned)(s * 128 * WPU + 64 * k + l));
        };
        const int id0 = block_id_t<PG>(a, b, blk0);
        load_codes(tile_k(id0), ra.k);
        load_codes(tile_v(id0), ra.v);
        load_aux(ra, id0);

        q_to_lds<NHX>(sm.q, a, qrow, g, l);
        for (int idx = l; idx < NH * 32; idx += 64)
            sm.qp[idx >> 5][3][(idx >> 4) & 1][idx & 15] = make_uint4(0u, 0u, 0u, 0u);
        if (X1 && l < 8) sm.qp4[X1 ? 3 : 0][l >> 2][l & 3] = make_uint4(0u, 0u, 0u, 0u);
        wave_sync();
        // q~ role: head 4*hg + G, channels 8n .. 8n + 7.  Two head groups: q stays in LDS, which keeps
        // 16 registers free for the tile loop.
        constexpr bool QLDS = NH == 2;
        float qr[8];
        if constexpr (!QLDS) {
#pragma unroll
            for (int k = 0; k < 8; ++k) qr[k] = sm.q[G][8 * n + k];
        }
        // extra head: channels 2l, 2l + 1
        const float qr4[2] = {X1 ? sm.q[NHX - 1][2 * l] : 0.f, X1 ? sm.q[NHX - 1][2 * l + 1] : 0.f};
        // source lane of the PV operand permutation (see above), as a byte address; for the
        // extra head the source row is the token block (tau), not the head
        const int perm_addr = (16 * h + 4 * G + j) * 4;
        // extra head: A row 4 h + 3 (h < 3) takes digit h from lane 4 G + h of token block tau
        const bool x1_row = X1 && j == 3 && h < 3;
        const int perm4 = (4 * G + h) * 4;

        // One tile: consume cur, prefetch tile id_next into nxt.
        // zoff is 0; the odd last tile passes it through an empty asm statement, so that its LDS
        // offsets are formed after the loop rather than held in registers across it (which spilled
        // them in the largest variant)
        auto step = [&](TileRegs& cur, TileRegs& nxt, int id_next, int zoff) {
            wave_sync();  // the previous tile is done with sm.aux / sm.qp / sm.hv
            // aux rows a_K, b_K, s2_K (keys: per channel), a_V, b_V, s2_V (values: per token)
            stage_half_aux<CMP>(sm.aux, 0, cur.ak, l);
            stage_half_aux<CMP>(sm.aux, 3, cur.av, l);
            load_aux(nxt, id_next);
            wave_sync();
            uint32_t kw[2][8 * WPU], vw[2][8 * WPU];
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int k = 0; k < 2 * WPU; ++k) {
                    kw[s][4 * k] = cur.k[s][k].x; kw[s][4 * k + 1] = cur.k[s][k].y;
                    kw[s][4 * k + 2] = cur.k[s][k].z; kw[s][4 * k + 3] = cur.k[s][k].w;
                    vw[s][4 * k] = cur.v[s][k].x; vw[s][4 * k + 1] = cur.v[s][k].y;
                    vw[s][4 * k + 2] = cur.v[s][k].z; vw[s][4 * k + 3] = cur.v[s][k].w;
                }
            // q~ = q_rot * a_K as fixed point on a per-head grid, then three digit planes; beta =
            // sum over channels of q_rot * b_K, the offsets' part of the logit (unscaled)
            {
                const float4 a0 = *reinterpret_cast<const float4*>(&sm.aux[0][8 * n]);
                const float4 a1 = *reinterpret_cast<const float4*>(&sm.aux[0][8 * n + 4]);
                const float4 b0 = *reinterpret_cast<const float4*>(&sm.aux[1][8 * n]);
                const float4 b1 = *reinterpret_cast<const float4*>(&sm.aux[1][8 * n + 4]);
                const float av[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
                const float bk[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
                // channels 8n .. 8n + 7 = kappa n / 8, group (n % 8) / 2, components 2 (n % 2) + {0, 1}
                const int kap = n >> 3, Gq = (n >> 1) & 3, half = n & 1;
#pragma unroll
                for (int hg = 0; hg < NH; ++hg) {
                    float qv[8], qt[8], mx = 0.f;
                    if constexpr (QLDS) {
                        const float4 x0 = *reinterpret_cast<const float4*>(&sm.q[4 * hg + G][8 * n]);
                        const float4 x1 = *reinterpret_cast<const float4*>(&sm.q[4 * hg + G][8 * n + 4]);
                        qv[0] = x0.x; qv[1] = x0.y; qv[2] = x0.z; qv[3] = x0.w;
                        qv[4] = x1.x; qv[5] = x1.y; qv[6] = x1.z; qv[7] = x1.w;
                    } else {
#pragma unroll
                        for (int k = 0; k < 8; ++k) qv[k] = qr[k];
                    }
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        qt[k] = qv[k] * av[k];
                        mx = fmaxf(mx, fabsf(qt[k]));
                    }
                    mx = row_max_nonneg(mx);
                    const float sc = mx > kTinyMax ? (float)QMAX * __builtin_amdgcn_rcpf(mx) : 0.f;
                    // channels 8n .. 8n + 3 sit in an even dword of the A operand, 8n + 4 ..
                    // 8n + 7 in an odd one
                    float bsum = 0.f;
                    uint32_t y[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const float yf = fmaf(qt[k], k < 4 ? sc * MUL : sc, MAGIC);
                        bsum = fmaf(qv[k], bk[k], bsum);
                        y[k] = __float_as_uint(yf) + (0x808080u - MAGIC_BITS);
                    }
                    const float bs = row_sum(bsum);
                    uint32_t d0, d1, d2, e0, e1, e2;
                    digits4(y[0], y[1], y[2], y[3], d0, d1, d2);
                    digits4(y[4], y[5], y[6], y[7], e0, e1, e2);
                    reinterpret_cast<uint2*>(&sm.qp[hg][0][kap][qslot(0, Gq, G)])[half] = make_uint2(d0, e0);
                    reinterpret_cast<uint2*>(&sm.qp[hg][1][kap][qslot(1, Gq, G)])[half] = make_uint2(d1, e1);
                    reinterpret_cast<uint2*>(&sm.qp[hg][2][kap][qslot(2, Gq, G)])[half] = make_uint2(d2, e2);
                    if (n == 0) {
                        sm.hv[4 * hg + G][0] = bs;
                        sm.hv[4 * hg + G][1] = mx * (1.0f / (MUL * (float)QMAX));
                    }
                }
                if constexpr (X1) {
                    // extra head: channels 2l, 2l + 1 = kappa l / 32, group (l / 8) % 4, bytes
                    // 2 (l % 8) + {0, 1} of that group (an even dword when (l / 2) % 2 == 0);
                    // grid, digits and beta as for the head groups, over the whole wave
                    const float2 a2 = *reinterpret_cast<const float2*>(&sm.aux[0][2 * l]);
                    const float2 b2 = *reinterpret_cast<const float2*>(&sm.aux[1][2 * l]);
                    const float qt0 = qr4[0] * a2.x, qt1 = qr4[1] * a2.y;
                    const float mx = wave_max_nonneg(fmaxf(fabsf(qt0), fabsf(qt1)));
                    const float sc = mx > kTinyMax ? (float)QMAX * __builtin_amdgcn_rcpf(mx) : 0.f;
                    const bool even = ((l >> 1) & 1) == 0;
                    const float y0f = fmaf(qt0, even ? sc * MUL : sc, MAGIC);
                    const float y1f = fmaf(qt1, even ? sc * MUL : sc, MAGIC);
                    const float bs = wave_sum(fmaf(qr4[1], b2.y, qr4[0] * b2.x));
                    const uint32_t y0 = __float_as_uint(y0f) + (0x808080u - MAGIC_BITS);
                    const uint32_t y1 = __float_as_uint(y1f) + (0x808080u - MAGIC_BITS);
                    const uint32_t d01 = perm(y1, y0, 0x05010400u) ^ 0x80808080u;  // digit 0 | digit 1 pairs
                    const uint32_t d2 = perm(y1, y0, 0x0c0c0602u) ^ 0x8080u;       // digit 2 pair
                    const int kp = l >> 5, gq = (l >> 3) & 3, e = l & 7;
                    reinterpret_cast<uint16_t*>(&sm.qp4[0][kp][gq])[e] = (uint16_t)(d01 & 0xFFFFu);
                    reinterpret_cast<uint16_t*>(&sm.qp4[X1 ? 1 : 0][kp][gq])[e] = (uint16_t)(d01 >> 16);
                    reinterpret_cast<uint16_t*>(&sm.qp4[X1 ? 2 : 0][kp][gq])[e] = (uint16_t)d2;
                    if (l == 0) {
                        sm.hv[NHX - 1][0] = bs;
                        sm.hv[NHX - 1][1] = mx * (1.0f / (MUL * (float)QMAX));
                    }
                }
            }
            wave_sync();

            // logits of head 4*hg + G, token 64*sg + 16*tau + n.  Tokens outer, head groups
            // inner: the code planes of a token block are extracted once and used at once.
            float lg[NH][8];
            v4i aq[NH][2];
            float bq[NH], fqs[NH];  // beta and the q~ grid step in logit units (log2, scaled)
#pragma unroll
            for (int hg = 0; hg < NH; ++hg) {
#pragma unroll
                for (int kap = 0; kap < 2; ++kap) {
                    // X1: rows 3, 7, 11 (slot 3 of heads 0-2) take the extra head's digits 0-2
                    const int jq = j + zoff;
                    const uint4 u = X1 && j == 3 && h < 3 ? sm.qp4[X1 ? h : 0][kap][G] : sm.qp[hg][jq][kap][qslot(jq, G, h)];
                    aq[hg][kap] = v4i{(int)u.x, (int)u.y, (int)u.z, (int)u.w};
                }
                fqs[hg] = sm.hv[4 * hg + G][1] * a.scale_log2;
                bq[hg] = sm.hv[4 * hg + G][0] * a.scale_log2;
            }
            // X1: accumulator 3 holds the extra head's digit-G partial (row group 3: zero)
            uint32_t x4[2][4];
#pragma unroll
            for (int sg = 0; sg < 2; ++sg)
#pragma unroll
                for (int tau = 0; tau < 4; ++tau) {
                    const v4i b0 = unit_planes<BITS>(&kw[sg][(2 * tau) * WPU]);
                    const v4i b1 = unit_planes<BITS>(&kw[sg][(2 * tau + 1) * WPU]);
                    const float s2k = sm.aux[2][64 * sg + 16 * tau + n];
#pragma unroll
                    for (int hg = 0; hg < NH; ++hg) {
                        v4i c = mfma_i8(aq[hg][0], b0, v4i{0, 0, 0, 0});
                        c = mfma_i8(aq[hg][1], b1, c);
                        lg[hg][4 * sg + tau] = fmaf((float)digit_sum(c), fqs[hg], bq[hg]) * s2k;
                        if (X1 && hg == 0) x4[sg][tau] = (uint32_t)c[3];
                    }
                }
            float lg4[2] = {0.f, 0.f};  // extra head, tokens 64 sg + 16 G + n
            if constexpr (X1) {
                const float fqs4 = sm.hv[NHX - 1][1] * a.scale_log2, bq4 = sm.hv[NHX - 1][0] * a.scale_log2;
#pragma unroll
                for (int sg = 0; sg < 2; ++sg) {
                    const uint32_t raw = rows_digit_reduce_scatter4(x4[sg][0], x4[sg][1], x4[sg][2], x4[sg][3]);
                    lg4[sg] = fmaf((float)(int)raw, fqs4, bq4) * sm.aux[2][64 * sg + 16 * G + n];
                }
            }
            load_codes(tile_k(id_next), nxt.k);

            // extra head: lane (G, n) holds token 64 sg + 16 G + n, i.e. token block tau = G of
            // each sg; its digit words are byte-transposed like the head groups' and reach A rows
            // 3, 7, 11 (digit h in row 4 h + 3) from the lanes of token block tau
            float alpha4 = 0.f, gam4 = 0.f, fp4 = 0.f;
            uint32_t t4[2] = {0u, 0u};
            if constexpr (X1) {
                alpha4 = softmax_wave(lg4, false, m4, l4);
                // the offsets' part of the output: sum over tokens of p * b_V
                gam4 = wave_sum(fmaf(lg4[1], sm.aux[4][64 + 16 * G + n], lg4[0] * sm.aux[4][16 * G + n]));
                lg4[0] *= sm.aux[3][16 * G + n];
                lg4[1] *= sm.aux[3][64 + 16 * G + n];
                const float pmx = wave_max_nonneg(fmaxf(lg4[0], lg4[1]));
                const float psc = pmx > kTinyMax ? (float)QMAX * __builtin_amdgcn_rcpf(pmx) : 0.f;
                const float ps = (G & 1) ? psc : psc * MUL;
#pragma unroll
                for (int sg = 0; sg < 2; ++sg) {
                    const float yf = fmaf(lg4[sg], ps, MAGIC);
                    t4[sg] = quad_transpose_bytes(__float_as_uint(yf) + (0x80808080u - MAGIC_BITS), j);
                }
                fp4 = pmx * (1.0f / (MUL * (float)QMAX));
            }
            v4i ap[NH][2];
            float alpha[NH], gam[NH], fp[NH];  // gam: the offset term in output units
#pragma unroll
            for (int hg = 0; hg < NH; ++hg) {
                alpha[hg] = softmax_update(lg[hg], false, m_run[hg], l_run[hg]);
                // the offsets' part of the output, sum over tokens of p * b_V; then p * a_V, the
                // real-valued side of the code products
                float pmx = 0.f, gsum = 0.f;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int tok = 64 * (k >> 2) + 16 * (k & 3) + n;
                    gsum = fmaf(lg[hg][k], sm.aux[4][tok], gsum);
                    lg[hg][k] *= sm.aux[3][tok];
                    pmx = fmaxf(pmx, lg[hg][k]);
                }
                pmx = row_max_nonneg(pmx);
                const float psc = pmx > kTinyMax ? (float)QMAX * __builtin_amdgcn_rcpf(pmx) : 0.f;
#pragma unroll
                for (int sg = 0; sg < 2; ++sg) {
                    uint32_t D[4];
#pragma unroll
                    for (int tau = 0; tau < 4; ++tau) {
                        const float yf = fmaf(lg[hg][4 * sg + tau], (tau & 1) ? psc : psc * MUL, MAGIC);
                        const uint32_t y = __float_as_uint(yf) + (0x80808080u - MAGIC_BITS);
                        const uint32_t t = quad_transpose_bytes(y, j);
                        uint32_t d = (uint32_t)__builtin_amdgcn_ds_bpermute(perm_addr, (int)t);
                        if (X1 && hg == 0) {
                            const uint32_t d4 = (uint32_t)__builtin_amdgcn_ds_bpermute(perm4 + 64 * tau, (int)t4[sg]);
                            d = x1_row ? d4 : d;
                        }
                        D[tau] = d ^ 0x80808080u;
                    }
                    ap[hg][sg] = v4i{(int)D[0], (int)D[1], (int)D[2], (int)D[3]};
                }
                fp[hg] = pmx * (1.0f / (MUL * (float)QMAX));
                gam[hg] = row_sum(gsum);
            }
            uint32_t x5[8];  // X1: accumulator 3, the extra head's digit-G partial of channel block mt
#pragma unroll
            for (int mt = 0; mt < 8; ++mt) {
                const v4i v0 = unit_planes<BITS>(&vw[0][mt * WPU]);
                const v4i v1 = unit_planes<BITS>(&vw[1][mt * WPU]);
                const float s2v = sm.aux[5][16 * mt + n];
#pragma unroll
                for (int hg = 0; hg < NH; ++hg) {
                    v4i acc = mfma_i8(ap[hg][0], v0, v4i{0, 0, 0, 0});
                    acc = mfma_i8(ap[hg][1], v1, acc);
                    orot[hg][mt] = fmaf(fmaf((float)digit_sum(acc), fp[hg], gam[hg]), s2v, orot[hg][mt] * alpha[hg]);
                    if (X1 && hg == 0) x5[mt] = (uint32_t)acc[3];
                }
            }
            if constexpr (X1) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const uint32_t raw = rows_digit_reduce_scatter4(x5[4 * q], x5[4 * q + 1], x5[4 * q + 2], x5[4 * q + 3]);
                    orot4[q] = fmaf(fmaf((float)(int)raw, fp4, gam4), sm.aux[5][16 * (4 * q + G) + n], orot4[q] * alpha4);
                }
            }
            load_codes(tile_v(id_next), nxt.v);
        };
        // Tiles in pairs, alternating the buffers, so that no register copy (and no wait for a
        // prefetch) is needed between iterations.
        int blk = blk0;
        int id_n = block_id_t<PG>(a, b, min(blk0 + 1, blk1 - 1));
        for (; blk + 1 < blk1; blk += 2) {
            const int id_nn = block_id_t<PG>(a, b, min(blk + 2, blk1 - 1));
            step(ra, rb, id_n, 0);
            id_n = block_id_t<PG>(a, b, min(blk + 3, blk1 - 1));
            step(rb, ra, id_nn, 0);
        }
        if (blk < blk1) {
            int z = 0;
            asm volatile("" : "+v"(z));
            step(ra, rb, id_n, z);
        }
    }

    // ---- sink and residual (bf16, unrotated) -------------------------------------------------
    // In chunks of kRC tokens: the sink's, then the residual's (no chunk spans both).  A chunk's key
    // rows (bf16 MFMA operands) and value rows (one dword per lane and row) are loaded together,
    // one memory round trip per chunk.
    float oplain[NHX][2];  // head hh, channel 2*l + jj (unrotated)
#pragma unroll
    for (int hh = 0; hh < NHX; ++hh) oplain[hh][0] = oplain[hh][1] = 0.f;
    if (c0 < c1) {
        // A operand of group hg: row 4h holds q of head 4*hg + h rounded to bf16, row 4h + 1 the
        // remainder (zero for bf16 q), rows 4h + 2, 4h + 3 zero; lane (G, 4h + j) holds
        // q[.][32k + 8G ..].  Loads are clamped to a valid head, then masked.
        v8bf aqs[NH][4];
        {
            size_t qi[4 * NH];
            float qv[4 * NH][8];
#pragma unroll
            for (int hg = 0; hg < NH; ++hg)
#pragma unroll
                for (int k = 0; k < 4; ++k) qi[4 * hg + k] = (qrow + min(4 * hg + h, g - 1)) * kD + 32 * k + 8 * G;
            load_q_runs<4 * NH>(a, qi, qv);
#pragma unroll
            for (int hg = 0; hg < NH; ++hg) {
                const bool use = 4 * hg + h < g && j < 2;
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float v = use ? qv[4 * hg + k][e] : 0.f;
                        const __bf16 hi = (__bf16)v;
                        aqs[hg][k][e] = j == 0 ? hi : (__bf16)(v - (float)hi);
                    }
            }
        }
        // extra head: the same rows (hi, lo) of its q, placed in row group tau at use
        v8bf aqs4[4];
        if constexpr (X1) {
            size_t qi[4];
            float qv[4][8];
#pragma unroll
            // (clamped to a head of the chunk: the extra slot may be empty in a chunk of a larger
            // group, and its results are then not written)
            for (int k = 0; k < 4; ++k) qi[k] = (qrow + min(NHX - 1, g - 1)) * kD + 32 * k + 8 * G;
            load_q_runs<4>(a, qi, qv);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float v = j < 2 ? qv[k][e] : 0.f;
                    const __bf16 hi = (__bf16)v;
                    aqs4[k][e] = j == 0 ? hi : (__bf16)(v - (float)hi);
                }
        }
        for (int c = c0; c < c1; ++c) {
            const bool in_sink = c < nsc;
            const int t0 = kRC * (in_sink ? c : c - nsc);
            const int cn = min(kRC, (in_sink ? ns : nr) - t0);
            const size_t row0 = in_sink ? (size_t)stream * a.n_sink + t0 : (size_t)stream * kG + t0;
            const uint16_t* Kp = (in_sink ? a.k_sink : a.k_resid) + row0 * kD;
            const uint16_t* Vp = (in_sink ? a.v_sink : a.v_resid) + row0 * kD;
            // A fused append's token is the residual's last row (of the last chunk): read from
            // the input (an fp32 one is rounded and put in the row's place below), and stored into the
            // residual below.
            const bool new_row = a.step_len > 0 && c == nch - 1, new_bf16 = new_row && !NEW32;
            const uint16_t* Klast = new_bf16 ? static_cast<const uint16_t*>(a.k_new) + (size_t)stream * kD : Kp + (size_t)(cn - 1) * kD;
            const uint16_t* Vlast = new_bf16 ? static_cast<const uint16_t*>(a.v_new) + (size_t)stream * kD : Vp + (size_t)(cn - 1) * kD;
            // (with the chunk's rows: the check below then waits for no memory round trip of its own)
            int stored = 0;
            if (!NEW32 && new_row && chunk == 0) stored = __hip_atomic_load(a.seq_len + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // Rows past the chunk read its last row (in bounds) and are masked (p = 0).
            v8bf B[2][4];  // key rows 16 tau + n, channels 32 k + 8 G ..
#pragma unroll
            for (int tau = 0; tau < 2; ++tau) {
                const int i = 16 * tau + n;
                const uint16_t* kr = (i < cn - 1 ? Kp + (size_t)i * kD : Klast) + 8 * G;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint4 u = *reinterpret_cast<const uint4*>(kr + 32 * k);
                    __builtin_memcpy(&B[tau][k], &u, 16);
                }
            }
            uint32_t v2[kRC];  // value row t, channels 2 l, 2 l + 1
#pragma unroll
            for (int t = 0; t < kRC; ++t) v2[t] = reinterpret_cast<const uint32_t*>(t < cn - 1 ? Vp + (size_t)t * kD : Vlast)[l];
            uint32_t new_k = 0, new_v = 0;  // NEW32: the new row's channels 2 l, 2 l + 1
            if (NEW32 && new_row) {
                auto pair = [](float2 x) { return (uint32_t)f32_to_bf16(x.x) | (uint32_t)f32_to_bf16(x.y) << 16; };
                new_k = pair(reinterpret_cast<const float2*>(static_cast<const float*>(a.k_new) + (size_t)stream * kD)[l]);
                new_v = pair(reinterpret_cast<const float2*>(static_cast<const float*>(a.v_new) + (size_t)stream * kD)[l]);
                wave_sync();  // the previous chunk is done with sm.p
                uint32_t* row = reinterpret_cast<uint32_t*>(&sm.p[0][0]);
                row[l] = new_k;
                wave_sync();
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    v8bf x;
                    __builtin_memcpy(&x, row + 16 * k + 4 * G, 16);
#pragma unroll
                    for (int tau = 0; tau < 2; ++tau) B[tau][k] = 16 * tau + n < cn - 1 ? B[tau][k] : x;
                }
#pragma unroll
                for (int t = 0; t < kRC; ++t) v2[t] = t < cn - 1 ? v2[t] : new_v;
            }
            if (new_row && chunk == 0) {
                // The token into the residual (one head chunk writes it), and the step's length (kv
                // head 0 of the sequence writes it).  The stored length must be the one before the
                // append, or the one after it (kv head 0 may have stored it already); else the
                // sequence is left as it is and bit 2 of err_word is set.
                if (NEW32) stored = __hip_atomic_load(a.seq_len + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (stored == a.step_len - 1 || stored == a.step_len) {
                    reinterpret_cast<uint32_t*>(a.k_resid + (row0 + cn - 1) * kD)[l] = NEW32 ? new_k : reinterpret_cast<const uint32_t*>(Klast)[l];
                    reinterpret_cast<uint32_t*>(a.v_resid + (row0 + cn - 1) * kD)[l] = NEW32 ? new_v : reinterpret_cast<const uint32_t*>(Vlast)[l];
                    if (kvh == 0 && l == 0) __hip_atomic_store(a.seq_len + b, a.step_len, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else if (l == 0 && a.err_word) {
                    __hip_atomic_fetch_or(a.err_word, 4u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            wave_sync();  // the previous chunk is done with sm.p / sm.hv
            // logits of head 4*hg + G, token 16*tau + n
            float lg[NH][2];
            v4f r4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int tau = 0; tau < 2; ++tau) {
#pragma unroll
                for (int hg = 0; hg < NH; ++hg) {
                    v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int k = 0; k < 4; ++k) acc = mfma_bf16(aqs[hg][k], B[tau][k], acc);
                    lg[hg][tau] = 16 * tau + n < cn ? (acc[0] + acc[1]) * a.scale_log2 : -INFINITY;
                }
                if constexpr (X1) {
                    // token block tau lands in lanes G == tau of the accumulator
                    const bool mine = h == tau;
                    const v8bf zb = {};
#pragma unroll
                    for (int k = 0; k < 4; ++k) r4 = mfma_bf16(mine ? aqs4[k] : zb, B[tau][k], r4);
                }
            }
            if constexpr (X1) {
                // extra head, token 16 G + n (G < 2)
                float lgx[2] = {G < 2 && 16 * G + n < cn ? (r4[0] + r4[1]) * a.scale_log2 : -INFINITY, -INFINITY};
                const float alpha = softmax_wave(lgx, true, m4, l4);
                orot4[0] *= alpha;
                orot4[1] *= alpha;
                if (G < 2) sm.p[NHX - 1][16 * G + n] = lgx[0];
                if (l == 0) sm.hv[NHX - 1][2] = alpha;
            }
#pragma unroll
            for (int hg = 0; hg < NH; ++hg) {
                const float alpha = softmax_update(lg[hg], true, m_run[hg], l_run[hg]);
#pragma unroll
                for (int mt = 0; mt < 8; ++mt) orot[hg][mt] *= alpha;
                // every head slot writes its row (slots past g: p = 0, alpha = 1), so that the
                // PV loop below runs over all slots without a branch per head and token
                const bool real = 4 * hg + G < g;
#pragma unroll
                for (int tau = 0; tau < 2; ++tau) sm.p[4 * hg + G][16 * tau + n] = real ? lg[hg][tau] : 0.f;
                if (n == 0) sm.hv[4 * hg + G][2] = real ? alpha : 1.f;
            }
            wave_sync();
            // o_plain[h] = alpha o_plain[h] + sum over the chunk's rows of p[h][t] V[t]
#pragma unroll
            for (int hh = 0; hh < NHX; ++hh) {
                const float al = sm.hv[hh][2];
                oplain[hh][0] *= al;
                oplain[hh][1] *= al;
#pragma unroll
                for (int t = 0; t < kRC; t += 4) {
                    const float4 ph = *reinterpret_cast<const float4*>(&sm.p[hh][t]);
                    const float pv[4] = {ph.x, ph.y, ph.z, ph.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        oplain[hh][0] = fmaf(pv[i], __uint_as_float(v2[t + i] << 16), oplain[hh][0]);
                        oplain[hh][1] = fmaf(pv[i], __uint_as_float(v2[t + i] & 0xFFFF0000u), oplain[hh][1]);
                    }
                }
            }
        }
    }

    // ---- finish ------------------------------------------------------------------------------
    // Every wave leaves its part in its own LDS block: [NHX][kD] rotated output, [NHX][kD] plain
    // output, [NHX] m, [NHX] l.  Then the workgroup's waves take the heads in turn: log-sum-exp of the
    // waves' parts in wave order (lane l holds channels 2l, 2l + 1), and either the output (inverse
    // rotation in registers, normalisation) or, where the stream has several workgroups, the
    // workgroup's partial.
    auto part = [&](int w) { return reinterpret_cast<float*>(reinterpret_cast<Smem4<NH, X1>*>(dyn_lds) + w); };
    constexpr int XP = NHX * kD, XM = 2 * NHX * kD, XL = XM + NHX;
    static_assert(sizeof(Smem4<NH, X1>) >= sizeof(float) * (2 * NHX * kD + 2 * NHX), "exchange area");
    wave_sync();  // this wave is done with sm
    {
        float* xb = part(wave);
#pragma unroll
        for (int hg = 0; hg < NH; ++hg) {
            const float lt = row_sum(l_run[hg]);
#pragma unroll
            for (int mt = 0; mt < 8; ++mt) xb[(4 * hg + G) * kD + 16 * mt + n] = orot[hg][mt];
            if (n == 0) {
                xb[XM + 4 * hg + G] = m_run[hg];
                xb[XL + 4 * hg + G] = lt;
            }
        }
        if constexpr (X1) {
            const float lt4 = wave_sum(l4);
#pragma unroll
            for (int q = 0; q < 2; ++q) xb[(NHX - 1) * kD + 16 * (4 * q + G) + n] = orot4[q];
            if (l == 0) {
                xb[XM + NHX - 1] = m4;
                xb[XL + NHX - 1] = lt4;
            }
        }
#pragma unroll
        for (int hh = 0; hh < NHX; ++hh)
            *reinterpret_cast<float2*>(xb + XP + hh * kD + 2 * l) = make_float2(oplain[hh][0], oplain[hh][1]);
    }
    __syncthreads();
    const float rs = a.rotate ? kInvSqrt128 : 1.f;
    for (int hh = wave; hh < g; hh += a.group) {
        // lane w: the weight of wave w's part (waves past the last repeat it and count for nothing)
        const float m = part(min(l, a.group - 1))[XM + hh];
        const float lw = l < a.group ? part(min(l, a.group - 1))[XL + hh] : 0.f;
        const float M = wave_max(m);
        const float ww = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
        const float L = wave_sum(ww * lw);
        float acc[2] = {0.f, 0.f}, pl[2] = {0.f, 0.f};
        for (int w = 0; w < a.group; ++w) {
            const float* xb = part(w);
            const float wt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ww), w));
            const float2 x = *reinterpret_cast<const float2*>(xb + hh * kD + 2 * l);
            const float2 y = *reinterpret_cast<const float2*>(xb + XP + hh * kD + 2 * l);
            acc[0] = fmaf(wt, x.x, acc[0]);
            acc[1] = fmaf(wt, x.y, acc[1]);
            pl[0] = fmaf(wt, y.x, pl[0]);
            pl[1] = fmaf(wt, y.y, pl[1]);
        }
        if (a.n_wg > 1) {
            float* P = a.ws + ((qrow + hh) * a.n_wg + wgi) * kPart;
            if (l == 0) *reinterpret_cast<float2*>(P) = make_float2(M, L);
            *reinterpret_cast<float2*>(P + 4 + 2 * l) = make_float2(acc[0], acc[1]);
            *reinterpret_cast<float2*>(P + 132 + 2 * l) = make_float2(pl[0], pl[1]);
            continue;
        }
        if (a.rotate) fwht128(acc, l);
        float o0 = acc[0] * rs + pl[0], o1 = acc[1] * rs + pl[1];
        o0 = L > 0.f ? o0 / L : 0.f;
        o1 = L > 0.f ? o1 / L : 0.f;
        const size_t idx = (qrow + hh) * kD + 2 * l;
        if (a.out_bf16)
            reinterpret_cast<uint32_t*>(a.out)[idx >> 1] = (uint32_t)f32_to_bf16(o0) | ((uint32_t)f32_to_bf16(o1) << 16);
        else
            *reinterpret_cast<float2*>(static_cast<float*>(a.out) + idx) = make_float2(o0, o1);
    }
}

// Merge of the workgroups' partials of a (sequence, query head): log-sum-exp weights, the inverse
// rotation of the body part in registers (lane l holds channels 2l, 2l + 1), normalisation.
// W waves per (sequence, query head), 256 threads per workgroup: W = 1 (four heads per
// workgroup) for few partials; W = 4 for many (a plan makes at most 32), wave w summing partials w,
// w + 4, ... and wave 0 adding the four sums in a fixed order.
constexpr int kMergeWide = 9;  // from this many partials on, four waves per head

template <int W>
__global__ __launch_bounds__(256) void k_decode_merge(DecodeArgs a) {
    static_assert(W == 1 || W == 4, "one or four waves per head");
    constexpr int HPB = 4 / W;          // heads per workgroup
    constexpr int U = W == 1 ? 8 : 16;  // partials with loads in flight per wave
    __shared__ float red[W > 1 ? W - 1 : 1][2 * kD + 2];
    const int l = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = wv % W;
    asm volatile("" ::"s"(a.ws), "s"(a.out), "s"(a.n_wg), "s"(a.n_rows), "s"(a.out_bf16), "s"(a.rotate));  // (one round of scalar loads)
    const size_t bh = (size_t)blockIdx.x * HPB + wv / W;
    // W > 1: one head per workgroup, so every wave leaves here or none does.
    if (bh >= (size_t)a.n_rows) return;
    const float* P = a.ws + bh * a.n_wg * kPart;
    const int S = a.n_wg;
    // Log-sum-exp over this wave's partials, U of them with every load in flight (indices past the
    // last one are clamped, their values unused), the sums kept relative to the running
    // maximum M of the partials that hold a probability mass.
    float M = -INFINITY, L = 0.f, acc[2] = {0.f, 0.f}, pl[2] = {0.f, 0.f};
    for (int s0 = part; s0 < S; s0 += U * W) {
        float mm[U], ll[U];
        float2 ov[U], pv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float* Ps = P + (size_t)min(s0 + u * W, S - 1) * kPart;
            mm[u] = Ps[0];
            ll[u] = Ps[1];
            ov[u] = *reinterpret_cast<const float2*>(Ps + 4 + 2 * l);
            pv[u] = *reinterpret_cast<const float2*>(Ps + 132 + 2 * l);
        }
        float mb = M;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (s0 + u * W < S && ll[u] > 0.f) mb = fmaxf(mb, mm[u]);
        if (mb == -INFINITY) continue;  // no mass so far
        const float r = exp2f(M - mb);  // 0 while M is still -inf
        L *= r;
        acc[0] *= r;
        acc[1] *= r;
        pl[0] *= r;
        pl[1] *= r;
        M = mb;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + u * W < S && ll[u] > 0.f) {
                const float w = exp2f(mm[u] - M);
                L += w * ll[u];
                acc[0] += w * ov[u].x;
                acc[1] += w * ov[u].y;
                pl[0] += w * pv[u].x;
                pl[1] += w * pv[u].y;
            }
        }
    }
    if constexpr (W > 1) {
        // waves 1..W-1 hand (M, L, sums) to wave 0, which rescales them to the common maximum
        // and adds them in wave order
        if (part > 0) {
            float* rw = red[part - 1];
            *reinterpret_cast<float2*>(rw + 2 * l) = make_float2(acc[0], acc[1]);
            *reinterpret_cast<float2*>(rw + kD + 2 * l) = make_float2(pl[0], pl[1]);
            if (l == 0) {
                rw[2 * kD] = M;
                rw[2 * kD + 1] = L;
            }
        }
        __syncthreads();
        if (part > 0) return;
        float Mw[W - 1];
        float Mt = M;
#pragma unroll
        for (int w = 0; w < W - 1; ++w) {
            Mw[w] = red[w][2 * kD];
            Mt = fmaxf(Mt, Mw[w]);
        }
        if (Mt != -INFINITY) {
            const float r = exp2f(M - Mt);
            L *= r;
            acc[0] *= r;
            acc[1] *= r;
            pl[0] *= r;
            pl[1] *= r;
#pragma unroll
            for (int w = 0; w < W - 1; ++w) {
                const float rw = exp2f(Mw[w] - Mt);  // 0 for a wave without mass
                const float2 x = *reinterpret_cast<const float2*>(red[w] + 2 * l);
                const float2 y = *reinterpret_cast<const float2*>(red[w] + kD + 2 * l);
                acc[0] += rw * x.x;
                acc[1] += rw * x.y;
                pl[0] += rw * y.x;
                pl[1] += rw * y.y;
                L += rw * red[w][2 * kD + 1];
            }
        }
    }
    if (a.rotate) fwht128(acc, l);
    const float rs = a.rotate ? kInvSqrt128 : 1.f;
    float o[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        o[e] = acc[e] * rs + pl[e];
        o[e] = L > 0.f ? o[e] / L : 0.f;
    }
    const size_t idx = bh * kD + 2 * l;
    if (a.out_bf16)
        reinterpret_cast<uint32_t*>(a.out)[idx >> 1] = (uint32_t)f32_to_bf16(o[0]) | ((uint32_t)f32_to_bf16(o[1]) << 16);
    else
        *reinterpret_cast<float2*>(static_cast<float*>(a.out) + idx) = make_float2(o[0], o[1]);
}

template <int BITS, int GQ, int CMP>
hipError_t launch_cfg(const DecodeArgs& a, int batch, hipStream_t stream) {
    const int streams = batch * a.n_kv;
    const int wpg = a.group;
    const dim3 grid((unsigned)(streams * a.n_chunk * a.n_wg)), block(64 * wpg);
    const bool pg = a.block_table != nullptr;
    if (pg && a.new_f32) return hipErrorInvalidValue;  // (no such kernel: the paged ones read the token as bf16)
    constexpr int NH = GQ == 8 ? 2 : 1, X1 = GQ == 5 ? 1 : 0;
    const size_t lds = wpg * sizeof(Smem4<NH, X1>);
    if (pg) hipLaunchKernelGGL((k_decode4<BITS, NH, CMP, 1, X1, 0>), grid, block, lds, stream, a);
    else if (a.new_f32) hipLaunchKernelGGL((k_decode4<BITS, NH, CMP, 0, X1, 1>), grid, block, lds, stream, a);
    else hipLaunchKernelGGL((k_decode4<BITS, NH, CMP, 0, X1, 0>), grid, block, lds, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.n_wg == 1) return e;
    const size_t heads = (size_t)batch * a.n_q;
    if (a.n_wg >= kMergeWide)
        hipLaunchKernelGGL(k_decode_merge<4>, dim3((unsigned)heads), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL(k_decode_merge<1>, dim3((unsigned)((heads + 3) / 4)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

template <int BITS, int CMP>
hipError_t launch_bits(const DecodeArgs& a, int batch, hipStream_t stream) {
    if (a.g_chunk <= 4) return launch_cfg<BITS, 4, CMP>(a, batch, stream);
    if (a.g_chunk == 5) return launch_cfg<BITS, 5, CMP>(a, batch, stream);
    return launch_cfg<BITS, 8, CMP>(a, batch, stream);
}

}  // namespace

size_t decode_workspace_bytes(int batch, int n_q, const DecodePlan& plan) {
    return (size_t)batch * n_q * plan.ws_parts * kPart * sizeof(float);
}

hipError_t launch_decode(const kvarn_cache& c, int bits, int compact, int rotate, int n_sink, int n_q, const void* q,
                         bool q_bf16, void* out, bool out_bf16, float sm_scale, const DecodePlan& plan, float* ws,
                         hipStream_t stream, const StepAppend* step) {
    DecodeArgs a;
    a.rotate = rotate;
    a.block_table = c.block_table;
    a.n_phys = c.n_phys;
    a.err_word = c.err_word;
    a.k_body = static_cast<const uint8_t*>(c.k_body);
    a.v_body = static_cast<const uint8_t*>(c.v_body);
    a.k_resid = static_cast<uint16_t*>(c.k_resid);
    a.v_resid = static_cast<uint16_t*>(c.v_resid);
    a.k_sink = static_cast<const uint16_t*>(c.k_sink);
    a.v_sink = static_cast<const uint16_t*>(c.v_sink);
    a.seq_len = c.seq_len;
    a.q = q;
    a.q_bf16 = q_bf16 ? 1 : 0;
    a.out = out;
    a.out_bf16 = out_bf16 ? 1 : 0;
    a.n_kv = c.n_kv;
    a.n_q = n_q;
    a.g = n_q / c.n_kv;
    a.max_blocks = c.max_blocks;
    a.n_sink = n_sink;
    a.scale_log2 = sm_scale * kLog2e;
    a.n_wg = plan.n_wg;
    a.group = plan.group;
    a.order = plan.order;
    a.inv_waves = 1.f / (float)(plan.n_wg * plan.group);
    a.n_streams = c.batch * c.n_kv;
    a.n_rows = c.batch * n_q;
    a.n_chunk = plan.n_chunk;
    a.g_chunk = plan.g_chunk;
    a.ws = ws;
    a.step_len = step ? step->len_before + 1 : 0;
    a.new_f32 = step && step->f32;
    a.k_new = step ? step->k_new : nullptr;
    a.v_new = step ? step->v_new : nullptr;
    if (compact) return bits == 2 ? launch_bits<2, 1>(a, c.batch, stream) : launch_bits<4, 1>(a, c.batch, stream);
    return bits == 2 ? launch_bits<2, 0>(a, c.batch, stream) : launch_bits<4, 0>(a, c.batch, stream);
}

}  // namespace kvarn
