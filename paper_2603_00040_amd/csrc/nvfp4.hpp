// phi of the NVFP4 format (Eq. 1 / Eq. 2, blocks of 16 along d), shared by the preparing kernels and the decode path.
#pragma once
#include "common.hpp"

namespace aq {

// A quantized block of 16: the E2M1 codes, element 2k in the low nibble of byte k of {clo, chi}, and the E4M3 scale as a value, with its byte in
// the two low bytes of sc (of which one conversion makes an fp16 pair).
struct Nv16 { uint32_t clo, chi, sc; float s; };

// phi of one block of 16 values that are bf16 numbers (Eq. 1).
// Scale: RNE_E4M3(amax / 6).  amax has 8 significant bits, so amax / 6 is on a rounding boundary of the E4M3 grid (at most 5 significant bits) or at least
// 2^-13 (relative) away from every one; amax * (1/6) is within 2^-23 of the quotient, and rounding it to 16 significant bits (by at most 2^-16) puts
// a tie back on its boundary exactly and moves nothing else across one.  The rounding to E4M3 (nearest, ties to even, subnormals kept) then is the
// hardware conversion.
// Codes: RNE of the real quotient x / s without a division per element.  |x| has 8 significant bits and s has 4, so a quotient that is not on a rounding
// boundary of the E2M1 grid is at least 2^-9 (relative) away from it, and one that is on a boundary (a tie) has at most 3 significant bits.  x * (1/s) with
// the approximate reciprocal is within 2^-21 of the quotient; rounding that product to fp16 (11 significant bits, by at most 2^-11; quotients below
// 2^-14, where it is more, are far below the least boundary, 0.25) does the same for it, two elements per instruction.  The rounding to E2M1 (nearest,
// ties to even, saturating at 6, sign kept) is the hardware conversion of the pair, which leaves the codes packed as the public layout wants them.
// (About 70 vector instructions a block.  With an IEEE division and the grid rounding of common.hpp for the scale and two integer instructions per element to
// round the quotient it was 130; these bound the preparing launches of small problems and the cache writes: training step of 2 heads,
// L = 256, d = 64 24.95 -> 24.55 us, 12 heads, L = 1560 131.0 -> 129.9 us, inference 32 heads, L = 777 24.9 -> 24.7 us.)
__device__ __forceinline__ void nv16_scale(float amax, uint32_t& sc, float& s, float& inv)
{
    typedef short short2v __attribute__((ext_vector_type(2)));
    const float q = __uint_as_float((__float_as_uint(amax * (1.0f / 6.0f)) + 0x80u) & 0xFFFFFF00u), qs = fminf(q, 448.0f);
    sc = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(short2v{0, 0}, qs, qs, 1.0f, false));
    s = __builtin_amdgcn_cvt_scalef32_f32_fp8(sc, 1.0f, 0);
    inv = s > 0.0f ? __builtin_amdgcn_rcpf(s) : 0.0f;      // s = 0: every quotient 0, every code 0
}
__device__ inline Nv16 phi_block16_bf16(const float (&v)[16])
{
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) amax = fmaxf(amax, fabsf(v[i]));
    Nv16 b;
    float inv;
    nv16_scale(amax, b.sc, b.s, inv);
    // (where the scale is saturated a quotient may be beyond fp16: infinity, which becomes 6)
    auto pair = [&](int i) __attribute__((always_inline)) { return half2v{(half_t)(v[2 * i] * inv), (half_t)(v[2 * i + 1] * inv)}; };
    b.clo = any_register(); b.chi = any_register();
#define AQ_PAIR(W, PR, SEL) W = __builtin_amdgcn_cvt_scalef32_pk_fp4_f16(W, pair(PR), 1.0f, SEL)
    AQ_PAIR(b.clo, 0, 0); AQ_PAIR(b.clo, 1, 1); AQ_PAIR(b.clo, 2, 2); AQ_PAIR(b.clo, 3, 3);
    AQ_PAIR(b.chi, 4, 0); AQ_PAIR(b.chi, 5, 1); AQ_PAIR(b.chi, 6, 2); AQ_PAIR(b.chi, 7, 3);
#undef AQ_PAIR
    return b;
}
// A block whose codes and scale byte come from memory.
__device__ inline Nv16 nv16_of(uint32_t clo, uint32_t chi, uint32_t scale_byte) {
    Nv16 b;
    b.clo = clo; b.chi = chi; b.sc = scale_byte * 0x0101u;
    b.s = __builtin_amdgcn_cvt_scalef32_f32_fp8(b.sc, 1.0f, 0);
    return b;
}

// The 16 values of a block (exact: <= 6 significant bits), as floats or as eight fp16 pairs.
__device__ inline void dequant_block16(const Nv16& b, float (&xf)[16])
{
    typedef float float2v __attribute__((ext_vector_type(2)));
#define AQ_BACK(W, PR, SEL) { const float2v cv = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(W, 1.0f, SEL); xf[2 * (PR)] = cv[0] * b.s; xf[2 * (PR) + 1] = cv[1] * b.s; }
    AQ_BACK(b.clo, 0, 0) AQ_BACK(b.clo, 1, 1) AQ_BACK(b.clo, 2, 2) AQ_BACK(b.clo, 3, 3)
    AQ_BACK(b.chi, 4, 0) AQ_BACK(b.chi, 5, 1) AQ_BACK(b.chi, 6, 2) AQ_BACK(b.chi, 7, 3)
#undef AQ_BACK
}
__device__ inline void dequant_block16_f16(const Nv16& b, uint32_t (&w)[8])
{
    const half2v sc = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(b.sc, 1.0f, false);
#define AQ_BACK(W, PR, SEL) w[PR] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(W, 1.0f, SEL) * sc);
    AQ_BACK(b.clo, 0, 0) AQ_BACK(b.clo, 1, 1) AQ_BACK(b.clo, 2, 2) AQ_BACK(b.clo, 3, 3)
    AQ_BACK(b.chi, 4, 0) AQ_BACK(b.chi, 5, 1) AQ_BACK(b.chi, 6, 2) AQ_BACK(b.chi, 7, 3)
#undef AQ_BACK
}

// phi, and back to fp16, of two blocks of bf16 values shared by the lanes l and l + 32: a lane has 8 values of block a in a and 8 of block b in b.  The
// bits of phi_block16_bf16 and dequant_block16_f16.  One half forms the scale of a, the other that of b.
__device__ __forceinline__ void phi_half_blocks(uint4v& a, uint4v& b)
{
    float v[2][8], m[2] = {0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[0][2 * i] = __uint_as_float(a[i] << 16); v[0][2 * i + 1] = __uint_as_float(a[i] & 0xFFFF0000u);
        v[1][2 * i] = __uint_as_float(b[i] << 16); v[1][2 * i + 1] = __uint_as_float(b[i] & 0xFFFF0000u);
    }
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int i = 0; i < 8; ++i) m[g] = fmaxf(m[g], fabsf(v[g][i]));
    uint32_t sc;
    float s, inv;
    nv16_scale(xhalf_max_pair(m[0], m[1]), sc, s, inv);
    const auto sc2 = __builtin_amdgcn_permlane32_swap(sc, sc, false, false);
    const auto inv2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(inv), __float_as_uint(inv), false, false);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const float iv = __uint_as_float(inv2[g]);
        const half2v sh = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(sc2[g], 1.0f, false);
        uint32_t c = any_register();
        uint4v& w = g ? b : a;
#define AQ_PAIR(I) c = __builtin_amdgcn_cvt_scalef32_pk_fp4_f16(c, half2v{(half_t)(v[g][2 * I] * iv), (half_t)(v[g][2 * I + 1] * iv)}, 1.0f, I);
        AQ_PAIR(0) AQ_PAIR(1) AQ_PAIR(2) AQ_PAIR(3)
#undef AQ_PAIR
#define AQ_BACK(I) w[I] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, I) * sh);
        AQ_BACK(0) AQ_BACK(1) AQ_BACK(2) AQ_BACK(3)
#undef AQ_BACK
    }
}

}  // namespace aq
