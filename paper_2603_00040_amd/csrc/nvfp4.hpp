// phi of the NVFP4 format (Eq. 1 / Eq. 2, blocks of 16 along d), shared by the preparing kernels and the decode path.
#pragma once
#include "common.hpp"

namespace aq {

// phi of one block of 16 values that are bf16 numbers (Eq. 1): the E4M3 scale s and the 16 E2M1 codes, element 2k in the low
// nibble of byte k of {clo, chi}.
// RNE of the real quotient x / s without a division per element (ten vector instructions each, which bound the streaming
// kernels).  |x| has 8 significant bits and s has 4, so a quotient that is not on a rounding boundary of the E2M1 grid is at
// least 2^-9 (relative) away from it, and one that is on a boundary (a tie) has at most 3 significant bits.  x * (1/s) with the
// approximate reciprocal is within 2^-21 of the quotient; rounding that product to 12 significant bits puts a tie back on its
// boundary exactly and moves nothing else across one (it moves a value by at most 2^-12).  The rounding to E2M1 itself
// (nearest, ties to even, saturating at 6, sign kept) then is the hardware conversion, two elements per instruction, which
// leaves the codes packed as the public layout wants them.
__device__ inline void phi_block16_bf16(const float (&v)[16], float& s, uint32_t& clo, uint32_t& chi)
{
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) amax = fmaxf(amax, fabsf(v[i]));
    s = block_scale_exact(amax);
    const float inv_s = s > 0.0f ? __builtin_amdgcn_rcpf(s) : 0.0f;      // s = 0: every quotient 0, every code 0
    auto snap = [](float r) __attribute__((always_inline)) {
        return __uint_as_float((__float_as_uint(r) + 0x800u) & 0xFFFFF000u);
    };
    clo = 0; chi = 0;
#define AQ_PAIR(W, PR, SEL) W = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(W, snap(v[2 * (PR)] * inv_s), snap(v[2 * (PR) + 1] * inv_s), 1.0f, SEL)
    AQ_PAIR(clo, 0, 0); AQ_PAIR(clo, 1, 1); AQ_PAIR(clo, 2, 2); AQ_PAIR(clo, 3, 3);
    AQ_PAIR(chi, 4, 0); AQ_PAIR(chi, 5, 1); AQ_PAIR(chi, 6, 2); AQ_PAIR(chi, 7, 3);
#undef AQ_PAIR
}

// The 16 values of a block from its codes and its scale (exact: <= 6 significant bits).
__device__ inline void dequant_block16(uint32_t clo, uint32_t chi, float s, float (&xf)[16])
{
    typedef float float2v __attribute__((ext_vector_type(2)));
#define AQ_BACK(W, PR, SEL) { const float2v cv = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(W, 1.0f, SEL); xf[2 * (PR)] = cv[0] * s; xf[2 * (PR) + 1] = cv[1] * s; }
    AQ_BACK(clo, 0, 0) AQ_BACK(clo, 1, 1) AQ_BACK(clo, 2, 2) AQ_BACK(clo, 3, 3)
    AQ_BACK(chi, 4, 0) AQ_BACK(chi, 5, 1) AQ_BACK(chi, 6, 2) AQ_BACK(chi, 7, 3)
#undef AQ_BACK
}

}  // namespace aq
