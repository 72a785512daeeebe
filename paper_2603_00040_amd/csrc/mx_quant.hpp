// phi of the MX format (blocks of 32, one power-of-two E8M0 scale) and the layouts its codes take in memory: device code shared by
// the public quantizers, the preparing kernels and the attention kernels.
#pragma once
#include "common.hpp"

namespace aq {

// 32 values -> 4 registers of E2M1 codes (value i in nibble i), RNE on v / scale, saturating.
__device__ inline uint4v mx_codes32(const float (&v)[32], float scale) {
    uint4v c;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        uint32_t r = any_register();
        r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * w + 0], v[8 * w + 1], scale, 0);
        r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * w + 2], v[8 * w + 3], scale, 1);
        r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * w + 4], v[8 * w + 5], scale, 2);
        r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * w + 6], v[8 * w + 7], scale, 3);
        c[w] = r;
    }
    return c;
}

__device__ inline float e2m1_value_of(uint32_t code) {
    const uint32_t m = code & 7u;
    const float v = m < 2u ? 0.5f * (float)m : __uint_as_float(((m >> 1) + 126u) << 23 | (m & 1u) << 22);
    return (code & 8u) ? -v : v;
}

// Bytes of one 64-key record of a kv head: K operands, V^T operands, K scales, V scales.
__host__ __device__ constexpr int mx_rec_bytes(int D, bool fp8v = false) { return 2 * (D / 64) * 1024 + (D / 32) * (fp8v ? 2048 : 1024) + 512; }

// 32 values -> 8 registers of E4M3 bytes (value i in byte i), RNE on v / scale; |v| / scale <= 448 by the scale rule.
typedef short short2v __attribute__((ext_vector_type(2)));
__device__ inline void mx_codes32_fp8(const float (&v)[32], float scale, uint32_t (&c)[8]) {
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        short2v r = __builtin_bit_cast(short2v, any_register());
        r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, v[4 * w + 0], v[4 * w + 1], scale, false);
        r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, v[4 * w + 2], v[4 * w + 3], scale, true);
        c[w] = __builtin_bit_cast(uint32_t, r);
    }
}
__device__ inline float e4m3_value_of(uint32_t byte) {
    const uint32_t e = (byte >> 3) & 15u, m = byte & 7u;
    const float v = e == 0u ? (float)m * 0.001953125f : __uint_as_float((e + 120u) << 23 | m << 20);
    return (byte & 0x80u) ? -v : v;
}

// Where the 64-key record `tile` of kv head `head` lives.  Contiguous: records of a head one after another.  Paged (a
// KV cache): a page holds two records (128 keys) of every kv head, page_ids[tile / 2] names the page of this sequence.
// A page id outside [0, num_pages) gives null: the writer leaves that record out instead of touching memory outside the cache.
__device__ inline unsigned char* mx_record_of(unsigned char* base, const int* page_ids, int num_pages, int head, int nheads, int Lp, int tile, int rec_bytes) {
    if (page_ids) {
        const int page = page_ids[tile >> 1];
        if (page < 0 || page >= num_pages) return nullptr;
        return base + (((size_t)page * nheads + head) * 2 + (tile & 1)) * rec_bytes;
    }
    return base + ((size_t)head * (Lp / 64) + tile) * rec_bytes;
}

// Row of S^T product t (0/1) that holds key kk (0..63) of a tile, and the lane half that ends up owning it:
// the accumulator register r of a lane in half h is row 8 (r/4) + 4 h + r % 4; key 32 h + 16 t + r goes there.
__device__ inline int mx_srow_of_key(int kk) { const int w = kk & 15; return 8 * (w >> 2) + 4 * (kk >> 5) + (w & 3); }

// Codes and scale byte of 32 values.
template <bool FP8>
__device__ inline void mx_block_codes(const float (&v)[32], uint32_t& byte, uint32_t (&c)[8]) {
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 32; ++i) amax = fmaxf(amax, fabsf(v[i]));
    byte = FP8 ? e8m0_of_amax_fp8(amax) : e8m0_of_amax(amax);
    const float s = e8m0_as_f32(byte);
    if constexpr (FP8) {
        mx_codes32_fp8(v, s, c);
    } else {
        const uint4v c4 = mx_codes32(v, s);
#pragma unroll
        for (int i = 0; i < 4; ++i) { c[i] = c4[i]; c[4 + i] = 0u; }
    }
}

// Block blk of row `row` of x [BH, L, D] (zeros from row L on).
template <int D>
__device__ inline uint4v mx_block_of_row(const uint16_t* __restrict__ x, int bh, int row, int blk, int L, uint32_t& byte) {
    float v[32];
    if (row < L) {
        const uint4v* src = reinterpret_cast<const uint4v*>(x + ((size_t)bh * L + row) * D + blk * 32);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint4v a = src[j];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[8 * j + 2 * i]     = __uint_as_float(a[i] << 16);
                v[8 * j + 2 * i + 1] = __uint_as_float(a[i] & 0xFFFF0000u);
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = 0.0f;
    }
    uint32_t c[8];
    mx_block_codes<false>(v, byte, c);
    uint4v r; r[0] = c[0]; r[1] = c[1]; r[2] = c[2]; r[3] = c[3];
    return r;
}

// Q as the B operand of the scaled MFMA for 32 rows: lane (row, half) has the codes of d-slots 64 ks + 32 half .. + 31 of its row and a dword of
// scale bytes (byte ks; unused bytes are 1).  The attention kernels quantize Q themselves where they can (qsc null: src is Q [BH, L, D] bf16): it is
// read once and never written, and a decode step has a launch less.  Otherwise src and qsc are what mx_put_operand made, group grp of 32 rows.
// NT threads (a wave, or the waves that share the rows) read the rows in whole lines, eight values a thread; four neighbouring threads
// form the scale of a block and a register of codes each, which they hand out through LDS (a lane that read its own 64 bytes made every load touch 64
// lines: a decode step of 32 sequences 117 -> 122 us).  fetch() asks for the values, quantize() writes kMxQOps<D> bytes to LDS, scale bytes
// apart; a barrier of the NT threads; read() takes the operand.  Between fetch() and quantize() a kernel asks for its first keys.
// Operands from the preparing launch -> here: block-sparse 32/8 heads, L = 8192 136 -> 129 us; 2 x 12 heads, L = 32760 6.01 -> 5.92 ms (of it four
// moves per tile of mx_codes32); chunks of 512 of 8 sequences 319 -> 312 us; decode steps: one sequence of 3000 keys 16.7 -> 14.6 us, 4 sequences, d = 64
// 16.3 -> 13.2 us, 32 sequences of 4k - 16k keys, walked, d = 64 111.5 -> 99.4 us (of it 23 moves per page that the compiler no longer makes), d = 128 117.4 -> 118.0 us.
template <int D> constexpr int kMxQOps = (D / 64) * 1024;
template <int D, int NT>
struct MxQ {
    static constexpr int KS = D / 64, CH = D / 8 /* pieces of 8 values per row */, N = (32 * CH + NT - 1) / NT;
    uint4v op[KS];
    uint32_t sc;
    uint4v raw[N];
    // tid: of the NT threads; row0: the group's first row
    __device__ __forceinline__ void fetch(const void* __restrict__ src, const uint32_t* __restrict__ qsc, int bh, int row0, size_t grp, int tid, int L) {
#pragma unroll
        for (int i = 0; i < N; ++i) raw[i] = uint4v{0u, 0u, 0u, 0u};
        if (qsc) return;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int c = tid + i * NT, row = row0 + c / CH;
            if ((32 * CH % NT == 0 || c < 32 * CH) && row < L)
                raw[i] = *reinterpret_cast<const uint4v*>(static_cast<const uint16_t*>(src) + ((size_t)bh * L + row) * D + 8 * (c % CH));
        }
    }
    // What fetch() asked for has arrived.
    __device__ __forceinline__ void arrived() {
#pragma unroll
        for (int i = 0; i < N; ++i) asm volatile("" : "+v"(raw[i]));
    }
    // ops: LDS address of kMxQOps<D> bytes, scs: of 256 bytes
    __device__ __forceinline__ void quantize(const uint32_t* __restrict__ qsc, uint32_t ops, uint32_t scs, int tid) {
        if (qsc) return;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int c = tid + i * NT, row = c / CH, p = c % CH;
            float v[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[2 * e] = __uint_as_float(raw[i][e] << 16); v[2 * e + 1] = __uint_as_float(raw[i][e] & 0xFFFF0000u); }
            float amax = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(v[e]));
            // the four threads of a block (quad_perm 1,0,3,2 and 2,3,0,1)
            amax = fmaxf(amax, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(amax), 0xB1, 0xF, 0xF, true)));
            amax = fmaxf(amax, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(amax), 0x4E, 0xF, 0xF, true)));
            const uint32_t byte = e8m0_of_amax(amax);
            const float s = e8m0_as_f32(byte);
            uint32_t w = any_register();
            w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, v[0], v[1], s, 0);
            w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, v[2], v[3], s, 1);
            w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, v[4], v[5], s, 2);
            w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, v[6], v[7], s, 3);
            if (32 * CH % NT == 0 || c < 32 * CH) {
                const uint32_t slot = (uint32_t)(((p >> 2) & 1) * 32 + row);              // lane (row, half)
                *(__attribute__((address_space(3))) uint32_t*)(uintptr_t)(ops + ((uint32_t)(p >> 3) * 64 + slot) * 16 + 4 * (p & 3)) = w;
                if ((p & 3) == 0) *(__attribute__((address_space(3))) unsigned char*)(uintptr_t)(scs + slot * 4 + (p >> 3)) = (unsigned char)byte;
            }
        }
    }
    __device__ __forceinline__ void read(const void* __restrict__ src, const uint32_t* __restrict__ qsc, size_t grp, int lane, uint32_t ops, uint32_t scs) {
        if (qsc) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) op[ks] = *reinterpret_cast<const uint4v*>(static_cast<const unsigned char*>(src) + ((grp * KS + ks) * 64 + lane) * 16);
            sc = qsc[grp * 64 + lane];
        } else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) op[ks] = lds_read16_at(ops + (uint32_t)((ks * 64 + lane) * 16));
            const uint32_t x = *(const __attribute__((address_space(3))) uint32_t*)(uintptr_t)(scs + 4u * (uint32_t)lane);
            sc = KS == 1 ? (x & 0xFFu) | 0x01010100u : (x & 0xFFFFu) | 0x01010000u;
        }
        // (arrived: the LDS may be written again behind the next barrier)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(op[ks]));
        asm volatile("" : "+v"(sc));
    }
};
// Between quantize() and read() where the NT threads are a wave.
__device__ __forceinline__ void mx_q_wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// put(i, value 2 i, value 2 i + 1) for the 32 values of a block: code * 2^e, at most 2 significant bits, exact in bf16 wherever
// it is a normal number.
template <class F>
__device__ inline void mx_dequant32(const uint4v& c, float s, F&& put) {
    typedef float float2v __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float2v a = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c[w], 1.0f, 0), b = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c[w], 1.0f, 1);
        const float2v d = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c[w], 1.0f, 2), e = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(c[w], 1.0f, 3);
        put(4 * w, a[0] * s, a[1] * s); put(4 * w + 1, b[0] * s, b[1] * s); put(4 * w + 2, d[0] * s, d[1] * s); put(4 * w + 3, e[0] * s, e[1] * s);
    }
}

}  // namespace aq
