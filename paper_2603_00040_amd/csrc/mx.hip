// MX variant of the quantizer and of the inference forward (Alg. 1) on the scaled FP4 MFMA of gfx950.
// (The MX training forward and backward are variants of the 16-bit kernels in fwd.hip and bwd.hip.)
//
// Format (the OCP microscaling FP4 that Sec. 2.1 names beside NVFP4): E2M1 elements in blocks of 32
// with one power-of-two E8M0 scale, the smallest 2^e (e >= -126) with 6 * 2^e >= max|X|: the
// power-of-two counterpart of Eq. 1, no element saturates.  Q and K are blocked along d, P-tilde and
// V along the keys, so both products of Alg. 1 contract over the blocked axis and run on
// v_mfma_scale_f32_32x32x64_f8f6f4 with the FP4 codes and the scale bytes as they are: there is no
// dequantization anywhere, and phi(P-tilde) is one exponent extraction plus the hardware converts.
//
// Operand layout of that instruction with FP4 on both sides (checked on the device against a
// scalar evaluation): lane l holds row (A) or column (B) l % 32 and the 32 contraction indices
// 32 * (l / 32) .. + 31 as 32 nibbles in 4 registers, low nibble first, plus one scale byte for
// exactly those 32 indices: one MX block per lane.
//
//   S^T[key, query]  = K codes (A, from LDS) x Q codes (B, registers), contraction over d
//   O^T[d, query]   += V^T codes (A, from LDS) x P-tilde codes (B, registers), contraction over keys
//
// Mixed recipe (Sec. 2.5: FP4 for Q K^T, FP8 for P V): the FP8PV variants keep Q and K in MXFP4 and hold V and
// P-tilde in MXFP8 (E4M3 elements, the same blocks of 32 keys and E8M0 scales; scale = smallest 2^e with
// 448 * 2^e >= max|X|).  The P.V product then runs the same instruction with FP8 operands, whose layout differs
// (measured): the 32 bytes of lane l are contraction indices 16 (l/32) .. + 15 and 32 + 16 (l/32) .. + 15, and the
// scale of indices 32 b .. + 31 comes from lane l % 32 + 32 b.
//
// The rows of the two S^T products of a 64-key tile are assigned to keys so that the 32 accumulator
// registers of a lane are the 32 consecutive keys 32 * (lane / 32) .. + 31 of the tile: one P block,
// whose maximum, scale and codes never leave the lane, and whose 4 code registers already are the
// B operand of the P.V product.
#include "common.hpp"
#include "kernels.hpp"
#include "mx_quant.hpp"

namespace aq {

#ifndef AQ_DECODE_NP
#define AQ_DECODE_NP 1     // pages per iteration of the decode kernel (4 waves per page)
#endif

typedef int int8v __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------------------------------------
// The public quantizer along d (blocks of 32), one thread per block: codes [rows, D/2], scales [rows, D/32], optional bf16 xf.
template <int D>
__global__ __launch_bounds__(256) void mx_quant_d_kernel(
    const uint16_t* __restrict__ x, int L, unsigned char* __restrict__ codes, unsigned char* __restrict__ scales, uint16_t* __restrict__ xf)
{
    constexpr int NB = D / 32;
    const int bh = blockIdx.y;
    const int gid = blockIdx.x * 256 + threadIdx.x;
    const int row = gid / NB, blk = gid % NB;
    uint32_t byte;
    const uint4v c = mx_block_of_row<D>(x, bh, row, blk, L, byte);
    if (row < L) {
        if (codes) *reinterpret_cast<uint4v*>(codes + ((size_t)bh * L + row) * (D / 2) + blk * 16) = c;
        if (scales) scales[((size_t)bh * L + row) * NB + blk] = (unsigned char)byte;
    }
    if (xf) {
        uint32_t o[16];
        mx_dequant32(c, e8m0_as_f32(byte), [&](int i, float lo, float hi) { o[i] = pack_bf16x2_rne(lo, hi); });
        // 4 x 4 transpose of 16-byte pieces in every group of four lanes: store j then writes the 64 bytes of the group's block j at
        // once.  (A lane that wrote its own block wrote 16 bytes out of every 64 per store: HBM bound, 24 heads, L = 32760, d = 128
        // 93 us, 84 us so; without codes 85 and 72 us.)
        const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t &p = o[8 * t + i], &q = o[8 * t + 4 + i];
                const uint32_t give = b0 ? p : q, got = (uint32_t)__builtin_amdgcn_mov_dpp((int)give, 0xB1, 0xF, 0xF, true);
                if (b0) p = got; else q = got;
            }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t &p = o[4 * t + i], &q = o[8 + 4 * t + i];
                const uint32_t give = b1 ? p : q, got = (uint32_t)__builtin_amdgcn_mov_dpp((int)give, 0x4E, 0xF, 0xF, true);
                if (b1) p = got; else q = got;
            }
        const int q0 = gid & ~3, q = gid & 3;
        uint4v* dst = reinterpret_cast<uint4v*>(xf + (size_t)bh * L * D) + (size_t)q0 * 4 + q;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((q0 + j) / NB < L) { uint4v w; w[0] = o[4 * j]; w[1] = o[4 * j + 1]; w[2] = o[4 * j + 2]; w[3] = o[4 * j + 3]; dst[4 * j] = w; }
    }
}

// The public quantizer along the sequence (blocks of 32 positions, zero padded): how V is blocked.  One thread per (block, d index);
// FP8: E4M3 elements (one byte each) instead of E2M1.  codes [BH, D, Lc/2] (FP8: [BH, D, Lc]), scales [BH, D, Lc/32] with
// Lc = round_up(L, 32); optional bf16 xf [BH, L, D].
template <int D, bool FP8>
__global__ __launch_bounds__(D) void mx_quant_l_kernel(
    const uint16_t* __restrict__ x, int L, unsigned char* __restrict__ codes, unsigned char* __restrict__ scales, uint16_t* __restrict__ xf)
{
    const int bh = blockIdx.y, kb = blockIdx.x, dd = threadIdx.x;
    const uint16_t* src = x + (size_t)bh * L * D + dd;
    float v[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const int l = kb * 32 + i;
        v[i] = l < L ? bf16_to_f32(src[(size_t)l * D]) : 0.0f;
    }
    uint32_t byte, c[8];
    mx_block_codes<FP8>(v, byte, c);
    const float s = e8m0_as_f32(byte);
    constexpr int NW = FP8 ? 8 : 4;                 // code registers per block
    const int Lc = round_up(L, 32);
    if (codes) {
        uint4v* dst = reinterpret_cast<uint4v*>(codes + (((size_t)bh * D + dd) * (Lc / 32) + kb) * (4 * NW));
#pragma unroll
        for (int i = 0; i < NW / 4; ++i) { uint4v o; o[0] = c[4 * i]; o[1] = c[4 * i + 1]; o[2] = c[4 * i + 2]; o[3] = c[4 * i + 3]; dst[i] = o; }
    }
    if (scales) scales[((size_t)bh * D + dd) * (Lc / 32) + kb] = (unsigned char)byte;
    if (xf) {
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const int l = kb * 32 + i;
            const float val = FP8 ? e4m3_value_of((c[i >> 2] >> (8 * (i & 3))) & 255u) : e2m1_value_of((c[i >> 3] >> (4 * (i & 7))) & 15u);
            if (l < L) xf[((size_t)bh * L + l) * D + dd] = f32_to_bf16_rne(val * s);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Alg. 1 on the MX operands.  A workgroup of 4 waves owns 128 query rows of one head, a wave 32 of
// them, a lane one row and one of the two 32-key blocks of every 64-key tile (B_k = 64).
// kv records arrive in stages of two tiles, copied global->LDS directly into a ring of three stage
// buffers; one barrier per stage.  The S^T products of tile j+1 are issued before the softmax of
// tile j, so the matrix unit works under the wave's own vector instructions.
// PAGED: the kv records come from a KV cache (pages of 128 keys = one stage per kv head, located through
// page_table [B, max_pages]), every sequence has its own number of keys kv_lens[b] >= L, and the L queries are the
// LAST positions of the sequence.  lq_inner: the rows of a head are the G query heads of a kv group one after another,
// lq_inner positions each (L = G * lq_inner; a kv head's queries are contiguous in [B,Hq,Lq,d], so grouped-query
// heads with few positions share one tile and one pass over the pages); lq_inner == L: plain rows.  Under the causal
// mask the query at position i of its head sees keys 0 .. kv_len - lq_inner + i.
//
// KVM == 2, block-sparse attention on contiguous kv records: the workgroup visits only the 128-key blocks listed for its
// 128 query rows (page_table then is the list [B*Hq*ceil(L/128), max_pages] of block indices in increasing order and
// kv_lens the number of entries per row of that list); a row that ends up without any key gets O = 0 and L = -inf.
template <int D, bool CAUSAL, bool FP8PV, int KVM /* 0 contiguous, 1 paged KV cache, 2 block-sparse, 3 paged, by sequence length */>
__global__ __launch_bounds__(256, 2) void fwd_mx_kernel(
    const void* __restrict__ qops, const uint32_t* __restrict__ qsc, const unsigned char* __restrict__ kv,
    uint16_t* __restrict__ O, float* __restrict__ lse, int L, int Lp, int Hq, int G, float c /* log2(e)/sqrt(d) */,
    const int* __restrict__ page_table, const int* __restrict__ kv_lens, int max_pages, int num_pages, int lq_inner, int B)
{
    constexpr int KS = D / 64, MT = D / 32;
    constexpr bool PAGED = KVM == 1 || KVM == 3, SPARSE = KVM == 2;
    constexpr int KOPS = 2 * KS * 1024, VOPS = MT * (FP8PV ? 2048 : 1024), REC = mx_rec_bytes(D, FP8PV), STAGE = 2 * REC, NCH = STAGE / 1024;
    static_assert(STAGE % 1024 == 0, "a stage is a whole number of 1 KiB wave copies");
    extern __shared__ __align__(16) unsigned char smem[];          // 3 stage buffers

    const int nqt = Lp / 128;
    int bh, qt;
    // (gridDim.x / nqt: the number of heads; taken as B * Hq it left this kernel 1 - 1.6 % slower, with the same instructions at another
    // place: 2 x 12/3 heads, L = 33818 6.34 against 6.44 ms, 2 x 12 heads, L = 32760 6.00 against 6.07 ms)
    // In order of length: measured against head after head, 2 x 16/4 heads, L = 3001 causal 87 -> 66 us, 4 x 32/8 heads, L = 4096
    // 416 -> 374 us, L = 8192 364 -> 323 us, 64/8 heads, L = 32768 8.84 ms either way; block-sparse 32/8 heads, L = 8192 148 -> 130 us.
    // (sequences of 2k - 16k keys, 512-position chunks of 8 of them: 392 -> 317 us)
    if constexpr (KVM == 3) {
        if (!varlen_item(blockIdx.x, kv_lens, B, Hq, G, nqt, bh, qt)) return;
    } else if (CAUSAL && !PAGED) longest_first(blockIdx.x, B * Hq, nqt, bh, qt);
    else head_tile_of_block(blockIdx.x, gridDim.x / nqt, nqt, bh, qt);
    if (CAUSAL) qt = nqt - 1 - qt;
    const int b = bh / Hq, h = bh % Hq;
    const int bhkv = b * (Hq / G) + h / G;
    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0_w = qt * 128 + wave * 32;
    const int q_row = row0_w + ln;
    const int wave_qmax = row0_w + 31;

    // Q operands of this lane: codes of its row for d-slots 64 ks + 32 hf .. + 31, scale bytes by ks
    MxQ<D, 64> Q;
    const size_t grp = (size_t)bh * (Lp / 32) + (row0_w >> 5);
    Q.fetch(qops, qsc, bh, row0_w, grp, lane, L);

    const int Lk = PAGED ? __builtin_amdgcn_readfirstlane(kv_lens[b]) : L;      // keys of this sequence
    const int koff = PAGED ? Lk - lq_inner : 0;                    // key index of position 0's diagonal
    const bool packed = PAGED && lq_inner != L;                    // several heads' positions in this tile
    const int nkt_all = PAGED ? min((Lk + 63) / 64, 2 * max_pages) : (Lk + 63) / 64;   // never past the page table
    // block-sparse: the blocks of this workgroup's row of the list, and the first key of the block visited s-th
    const int* blk_row = SPARSE ? page_table + ((size_t)bh * nqt + qt) * max_pages : nullptr;
    const int nblk = SPARSE ? min(max(__builtin_amdgcn_readfirstlane(kv_lens[(size_t)bh * nqt + qt]), 0), max_pages) : 0;
    auto blk_of = [&](int s) __attribute__((always_inline)) -> int {
        return min(max(__builtin_amdgcn_readfirstlane(blk_row[s]), 0), Lp / 128 - 1);      // a bad entry reads a wrong block, never outside
    };
    const int nkt = SPARSE ? 2 * nblk
                  : (CAUSAL && !packed) ? min((koff + qt * 128 + 128 + 63) / 64, nkt_all) : nkt_all;   // tiles this workgroup visits
    const int nst = (nkt + 1) / 2;
    auto k0_of = [&](int j) __attribute__((always_inline)) -> int { return SPARSE ? blk_of(j >> 1) * 128 + (j & 1) * 64 : j * 64; };
    const unsigned char* kv_head = kv + (size_t)bhkv * (Lp / 64) * REC;
    const int Hkv = Hq / G;
    auto issue_stage = [&](int s) __attribute__((always_inline)) {
        const unsigned char* src = kv_head + (size_t)(SPARSE ? blk_of(s) : s) * STAGE;
        if constexpr (PAGED) {
            int page = __builtin_amdgcn_readfirstlane(page_table[(size_t)b * max_pages + s]);
            page = min(max(page, 0), num_pages - 1);               // a bad table entry reads a wrong page, never outside the cache
            src = kv + ((size_t)page * Hkv + (h / G)) * STAGE;
        }
        unsigned char* dst = smem + (s % 3) * STAGE;
        for (int i = wave; i < NCH; i += 4) async_copy16(src, (uint32_t)(i * 1024 + lane * 16), dst + i * 1024);
    };
    auto rec_of = [&](int j) __attribute__((always_inline)) -> const unsigned char* {
        return smem + ((j >> 1) % 3) * STAGE + (j & 1) * REC;
    };

    floatx16 o[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[mt][i] = 0.0f;
    float m = -INFINITY, lsum = 0.0f;

    auto as8 = [](const uint4v& x) __attribute__((always_inline)) -> int8v {
        int8v r = {(int)x[0], (int)x[1], (int)x[2], (int)x[3], 0, 0, 0, 0};
        return r;
    };
    // S^T of one tile: product t covers keys {16 t .. 16 t + 15} of both 32-key blocks
    auto scores = [&](const unsigned char* rec, floatx16 (&s)[2]) __attribute__((always_inline)) {
        const uint32_t ksc = lds_read4(rec + KOPS + VOPS + lane * 4);
        uint4v a[2][KS];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) a[t][ks] = lds_read16(rec + ((t * KS + ks) * 64 + lane) * 16);
        // (a constant zero accumulator is encoded in the instruction: no registers to clear)
        const floatx16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[0][0]), as8(Q.op[0]), zero, 4, 4, 0, ksc, 0, Q.sc);
        s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[1][0]), as8(Q.op[0]), zero, 4, 4, KS, ksc, 0, Q.sc);
        if constexpr (KS == 2) {
            s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[0][1]), as8(Q.op[1]), s[0], 4, 4, 1, ksc, 1, Q.sc);
            s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[1][1]), as8(Q.op[1]), s[1], 4, 4, 3, ksc, 1, Q.sc);
        }
    };
    // online softmax of one tile (Alg. 1 inner loop), phi of this lane's P-tilde block, O += V^F^T P-tilde^F
    auto softmax_pv = [&](int j, const unsigned char* rec, floatx16 (&s)[2]) __attribute__((always_inline)) {
        const int k0 = k0_of(j);
        const bool need_mask = (k0 + 64 > Lk) || (CAUSAL && k0 + 63 > koff + (packed ? 0 : row0_w));
        if (__builtin_expect(need_mask, 0)) {
            const int klim = CAUSAL ? min(Lk - 1, koff + (packed ? q_row % lq_inner : q_row)) : Lk - 1;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (k0 + 32 * hf + 16 * t + i > klim) s[t][i] = -INFINITY;
        }
        float mp[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) mp[t] = max_raw(s[0][t], s[1][t]);
#pragma unroll
        for (int i = 4; i < 16; ++i) mp[i & 3] = max_nc(max_nc(mp[i & 3], s[0][i]), s[1][i]);
        const float mown = max_nc(max_nc(mp[0], mp[1]), max_nc(mp[2], mp[3]));      // maximum of this lane's block
        const float mnew = max_nc(m, xhalf_max(mown));
        // (block-sparse: the first blocks a row meets may lie entirely in its causal future; until it has seen a key
        //  its maximum is -inf, and a finite stand-in keeps the two expressions below free of inf - inf)
        const float mref = (SPARSE && mnew == -INFINITY) ? 0.0f : mnew;
        const float alpha = __builtin_amdgcn_exp2f((m - mref) * c);
        const float ms = mref * c;
        m = mnew;
        float p[32];
        float rp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                p[16 * t + i] = __builtin_amdgcn_exp2f(fmaf(s[t][i], c, -ms));
                rp[i & 3] += p[16 * t + i];
            }
        lsum = lsum * alpha + ((rp[0] + rp[1]) + (rp[2] + rp[3]));                  // un-quantized P-tilde
        // block maximum of P-tilde: exp2 of the block's largest score, the same instructions on the same inputs
        const float amax = __builtin_amdgcn_exp2f(fmaf(mown, c, -ms));
        const uint32_t pbyte = FP8PV ? e8m0_of_amax_fp8(amax) : e8m0_of_amax(amax);
        uint32_t pc[8];
        if constexpr (FP8PV) {
            // E4M3 bytes of this lane's block, then the exchange that the FP8 operand layout asks for: registers 0-3 of
            // lane (row, h) hold keys 16 h .. + 15 of the tile and registers 4-7 keys 32 + 16 h .. + 15, so the lower
            // half-wave hands the second half of its block to the upper one and takes the first half of the upper's
            uint32_t own[8];
            mx_codes32_fp8(p, e8m0_as_f32(pbyte), own);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                auto r = __builtin_amdgcn_permlane32_swap(own[i], own[4 + i], false, false);
                pc[i] = r[0]; pc[4 + i] = r[1];
            }
        } else {
            const uint4v c4 = mx_codes32(p, e8m0_as_f32(pbyte));
#pragma unroll
            for (int i = 0; i < 4; ++i) { pc[i] = c4[i]; pc[4 + i] = 0u; }
        }
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0, 0)) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[mt][i] *= alpha;
        }
        const uint32_t vsc = lds_read4(rec + KOPS + VOPS + 256 + lane * 4);
        const int8v pb = {(int)pc[0], (int)pc[1], (int)pc[2], (int)pc[3], (int)pc[4], (int)pc[5], (int)pc[6], (int)pc[7]};
        if constexpr (FP8PV) {
            int8v va[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const uint4v lo = lds_read16(rec + KOPS + ((2 * mt) * 64 + lane) * 16), hi = lds_read16(rec + KOPS + ((2 * mt + 1) * 64 + lane) * 16);
                va[mt] = int8v{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
            }
            o[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va[0], pb, o[0], 0, 0, 0, vsc, 0, pbyte);
            o[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va[1], pb, o[1], 0, 0, 1, vsc, 0, pbyte);
            if constexpr (MT == 4) {
                o[2] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va[2], pb, o[2], 0, 0, 2, vsc, 0, pbyte);
                o[3] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va[3], pb, o[3], 0, 0, 3, vsc, 0, pbyte);
            }
        } else {
            uint4v va[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) va[mt] = lds_read16(rec + KOPS + (mt * 64 + lane) * 16);
            o[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(va[0]), pb, o[0], 4, 4, 0, vsc, 0, pbyte);
            o[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(va[1]), pb, o[1], 4, 4, 1, vsc, 0, pbyte);
            if constexpr (MT == 4) {
                o[2] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(va[2]), pb, o[2], 4, 4, 2, vsc, 0, pbyte);
                o[3] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(va[3]), pb, o[3], 4, 4, 3, vsc, 0, pbyte);
            }
        }
    };
    auto wave_sees = [&](int j) __attribute__((always_inline)) -> bool { return !CAUSAL || packed || k0_of(j) <= koff + wave_qmax; };
    // One tile: at odd j the next stage becomes visible (and the buffer two stages back becomes free).
    auto tile_step = [&](int j, floatx16 (&scur)[2], floatx16 (&snext)[2]) __attribute__((always_inline)) {
        if (j & 1) {
            __builtin_amdgcn_s_waitcnt(0);                 // this wave's part of stage (j+1)/2 is in LDS
            __builtin_amdgcn_s_barrier();                  // ... everyone's is, and everyone is past tile j-1
            if ((j >> 1) + 2 < nst) issue_stage((j >> 1) + 2);
        }
        if (j + 1 < nkt && wave_sees(j + 1)) scores(rec_of(j + 1), snext);
        if (wave_sees(j)) softmax_pv(j, rec_of(j), scur);
    };

    issue_stage(0);
    if (nst > 1) issue_stage(1);
    // (phi(Q) through the third stage buffer, which is not asked for yet)
    const uint32_t q_ops = lds_addr_of(smem) + (uint32_t)(2 * STAGE + wave * (kMxQOps<D> + 256));
    static_assert(4 * (kMxQOps<D> + 256) <= STAGE);
    Q.quantize(qsc, q_ops, q_ops + kMxQOps<D>, lane);
    mx_q_wave_fence();
    Q.read(qops, qsc, grp, lane, q_ops, q_ops + kMxQOps<D>);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    floatx16 sa[2], sb[2];
    scores(rec_of(0), sa);
    for (int j = 0; j < nkt; j += 2) {
        tile_step(j, sa, sb);
        if (j + 1 < nkt) tile_step(j + 1, sb, sa);
    }

    // ---- epilogue: O /= l, L = m + log l
    const float l = xhalf_sum(lsum);
    const float inv_l = ((PAGED || SPARSE) && !(l > 0.0f)) ? 0.0f : 1.0f / l;         // a row without keys: O = 0, L = -inf
    if (q_row < L) {
        const size_t row = (size_t)bh * L + q_row;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int d0 = 32 * mt + 8 * t + 4 * hf;
                uint2v w;
                w[0] = pack_bf16x2_rne(o[mt][4 * t] * inv_l, o[mt][4 * t + 1] * inv_l);
                w[1] = pack_bf16x2_rne(o[mt][4 * t + 2] * inv_l, o[mt][4 * t + 3] * inv_l);
                *reinterpret_cast<uint2v*>(O + row * D + d0) = w;
            }
        if (hf == 0) lse[row] = m * (c * 0.6931471805599453f) + logf(l);   // m is in raw q.k units
    }
}

// The same where there are too few query rows to fill the chip (see fwd_split_kernel in fwd.hip): a workgroup owns 32 rows, its four waves take
// four key tiles at a time, wave w tile 4 n + w for the scores, the softmax and phi(P-tilde), and block w of 32 d of O for the products of
// all four.  P crosses LDS as the codes and scale bytes that the instruction takes (1.25 KiB per tile), K and V operands go straight to
// registers.  All sums keep their order: the bits of fwd_mx_kernel.  KVM: 0 contiguous, 1 paged, 2 block-sparse, as there.
template <int D, bool CAUSAL, bool FP8PV, int KVM>
__global__ __launch_bounds__(256, 2) void fwd_mx_split_kernel(
    const void* __restrict__ qops, const uint32_t* __restrict__ qsc, const unsigned char* __restrict__ kv,
    uint16_t* __restrict__ O, float* __restrict__ lse, int L, int Lp, int Hq, int G, float c /* log2(e)/sqrt(d) */,
    const int* __restrict__ page_table, const int* __restrict__ kv_lens, int max_pages, int num_pages, int lq_inner, int B)
{
    constexpr int KS = D / 64, MT = D / 32, NT = 4, VW = FP8PV ? 2 : 1;     // VW: 16-byte pieces of a lane's V operand and of its codes of P
    constexpr bool PAGED = KVM == 1, SPARSE = KVM == 2;
    constexpr int KOPS = 2 * KS * 1024, VOPS = MT * VW * 1024, REC = mx_rec_bytes(D, FP8PV);
    __shared__ __align__(16) uint4v p_codes[NT][VW][64];
    __shared__ uint32_t p_byte[NT][64];
    __shared__ float x_max[NT][32], x_alpha[NT][32], x_sum[NT][64];

    const int n32 = (L + 31) / 32, nqt = Lp / 128;
    int bh, qt;
    if (CAUSAL && !PAGED) { longest_first(blockIdx.x, B * Hq, n32, bh, qt); qt = n32 - 1 - qt; }
    else head_tile_of_block(blockIdx.x, B * Hq, n32, bh, qt);
    const int b = bh / Hq, h = bh % Hq, bhkv = b * (Hq / G) + h / G, Hkv = Hq / G;
    const int lane = threadIdx.x & 63, ln = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int row0 = qt * 32, q_row = row0 + ln;
    MxQ<D, 256> Q;
    const size_t grp = (size_t)bh * (Lp / 32) + qt;
    Q.fetch(qops, qsc, bh, row0, grp, (int)threadIdx.x, L);

    const int Lk = PAGED ? __builtin_amdgcn_readfirstlane(kv_lens[b]) : L;
    const int koff = PAGED ? Lk - lq_inner : 0;
    const bool packed = PAGED && lq_inner != L;
    const int nkt_all = PAGED ? min((Lk + 63) / 64, 2 * max_pages) : (Lk + 63) / 64;
    // block-sparse: the list of this row block, and how many of its blocks these rows see at least in part (they are in increasing order)
    const int* blk_row = SPARSE ? page_table + ((size_t)bh * nqt + (qt >> 2)) * max_pages : nullptr;
    int nkt;
    if constexpr (SPARSE) {
        const int listed = min(max(__builtin_amdgcn_readfirstlane(kv_lens[(size_t)bh * nqt + (qt >> 2)]), 0), max_pages);
        int seen = 0;
        for (int i = 0; i < listed; i += 64)
            seen += __popcll(__builtin_amdgcn_ballot_w64(i + lane < listed && (!CAUSAL || blk_row[min(i + lane, listed - 1)] * 128 <= row0 + 31)));
        nkt = 2 * seen;
    } else nkt = CAUSAL && !packed ? min((koff + row0 + 31) / 64 + 1, nkt_all) : nkt_all;
    auto blk_of = [&](int s) __attribute__((always_inline)) -> int {
        return min(max(__builtin_amdgcn_readfirstlane(blk_row[s]), 0), Lp / 128 - 1);      // a bad entry reads a wrong block, never outside
    };
    auto k0_of = [&](int j) __attribute__((always_inline)) -> int { return SPARSE ? blk_of(j >> 1) * 128 + (j & 1) * 64 : j * 64; };
    if (SPARSE && CAUSAL && nkt > 0 && k0_of(nkt - 1) > row0 + 31) --nkt;                   // (the last block's second half)
    const unsigned char* kv_head = kv + (size_t)bhkv * (Lp / 64) * REC;
    auto rec_of = [&](int j_) __attribute__((always_inline)) -> const unsigned char* {      // (beyond the last tile: the last one)
        const int j = min(j_, nkt - 1);
        if constexpr (PAGED) {
            int page = __builtin_amdgcn_readfirstlane(page_table[(size_t)b * max_pages + (j >> 1)]);
            page = min(max(page, 0), num_pages - 1);               // a bad table entry reads a wrong page, never outside the cache
            return kv + (((size_t)page * Hkv + (h / G)) * 2 + (j & 1)) * REC;
        }
        return kv_head + (size_t)(SPARSE ? 2 * blk_of(j >> 1) + (j & 1) : j) * REC;
    };
    auto as8 = [](const uint4v& x) __attribute__((always_inline)) -> int8v {
        int8v r = {(int)x[0], (int)x[1], (int)x[2], (int)x[3], 0, 0, 0, 0};
        return r;
    };
    const bool has_o = wave < MT;
    const int mt = has_o ? wave : 0;
    uint4v kr[2 * KS], vr[NT][VW];
    uint32_t ksc = 0u, vsc[NT];
    auto load_k = [&](const unsigned char* rec) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2 * KS; ++i) kr[i] = *reinterpret_cast<const uint4v*>(rec + 1024 * i + 16 * lane);
        ksc = *reinterpret_cast<const uint32_t*>(rec + KOPS + VOPS + 4 * lane);
    };
    auto load_v = [&](int t, const unsigned char* rec) __attribute__((always_inline)) {
#pragma unroll
        for (int w = 0; w < VW; ++w) vr[t][w] = *reinterpret_cast<const uint4v*>(rec + KOPS + ((mt * VW + w) * 64 + lane) * 16);
        vsc[t] = *reinterpret_cast<const uint32_t*>(rec + KOPS + VOPS + 256 + 4 * lane) >> (8 * mt);
    };
    auto lds_barrier = [&]() __attribute__((always_inline)) {       // what was written to LDS is there, what was read has arrived
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC07F);                         // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    floatx16 o;
#pragma unroll
    for (int i = 0; i < 16; ++i) o[i] = 0.0f;
    float m = -INFINITY, lsum = 0.0f;
    if (nkt > 0) {
        load_k(rec_of(wave));
#pragma unroll
        for (int t = 0; t < NT; ++t) load_v(t, rec_of(t));
    }
    // (phi(Q) through the room of P, which is first written behind the barrier in the loop)
    static_assert(kMxQOps<D> <= sizeof(p_codes) && 256 <= sizeof(p_byte));
    Q.quantize(qsc, lds_addr_of(&p_codes[0][0][0]), lds_addr_of(&p_byte[0][0]), (int)threadIdx.x);
    lds_barrier();
    Q.read(qops, qsc, grp, lane, lds_addr_of(&p_codes[0][0][0]), lds_addr_of(&p_byte[0][0]));
    for (int j0 = 0; j0 < nkt; j0 += NT) {
        const int j = j0 + wave, nt = min(nkt - j0, NT);
        const bool active = wave < nt;
        floatx16 s[2];
        if (active) {
            const floatx16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr[0]), as8(Q.op[0]), zero, 4, 4, 0, ksc, 0, Q.sc);
            s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr[KS]), as8(Q.op[0]), zero, 4, 4, KS, ksc, 0, Q.sc);
            if constexpr (KS == 2) {
                s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr[1]), as8(Q.op[1]), s[0], 4, 4, 1, ksc, 1, Q.sc);
                s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr[3]), as8(Q.op[1]), s[1], 4, 4, 3, ksc, 1, Q.sc);
            }
            mfma_scale_settle(s[0], s[1]);
        }
        const bool more = j0 + NT < nkt;
        if (more) load_k(rec_of(j + NT));
        float mown = -INFINITY;
        if (active) {
            const int k0 = k0_of(j);
            if ((k0 + 64 > Lk) || (CAUSAL && k0 + 63 > koff + (packed ? 0 : row0))) {
                const int klim = CAUSAL ? min(Lk - 1, koff + (packed ? q_row % lq_inner : q_row)) : Lk - 1;
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (k0 + 32 * hf + 16 * t + i > klim) s[t][i] = -INFINITY;
            }
            float mp[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) mp[t] = max_raw(s[0][t], s[1][t]);
#pragma unroll
            for (int i = 4; i < 16; ++i) mp[i & 3] = max_nc(max_nc(mp[i & 3], s[0][i]), s[1][i]);
            mown = max_nc(max_nc(mp[0], mp[1]), max_nc(mp[2], mp[3]));              // maximum of this lane's block
            const float mt_ = xhalf_max(mown);
            if (hf == 0) x_max[wave][ln] = mt_;
        }
        lds_barrier();
        float m_next = m, m_prev = m, mnew = m;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float x = x_max[t][ln];
            if (t < wave) m_prev = max_nc(m_prev, x);
            if (t <= wave) mnew = max_nc(mnew, x);
            if (t < nt) m_next = max_nc(m_next, x);
        }
        m = m_next;
        if (active) {
            // (block-sparse: see fwd_mx_kernel)
            const float mref = (SPARSE && mnew == -INFINITY) ? 0.0f : mnew;
            const float alpha = __builtin_amdgcn_exp2f((m_prev - mref) * c);
            const float ms = mref * c;
            float p[32];
            float rp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    p[16 * t + i] = __builtin_amdgcn_exp2f(fmaf(s[t][i], c, -ms));
                    rp[i & 3] += p[16 * t + i];
                }
            x_sum[wave][lane] = (rp[0] + rp[1]) + (rp[2] + rp[3]);                      // un-quantized P-tilde
            if (hf == 0) x_alpha[wave][ln] = alpha;
            const float amax = __builtin_amdgcn_exp2f(fmaf(mown, c, -ms));
            const uint32_t pbyte = FP8PV ? e8m0_of_amax_fp8(amax) : e8m0_of_amax(amax);
            if constexpr (FP8PV) {
                uint32_t own[8];
                mx_codes32_fp8(p, e8m0_as_f32(pbyte), own);
                uint4v lo, hi;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    auto r = __builtin_amdgcn_permlane32_swap(own[i], own[4 + i], false, false);
                    lo[i] = r[0]; hi[i] = r[1];
                }
                p_codes[wave][0][lane] = lo;
                p_codes[wave][VW - 1][lane] = hi;
            } else p_codes[wave][0][lane] = mx_codes32(p, e8m0_as_f32(pbyte));
            p_byte[wave][lane] = pbyte;
        }
        lds_barrier();                                              // P, alpha and the sums are in LDS
        uint4v pc[NT][VW];
        uint32_t pb[NT];
        float al[NT], sm[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            al[t] = x_alpha[t][ln]; sm[t] = x_sum[t][lane]; pb[t] = p_byte[t][lane];
#pragma unroll
            for (int w = 0; w < VW; ++w) pc[t][w] = p_codes[t][w][lane];
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (t < nt) {
                lsum = lsum * al[t] + sm[t];                        // l in tile order
                if (has_o) {
                    if (__builtin_amdgcn_ballot_w64(al[t] != 1.0f) != 0) {
#pragma unroll
                        for (int i = 0; i < 16; ++i) o[i] *= al[t];
                    }
                    if constexpr (FP8PV) {
                        const int8v va = {(int)vr[t][0][0], (int)vr[t][0][1], (int)vr[t][0][2], (int)vr[t][0][3],
                                          (int)vr[t][VW - 1][0], (int)vr[t][VW - 1][1], (int)vr[t][VW - 1][2], (int)vr[t][VW - 1][3]};
                        const int8v pv = {(int)pc[t][0][0], (int)pc[t][0][1], (int)pc[t][0][2], (int)pc[t][0][3],
                                          (int)pc[t][VW - 1][0], (int)pc[t][VW - 1][1], (int)pc[t][VW - 1][2], (int)pc[t][VW - 1][3]};
                        o = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va, pv, o, 0, 0, 0, vsc[t], 0, pb[t]);
                    } else o = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(vr[t][0]), as8(pc[t][0]), o, 4, 4, 0, vsc[t], 0, pb[t]);
                }
            }
        }
        mfma_scale_settle(o);
        if (more && has_o) {
#pragma unroll
            for (int t = 0; t < NT; ++t) load_v(t, rec_of(j0 + NT + t));
        }
    }
    const float l = xhalf_sum(lsum);
    const float inv_l = ((PAGED || SPARSE) && !(l > 0.0f)) ? 0.0f : 1.0f / l;         // a row without keys: O = 0, L = -inf
    if (q_row < L && has_o) {
        const size_t row = (size_t)bh * L + q_row;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint2v w;
            w[0] = pack_bf16x2_rne(o[4 * t] * inv_l, o[4 * t + 1] * inv_l);
            w[1] = pack_bf16x2_rne(o[4 * t + 2] * inv_l, o[4 * t + 3] * inv_l);
            *reinterpret_cast<uint2v*>(O + row * D + 32 * mt + 8 * t + 4 * hf) = w;
        }
        if (hf == 0 && wave == 0) lse[row] = m * (c * 0.6931471805599453f) + logf(l);
    }
}

// ---------------------------------------------------------------------------------------------
// Decode form of the paged forward: at most 32 query rows per (sequence, kv head) — one position, or a few, of the G
// query heads of a group — against a long sequence.  fwd_mx_kernel would leave three of its four waves without rows
// and walk the pages with one; here the waves of a workgroup share the KEYS: an iteration takes NP pages (a page: two
// 64-key tiles), and wave w takes the product t = w % 2 of tile T = (w / 2) % 2 of page w / 4 of the iteration, i.e.
// keys {32 hf + 16 t .. + 15} of that tile (16 of each of its two 32-key blocks), for all 32 rows.  What Alg. 1 makes
// sequential is only the running maximum, and that needs no more than the waves' partial row maxima of S: they go
// through LDS once per iteration, after which every wave knows the maximum after each of the 2 NP tiles and the largest
// score of its two blocks (exp2 of it, by the same instructions as that element's P-tilde, is the block's amax, so both
// waves of a block derive the same scale).  Each wave then quantizes its 16 keys per row against the maximum after ITS
// tile, exactly as the tile order of Alg. 1 prescribes, and accumulates its own O and l against its own reference
// maximum; the partial results are brought to the final maximum and added at the end.
constexpr int kMxDecRows = 32;                       // most rows of a head
template <int D, bool CAUSAL, int NP /* pages per iteration: 4 NP waves */>
__global__ __launch_bounds__(256 * NP, NP == 1 ? 2 : 1) void fwd_mx_decode_kernel(
    const void* __restrict__ qops, const uint32_t* __restrict__ qsc, const unsigned char* __restrict__ kv,
    uint16_t* __restrict__ O, float* __restrict__ lse, int L /* rows, <= 32 */, int Hq, int G, float c /* log2(e)/sqrt(d) */,
    const int* __restrict__ page_table, const int* __restrict__ kv_lens, int max_pages, int num_pages, int lq_inner)
{
    constexpr int KS = D / 64, MT = D / 32, NW = 4 * NP;
    constexpr int NIT = NP == 1 ? 4 : NP == 2 ? 3 : 2;   // iterations whose pages the LDS ring holds (NIT - 1 of them in flight)
    constexpr int NR = NIT * NP;                     // ... in pages
    constexpr int KOPS = 2 * KS * 1024, VOPS = MT * 1024, REC = mx_rec_bytes(D, false), STAGE = 2 * REC, NCH = STAGE / 1024;
    constexpr int NV = MT * 16 + 1;                  // floats per lane in the final reduction
    static_assert(STAGE % 1024 == 0 && NR * STAGE >= (NW / 2) * NV * 256, "the ring also holds the final reduction");
    extern __shared__ __align__(16) unsigned char smem[];          // NR page buffers, then NW x 64 floats of partial maxima
    float* xchg = reinterpret_cast<float*>(smem + NR * STAGE);

    const int bh = blockIdx.x;
    const int b = bh / Hq, h = bh % Hq;
    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pi = wave >> 2, T = (wave >> 1) & 1, t = wave & 1;
    const int q_row = ln;
    const int Hkv = Hq / G;

    // Q operands of row block 0 (rows 0..31 of this head's only tile; rows >= L are zero)
    MxQ<D, 64 * NW> Q;
    Q.fetch(qops, qsc, bh, 0, (size_t)bh * 4, tid, L);

    const int Lk = __builtin_amdgcn_readfirstlane(kv_lens[b]);
    const int koff = Lk - lq_inner;
    const bool packed = lq_inner != L;
    const int nst = min((Lk + 127) / 128, max_pages);              // pages of this sequence
    const int nit = (nst + NP - 1) / NP;
    const int klim = CAUSAL ? min(Lk - 1, koff + (packed ? q_row % lq_inner : q_row)) : Lk - 1;

    // The pages of iteration it: NP * NCH copies of 1 KiB, dealt out to the waves in turn
    auto issue_iter = [&](int it) __attribute__((always_inline)) {
#pragma unroll
        for (int pp = 0; pp < NP; ++pp) {
            const int st = it * NP + pp;
            if (st < nst) {
                int page = __builtin_amdgcn_readfirstlane(page_table[(size_t)b * max_pages + st]);
                page = min(max(page, 0), num_pages - 1);           // a bad table entry reads a wrong page, never outside the cache
                const unsigned char* src = kv + ((size_t)page * Hkv + (h / G)) * STAGE;
                unsigned char* dst = smem + (st % NR) * STAGE;
                // copy g = pp * NCH + ch of the iteration goes to wave g mod NW
                for (int ch = (wave + NW - (pp * NCH) % NW) % NW; ch < NCH; ch += NW)
                    async_copy16(src, (uint32_t)(ch * 1024 + lane * 16), dst + ch * 1024);
            }
        }
    };
    // Wait until all but the copies of the `newer` most recent iterations have landed (vector-memory operations complete
    // in order).  Only meaningful while those iterations are whole: a wave issues (NP * NCH) / NW copies per iteration,
    // the first (NP * NCH) % NW waves one more.  s_waitcnt takes an immediate, hence the branches.
    constexpr int CLO = (NP * NCH) / NW, NHI = (NP * NCH) % NW;
    static_assert(NIT <= 4 && 2 * (CLO + 1) < 16, "at most two newer iterations in flight at a wait; the immediate below has 4 bits");
    auto wait_all_but = [&](int newer) __attribute__((always_inline)) {
#define AQ_VM(N) __builtin_amdgcn_s_waitcnt((N) | 0x70)
        if (newer >= 2)      { if (wave < NHI) AQ_VM(2 * (CLO + 1)); else AQ_VM(2 * CLO); }
        else if (newer == 1) { if (wave < NHI) AQ_VM(CLO + 1); else AQ_VM(CLO); }
        else                 __builtin_amdgcn_s_waitcnt(0);
#undef AQ_VM
    };
    auto as8 = [](const uint4v& x) __attribute__((always_inline)) -> int8v {
        int8v r = {(int)x[0], (int)x[1], (int)x[2], (int)x[3], 0, 0, 0, 0};
        return r;
    };

    floatx16 o[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[mt][i] = 0.0f;
    float m_run = -INFINITY;         // maximum after the last iteration (the same in every wave)
    float mref = -INFINITY;          // maximum this wave's O and l refer to (after its tile of its last iteration)
    float lsum = 0.0f;

    // Q must have arrived before the copies start: the wait for an ordinary load issued after them would wait for them too
    Q.arrived();
    __builtin_amdgcn_s_waitcnt(0);
#pragma unroll
    for (int i = 0; i < NIT - 1; ++i)
        if (i < nit) issue_iter(i);
    // (phi(Q) through the buffers of iteration NIT - 1, which is asked for behind the first barrier of the loop)
    const uint32_t q_ops = lds_addr_of(smem) + (uint32_t)((NIT - 1) * NP * STAGE);
    Q.quantize(qsc, q_ops, q_ops + kMxQOps<D>, tid);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    Q.read(qops, qsc, (size_t)bh * 4, lane, q_ops, q_ops + kMxQOps<D>);

    for (int it = 0; it < nit; ++it) {
        // iteration it's pages are in LDS (the newer ones may be in flight if they are whole), everyone is past iteration it - 1
        const int issued = min(nit, it + NIT - 1);                            // iterations issued so far
        wait_all_but(issued * NP <= nst ? issued - 1 - it : 0);
        __builtin_amdgcn_s_barrier();
        if (it + NIT - 1 < nit) issue_iter(it + NIT - 1);                     // into the buffers of iteration it - 1
        const int st = it * NP + pi;                                          // this wave's page
        const bool valid = st < nst;                                          // (the last iteration may be short of pages)
        const unsigned char* rec = smem + (st % NR) * STAGE + T * REC;
        const int k0 = st * 128 + T * 64;
        // S^T of this wave's 32 keys
        floatx16 sv;
#pragma unroll
        for (int i = 0; i < 16; ++i) sv[i] = -INFINITY;
        if (valid) {
            const uint32_t ksc = lds_read4(rec + KOPS + VOPS + lane * 4);
            uint4v a[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) a[ks] = lds_read16(rec + ((t * KS + ks) * 64 + lane) * 16);
#pragma unroll
            for (int i = 0; i < 16; ++i) sv[i] = 0.0f;
            if (t == 0) {
                sv = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[0]), as8(Q.op[0]), sv, 4, 4, 0, ksc, 0, Q.sc);
                if constexpr (KS == 2) sv = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[1]), as8(Q.op[1]), sv, 4, 4, 1, ksc, 1, Q.sc);
            } else {
                sv = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[0]), as8(Q.op[0]), sv, 4, 4, KS, ksc, 0, Q.sc);
                if constexpr (KS == 2) sv = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[1]), as8(Q.op[1]), sv, 4, 4, 3, ksc, 1, Q.sc);
            }
            const bool need_mask = (k0 + 64 > Lk) || (CAUSAL && k0 + 63 > koff);
            if (need_mask) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (k0 + 32 * hf + 16 * t + i > klim) sv[i] = -INFINITY;
            }
        }
        float pm[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) pm[i] = max_nc(max_nc(sv[i], sv[4 + i]), max_raw(sv[8 + i], sv[12 + i]));
        xchg[wave * 64 + lane] = max_nc(max_nc(pm[0], pm[1]), max_nc(pm[2], pm[3]));
        // (fences, not __syncthreads(): the copies in flight are not to be waited for here)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        // maxima after each of the iteration's 2 NP tiles (tile tau: waves 2 tau and 2 tau + 1, both half-waves)
        float mT = m_run, bm = -INFINITY, mt_run = m_run;
#pragma unroll
        for (int tau = 0; tau < 2 * NP; ++tau) {
            const float x0 = xchg[(2 * tau) * 64 + lane], x1 = xchg[(2 * tau + 1) * 64 + lane];
            const float y0 = xchg[(2 * tau) * 64 + (lane ^ 32)], y1 = xchg[(2 * tau + 1) * 64 + (lane ^ 32)];
            mt_run = max_nc(mt_run, max_nc(max_nc(x0, x1), max_nc(y0, y1)));
            if (tau == 2 * pi + T) { mT = mt_run; bm = max_nc(x0, x1); }     // wave-uniform: this wave's tile, this lane's block
        }
        m_run = mt_run;
        if (valid) {
            const float alpha = __builtin_amdgcn_exp2f((mref - mT) * c);
            const float ms = mT * c;
            mref = mT;
            float p[16];
            float rp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                p[i] = __builtin_amdgcn_exp2f(fmaf(sv[i], c, -ms));
                rp[i & 3] += p[i];
            }
            lsum = lsum * alpha + ((rp[0] + rp[1]) + (rp[2] + rp[3]));        // un-quantized P-tilde
            const float amax = __builtin_amdgcn_exp2f(fmaf(bm, c, -ms));
            const uint32_t pbyte = e8m0_of_amax(amax);
            const float psc = e8m0_as_f32(pbyte);
            uint32_t c0 = 0u, c1 = 0u;
            c0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c0, p[0], p[1], psc, 0);
            c0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c0, p[2], p[3], psc, 1);
            c0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c0, p[4], p[5], psc, 2);
            c0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c0, p[6], p[7], psc, 3);
            c1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c1, p[8], p[9], psc, 0);
            c1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c1, p[10], p[11], psc, 1);
            c1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c1, p[12], p[13], psc, 2);
            c1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c1, p[14], p[15], psc, 3);
            // B operand of O^T += V^F^T P^T: this lane's k-slots are keys 32 hf + 0..31 of the tile, 8 to a register;
            // the wave fills the 16 it has and leaves the other wave's at zero
            const int8v pb = t ? int8v{0, 0, (int)c0, (int)c1, 0, 0, 0, 0} : int8v{(int)c0, (int)c1, 0, 0, 0, 0, 0, 0};
            if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) o[mt][i] *= alpha;
            }
            const uint32_t vsc = lds_read4(rec + KOPS + VOPS + 256 + lane * 4);
            uint4v va[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) va[mt] = lds_read16(rec + KOPS + (mt * 64 + lane) * 16);
            o[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(va[0]), pb, o[0], 4, 4, 0, vsc, 0, pbyte);
            o[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(va[1]), pb, o[1], 4, 4, 1, vsc, 0, pbyte);
            if constexpr (MT == 4) {
                o[2] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(va[2]), pb, o[2], 4, 4, 2, vsc, 0, pbyte);
                o[3] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(va[3]), pb, o[3], 4, 4, 3, vsc, 0, pbyte);
            }
        }
        // (the partial maxima are read before the next iteration's barrier, which precedes the next writes)
    }

    // ---- the partial results, brought to the final maximum and added (a tree over the waves); O /= l, L = m + log l
    const float f = (mref == m_run) ? 1.0f : __builtin_amdgcn_exp2f((mref - m_run) * c);      // (also covers -inf - -inf)
    float l = xhalf_sum(lsum) * f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[mt][i] *= f;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();                                                          // everyone is done with the page buffers
    float* red = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int step = NW / 2; step >= 1; step >>= 1) {
        if (wave >= step && wave < 2 * step) {
            float* dst = red + (size_t)(wave - step) * NV * 64;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 16; ++i) dst[(mt * 16 + i) * 64 + lane] = o[mt][i];
            dst[(MT * 16) * 64 + lane] = l;
        }
        __syncthreads();
        if (wave < step) {
            const float* src = red + (size_t)wave * NV * 64;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[mt][i] += src[(mt * 16 + i) * 64 + lane];
            l += src[(MT * 16) * 64 + lane];
        }
        __syncthreads();
    }
    if (wave == 0) {
        const float inv_l = l > 0.0f ? 1.0f / l : 0.0f;                       // a sequence without keys: O = 0, L = -inf
        if (q_row < L) {
            const size_t row = (size_t)bh * L + q_row;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int tt = 0; tt < 4; ++tt) {
                    const int d0 = 32 * mt + 8 * tt + 4 * hf;
                    uint2v w;
                    w[0] = pack_bf16x2_rne(o[mt][4 * tt] * inv_l, o[mt][4 * tt + 1] * inv_l);
                    w[1] = pack_bf16x2_rne(o[mt][4 * tt + 2] * inv_l, o[mt][4 * tt + 3] * inv_l);
                    *reinterpret_cast<uint2v*>(O + row * D + d0) = w;
                }
            if (hf == 0) lse[row] = m_run * (c * 0.6931471805599453f) + logf(l);
        }
    }
}

// Few sequences: one workgroup per (sequence, kv head) walks all pages, a microsecond each, while most compute units idle.  The walk is then
// taken apart; every sum keeps its terms and their order, so the results have the bits of fwd_mx_decode_kernel, whatever runs beside a sequence:
//   mx_decode_max_kernel   the scores of a chunk of pages for their row maxima alone (P-tilde is quantized against the running maximum; on
//                          the FP4 instruction scores are cheap, and this reads the K half of the records only);
//   mx_decode_p_kernel     a workgroup per chunk, from the maximum in front of it: scores, softmax, phi(P-tilde).  Codes, scale byte, running
//                          maximum and the two parts of l that the walk's waves add go to memory, 36 bytes per row and 32 keys;
//   mx_decode_pv_kernel    a workgroup per (sequence, kv head) and block of 32 d: what is sequential about the walk, P V and l of each of
//                          its four waves page by page, with the loads of sixteen pages on their way: 0.12 us a page (10 KiB through
//                          the cache of one compute unit), 15.4 us for 16000 keys.
// The records of P have room for kMxDecPageHeads pages; longer sequences take the last two launches in several segments.
// A record of a page: 32 bytes per (tile, half of its keys, row), {codes, sum of P-tilde, maximum} of keys 0-15 and of keys 16-31 of the block
// of 32; then a dword each, the block's scale byte.
constexpr int kMxDecSlot = 32;
constexpr int kMxDecAhead = 16;                      // pages whose loads mx_decode_pv_kernel has on their way
struct MxDecSplit { int per /* pages of a chunk */, n /* chunks of a sequence */, seg /* pages of a segment */; float* cmax; float* state; unsigned char* rec; };
__host__ __device__ constexpr size_t mx_dec_rec_bytes(int L) { return (size_t)4 * L * (kMxDecSlot + 4); }
__device__ inline unsigned char* mx_dec_rec(const MxDecSplit& sp, int L, int bh, int page /* of the segment */) {
    return sp.rec + ((size_t)bh * sp.seg + page) * mx_dec_rec_bytes(L);
}

// Row maxima of the scores of every chunk but a sequence's last (nobody asks for that one's): blockIdx = (head, chunk).  Operands straight
// to registers, a page ahead; waves as in fwd_mx_decode_kernel: wave w has product w % 2 of tile w / 2 of each page.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(256) void mx_decode_max_kernel(
    const void* __restrict__ qops, const uint32_t* __restrict__ qsc, const unsigned char* __restrict__ kv, int L, int Hq, int G,
    const int* __restrict__ page_table, const int* __restrict__ kv_lens, int max_pages, int num_pages, int lq_inner, int per, int n, float* __restrict__ cmax)
{
    constexpr int KS = D / 64, MT = D / 32, KOPS = 2 * KS * 1024, VOPS = MT * 1024, REC = mx_rec_bytes(D, false), STAGE = 2 * REC;
    __shared__ float red[4][64];
    const int bh = blockIdx.x, ch = blockIdx.y, b = bh / Hq, h = bh % Hq, Hkv = Hq / G;
    const int lane = threadIdx.x & 63, ln = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), T = wave >> 1, t = wave & 1;
    const int Lk = __builtin_amdgcn_readfirstlane(kv_lens[b]);
    const int nst = min((Lk + 127) / 128, max_pages), p0 = ch * per;
    if (p0 + per >= nst) return;                                              // the last chunk, or none
    const int koff = Lk - lq_inner;
    const int klim = CAUSAL ? min(Lk - 1, koff + (lq_inner != L ? ln % lq_inner : ln)) : Lk - 1;
    MxQ<D, 256> Q;
    Q.fetch(qops, qsc, bh, 0, (size_t)bh * 4, (int)threadIdx.x, L);
    auto as8 = [](const uint4v& x) __attribute__((always_inline)) -> int8v {
        int8v r = {(int)x[0], (int)x[1], (int)x[2], (int)x[3], 0, 0, 0, 0};
        return r;
    };
    uint4v a[KS];
    uint32_t ksc;
    auto load = [&](int p) __attribute__((always_inline)) {
        const int page = min(max(__builtin_amdgcn_readfirstlane(page_table[(size_t)b * max_pages + p]), 0), num_pages - 1);
        const unsigned char* rec = kv + ((size_t)page * Hkv + h / G) * STAGE + T * REC;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) a[ks] = *reinterpret_cast<const uint4v*>(rec + ((t * KS + ks) * 64 + lane) * 16);
        ksc = *reinterpret_cast<const uint32_t*>(rec + KOPS + VOPS + lane * 4) >> (8 * t * KS);
    };
    float mx = -INFINITY;
    load(p0);
    __shared__ __align__(16) unsigned char q_lds[kMxQOps<D> + 256];
    Q.quantize(qsc, lds_addr_of(q_lds), lds_addr_of(q_lds) + kMxQOps<D>, (int)threadIdx.x);
    __syncthreads();
    Q.read(qops, qsc, (size_t)bh * 4, lane, lds_addr_of(q_lds), lds_addr_of(q_lds) + kMxQOps<D>);
    for (int p = p0; p < p0 + per; ++p) {
        floatx16 sv;
#pragma unroll
        for (int i = 0; i < 16; ++i) sv[i] = 0.0f;
        sv = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[0]), as8(Q.op[0]), sv, 4, 4, 0, ksc, 0, Q.sc);
        if constexpr (KS == 2) sv = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[1]), as8(Q.op[1]), sv, 4, 4, 1, ksc, 1, Q.sc);
        mfma_scale_settle(sv);
        if (p + 1 < p0 + per) load(p + 1);
        const int k0 = p * 128 + T * 64;
        if ((k0 + 64 > Lk) || (CAUSAL && k0 + 63 > koff)) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (k0 + 32 * hf + 16 * t + i > klim) sv[i] = -INFINITY;
        }
        float pm[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) pm[i] = max_nc(max_nc(sv[i], sv[4 + i]), max_raw(sv[8 + i], sv[12 + i]));
        mx = max_nc(mx, max_nc(max_nc(pm[0], pm[1]), max_nc(pm[2], pm[3])));
    }
    red[wave][lane] = xhalf_max(mx);
    __syncthreads();
    if (wave == 0 && hf == 0) cmax[((size_t)bh * n + ch) * kMxDecRows + ln] = fmaxf(fmaxf(red[0][lane], red[1][lane]), fmaxf(red[2][lane], red[3][lane]));
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(256) void mx_decode_p_kernel(
    const void* __restrict__ qops, const uint32_t* __restrict__ qsc, const unsigned char* __restrict__ kv, int L, int Hq, int G, float c,
    const int* __restrict__ page_table, const int* __restrict__ kv_lens, int max_pages, int num_pages, int lq_inner, MxDecSplit sp, int seg0 /* first page of the segment */)
{
    constexpr int KS = D / 64, MT = D / 32, KOPS = 2 * KS * 1024, VOPS = MT * 1024, REC = mx_rec_bytes(D, false), NT = 4;
    __shared__ float front[8][32], x_max[2][NT][32];
    const int bh = blockIdx.x, ch = seg0 / sp.per + (int)blockIdx.y, b = bh / Hq, h = bh % Hq, Hkv = Hq / G;
    const int lane = threadIdx.x & 63, ln = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int Lk = __builtin_amdgcn_readfirstlane(kv_lens[b]);
    const int p0 = ch * sp.per, nt_all = 2 * min(min((Lk + 127) / 128, max_pages) - p0, sp.per);      // tiles of this chunk
    if (nt_all <= 0) return;
    const int koff = Lk - lq_inner;
    const int klim = CAUSAL ? min(Lk - 1, koff + (lq_inner != L ? ln % lq_inner : ln)) : Lk - 1;
    uint4v kr[2 * KS];
    MxQ<D, 256> Q;
    uint32_t ksc;
    // tile j of the chunk (beyond the last one: the last one)
    auto page_of = [&](int j) __attribute__((always_inline)) { return page_table[(size_t)b * max_pages + p0 + (min(j, nt_all - 1) >> 1)]; };
    auto load_k = [&](int j, int id) __attribute__((always_inline)) {
        const int page = min(max(__builtin_amdgcn_readfirstlane(id), 0), num_pages - 1);           // a bad table entry reads a wrong page, never outside the cache
        const unsigned char* rec = kv + (((size_t)page * Hkv + h / G) * 2 + (min(j, nt_all - 1) & 1)) * REC;
#pragma unroll
        for (int i = 0; i < 2 * KS; ++i) kr[i] = *reinterpret_cast<const uint4v*>(rec + 1024 * i + 16 * lane);
        ksc = *reinterpret_cast<const uint32_t*>(rec + KOPS + VOPS + 4 * lane);
    };
    Q.fetch(qops, qsc, bh, 0, (size_t)bh * 4, (int)threadIdx.x, L);
    load_k(wave, page_of(wave));
    int id_next = page_of(wave + NT);
    auto as8 = [](const uint4v& x) __attribute__((always_inline)) -> int8v {
        int8v r = {(int)x[0], (int)x[1], (int)x[2], (int)x[3], 0, 0, 0, 0};
        return r;
    };
    auto lds_barrier = [&]() __attribute__((always_inline)) {       // (fences, not __syncthreads(): the loads of the next tile stay on their way)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    };
    // the maximum in front of the chunk: the half-waves take every eighth chunk
    float m = -INFINITY;
    for (int i = 2 * wave + hf; i < ch; i += 8) m = fmaxf(m, sp.cmax[((size_t)bh * sp.n + i) * kMxDecRows + ln]);
    front[2 * wave + hf][ln] = m;
    __shared__ __align__(16) unsigned char q_lds[kMxQOps<D> + 256];
    Q.quantize(qsc, lds_addr_of(q_lds), lds_addr_of(q_lds) + kMxQOps<D>, (int)threadIdx.x);
    lds_barrier();
#pragma unroll
    for (int i = 0; i < 8; ++i) m = fmaxf(m, front[i][ln]);
    Q.read(qops, qsc, (size_t)bh * 4, lane, lds_addr_of(q_lds), lds_addr_of(q_lds) + kMxQOps<D>);
    for (int j0 = 0, buf = 0; j0 < nt_all; j0 += NT, buf ^= 1) {
        const int j = j0 + wave;
        const bool active = j < nt_all;
        const floatx16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        floatx16 s[2];
        s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr[0]), as8(Q.op[0]), zero, 4, 4, 0, ksc, 0, Q.sc);
        s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr[KS]), as8(Q.op[0]), zero, 4, 4, KS, ksc, 0, Q.sc);
        if constexpr (KS == 2) {
            s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr[1]), as8(Q.op[1]), s[0], 4, 4, 1, ksc, 1, Q.sc);
            s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr[3]), as8(Q.op[1]), s[1], 4, 4, 3, ksc, 1, Q.sc);
        }
        mfma_scale_settle(s[0], s[1]);
        if (j0 + NT < nt_all) {
            load_k(j + NT, id_next);
            id_next = page_of(j + 2 * NT);
        }
        const int k0 = p0 * 128 + j * 64;
        if (active && ((k0 + 64 > Lk) || (CAUSAL && k0 + 63 > koff))) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (k0 + 32 * hf + 16 * t + i > klim) s[t][i] = -INFINITY;
        }
        float pm[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) pm[i] = max_raw(s[0][i], s[1][i]);
#pragma unroll
        for (int i = 4; i < 16; ++i) pm[i & 3] = max_nc(max_nc(pm[i & 3], s[0][i]), s[1][i]);
        const float bm = max_nc(max_nc(pm[0], pm[1]), max_nc(pm[2], pm[3]));      // maximum of this lane's block of 32 keys
        const float tm = xhalf_max(bm);
        if (hf == 0) x_max[buf][wave][ln] = tm;
        lds_barrier();
        float mT = m;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float x = x_max[buf][t][ln];
            if (t <= wave) mT = max_nc(mT, x);
            if (j0 + t < nt_all) m = max_nc(m, x);
        }
        if (active) {
            const float ms = mT * c;
            float p[32], sum[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                float rp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    p[16 * t + i] = __builtin_amdgcn_exp2f(fmaf(s[t][i], c, -ms));
                    rp[i & 3] += p[16 * t + i];
                }
                sum[t] = (rp[0] + rp[1]) + (rp[2] + rp[3]);                       // un-quantized P-tilde
            }
            const uint32_t pbyte = e8m0_of_amax(__builtin_amdgcn_exp2f(fmaf(bm, c, -ms)));
            const uint4v codes = mx_codes32(p, e8m0_as_f32(pbyte));
            if (ln < L) {
                unsigned char* rec = mx_dec_rec(sp, L, bh, p0 - seg0 + (j >> 1));
                const int slot = (2 * (j & 1) + hf) * L + ln;
                uint4v* dst = reinterpret_cast<uint4v*>(rec + (size_t)slot * kMxDecSlot);
                dst[0] = uint4v{codes[0], codes[1], __float_as_uint(sum[0]), __float_as_uint(mT)};
                dst[1] = uint4v{codes[2], codes[3], __float_as_uint(sum[1]), __float_as_uint(mT)};
                *reinterpret_cast<uint32_t*>(rec + (size_t)4 * L * kMxDecSlot + 4 * slot) = pbyte;
            }
        }
    }
}

// Waves as in fwd_mx_decode_kernel: wave w has the keys {32 hf + 16 t .. + 15} of tile T of every page, t = w % 2, T = w / 2.
template <int D>
__global__ __launch_bounds__(256, 2) void mx_decode_pv_kernel(
    const unsigned char* __restrict__ kv, uint16_t* __restrict__ O, float* __restrict__ lse, int L, int Hq, int G, float c,
    const int* __restrict__ page_table, const int* __restrict__ kv_lens, int max_pages, int num_pages, MxDecSplit sp, int seg0)
{
    constexpr int KS = D / 64, MT = D / 32, KOPS = 2 * KS * 1024, VOPS = MT * 1024, REC = mx_rec_bytes(D, false), PF = kMxDecAhead, NV = 17;
    __shared__ float red[2][NV][64];
    __shared__ __align__(16) uint32_t ids[kMxDecPageHeads + 2 * PF];
    const int bh = blockIdx.x, mt = blockIdx.y, b = bh / Hq, h = bh % Hq, Hkv = Hq / G;
    const int lane = threadIdx.x & 63, ln = lane & 31, hf = lane >> 5, row = min(ln, L - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), T = wave >> 1, t = wave & 1;
    const int nst = min((__builtin_amdgcn_readfirstlane(kv_lens[b]) + 127) / 128, max_pages);
    if (seg0 > 0 && nst <= seg0) return;                           // finished in a segment in front
    const int n = max(min(nst - seg0, sp.seg), 0);                 // its pages in this segment
    // the ids of the segment's pages, in LDS (scalar loads of them would be waited for page by page, all at once each time); behind the last
    // page: that one again
    if (n > 0) {
        for (int i = threadIdx.x; i < n + 2 * PF; i += 256)
            ids[i] = min(max(page_table[(size_t)b * max_pages + seg0 + min(i, n - 1)], 0), num_pages - 1);      // a bad table entry reads a wrong page, never outside the cache
    }
    __syncthreads();
    const unsigned char* v_head = kv + ((size_t)(h / G) * 2 + T) * REC;
    const uint32_t page_stride = (uint32_t)Hkv * 2 * REC, rec_stride = (uint32_t)mx_dec_rec_bytes(L);
    uint4v va[PF], pc[PF];                                         // V; codes, sum, maximum
    uint32_t vsc[PF], psc[PF];
    const int slot = (2 * T + hf) * L + row;
    const uint32_t v_lane = (uint32_t)(KOPS + (mt * 64 + lane) * 16), s_lane = (uint32_t)(KOPS + VOPS + 256 + 4 * lane);
    const uint32_t p_lane = (uint32_t)(slot * kMxDecSlot + 16 * t), b_lane = (uint32_t)(4 * L * kMxDecSlot + 4 * slot);
    const unsigned char* p_at = mx_dec_rec(sp, L, bh, 0);           // of the page that is loaded next
    auto load = [&](int u, uint32_t id) __attribute__((always_inline)) {
        va[u] = *reinterpret_cast<const uint4v*>(v_head + v_lane + (uint64_t)id * page_stride);
        vsc[u] = *reinterpret_cast<const uint32_t*>(v_head + s_lane + (uint64_t)id * page_stride);
        pc[u] = *reinterpret_cast<const uint4v*>(p_at + p_lane);
        psc[u] = *reinterpret_cast<const uint32_t*>(p_at + b_lane);
        p_at += rec_stride;
        __builtin_amdgcn_sched_barrier(0);
    };
    floatx16 o;
    float mref, lsum;
    float* state = sp.state + ((((size_t)bh * MT + mt) * 4 + wave) * 18 * 2 + hf) * L + row;       // [18][2][L]
    if (seg0 > 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) o[i] = state[i * 2 * L];
        mref = state[16 * 2 * L]; lsum = state[17 * 2 * L];
        asm volatile("" : "+v"(o), "+v"(mref), "+v"(lsum));        // (arrived: they would otherwise be waited for in the loop, every time)
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) o[i] = 0.0f;
        mref = -INFINITY; lsum = 0.0f;
    }
    const int keep_lo = t ? 0 : -1;
    auto page = [&](int u) __attribute__((always_inline)) {
        // (pinned copies and results: whatever of a page's registers lived on behind its next load would be copied, all of them at the end of
        //  the loop, where those loads would then be waited for)
        float mT;
        uint32_t vs;
        asm volatile("v_mov_b32 %0, %1" : "=v"(mT) : "v"(pc[u][3]));
        asm volatile("v_lshrrev_b32 %0, %1, %2" : "=v"(vs) : "s"(8 * mt), "v"(vsc[u]));
        const float alpha = __builtin_amdgcn_exp2f((mref - mT) * c);
        mref = mT;
        lsum = fmaf(lsum, alpha, __uint_as_float(pc[u][2]));
        asm volatile("" : "+v"(lsum));
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) o[i] *= alpha;
        }
        const int c0 = (int)pc[u][0], c1 = (int)pc[u][1];
        const int8v pb = {c0 & keep_lo, c1 & keep_lo, c0 & ~keep_lo, c1 & ~keep_lo, 0, 0, 0, 0};
        const int8v av = {(int)va[u][0], (int)va[u][1], (int)va[u][2], (int)va[u][3], 0, 0, 0, 0};
        o = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, pb, o, 4, 4, 0, vs, 0, psc[u]);
    };
    // the next PF pages
    auto load_all = [&](int i, auto between) __attribute__((always_inline)) {
        uint4v id[PF / 4];
#pragma unroll
        for (int u = 0; u < PF / 4; ++u) id[u] = *reinterpret_cast<const uint4v*>(&ids[i + 4 * u]);
#pragma unroll
        for (int u = 0; u < PF; ++u) { between(u); load(u, id[u / 4][u % 4]); }
    };
    if (n > 0) load_all(0, [](int) {});
    int i0 = 0;
    for (; i0 + PF <= n; i0 += PF) load_all(i0 + PF, page);
#pragma unroll
    for (int u = 0; u < PF; ++u)
        if (i0 + u < n) page(u);
    mfma_scale_settle(o);
    if (nst > seg0 + sp.seg) {                                      // the sequence goes on in the next segment
        if (ln < L) {
#pragma unroll
            for (int i = 0; i < 16; ++i) state[i * 2 * L] = o[i];
            state[16 * 2 * L] = mref; state[17 * 2 * L] = lsum;
        }
        return;
    }
    // the waves' sums brought to the last maximum and added, as in fwd_mx_decode_kernel
    const float m_run = n > 0 ? *reinterpret_cast<const float*>(mx_dec_rec(sp, L, bh, n - 1) + ((2 + hf) * L + row) * kMxDecSlot + 12) : -INFINITY;
    const float f = (mref == m_run) ? 1.0f : __builtin_amdgcn_exp2f((mref - m_run) * c);
    float l = xhalf_sum(lsum) * f;
#pragma unroll
    for (int i = 0; i < 16; ++i) o[i] *= f;
#pragma unroll
    for (int step = 2; step >= 1; step >>= 1) {
        if (wave >= step && wave < 2 * step) {
#pragma unroll
            for (int i = 0; i < 16; ++i) red[wave - step][i][lane] = o[i];
            red[wave - step][16][lane] = l;
        }
        __syncthreads();
        if (wave < step) {
#pragma unroll
            for (int i = 0; i < 16; ++i) o[i] += red[wave][i][lane];
            l += red[wave][16][lane];
        }
        __syncthreads();
    }
    if (wave == 0 && ln < L) {
        const float inv_l = l > 0.0f ? 1.0f / l : 0.0f;                       // a sequence without keys: O = 0, L = -inf
        const size_t at = (size_t)bh * L + ln;
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            uint2v w;
            w[0] = pack_bf16x2_rne(o[4 * tt] * inv_l, o[4 * tt + 1] * inv_l);
            w[1] = pack_bf16x2_rne(o[4 * tt + 2] * inv_l, o[4 * tt + 3] * inv_l);
            *reinterpret_cast<uint2v*>(O + at * D + 32 * mt + 8 * tt + 4 * hf) = w;
        }
        if (hf == 0 && mt == 0) lse[at] = m_run * (c * 0.6931471805599453f) + logf(l);
    }
}

// How the pages are cut for `heads` (sequence, kv head)s; n = 1: not at all.  Up to four workgroups per compute unit, of two pages at least.  The
// walk takes 0.85 us a page, two more launches what 12 pages take.  Whole step, d = 128, 8 kv heads, walk -> in parts: one sequence of 3000
// keys 26.9 -> 15.5 us, of 16000 111 -> 25.0, of 64000 429 -> 67; 8 of 500 - 1700 18.5 -> 14.4, of 2000 - 8000 60 -> 27.2; 16 of 256 - 2000 20.5 ->
// 19.2, of 2000 - 8000 60 -> 40.7.  In several segments: 14 of 4000 - 16000 (112 heads) 113 -> 79, but 20 of them 113 -> 130 and 20 of
// 2000 - 8000 61 -> 68: up to 128 heads.  (Chunks added up each by itself, whose bits then depend on how many there are: one sequence 13.6,
// 19.0 and 38 us, the others the same.)
static int mx_decode_room(int L) { return min(kMxDecPageHeads, (int)((16u << 20) / mx_dec_rec_bytes(L))); }      // pages times heads
static MxDecSplit mx_decode_split(int heads, int L, int max_pages)
{
    MxDecSplit sp{};
    sp.n = 1;
    const int room = mx_decode_room(L) / heads / 2 * 2, want = min((max_pages + 1) / 2, 1024 / heads);
    if (room < 2 || want < 3 || (long long)max_pages * (want - 1) < 12ll * want) return sp;
    const int n = max(want, (max_pages + room - 1) / room);
    if ((long long)n * heads > kMxDecUnits || (max_pages > room && heads > 128)) return sp;
    sp.per = ((max_pages + n - 1) / n + 1) / 2 * 2;                           // (the kernel of P takes two pages at a time)
    sp.n = (max_pages + sp.per - 1) / sp.per;
    sp.seg = min(room, sp.n * sp.per) / sp.per * sp.per;
    return sp;
}
static size_t mx_decode_state_bytes(int heads, int L, int D) { return (size_t)heads * (D / 32) * 4 * 18 * 2 * L * 4; }
size_t mx_decode_part_bytes(int heads, int L, int D)
{
    if (L > kMxDecRows || heads > 170) return 0;
    return (size_t)kMxDecUnits * kMxDecRows * 4 + mx_decode_state_bytes(heads, L, D) + (size_t)(mx_decode_room(L) + kMxDecAhead) * mx_dec_rec_bytes(L);
}

// ---------------------------------------------------------------------------------------------
int launch_mx_quant(const void* x, int BH, int L, int D, int axis, bool fp8, unsigned char* codes, unsigned char* scales, void* xf, hipStream_t st)
{
    if (BH > 65535 || (axis == 0 && fp8) || (D != 64 && D != 128)) return -1;
    const dim3 grid_d((unsigned)(((size_t)L * (D / 32) + 255) / 256), (unsigned)BH), grid_l((unsigned)((L + 31) / 32), (unsigned)BH);
#define AQ_Q(KERN, GRID, BLOCK) hipLaunchKernelGGL((KERN), GRID, dim3(BLOCK), 0, st, (const uint16_t*)x, L, codes, scales, (uint16_t*)xf)
    if (axis == 0) { if (D == 128) AQ_Q(mx_quant_d_kernel<128>, grid_d, 256); else AQ_Q(mx_quant_d_kernel<64>, grid_d, 256); }
    else if (fp8)  { if (D == 128) AQ_Q((mx_quant_l_kernel<128, true>), grid_l, 128); else AQ_Q((mx_quant_l_kernel<64, true>), grid_l, 64); }
    else           { if (D == 128) AQ_Q((mx_quant_l_kernel<128, false>), grid_l, 128); else AQ_Q((mx_quant_l_kernel<64, false>), grid_l, 64); }
#undef AQ_Q
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

size_t mx_kv_bytes(int BHkv, int L, int D, bool fp8v) { return (size_t)BHkv * (round_up(L, kRowPad) / 64) * mx_rec_bytes(D, fp8v); }
size_t mx_ktrain_bytes(int BHkv, int L, int D) { return (size_t)BHkv * (round_up(L, kRowPad) / 64) * mx_ktrain_rec_bytes(D); }
size_t mx_qops_bytes(int BHq, int L, int D) { return (size_t)BHq * round_up(L, kRowPad) * (D / 2); }
size_t mx_qsc_bytes(int BHq, int L) { return (size_t)BHq * (round_up(L, kRowPad) / 32) * 64 * 4; }
size_t mx_page_bytes(int D) { return 2 * (size_t)mx_rec_bytes(D, false); }

// Whether the key tiles are shared (fwd_mx_split_kernel): by the number of 32-row groups per compute unit, as split_key_tiles in fwd.hip.  Rows of
// one length: three, as many as share a unit (two in the mixed recipe): d = 128, 8 heads, L = 2000 (504 groups) 34.8 -> 25.3 us, L = 3000 (752)
// 47.6 -> 41.1 us, 32 heads, L = 777 (800) 22.7 -> 26.5 us; mixed recipe 37.0 -> 27.9 us, 51 -> 59 us; chunks of a prefill, 8 sequences of
// 2000 - 8000 (512) 101 -> 70 us.  Causal: five, fewer for short rows: 12 heads, L = 2300 (864) 41.7 -> 30.2 us, 8 heads, L = 5000 (1256)
// 76 -> 56 us, 64 heads, L = 256 (512) 12.8 -> 11.4 us, L = 500 (1024) 18.7 -> 19.2 us, 32 heads, L = 2500 (2528) 54 -> 63 us; four in the mixed recipe
// (40 heads, L = 1000 (1280) 29.3 -> 32.3 us; 9 heads, L = 4000 (1125) 1.14 times).  Block-sparse under it (0.3 of the blocks): six: 32 heads,
// L = 1500 (1504) 30.5 -> 27.0 us, L = 2500 (2528) 42.4 -> 44.9 us.  Contiguous heads whose number does not let them stay on one XCD: fewer for short rows
// without a mask (60 heads, L = 320 (600) 16.1 -> 17.8 us, 52 heads, L = 256 (416), mixed 14.2 -> 15.5 us) and in the mixed recipe (46 heads, L = 500 (736)
// causal 21.1 -> 23.5 us).
static bool mx_split_key_tiles(int heads, int L, bool causal, bool fp8pv, bool sparse, bool paged)
{
    const int n32 = (L + 31) / 32;
    const bool spread = heads % 8 != 0 && !sparse && !paged;
    int quarters = 4 * (causal ? min(sparse ? 6 : 5, 1 + n32 / 8) : fp8pv ? 2 : 3);      // of a group per compute unit
    if (causal && fp8pv && n32 < 100) quarters = min(quarters, !spread || n32 >= 32 ? 16 : n32 < 20 ? 8 : 12);
    if (!causal && spread && n32 < 16) quarters = fp8pv ? 5 : 7;
    return (long long)heads * n32 * 4 <= (long long)device_cu_count() * quarters;
}

template <int D, bool CAUSAL, bool FP8PV, int KVM>
static int launch_fwd_mx_t(const void* qops, const void* qsc, const void* kv, int B, int Hq, int Hkv, int L,
                           void* o, float* lse, const int* page_table, const int* kv_lens, int max_pages, int num_pages, int lq_inner,
                           hipStream_t st)
{
    const int Lp = round_up(L, kRowPad);
    const size_t smem = 3 * 2 * (size_t)mx_rec_bytes(D, FP8PV);
    const float c = 1.4426950408889634f / sqrtf((float)D);
    if constexpr (KVM != 3) {
        if (mx_split_key_tiles(B * Hq, L, CAUSAL && KVM != 1, FP8PV, KVM == 2, KVM == 1)) {
            hipLaunchKernelGGL((fwd_mx_split_kernel<D, CAUSAL, FP8PV, KVM>), dim3((unsigned)(B * Hq * ((L + 31) / 32))), dim3(256), 0, st,
                               qops, (const uint32_t*)qsc, (const unsigned char*)kv,
                               (uint16_t*)o, lse, L, Lp, Hq, Hq / Hkv, c, page_table, kv_lens, max_pages, num_pages, lq_inner, B);
            return hipGetLastError() == hipSuccess ? 0 : -1;
        }
    }
    auto kern = fwd_mx_kernel<D, CAUSAL, FP8PV, KVM>;
    static unsigned long long lds_set = 0;          // one per instantiation
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)smem, lds_set)) return -1;
    const int groups = KVM == 3 ? round_up(B * Hkv, 8) : B * Hkv;       // (see varlen_item)
    hipLaunchKernelGGL(kern, dim3((unsigned)(groups * (Hq / Hkv) * (Lp / 128))), dim3(256), smem, st,
                       qops, (const uint32_t*)qsc, (const unsigned char*)kv,
                       (uint16_t*)o, lse, L, Lp, Hq, Hq / Hkv, c, page_table, kv_lens, max_pages, num_pages, lq_inner, B);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
template <int D, bool FP8PV>
static int launch_fwd_mx_d(const void* qops, const void* qsc, const void* kv, int B, int Hq, int Hkv, int L, bool causal,
                           void* o, float* lse, hipStream_t st)
{
    return causal ? launch_fwd_mx_t<D, true, FP8PV, 0>(qops, qsc, kv, B, Hq, Hkv, L, o, lse, nullptr, nullptr, 0, 0, L, st)
                  : launch_fwd_mx_t<D, false, FP8PV, 0>(qops, qsc, kv, B, Hq, Hkv, L, o, lse, nullptr, nullptr, 0, 0, L, st);
}

int launch_fwd_mx(const void* qops, const void* qsc, const void* kv, int B, int Hq, int Hkv, int L, int D, bool causal, bool fp8pv,
                  void* o, float* lse, hipStream_t st)
{
    if (D == 128) return fp8pv ? launch_fwd_mx_d<128, true>(qops, qsc, kv, B, Hq, Hkv, L, causal, o, lse, st)
                               : launch_fwd_mx_d<128, false>(qops, qsc, kv, B, Hq, Hkv, L, causal, o, lse, st);
    if (D == 64)  return fp8pv ? launch_fwd_mx_d<64, true>(qops, qsc, kv, B, Hq, Hkv, L, causal, o, lse, st)
                               : launch_fwd_mx_d<64, false>(qops, qsc, kv, B, Hq, Hkv, L, causal, o, lse, st);
    return -1;
}

int launch_fwd_mx_paged(const void* qops, const void* qsc, const void* cache, int B, int Hq, int Hkv, int Lq, int D, bool causal,
                        const int* page_table, const int* kv_lens, int max_pages, int num_pages, int lq_inner,
                        unsigned char* part, void* o, float* lse, hipStream_t st)
{
    if (Lq <= kMxDecRows) {
        // a step of decoding: the four waves of a workgroup share the keys of a page
        const float c = 1.4426950408889634f / sqrtf((float)D);
        MxDecSplit sp{};
        if (part) sp = mx_decode_split(B * Hq, Lq, max_pages);
        if (sp.n > 1) {
            sp.cmax = reinterpret_cast<float*>(part);
            sp.rec = part + (size_t)kMxDecUnits * kMxDecRows * 4;
            sp.state = reinterpret_cast<float*>(sp.rec + (size_t)(mx_decode_room(Lq) + kMxDecAhead) * mx_dec_rec_bytes(Lq));
#define AQ_SPLIT(DD, CC) do { \
            hipLaunchKernelGGL((mx_decode_max_kernel<DD, CC>), dim3((unsigned)(B * Hq), (unsigned)(sp.n - 1)), dim3(256), 0, st, qops, (const uint32_t*)qsc, \
                               (const unsigned char*)cache, Lq, Hq, Hq / Hkv, page_table, kv_lens, max_pages, num_pages, lq_inner, sp.per, sp.n, sp.cmax); \
            for (int seg0 = 0; seg0 < max_pages; seg0 += sp.seg) { \
                hipLaunchKernelGGL((mx_decode_p_kernel<DD, CC>), dim3((unsigned)(B * Hq), (unsigned)(min(sp.seg, max_pages - seg0) + sp.per - 1) / sp.per), dim3(256), 0, st, \
                                   qops, (const uint32_t*)qsc, (const unsigned char*)cache, Lq, Hq, Hq / Hkv, c, page_table, kv_lens, max_pages, num_pages, lq_inner, sp, seg0); \
                hipLaunchKernelGGL((mx_decode_pv_kernel<DD>), dim3((unsigned)(B * Hq), DD / 32), dim3(256), 0, st, (const unsigned char*)cache, (uint16_t*)o, lse, \
                                   Lq, Hq, Hq / Hkv, c, page_table, kv_lens, max_pages, num_pages, sp, seg0); \
            } \
            return hipGetLastError() == hipSuccess ? 0 : -1; } while (0)
            if (D == 128) { if (causal) AQ_SPLIT(128, true); else AQ_SPLIT(128, false); }
            if (D == 64)  { if (causal) AQ_SPLIT(64, true); else AQ_SPLIT(64, false); }
#undef AQ_SPLIT
            return -1;
        }
#define AQ_DECODE(DD, CC) do { \
        constexpr int NP = AQ_DECODE_NP; \
        constexpr size_t smem = (NP == 1 ? 4 : NP == 2 ? 3 : 2) * NP * 2 * (size_t)mx_rec_bytes(DD, false) + 4 * NP * 256; \
        auto kern = fwd_mx_decode_kernel<DD, CC, NP>; \
        static unsigned long long lds_set = 0; \
        if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)smem, lds_set)) return -1; \
        hipLaunchKernelGGL(kern, dim3((unsigned)(B * Hq)), dim3(256 * NP), smem, st, qops, (const uint32_t*)qsc, \
                           (const unsigned char*)cache, (uint16_t*)o, lse, Lq, Hq, Hq / Hkv, c, page_table, kv_lens, max_pages, num_pages, lq_inner); \
        return hipGetLastError() == hipSuccess ? 0 : -1; } while (0)
        if (D == 128) { if (causal) AQ_DECODE(128, true); else AQ_DECODE(128, false); }
        if (D == 64)  { if (causal) AQ_DECODE(64, true); else AQ_DECODE(64, false); }
#undef AQ_DECODE
        return -1;
    }
    // With no more workgroups than compute units each has one of its own, and no order is worth looking up.  A kernel of its own: with
    // both in one the key loop came out 1.5 - 2 % slower, of the same instructions in other registers (16/2 heads, 500 positions over
    // 15k keys: 112.2 -> 114.4 us; 8 sequences of 16/4 heads, 98 positions over 2k - 7k keys: 87.4 -> 88.8 us).
    // (few query rows: the kernel in which four waves share the key tiles takes the plain order, too)
    const bool by_length = (long long)B * Hq * (round_up(Lq, kRowPad) / 128) > device_cu_count() && !mx_split_key_tiles(B * Hq, Lq, false, false, false, true);
#define AQ_PAGED_K(DD, CC, KK) launch_fwd_mx_t<DD, CC, false, KK>(qops, qsc, cache, B, Hq, Hkv, Lq, o, lse, page_table, kv_lens, max_pages, num_pages, lq_inner, st)
#define AQ_PAGED(DD, CC) (by_length ? AQ_PAGED_K(DD, CC, 3) : AQ_PAGED_K(DD, CC, 1))
    if (D == 128) return causal ? AQ_PAGED(128, true) : AQ_PAGED(128, false);
    if (D == 64)  return causal ? AQ_PAGED(64, true) : AQ_PAGED(64, false);
#undef AQ_PAGED
#undef AQ_PAGED_K
    return -1;
}

int launch_fwd_mx_sparse(const void* qops, const void* qsc, const void* kv, int B, int Hq, int Hkv, int L, int D, bool causal,
                         const int* list, const int* cnt, void* o, float* lse, hipStream_t st)
{
    const int nb = round_up(L, kRowPad) / 128;
#define AQ_SPARSE(DD, CC) launch_fwd_mx_t<DD, CC, false, 2>(qops, qsc, kv, B, Hq, Hkv, L, o, lse, list, cnt, nb, 0, L, st)
    if (D == 128) return causal ? AQ_SPARSE(128, true) : AQ_SPARSE(128, false);
    if (D == 64)  return causal ? AQ_SPARSE(64, true) : AQ_SPARSE(64, false);
#undef AQ_SPARSE
    return -1;
}

}  // namespace aq
