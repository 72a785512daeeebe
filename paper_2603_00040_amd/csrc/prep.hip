// phi of Eq. 1 / Eq. 2 (Sec. 2.1) as a streaming kernel, plus the layout copies the
// attention kernels read: the first line of Alg. 1 (phi(Q), phi(K), phi(V)) and of
// Alg. 2 (Q^F, K^F, V^F).  HBM-bandwidth bound.
//
// One thread owns one block of 16 consecutive d-elements (32 bytes in).  A workgroup
// covers 64 sequence positions; the optional transposed copy goes through LDS so that
// both the row-major and the transposed stores are 16-byte vectors.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "prep.hpp"
#include "nvfp4.hpp"

namespace aq {

// Position p (0..15) inside a group of 16 sequence positions of a transposed copy holds
// sequence index perm16(p): quads 1 and 2 are exchanged.  A lane of a 32x32x16 MFMA
// accumulator owns sequence indices {0-3, 8-11} (lanes 0-31) or {4-7, 12-15} (lanes
// 32-63) of such a group, so with this order its 8 values pair with one contiguous
// 16-byte run of the transposed operand.
__host__ __device__ inline int perm16(int p) { return (p & ~12) | ((p & 4) << 1) | ((p & 8) >> 1); }

// The NVFP4 KV cache: a page holds 128 consecutive positions of one sequence for all kv heads; per kv head, in this order,
// K codes [128][D/2], K scale bytes [128][D/16], V codes [128][D/2], V scale bytes [128][D/16]: the public layout of
// attnqat_quantize cut into pages.  Blocks run along d, so positions are independent of each other: a sequence grows by
// writing its new positions only.
__host__ __device__ inline size_t nvfp4_page_head_bytes(int D) { return (size_t)2 * 128 * (D / 2 + D / 16); }
// Codes and scale byte of block cb of position l (nullptr for a page id outside the cache).
__device__ inline const unsigned char* nvfp4_page_part(const unsigned char* cache, int page, int num_pages, int Hkv, int h, int D, int which) {
    if (page < 0 || page >= num_pages) return nullptr;
    return cache + ((size_t)page * Hkv + h) * nvfp4_page_head_bytes(D) + (size_t)which * 128 * (D / 2 + D / 16);
}

// The 64 positions l0 .. l0 + 63 of head bh, by one workgroup.
// PACKED (with QUANT = false): the input is not x but an already quantized tensor, codes [BH, L, D/2] and E4M3 scale bytes
// [BH, L, D/16] in the public layout of attnqat_quantize (read through `codes` and `scales`); the kernel writes the
// dequantized layout copies, the same values the quantizing variant writes for the tensor those codes came from.
// PAGED (with PACKED): the quantized tensor is the K or the V part of the pages of an NVFP4 KV cache; bh = sequence * Hkv + kv
// head, position l of sequence b is slot l % 128 of page table[b][l / 128], positions from kv_lens[b] on read as zeros, and
// L is the capacity max_pages * 128 that the copies are laid out for.
// NORM: n2 becomes the largest squared norm of the rows seen so far (in the lanes that hold a row's first block).
// KOPS: the rows (xr) are written in the order of the forward's K operands.
// The public outputs (codes, scales, xf_pub) are those of the public quantizer alone, which has bf16 copies and no bound (PUBLIC); sub (K smoothing), whose values
// have no codes here, is for the others.
template <int D, bool QUANT, bool OUT_F16, bool PACKED, bool PAGED, bool NORM, bool KOPS = false>
__device__ __forceinline__ void prep_tile_d(
    uint16_t (*tile)[128 + 2], int bh, int l0, const uint16_t* __restrict__ x, int L, int Lp,
    uint8_t* __restrict__ codes, uint8_t* __restrict__ scales, uint16_t* __restrict__ xf_pub,
    uint16_t* __restrict__ xr, uint16_t* __restrict__ xt, const float* __restrict__ sub, const PagedSrc& ps, float& n2)
{
    static_assert(!(QUANT && PACKED), "a packed input is already quantized");
    static_assert(!PAGED || PACKED, "pages hold quantized tensors");
    constexpr bool PUBLIC = QUANT && !OUT_F16 && !NORM;
    constexpr int nb = D / 16, NI = nb / 4;      // 16-element blocks per row, and of the 64 rows per thread
    const size_t in_base = (size_t)bh * L * D;
    int Lseq = L;
    const unsigned char* page_part[PAGED ? 1 : 1] = {nullptr};
    if constexpr (PAGED) {
        const int b = bh / ps.Hkv;
        const int page = ps.table[(size_t)b * ps.max_pages + (l0 >> 7)];      // a workgroup's 64 positions lie in one page
        Lseq = max(0, min(ps.kv_lens[b], L));
        if (l0 >= Lseq) return;                  // key tiles that start beyond the sequence are never read
        page_part[0] = nvfp4_page_part(ps.cache, page, ps.num_pages, ps.Hkv, bh % ps.Hkv, D, ps.which);
    }

    // The loads of all blocks of a thread first: one trip to memory instead of one per block.  With d as a constant (no divisions), 8
    // sequences of 2k - 16k keys in pages, 8 kv heads, 512 rows each, whole step 662 -> 646 us; 32 heads, L = 777 25.5 -> 25.15 us.
    // (opaque: the addresses of every variant would otherwise be formed in front of the loop over tiles and held in registers)
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int cb = (int)(tid % nb), row0 = (int)(tid / nb);
    uint4v xa[PACKED ? 1 : NI], xb[PACKED ? 1 : NI];
    uint2v cw[PACKED ? NI : 1];
    uint32_t sw[PACKED ? NI : 1];
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const int row = row0 + it * (256 / nb), l = l0 + row;
        if constexpr (PACKED) {
            const unsigned char* cp = nullptr; const unsigned char* sp = nullptr;
            if constexpr (PAGED) {
                if (l < Lseq && page_part[0]) {
                    cp = page_part[0] + (size_t)(l & 127) * (D / 2) + cb * 8;
                    sp = page_part[0] + (size_t)128 * (D / 2) + (size_t)(l & 127) * nb + cb;
                }
            } else if (l < L) {
                cp = codes + ((size_t)bh * L + l) * (D / 2) + cb * 8;
                sp = scales + ((size_t)bh * L + l) * nb + cb;
            }
            cw[it][0] = cw[it][1] = sw[it] = 0u;          // (reads as zeros)
            if (cp) { cw[it] = *reinterpret_cast<const uint2v*>(cp); sw[it] = *sp; }
        } else {
            xa[it] = xb[it] = uint4v{0u, 0u, 0u, 0u};
            if (l < L) {
                const uint4v* src = reinterpret_cast<const uint4v*>(x + in_base + (size_t)l * D + cb * 16);
                xa[it] = src[0]; xb[it] = src[1];
            }
        }
    }
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        __builtin_amdgcn_sched_barrier(0);         // (one block after the other: the registers of two at once would cost wavefronts)
        const int row = row0 + it * (256 / nb), l = l0 + row;
        float v[16];
        Nv16 q = nv16_of(0u, 0u, 0u);
        if constexpr (PACKED) {
            q = nv16_of(cw[it][0], cw[it][1], sw[it]);
        } else {
            const uint4v a = xa[it], b = xb[it];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[2 * i]         = __uint_as_float(a[i] << 16);
                v[2 * i + 1]     = __uint_as_float(a[i] & 0xFFFF0000u);
                v[8 + 2 * i]     = __uint_as_float(b[i] << 16);
                v[8 + 2 * i + 1] = __uint_as_float(b[i] & 0xFFFF0000u);
            }
            if (!PUBLIC && sub && l < L) {  // K smoothing: minus the token mean of the channel, an fp32 subtraction.
                // The inputs of phi then have 24 significant bits: the two "IEEE division == real quotient" arguments
                // below hold up to a double rounding that can move a value sitting within 2^-24 of a rounding boundary.
                const float* sp = sub + (size_t)bh * D + cb * 16;
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] -= sp[i];
            }
        }

        float xf[16];
        bool direct = true;                              // the values are those of q
        if constexpr (QUANT) {
            if (!PUBLIC && sub) {
                direct = false;
                float amax = 0.0f;
#pragma unroll
                for (int i = 0; i < 16; ++i) amax = fmaxf(amax, fabsf(v[i]));
                q.s = block_scale_exact(amax);
                // (inputs with 24 significant bits, after the K smoothing subtraction: IEEE division and the grid rounding
                //  of common.hpp; the short cuts of phi_block16_bf16 rely on bf16 inputs)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const uint32_t sign = __float_as_uint(v[i]) >> 31;
                    float r = 0.0f;
                    if (q.s > 0.0f) {
                        r = fabsf(v[i]) / q.s;
                        r = rne_e2m1_grid(r < 6.0f ? r : 6.0f);
                    }
                    const float d = r * q.s;                 // exact: <= 6 significant bits
                    xf[i] = sign ? -d : d;
                }
            } else q = phi_block16_bf16(v);
            if (PUBLIC && l < L && codes) {
                uint2v c2; c2[0] = q.clo; c2[1] = q.chi;
                *reinterpret_cast<uint2v*>(codes + ((size_t)bh * L + l) * (D / 2) + cb * 8) = c2;
            }
            if (PUBLIC && scales) {
                // four neighbouring blocks of a row (four neighbouring lanes: nb is 4 or 8 and a wave starts at a multiple
                // of 64 blocks) write their scale bytes as one dword; rows beyond L take part in the exchange and write nothing
                uint32_t sb = q.sc & 0xFFu;
                sb |= lane_down<1>(sb) << 8;
                sb |= lane_down<2>(sb) << 16;
                if (l < L && (cb & 3) == 0) *reinterpret_cast<uint32_t*>(scales + ((size_t)bh * L + l) * nb + cb) = sb;
            }
        }
        // the values as floats where more than the fp16 copy is made of them
        constexpr bool FLOATS = NORM || !OUT_F16;
        if constexpr (FLOATS) {
            if constexpr (QUANT || PACKED) { if (direct) dequant_block16(q, xf); }
            else
#pragma unroll
                for (int i = 0; i < 16; ++i) xf[i] = v[i];
        }

        if constexpr (NORM) {                            // |row|^2: nb neighbouring lanes hold a row
            float acc = 0.0f;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc = fmaf(xf[i], xf[i], acc);
            acc = lanes_sum<nb / 2, 1>(acc);
            n2 = fmaxf(n2, acc);
        }
        // public copy (bf16, un-padded) and workspace copies (fp16 or bf16); both formats hold s*c exactly
        uint32_t w[8];
        if constexpr (OUT_F16) {
            static_assert(QUANT || PACKED);
            if (direct) dequant_block16_f16(q, w);
            else
#pragma unroll
                for (int i = 0; i < 8; ++i) w[i] = pack_f16x2(xf[2 * i], xf[2 * i + 1]);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = pack_bf16x2_cvt(xf[2 * i], xf[2 * i + 1]);
            if (PUBLIC && xf_pub && l < L) {
                uint4v o0, o1;
#pragma unroll
                for (int i = 0; i < 4; ++i) { o0[i] = w[i]; o1[i] = w[4 + i]; }
                uint4v* dst = reinterpret_cast<uint4v*>(xf_pub + in_base + (size_t)l * D + cb * 16);
                dst[0] = o0; dst[1] = o1;
            }
        }
        if (xr) {                                        // rows padded to Lp with zeros
            uint4v o0, o1;
#pragma unroll
            for (int i = 0; i < 4; ++i) { o0[i] = w[i]; o1[i] = w[4 + i]; }
            uint16_t* dst = xr + (size_t)bh * Lp * D + (KOPS ? k_operand_offset(l, cb, 0, D) : (size_t)l * D + cb * 16);
            *reinterpret_cast<uint4v*>(dst) = o0;
            *reinterpret_cast<uint4v*>(dst + (KOPS ? 32 * 8 : 8)) = o1;
        }
        if (xt) {
#pragma unroll
            for (int i = 0; i < 8; ++i) reinterpret_cast<uint32_t*>(&tile[row][cb * 16])[i] = w[i];      // (rows are 4-byte aligned)
        }
    }
    if (xt) {
        __syncthreads();
        // transposed copy: 8 positions (16 bytes) per store; a thread takes them of two neighbouring columns, which lie in one LDS
        // word and whose operands are neighbours in memory
#pragma unroll
        for (int ch = (int)tid; ch < D * 4; ch += 256) {
            const int c = 2 * (ch % (D / 2)), kc = ch / (D / 2);
            uint32_t x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int p = kc * 8 + j;
                x[j] = *reinterpret_cast<const uint32_t*>(&tile[(p & ~15) | perm16(p & 15)][c]);
            }
            uint4v lo, hi;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                lo[j] = __builtin_amdgcn_perm(x[2 * j + 1], x[2 * j], 0x05040100u);
                hi[j] = __builtin_amdgcn_perm(x[2 * j + 1], x[2 * j], 0x07060302u);
            }
            uint16_t* dst = xt + (size_t)bh * Lp * D + v_operand_offset((l0 >> 4) + (kc >> 1), c, kc & 1, D);
            *reinterpret_cast<uint4v*>(dst) = lo;
            *reinterpret_cast<uint4v*>(dst + 8) = hi;
        }
    }
}

// (The head dimension as a constant: no divisions by it, and the blocks of a thread side by side.)
template <bool QUANT, bool OUT_F16, bool PACKED, bool PAGED, bool NORM, bool KOPS = false>
__device__ __forceinline__ void prep_tile(
    uint16_t (*tile)[128 + 2], int bh, int l0, const uint16_t* __restrict__ x, int L, int Lp, int D,
    uint8_t* __restrict__ codes, uint8_t* __restrict__ scales, uint16_t* __restrict__ xf_pub,
    uint16_t* __restrict__ xr, uint16_t* __restrict__ xt, const float* __restrict__ sub, const PagedSrc& ps, float& n2)
{
    if (D == 128) prep_tile_d<128, QUANT, OUT_F16, PACKED, PAGED, NORM, KOPS>(tile, bh, l0, x, L, Lp, codes, scales, xf_pub, xr, xt, sub, ps, n2);
    else          prep_tile_d<64, QUANT, OUT_F16, PACKED, PAGED, NORM, KOPS>(tile, bh, l0, x, L, Lp, codes, scales, xf_pub, xr, xt, sub, ps, n2);
}

// The public quantizer: codes, scales and dequantized values of one tensor.
__global__ __launch_bounds__(256) void quantize_kernel(const uint16_t* __restrict__ x, int L, int Lp, int D,
                                                       uint8_t* __restrict__ codes, uint8_t* __restrict__ scales, uint16_t* __restrict__ xf)
{
    float n2 = 0.0f;
    prep_tile<true, false, false, false, false>(nullptr, blockIdx.y, blockIdx.x * 64, x, L, Lp, D, codes, scales, xf, nullptr, nullptr, nullptr, PagedSrc{}, n2);
}

// All tensors that a forward or a backward prepares, as one launch.  Bound by HBM on large problems; on small ones a launch takes
// 3 - 5 us whatever its size (start, first loads, last stores), and a forward had three of them, a backward six.
// The maxima that bound |dS| come out of the same reads (V^F from its registers, dO and D as they
// are formed) instead of a second pass over the copies, and dO is not copied where its rows need no padding.  Measured, one launch
// per tensor -> one: training step of 2 heads, L = 256, d = 64 55.4 -> 37.0 us; 12 heads, L = 1560 199 -> 175 us; 4 x 32 heads of
// 8 kv heads, L = 4096 3.22 -> 3.10 ms; inference on 32 heads, L = 777 36.6 -> 30.0 us.
// A workgroup takes 64 positions of one head of one tensor; where a maximum is wanted (V and dO of a backward) it takes the
// head's chunk of them, at most kBoundParts chunks per head, and writes the chunk's maxima; unused chunks are written as 0.
// SRC: 0 Q, K, V in bf16; 1 all three packed (codes and scales); 2 K and V in the pages of the cache.  A forward's attention kernel quantizes Q
// itself: with bf16 Q a forward's launch does no more than copy it, where a result lies over it (32/8 heads, L = 777 causal, inference with O over Q 25.6 us, with the copy as a
// command of its own 28.0; O elsewhere 22.4).
// VQUANT false: V only changes layout (bf16).  BWD: V as bf16 rows with its bound, and the dO / O' part; else V transposed.
template <int SRC, bool VQUANT, bool BWD>
__global__ __launch_bounds__(256) void prep_group_kernel(PrepGroup g, unsigned nblocks)
{
    __shared__ uint16_t tile[BWD ? 1 : 64][128 + 2];
    __shared__ float red[4];
    constexpr bool VF16 = VQUANT && !BWD;
    const int tiles_q = g.Lp / 64, tiles_kv = g.Lp_kv / 64;
    const int per_g = bound_chunk_tiles(tiles_q), nch_g = (tiles_q + per_g - 1) / per_g;        // 64-row tiles per chunk, chunks
    const int per_v = BWD ? bound_chunk_tiles(tiles_kv) : 1, nch_v = (tiles_kv + per_v - 1) / per_v;
    const unsigned n_g = BWD ? (unsigned)g.BHq * nch_g : 0u, n_v = (unsigned)g.BHkv * nch_v;
    constexpr bool QPHI = BWD || SRC == 1;               // phi(Q); else at most a copy of Q
    const unsigned n_q = QPHI ? (unsigned)g.BHq * tiles_q : g.q_out ? (unsigned)(((size_t)g.BHq * g.L + 63) / 64) : 0u;
    for (unsigned blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
        unsigned i = blk;
        float n2 = 0.0f;
        if (BWD && i < n_g) {
            grad_chunk(g.grad, (int)(i / nch_g), (int)(i % nch_g), per_g, nch_g, g.BHq, g.L, g.Lp, g.D, red);
            continue;
        }
        i -= n_g;
        if (i < n_v) {
            const int bh = (int)(i / nch_v), ch = (int)(i % nch_v);
            PagedSrc ps = g.ps;
            ps.which = 1;
            for (int t = ch * per_v; t < min(tiles_kv, (ch + 1) * per_v); ++t)
                prep_tile<VQUANT && SRC == 0, VF16, SRC != 0, SRC == 2, BWD>(tile, bh, t * 64, g.v, g.L_kv, g.Lp_kv, g.D, const_cast<uint8_t*>(g.codes[2]),
                    const_cast<uint8_t*>(g.scales[2]), nullptr, BWD ? g.v_out : nullptr, BWD ? nullptr : g.v_out, nullptr, ps, n2);
            if constexpr (BWD) write_bound(g.grad.bounds + (size_t)bh * kBoundParts, ch, nch_v, sqrtf(wg_max(n2, red)) * 1.0001f);
            else if (gridDim.x < nblocks) __syncthreads();              // the next tile of this workgroup takes the LDS tile
            continue;
        }
        i -= n_v;
        const bool is_q = i < n_q;
        if (!is_q) i -= n_q;
        auto rows = [&](auto k_ops) __attribute__((always_inline)) {      // Q, or a backward's K: rows
            const int per = is_q ? tiles_q : tiles_kv, w = is_q ? 0 : 1;
            prep_tile<SRC != 1, true, SRC == 1, false, false, decltype(k_ops)::value>(tile, (int)(i / per), (int)(i % per) * 64, is_q ? g.q : g.k, is_q ? g.L : g.L_kv, is_q ? g.Lp : g.Lp_kv, g.D,
                const_cast<uint8_t*>(g.codes[w]), const_cast<uint8_t*>(g.scales[w]), nullptr, is_q ? g.q_out : g.k_out, nullptr, is_q ? nullptr : g.k_sub, PagedSrc{}, n2);
        };
        if constexpr (!QPHI) {
            if (is_q) {
                if (g.D == 128) copy_rows64<128>(g.q, g.q_out, (size_t)g.BHq * g.L, i);
                else            copy_rows64<64>(g.q, g.q_out, (size_t)g.BHq * g.L, i);
                continue;
            }
        }
        if (BWD || (SRC == 1 && is_q)) rows(std::false_type{});
        else if constexpr (SRC == 2) {
            PagedSrc ps = g.ps;
            ps.which = 0;
            prep_tile<false, true, true, true, false, true>(tile, (int)(i / tiles_kv), (int)(i % tiles_kv) * 64, nullptr, g.L_kv, g.Lp_kv, g.D, nullptr, nullptr, nullptr,
                g.k_out, nullptr, nullptr, ps, n2);
        } else rows(std::true_type{});
    }
}

int launch_prep_group(const PrepGroup& g, hipStream_t st)
{
    const int tiles_q = g.Lp / 64, tiles_kv = g.Lp_kv / 64;
    const bool bwd = g.grad.d_o != nullptr;
    auto chunks = [](int tiles) { const int per = bound_chunk_tiles(tiles); return (tiles + per - 1) / per; };
    long long n = (long long)g.BHkv * (bwd ? chunks(tiles_kv) : tiles_kv);
    const bool packed = g.codes[2] != nullptr, paged = g.ps.cache != nullptr;
    if (bwd || packed) n += (long long)g.BHq * tiles_q;
    else if (g.q_out) n += ((long long)g.BHq * g.L + 63) / 64;
    if (g.k_out) n += (long long)g.BHkv * tiles_kv;
    if (bwd) n += (long long)g.BHq * chunks(tiles_q);
    if (n > 0x7FFFFFFFLL) return -1;
    const unsigned nblocks = (unsigned)n, grid = min(nblocks, 1u << 22);       // (a grid has fewer than 2^32 threads)
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, st, g, nblocks); };
    if (bwd)          { if (packed) go(prep_group_kernel<1, true, true>); else go(prep_group_kernel<0, true, true>); }
    else if (paged)   go(prep_group_kernel<2, true, false>);
    else if (packed)  go(prep_group_kernel<1, true, false>);
    else if (g.v_quant) go(prep_group_kernel<0, true, false>);
    else              go(prep_group_kernel<0, false, false>);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Writer of the NVFP4 KV cache: phi of n new positions pos0 .. pos0 + n - 1 of one sequence, k and v [Hkv, n, D] bf16, into
// the pages page_ids[pos / 128] (the sequence's page list).  The slots between the last new position and the end of its page
// are cleared (codes and scales 0: they read as zeros until the sequence grows into them).  A page id outside [0, num_pages)
// is left out.  One thread per block of 16 elements, in one pass (a call is as long as its chain of loads); grid (groups of
// 256 blocks, Hkv, 2: K then V).
template <int D>
__global__ __launch_bounds__(256) void kv_page_write_kernel(
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v, int n, int pos0, int Hkv,
    unsigned char* __restrict__ cache, int num_pages, const int* __restrict__ page_ids)
{
    constexpr int nb = D / 16;
    const int h = blockIdx.y, which = blockIdx.z;
    const uint16_t* x = (which ? v : k) + (size_t)h * n * D;
    const int rows_total = ((pos0 + n + 127) & ~127) - pos0;
    const int row = blockIdx.x * (256 / nb) + threadIdx.x / nb, cb = threadIdx.x % nb;
    const int pos = pos0 + min(row, rows_total - 1);
    const int page = page_ids[pos >> 7];
    Nv16 q = nv16_of(0u, 0u, 0u);
    if (row < n) {
        const uint4v* src = reinterpret_cast<const uint4v*>(x + (size_t)row * D + cb * 16);
        const uint4v a = src[0], b = src[1];
        float val[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            val[2 * i]         = __uint_as_float(a[i] << 16);
            val[2 * i + 1]     = __uint_as_float(a[i] & 0xFFFF0000u);
            val[8 + 2 * i]     = __uint_as_float(b[i] << 16);
            val[8 + 2 * i + 1] = __uint_as_float(b[i] & 0xFFFF0000u);
        }
        q = phi_block16_bf16(val);
    }
    // the scale bytes of four neighbouring blocks of a row as one dword (rows beyond the page end take part and write nothing)
    uint32_t sb = q.sc & 0xFFu;
    sb |= lane_down<1>(sb) << 8;
    sb |= lane_down<2>(sb) << 16;
    unsigned char* part = const_cast<unsigned char*>(nvfp4_page_part(cache, page, num_pages, Hkv, h, D, which));
    if (row >= rows_total || !part) return;
    uint2v c2; c2[0] = q.clo; c2[1] = q.chi;
    *reinterpret_cast<uint2v*>(part + (size_t)(pos & 127) * (D / 2) + cb * 8) = c2;
    if ((cb & 3) == 0) *reinterpret_cast<uint32_t*>(part + (size_t)128 * (D / 2) + (size_t)(pos & 127) * nb + cb) = sb;
}

size_t nvfp4_page_bytes(int Hkv, int D) { return (size_t)Hkv * nvfp4_page_head_bytes(D); }

int launch_kv_page_write(const void* k, const void* v, int Hkv, int n, int D, int pos0,
                         void* cache, int num_pages, const int* page_ids, hipStream_t st)
{
    if (Hkv > 65535 || (D != 64 && D != 128) || n < 1 || pos0 < 0) return -1;
    const int rows_total = ((pos0 + n + 127) & ~127) - pos0;
    const int per = 256 / (D / 16);
    dim3 grid((rows_total + per - 1) / per, Hkv, 2);
    if (D == 128) hipLaunchKernelGGL((kv_page_write_kernel<128>), grid, dim3(256), 0, st, (const uint16_t*)k, (const uint16_t*)v, n, pos0, Hkv,
                                     (unsigned char*)cache, num_pages, page_ids);
    else          hipLaunchKernelGGL((kv_page_write_kernel<64>), grid, dim3(256), 0, st, (const uint16_t*)k, (const uint16_t*)v, n, pos0, Hkv,
                                     (unsigned char*)cache, num_pages, page_ids);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Token mean of every channel, for K smoothing: fp64 partial sums of NCHUNK row ranges, then their sum in a fixed
// order, divided by L and rounded to fp32.  Deterministic; x [BH, L, D] bf16.
constexpr int kMeanChunks = 32;
template <int D>
__global__ __launch_bounds__(256) void colsum_partial_kernel(const uint16_t* __restrict__ x, int L, double* __restrict__ part)
{
    constexpr int NS = 256 / D;                       // row slices per block
    __shared__ double red[256];
    const int bh = blockIdx.y, ch = blockIdx.x, c = threadIdx.x % D, sl = threadIdx.x / D;
    const int per = (L + kMeanChunks - 1) / kMeanChunks;
    const int r0 = ch * per, r1 = min(L, r0 + per);
    const uint16_t* src = x + (size_t)bh * L * D + c;
    double acc = 0.0;
    for (int r = r0 + sl; r < r1; r += NS) acc += (double)bf16_to_f32(src[(size_t)r * D]);
    red[threadIdx.x] = acc;
    __syncthreads();
    if (sl == 0) {
        double t = red[c];
#pragma unroll
        for (int i = 1; i < NS; ++i) t += red[i * D + c];
        part[((size_t)bh * kMeanChunks + ch) * D + c] = t;
    }
}
__global__ void colmean_kernel(const double* __restrict__ part, int L, int D, float* __restrict__ mean)
{
    const int bh = blockIdx.x, c = threadIdx.x;
    double t = 0.0;
    for (int ch = 0; ch < kMeanChunks; ++ch) t += part[((size_t)bh * kMeanChunks + ch) * D + c];
    mean[(size_t)bh * D + c] = (float)(t / (double)L);
}

size_t colmean_scratch_bytes(int BH, int D) { return (size_t)BH * kMeanChunks * D * sizeof(double); }

int launch_colmean(const void* x, int BH, int L, int D, double* scratch, float* mean, hipStream_t st)
{
    if (BH > 65535 || (D != 64 && D != 128)) return -1;
    if (D == 128) hipLaunchKernelGGL((colsum_partial_kernel<128>), dim3(kMeanChunks, BH), dim3(256), 0, st, (const uint16_t*)x, L, scratch);
    else          hipLaunchKernelGGL((colsum_partial_kernel<64>), dim3(kMeanChunks, BH), dim3(256), 0, st, (const uint16_t*)x, L, scratch);
    if (hipGetLastError() != hipSuccess) return -1;
    hipLaunchKernelGGL(colmean_kernel, dim3(BH), dim3(D), 0, st, (const double*)scratch, L, D, mean);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_quantize(const void* x, int BH, int L, int D, uint8_t* codes, uint8_t* scales, void* xf, hipStream_t st)
{
    const int Lp = round_up(L, kRowPad);
    hipLaunchKernelGGL(quantize_kernel, dim3(Lp / 64, BH), dim3(256), 0, st, (const uint16_t*)x, L, Lp, D, codes, scales, (uint16_t*)xf);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace aq
