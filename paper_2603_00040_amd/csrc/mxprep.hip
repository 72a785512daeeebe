// What the MX forward and backward prepare, in one launch (see launch_mx_group): phi of Q and K along d, of V along the keys, the
// layouts that the attention kernels read, and the statistics of dO.  Bound by HBM on large problems, by launches on small ones.
#include "common.hpp"
#include "kernels.hpp"
#include "prep.hpp"
#include "mx_quant.hpp"

namespace aq {

// Operand layout of the scaled MFMA for 32 rows (Q, or the keys of a dK/dV wave): ops [rows/32, D/64, 64 lanes, 16 B], sc
// [rows/32, 64 lanes] dwords of scale bytes (byte ks; unused bytes are 1).
template <int D>
__device__ inline void mx_put_operand(unsigned char* __restrict__ ops, unsigned char* __restrict__ sc, int bh, int row, int blk, int Lp, const uint4v& c, uint32_t byte) {
    constexpr int KS = D / 64;
    const int ks = blk >> 1, lane = (blk & 1) * 32 + (row & 31);
    const size_t grp = (size_t)bh * (Lp / 32) + (row >> 5);
    *reinterpret_cast<uint4v*>(ops + ((grp * KS + ks) * 64 + lane) * 16) = c;
    unsigned char* p = sc + (grp * 64 + lane) * 4;
    p[ks] = (unsigned char)byte;
    if (KS == 1) p[1] = 1;
    if (ks == 0) { p[2] = 1; p[3] = 1; }
}

// K records of the training forward and of the dQ pass (16-bit P V, scores on the FP4 instruction): per 64-key tile
// mx_ktrain_rec_bytes(D) bytes = ops [2 blocks of 32 keys][D/64][64 lanes][16 B] with the keys of a block in their natural order as
// operand rows (so that the score tile has the accumulator layout of the 16-bit kernels), then per lane one dword of scale bytes
// (byte = block * D/64 + ks), padded to a whole KiB.
template <int D>
__device__ inline void mx_put_krec(unsigned char* __restrict__ recs, int bh, int row, int blk, int Lp, const uint4v& c, uint32_t byte) {
    constexpr int KS = D / 64, REC = mx_ktrain_rec_bytes(D), KOPS = 2 * KS * 1024;
    const int kk = row & 63, kb = kk >> 5, ks = blk >> 1, lane = (blk & 1) * 32 + (kk & 31);
    unsigned char* rec = recs + ((size_t)bh * (Lp / 64) + (row >> 6)) * REC;
    *reinterpret_cast<uint4v*>(rec + ((kb * KS + ks) * 64 + lane) * 16) = c;
    rec[KOPS + lane * 4 + kb * KS + ks] = (unsigned char)byte;
    if (KS == 1 && kb == 0) { rec[KOPS + lane * 4 + 2] = 1; rec[KOPS + lane * 4 + 3] = 1; }
}

// K part of the kv records of the inference forward.
template <int D, bool FP8V>
__device__ inline void mx_put_kv_k(unsigned char* __restrict__ base, const int* __restrict__ page_ids, int num_pages, int bh, int nheads, int row, int blk, int Lp, const uint4v& c, uint32_t byte) {
    constexpr int NB = D / 32, KS = D / 64, REC = mx_rec_bytes(D, FP8V), KOPS = 2 * KS * 1024, VOPS = NB * (FP8V ? 2048 : 1024);
    const int kk = row & 63, t = (kk >> 4) & 1, ks = blk >> 1, lane = (blk & 1) * 32 + mx_srow_of_key(kk);
    unsigned char* rec = mx_record_of(base, page_ids, num_pages, bh, nheads, Lp, row >> 6, REC);
    if (!rec) return;
    *reinterpret_cast<uint4v*>(rec + ((t * KS + ks) * 64 + lane) * 16) = c;
    rec[KOPS + VOPS + lane * 4 + t * KS + ks] = (unsigned char)byte;
    if (KS == 1 && t == 0) { rec[KOPS + VOPS + lane * 4 + 2] = 1; rec[KOPS + VOPS + lane * 4 + 3] = 1; }
}

// V part: codes of (block kb of 32 keys, d index dd).  FP8: two 1 KiB halves per d-block, bytes 0-15 and 16-31 of every lane.
template <int D, bool FP8V>
__device__ inline void mx_put_kv_v(unsigned char* __restrict__ rec, int kb, int dd, const uint32_t (&c)[8], uint32_t byte) {
    constexpr int KS = D / 64, MT = D / 32, KOPS = 2 * KS * 1024, VOPS = MT * (FP8V ? 2048 : 1024);
    const int lane = kb * 32 + (dd & 31), mt = dd >> 5;
    if constexpr (FP8V) {
        // FP8 operands: registers 0-3 of lane (row, h) are contraction indices 16 h .. + 15, registers 4-7 are
        // 32 + 16 h .. + 15, and the scale of indices 32 b .. + 31 is taken from lane (row, b): the two halves of
        // this block of 32 keys go to the two lane halves, in the register group of the block
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint4v o; o[0] = c[4 * i]; o[1] = c[4 * i + 1]; o[2] = c[4 * i + 2]; o[3] = c[4 * i + 3];
            *reinterpret_cast<uint4v*>(rec + KOPS + ((mt * 2 + kb) * 64 + i * 32 + (dd & 31)) * 16) = o;
        }
    } else {
        uint4v o; o[0] = c[0]; o[1] = c[1]; o[2] = c[2]; o[3] = c[3];
        *reinterpret_cast<uint4v*>(rec + KOPS + (mt * 64 + lane) * 16) = o;
    }
    unsigned char* p = rec + KOPS + VOPS + 256 + lane * 4;
    p[mt] = (unsigned char)byte;
    if (MT == 2 && mt == 0) { p[2] = 1; p[3] = 1; }
}

// 64 positions of V, by one workgroup.  They come into LDS as 16-byte pieces of rows, a thread then takes a column of 32 (reading
// the column from memory, two bytes per lane and load, ran at a third of the bandwidth: 117 us for 24 heads, L = 32768 against 44 us
// for K).
template <int D, MxKind KIND>
__device__ __forceinline__ void mx_v_tile(uint16_t (*tile)[D + 2], const MxGroup& g, int bh, int t, float& n2)
{
    constexpr int CH = D / 8;                       // 16-byte pieces per row
    const int l0 = t * 64, L = g.L, Lp = g.Lp;
    const bool aligned = ((uintptr_t)g.v & 15) == 0;          // (V may lie at any address of a 16-bit value)
    for (int i = threadIdx.x; i < 64 * CH; i += 256) {
        const int row = i / CH, c = i % CH;
        uint4v a = {0u, 0u, 0u, 0u};
        if (l0 + row < L) {
            const uint16_t* src = g.v + ((size_t)bh * L + l0 + row) * D + 8 * c;
            if (aligned) a = *reinterpret_cast<const uint4v*>(src);
            else
#pragma unroll
                for (int j = 0; j < 4; ++j) a[j] = (uint32_t)src[2 * j] | ((uint32_t)src[2 * j + 1] << 16);
        }
        uint32_t* dst = reinterpret_cast<uint32_t*>(&tile[row][8 * c]);       // (rows are 4-byte aligned: D + 2 values)
#pragma unroll
        for (int j = 0; j < 4; ++j) dst[j] = a[j];
    }
    __syncthreads();
    if (threadIdx.x < 2 * D) {
        const int dd = threadIdx.x % D, kb = threadIdx.x / D;
        float v[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = bf16_to_f32(tile[kb * 32 + i][dd]);
        uint32_t byte, c[8];
        mx_block_codes<KIND == MX_INFER_FP8V>(v, byte, c);
        if constexpr (KIND == MX_INFER || KIND == MX_INFER_FP8V) {
            unsigned char* rec = mx_record_of(g.kv, g.page_ids, g.num_pages, bh, g.BHkv, Lp, t, mx_rec_bytes(D, KIND == MX_INFER_FP8V));
            if (rec) mx_put_kv_v<D, KIND == MX_INFER_FP8V>(rec, kb, dd, c, byte);
        } else {
            const uint4v c4 = {c[0], c[1], c[2], c[3]};
            const float s = e8m0_as_f32(byte);
            if constexpr (KIND == MX_TRAIN) {
                // transposed, in the order of the forward's operands: quads 1 and 2 of a group of 16 positions exchanged
                uint32_t o[16];
                mx_dequant32(c4, s, [&](int i, float lo, float hi) { o[i] = pack_f16x2(lo, hi); });
                uint16_t* dst = g.v_out + (size_t)bh * D * Lp;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint4v a, b;
                    a[0] = o[8 * h]; a[1] = o[8 * h + 1]; a[2] = o[8 * h + 4]; a[3] = o[8 * h + 5];
                    b[0] = o[8 * h + 2]; b[1] = o[8 * h + 3]; b[2] = o[8 * h + 6]; b[3] = o[8 * h + 7];
                    *reinterpret_cast<uint4v*>(dst + v_operand_offset((l0 >> 4) + 2 * kb + h, dd, 0, D)) = a;
                    *reinterpret_cast<uint4v*>(dst + v_operand_offset((l0 >> 4) + 2 * kb + h, dd, 1, D)) = b;
                }
            } else {
                mx_dequant32(c4, s, [&](int i, float lo, float hi) {
                    tile[kb * 32 + 2 * i][dd] = f32_to_bf16_rne(lo);
                    tile[kb * 32 + 2 * i + 1][dd] = f32_to_bf16_rne(hi);
                });
            }
        }
    }
    __syncthreads();
    if constexpr (KIND == MX_BWD) {
        for (int i = threadIdx.x; i < 64 * CH; i += 256) {
            const int row = i / CH, c = i % CH;
            const uint32_t* src = reinterpret_cast<const uint32_t*>(&tile[row][8 * c]);
            uint4v a;
            float acc = 0.0f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                a[j] = src[j];
                const float lo = __uint_as_float(a[j] << 16), hi = __uint_as_float(a[j] & 0xFFFF0000u);
                acc = fmaf(lo, lo, fmaf(hi, hi, acc));
            }
            acc = lanes_sum<CH / 2, 1>(acc);
            n2 = fmaxf(n2, acc);
            *reinterpret_cast<uint4v*>(g.v_out + ((size_t)bh * Lp + l0 + row) * D + 8 * c) = a;
        }
        __syncthreads();
    }
}

__device__ inline void mx_put_row16(uint16_t* __restrict__ rows, size_t row, int D, int blk, const uint4v& c, uint32_t byte) {
    uint32_t o[16];
    mx_dequant32(c, e8m0_as_f32(byte), [&](int i, float lo, float hi) { o[i] = pack_f16x2(lo, hi); });
    uint4v* dst = reinterpret_cast<uint4v*>(rows + row * D + blk * 32);
#pragma unroll
    for (int j = 0; j < 4; ++j) { uint4v w; w[0] = o[4 * j]; w[1] = o[4 * j + 1]; w[2] = o[4 * j + 2]; w[3] = o[4 * j + 3]; dst[j] = w; }
}

// Row r = (b * Hq + h) * nqb + query block of the mask [rows, nkb] (bytes, zero = the block is left out) -> the indices of its
// non-zero key blocks in increasing order, and their number.  One wave per row, 64 blocks at a time (one thread per row walked
// 64 bytes one after another: 12.8 us for 32 heads, L = 8192, more than all of phi(Q)).
__device__ inline void mx_block_list(const unsigned char* __restrict__ mask, int r, int nkb, int* __restrict__ list, int* __restrict__ count) {
    const int lane = threadIdx.x & 63;
    int n = 0;
    for (int k0 = 0; k0 < nkb; k0 += 64) {
        const bool on = k0 + lane < nkb && mask[(size_t)r * nkb + k0 + lane] != 0;
        const unsigned long long all = __builtin_amdgcn_ballot_w64(on);
        if (on) list[(size_t)r * nkb + n + __popcll(all & ((1ull << lane) - 1ull))] = k0 + lane;
        n += __popcll(all);
    }
    if (lane == 0) count[r] = n;
}

// A workgroup takes 64 positions of V (in a backward the chunk of a head's 64-row tiles that one partial maximum covers), 256 blocks
// of 32 values of Q or K, 64 rows of Q to copy (training forward), four rows of the mask, or a chunk of dO.
// (five wavefronts per SIMD: the loads of a backward's dO and O' together would otherwise take 101 registers, one wavefront less)
template <int D, MxKind KIND>
__global__ __launch_bounds__(256, 5) void mx_group_kernel(MxGroup g, unsigned nblocks)
{
    constexpr int NB = D / 32, RW = 256 / NB;       // blocks per row, rows of Q or K per workgroup
    __shared__ uint16_t tile[64][D + 2];
    __shared__ float red[4];
    const int tiles = g.Lp / 64, per = KIND == MX_BWD ? bound_chunk_tiles(tiles) : 1, nch = (tiles + per - 1) / per;
    const unsigned n_g = KIND == MX_BWD ? (unsigned)g.BHq * nch : 0u, n_v = g.v ? (unsigned)g.BHkv * nch : 0u;
    const unsigned per_qk = (unsigned)(g.Lp / RW), n_k = g.k ? (unsigned)g.BHkv * per_qk : 0u;
    const unsigned n_q = !g.q ? 0u : KIND == MX_TRAIN ? (unsigned)(((size_t)g.BHq * g.L + 63) / 64) : (unsigned)g.BHq * per_qk;
    for (unsigned b = blockIdx.x; b < nblocks; b += gridDim.x) {
        unsigned i = b;
        if (KIND == MX_BWD && i < n_g) {
            grad_chunk(g.grad, (int)(i / nch), (int)(i % nch), per, nch, g.BHq, g.L, g.Lp, D, red);
            continue;
        }
        i -= n_g;
        if (i < n_v) {
            const int bh = (int)(i / nch), ch = (int)(i % nch);
            float n2 = 0.0f;
            for (int t = ch * per; t < min(tiles, (ch + 1) * per); ++t) mx_v_tile<D, KIND>(tile, g, bh, t, n2);
            if constexpr (KIND == MX_BWD) write_bound(g.grad.bounds + (size_t)bh * kBoundParts, ch, nch, sqrtf(wg_max(n2, red)) * 1.0001f);
            continue;
        }
        i -= n_v;
        if (i < n_q + n_k) {
            const bool is_q = i < n_q;
            if constexpr (KIND == MX_TRAIN) {
                if (is_q) {
                    copy_rows64<D>(g.q, g.q_row, (size_t)g.BHq * g.L, i);
                    continue;
                }
            }
            if (!is_q) i -= n_q;
            const int bh = (int)(i / per_qk), row = (int)(i % per_qk) * RW + threadIdx.x / NB, blk = threadIdx.x % NB;
            uint32_t byte;
            const uint4v c = mx_block_of_row<D>(is_q ? g.q : g.k, bh, row, blk, g.L, byte);
            if (KIND != MX_TRAIN && is_q) mx_put_operand<D>(g.qops, g.qsc, bh, row, blk, g.Lp, c, byte);
            else if (KIND == MX_TRAIN || KIND == MX_BWD) mx_put_krec<D>(g.krec, bh, row, blk, g.Lp, c, byte);
            else mx_put_kv_k<D, KIND == MX_INFER_FP8V>(g.kv, g.page_ids, g.num_pages, bh, g.BHkv, row, blk, g.Lp, c, byte);
            if constexpr (KIND == MX_BWD) {
                if (!is_q) mx_put_operand<D>(g.kops, g.ksc, bh, row, blk, g.Lp, c, byte);
                mx_put_row16(is_q ? g.q_row : g.k_row, (size_t)bh * g.Lp + row, D, blk, c, byte);
            }
            continue;
        }
        if constexpr (KIND == MX_INFER) {
            const int nb = g.Lp / 128, r = (int)(i - n_q - n_k) * 4 + (threadIdx.x >> 6);
            if (r < g.BHq * nb) mx_block_list(g.mask, r, nb, g.list, g.list_count);
        }
    }
}

// Q alone (serving: K and V are in the cache): the group kernel's larger frame costs a decode step 1 us.  A head of at most 32 rows has
// one group of 32 (the decode kernel reads no other).  blockIdx.y is the head: with several heads in a workgroup the division by a
// head's blocks cost 0.3 us of 22 (7 sequences of 4 heads, d = 64).
template <int D>
__global__ __launch_bounds__(256) void mx_q_kernel(const uint16_t* __restrict__ q, unsigned char* __restrict__ qops, unsigned char* __restrict__ qsc,
                                                   int L, int Lp)
{
    constexpr int NB = D / 32;
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x), bh = (int)blockIdx.y, row = i / NB, blk = i % NB;
    uint32_t byte;
    const uint4v c = mx_block_of_row<D>(q, bh, row, blk, L, byte);
    mx_put_operand<D>(qops, qsc, bh, row, blk, Lp, c, byte);
}

int launch_mx_group(const MxGroup& g, MxKind kind, int D, hipStream_t st)
{
    if (D != 64 && D != 128) return -1;
    if (kind == MX_INFER && g.q && !g.k && !g.v && !g.mask) {
        // (the blocks of a head's rows, 32 or a multiple of 128 of them, fill whole workgroups; check_dims limits the heads to 65535)
        const unsigned n = (unsigned)(g.L <= 32 ? 32 : g.Lp) * (D / 32), block = n < 256 ? n : 256;
        const dim3 grid(n / block, (unsigned)g.BHq);
        if (D == 128) hipLaunchKernelGGL(mx_q_kernel<128>, grid, dim3(block), 0, st, g.q, g.qops, g.qsc, g.L, g.Lp);
        else          hipLaunchKernelGGL(mx_q_kernel<64>, grid, dim3(block), 0, st, g.q, g.qops, g.qsc, g.L, g.Lp);
        return hipGetLastError() == hipSuccess ? 0 : -1;
    }
    const int tiles = g.Lp / 64, per = kind == MX_BWD ? bound_chunk_tiles(tiles) : 1, nch = (tiles + per - 1) / per, per_qk = g.Lp / (256 / (D / 32));
    long long n = (kind == MX_BWD ? (long long)g.BHq * nch : 0) + (g.v ? (long long)g.BHkv * nch : 0) + (!g.q ? 0 : kind == MX_TRAIN ? ((long long)g.BHq * g.L + 63) / 64 : (long long)g.BHq * per_qk) + (g.k ? (long long)g.BHkv * per_qk : 0);
    if (g.mask) n += ((long long)g.BHq * (g.Lp / 128) + 3) / 4;
    if (n < 1 || n > 0x7FFFFFFFLL || (g.mask && kind != MX_INFER) || (g.page_ids && kind != MX_INFER)) return -1;
    const unsigned nblocks = (unsigned)n, grid = min(nblocks, 1u << 22);       // (a grid has fewer than 2^32 threads)
#define AQ_G(KIND) do { if (D == 128) hipLaunchKernelGGL((mx_group_kernel<128, KIND>), dim3(grid), dim3(256), 0, st, g, nblocks); \
                        else hipLaunchKernelGGL((mx_group_kernel<64, KIND>), dim3(grid), dim3(256), 0, st, g, nblocks); } while (0)
    if (kind == MX_INFER) AQ_G(MX_INFER);
    else if (kind == MX_INFER_FP8V) AQ_G(MX_INFER_FP8V);
    else if (kind == MX_TRAIN) AQ_G(MX_TRAIN);
    else AQ_G(MX_BWD);
#undef AQ_G
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace aq
