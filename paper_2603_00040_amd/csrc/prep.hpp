// The part of the backward's preparation that does not depend on the format of Q, K and V (device code shared by prep.hip and
// mxprep.hip).
#pragma once
#include "common.hpp"
#include "kernels.hpp"

namespace aq {

// 64-row tiles per chunk of the partial maxima: at most kBoundParts chunks per head.
__host__ __device__ inline int bound_chunk_tiles(int tiles) { return (tiles + kBoundParts - 1) / kBoundParts; }

// The statistics that the backward needs of 64 rows of dO and O' (Alg. 3, first line): rowstat = {L log2(e), D} with
// D = rowsum(dO o O') (padding rows hold {0, 0}), the largest |dO_i|^2 and |D_i| / sqrt(d) so far in n2 and dmax, and the zero-padded
// copy of dO where one is asked for (dob).  D is added up eight elements at a time (pairs 0, 2, 1, 3 of them), then over the groups of
// eight in a tree whose last level joins neighbours: which order the sum has is part of the result's bits, so the two groups of a
// thread stay apart until the end.
template <int D>
__device__ __forceinline__ void grad_tile(int bh, int l0, const uint16_t* __restrict__ dO, const void* __restrict__ o_acc, bool o_is_bf16,
                                          const float* __restrict__ lse, int L, int Lp, float rs,
                                          float2* __restrict__ rowstat, uint16_t* __restrict__ dob, float& n2, float& dmax)
{
    constexpr int nb = D / 16, NI = nb / 4;        // blocks of 16 elements per row, and of the 64 rows per thread
    // (opaque: the addresses of every variant would otherwise be formed in front of the loop over tiles and held in registers)
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int cb = (int)(tid % nb), row0 = (int)(tid / nb);
    // the loads of all blocks of a thread first: one trip to memory instead of one per block
    uint4v g_[NI][2] = {};
    floatx4 w_[NI][4] = {};
    float lse_[NI] = {};
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const int l = l0 + row0 + it * (256 / nb);
        if (l < L) {
            const size_t off = ((size_t)bh * L + l) * D + cb * 16;
            g_[it][0] = reinterpret_cast<const uint4v*>(dO + off)[0];
            g_[it][1] = reinterpret_cast<const uint4v*>(dO + off)[1];
            if (o_is_bf16) {                       // ablation: D from the low-precision output
#pragma unroll
                for (int t = 0; t < 2; ++t) w_[it][t] = reinterpret_cast<const floatx4*>(static_cast<const uint16_t*>(o_acc) + off)[t];
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) w_[it][t] = reinterpret_cast<const floatx4*>(static_cast<const float*>(o_acc) + off)[t];
            }
            if (cb == 0) lse_[it] = lse[(size_t)bh * L + l];
        }
    }
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        __builtin_amdgcn_sched_barrier(0);         // (one block after the other: the registers of two at once would cost wavefronts)
        const int l = l0 + row0 + it * (256 / nb);
        const uint4v (&g)[2] = g_[it];
        float dot8[2] = {0.0f, 0.0f}, nrm = 0.0f;
        if (l < L) {
            float o[16];
            if (o_is_bf16) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t w = __float_as_uint(w_[it][t][i]);
                        o[8 * t + 2 * i] = __uint_as_float(w << 16); o[8 * t + 2 * i + 1] = __uint_as_float(w & 0xFFFF0000u);
                    }
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[4 * t + i] = w_[it][t][i];
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                float lo[4], hi[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    lo[i] = __uint_as_float(g[t][i] << 16); hi[i] = __uint_as_float(g[t][i] & 0xFFFF0000u);
                    nrm = fmaf(lo[i], lo[i], fmaf(hi[i], hi[i], nrm));
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    dot8[t] += lo[i] * o[8 * t + 2 * i] + hi[i] * o[8 * t + 2 * i + 1];
                    dot8[t] += lo[2 + i] * o[8 * t + 4 + 2 * i] + hi[2 + i] * o[8 * t + 5 + 2 * i];
                }
            }
        }
        dot8[0] = lanes_sum<nb / 2, 1>(dot8[0]); dot8[1] = lanes_sum<nb / 2, 1>(dot8[1]); nrm = lanes_sum<nb / 2, 1>(nrm);
        const float dot = dot8[0] + dot8[1];
        if (cb == 0) rowstat[(size_t)bh * Lp + l] = make_float2(l < L ? lse_[it] * 1.4426950408889634f : 0.0f, dot);
        n2 = fmaxf(n2, nrm);
        dmax = fmaxf(dmax, fabsf(dot * rs));
        if (dob) {
            uint4v* dst = reinterpret_cast<uint4v*>(dob + ((size_t)bh * Lp + l) * D + cb * 16);
            dst[0] = g[0]; dst[1] = g[1];
        }
    }
}

// Copies rows 64 i .. of Q [rows, D] as they are: a forward whose results lie over Q reads this copy.
template <int D>
__device__ __forceinline__ void copy_rows64(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, size_t rows, size_t i)
{
    const uint4v* s = reinterpret_cast<const uint4v*>(src) + i * (64 * D / 8);
    uint4v* d = reinterpret_cast<uint4v*>(dst) + i * (64 * D / 8);
    const uint32_t n = (uint32_t)min((size_t)64, rows - 64 * i) * (D / 8);
#pragma unroll
    for (int p = 0; p < 64 * D / 8; p += 256)
        if (p + threadIdx.x < n) d[p + threadIdx.x] = s[p + threadIdx.x];
}

// Largest value of a workgroup; every thread gets it.  (The barriers also keep `red` from being overwritten too early.)
__device__ inline float wg_max(float v, float (&red)[4]) {
    v = lanes_max<32, 1>(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// Partial maximum `ch` of a head (nch of them); the unused ones are written as 0.  All threads hold the value.
__device__ inline void write_bound(float* part, int ch, int nch, float value) {
    if (threadIdx.x == 0) part[ch] = value;
    if (ch == 0 && (int)threadIdx.x >= nch && threadIdx.x < kBoundParts) part[threadIdx.x] = 0.0f;
}

// Chunk ch (of nch, `per` tiles of 64 rows each) of query head bh.
__device__ __forceinline__ void grad_chunk(const GradArgs& a, int bh, int ch, int per, int nch, int BHq, int L, int Lp, int D, float (&red)[4]) {
    float n2 = 0.0f, dmax = 0.0f;
    for (int t = ch * per; t < min(Lp / 64, (ch + 1) * per); ++t)
        if (D == 128) grad_tile<128>(bh, t * 64, a.d_o, a.o_acc, a.o_is_bf16, a.lse, L, Lp, a.rs, a.rowstat, a.dob, n2, dmax);
        else          grad_tile<64>(bh, t * 64, a.d_o, a.o_acc, a.o_is_bf16, a.lse, L, Lp, a.rs, a.rowstat, a.dob, n2, dmax);
    write_bound(a.bounds + ((size_t)BHq + bh) * kBoundParts, ch, nch, sqrtf(wg_max(n2, red)) * 1.0001f);      // rounded up a little: it is an upper bound
    write_bound(a.bounds + ((size_t)2 * BHq + bh) * kBoundParts, ch, nch, wg_max(dmax, red));
}

}  // namespace aq
