// Backward of Attn-QAT on gfx950 (Alg. 3), as two kernels behind the preparing one (prep_group_kernel: the copies of
// Q, K, V and dO, D = rowsum(dO o O') and the per-row {L, D} pairs, per-head maxima of |dO_i|, |V^F_j| and |D_i|):
//   bwd_dq     query-stationary: S, P, dP, dS, dQ += dS K^F
//   bwd_dkdv   key-stationary:   S, P, P^F, dP, dS, dV += P^F^T dO, dK += dS^T Q^F
// The paper's single loop nest accumulates dQ across key tiles; here dQ gets its own pass
// that recomputes S and dP instead of accumulating across workgroups with atomics (the
// two-pass form of the Triton tutorial kernel the paper extends), which keeps every
// output deterministic.
//
// MFMA: v_mfma_f32_32x32x16_{f16,bf16}.  Q^F, K^F, V^F and P^F are exact in both 16-bit
// formats and dO is bf16 input, so S (fp16 operands), dP and dV (bf16 operands) see exact
// operands.  dS is fp32 and the only rounded operand: it enters its two products (with K^F
// and with Q^F, both fp16) as fp16, 11 significant bits, after multiplication by a power of
// two chosen from an upper bound of |dS| so that nothing overflows and the values that matter
// stay clear of the subnormals:
//     |dS_ij| = P_ij |dP_ij - D_i| / sqrt(d) <= (|dO_i| max_j |V^F_j| + |D_i|) / sqrt(d)
// (P <= 1, Cauchy-Schwarz).  The dQ pass scales per query row, the dK/dV pass per kv head; the
// accumulators are divided by the same power of two at the end.  A single bf16 (8 bits)
// would by itself cost about 1.7e-3 relative L2 in dQ and dK.
//
// As in the forward, S and dP are computed transposed ([key, query]) so that a lane owns
// one query row: L_i, D_i are per-lane scalars and the 16-key blocks of phi(P) are
// register reductions plus one exchange between the 32-lane halves.  Tiles are copied
// global->LDS directly (XOR-swizzled rows); operands that a product needs transposed
// (K^T for dQ; Q and dO column-wise, P^F^T and dS^T for dK/dV) are read from the row-major
// tiles with the LDS transpose read, so no transposed copy exists anywhere.
//
// LDS reads are the scarce resource of these loops (one wave sustains about one 1 KiB read
// per 40 cycles, latency ~130 cycles), so every operand read is issued a few MFMAs ahead of
// its consumer and the scheduling groups pin that order.
#include <type_traits>
#include "common.hpp"
#include "kernels.hpp"

namespace aq {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
    bf16x2 h; h[0] = (__bf16)lo; h[1] = (__bf16)hi;              // RNE
    return __builtin_bit_cast(uint32_t, h);
}
__device__ inline float bf16_lo_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi_f32(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ inline floatx16 mfma_bf16(uint4v a, uint4v b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ inline floatx16 mfma_f16(uint4v a, uint4v b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
}
// Largest power of two <= kDsTop / bound (bound >= 0), kept inside [2^-60, 2^60]: the factor that dS
// is multiplied by before it is rounded to fp16.
constexpr float kDsTop = 49152.0f;
__device__ inline float ds_scale_for(float bound) {
    float t = kDsTop / fmaxf(bound, 1e-30f);
    t = fminf(fmaxf(t, 8.7e-19f), 1.15e18f);
    return __uint_as_float(__float_as_uint(t) & 0x7F800000u);
}
__device__ inline uint4v join(uint2v a, uint2v b) { uint4v r; r[0] = a[0]; r[1] = a[1]; r[2] = b[0]; r[3] = b[1]; return r; }

// One of the three maxima of a head: every lane gets the maximum of the head's partial values.
__device__ inline float bound_of(const float* __restrict__ part, int NHq, int which, int head) {
    float v = part[((size_t)which * NHq + head) * kBoundParts + (threadIdx.x & 63)];
    return lanes_max<32, 1>(v);
}

// ---- what the kernels of both passes share
// Largest P of group gq (16 keys) in this lane, of its 8 values of them.
__device__ __forceinline__ float nvfp4_group_max(const floatx16& s, int gq) {
    const float a0 = fmaxf(fmaxf(s[8 * gq], s[8 * gq + 1]), s[8 * gq + 2]), a1 = fmaxf(fmaxf(s[8 * gq + 3], s[8 * gq + 4]), s[8 * gq + 5]);
    return fmaxf(fmaxf(a0, a1), fmaxf(s[8 * gq + 6], s[8 * gq + 7]));
}
// Does a largest P of amax ask for products with P^F?  RNE_E4M3(amax / 6) is zero exactly when amax / 6 <= 2^-10 (half of the smallest
// subnormal, and the tie goes to the even neighbour, zero), and it grows with amax: some block of a tile has a non-zero scale iff some
// lane's largest P passes this test.  (The product is rounded to fp32 here and not in nvfp4_pair_scales: at the one P where they differ, 6 * 2^-10 itself, a
// tile is left out if no larger one is in it.)
__device__ __forceinline__ bool nvfp4_scale_nonzero(float amax) { return amax * (1.0f / 6.0f) > 0.0009765625f; }
// Block scales of phi(P) of the two groups, and their reciprocals.  Each half of the wave forms the scale of one group and hands it to the other, as in
// the forward (P <= 1: no saturation; a scale of 0 leaves any finite factor).  A scale is RNE_E4M3 of the unrounded product of the largest P with fp32's 1/6; the forward
// rounds that product to fp32 first, which differs at ties of the grid only.  (The hardware conversion would round it first here too, in three
// instructions instead of six: training step of 4 x 32/8 heads, L = 4096 causal 2800 us instead of 2813, but dV moves by 1e-4 of its norm.)
__device__ __forceinline__ void nvfp4_pair_scales(const float (&gmax)[2], float (&sc)[2], float (&inv)[2]) {
    const float own = rne_e4m3_grid_of_product(xhalf_max_pair(gmax[0], gmax[1]), 1.0f / 6.0f), r = fminf(__builtin_amdgcn_rcpf(own), 512.0f);
    const auto sb = __builtin_amdgcn_permlane32_swap(__float_as_uint(own), __float_as_uint(own), false, false);
    const auto ib = __builtin_amdgcn_permlane32_swap(__float_as_uint(r), __float_as_uint(r), false, false);
#pragma unroll
    for (int gq = 0; gq < 2; ++gq) { sc[gq] = __uint_as_float(sb[gq]); inv[gq] = __uint_as_float(ib[gq]); }
}
// phi^-1(phi(P)) of registers r0 .. r0 + 3 as bf16.
__device__ __forceinline__ uint2v nvfp4_pf_quad(const floatx16& s, int r0, float sc, float inv) {
    typedef float float2v __attribute__((ext_vector_type(2)));
    uint2v w;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const uint32_t codes = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(any_register(), s[r0 + 2 * u] * inv, s[r0 + 2 * u + 1] * inv, 1.0f, 0);
        const float2v q = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(codes, 1.0f, 0);
        w[u] = pack_bf16x2(q[0] * sc, q[1] * sc);
    }
    return w;
}
// The dQ pass: dS of a row goes to fp16 after multiplication by ds_scale = 2^k, k from the bound (|dO_i| max_j |V^F_j| + |D_i|) / sqrt(d) >= |dS_ij|.
// FOLD: the dO operand of the row is multiplied by 2^k, exactly, so that no rounding depends on the scale of the gradients (in the exponent of P it
// cost up to 1 % of dQ's error at |dO| = 2^-40); where that would leave the range of bf16 (V^F next to zero, |dO| beyond 2^40), it goes
// into the exponent (dq_row_exponent), and do_scale is 1.
template <bool FOLD, int DS>
__device__ __forceinline__ void dq_row_scale(uint4v (&doreg)[DS], float vmax, float Di, float rs, float& ds_scale, float& do_scale) {
    float n2 = 0.0f;
#pragma unroll
    for (int ds = 0; ds < DS; ++ds)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float lo = bf16_lo_f32(doreg[ds][i]), hi = bf16_hi_f32(doreg[ds][i]);
            n2 = fmaf(lo, lo, fmaf(hi, hi, n2));
        }
    n2 = xhalf_sum(n2);
    ds_scale = ds_scale_for((sqrtf(n2) * 1.0001f * vmax) * rs + fabsf(Di * rs));
    do_scale = 1.0f;
    if constexpr (FOLD) {
        if (sqrtf(n2) * ds_scale < 1e30f) do_scale = ds_scale;
#pragma unroll
        for (int ds = 0; ds < DS; ++ds)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                doreg[ds][i] = __builtin_amdgcn_perm(__float_as_uint(bf16_hi_f32(doreg[ds][i]) * do_scale), __float_as_uint(bf16_lo_f32(doreg[ds][i]) * do_scale), 0x07060302u);
    }
}
// L_i log2(e) - log2(1 / sqrt(d))  (3.5 and 3 are exact), and the part of k that dO does not carry
template <int D>
__device__ __forceinline__ float dq_row_exponent(float Llog2e, float ds_scale, float do_scale) {
    return Llog2e - ((float)((int)(__float_as_uint(ds_scale / do_scale) >> 23) - 127) - (D == 128 ? 3.5f : 3.0f));
}

static int g_bwd_waves = 0;           // waves per workgroup of the dQ and dK/dV passes, 0: chosen per problem; 4 / 8: forced (tests)
void set_bwd_waves(int waves) { __atomic_store_n(&g_bwd_waves, waves, __ATOMIC_RELAXED); }

// ------------------------------------------------------------------ dQ pass
template <int D, bool MXS>
struct DqSmem {
    uint16_t k[2][64 * D];       // K^F tile [key][d], fp16, swizzled
    uint16_t v[2][64 * D];       // V^F tile [key][d], bf16, swizzled
    unsigned char krec[MXS ? 2 : 1][MXS ? mx_ktrain_rec_bytes(D) : 16];      // MX: K operands of the FP4 instruction and their scales
};

typedef int int8v_t __attribute__((ext_vector_type(8)));
__device__ inline int8v_t fp4_opnd(const uint4v& x) {
    int8v_t r = {(int)x[0], (int)x[1], (int)x[2], (int)x[3], 0, 0, 0, 0};
    return r;
}

// MXS (the MX format): S^T = K^F Q^F^T is recomputed from the E2M1 codes and E8M0 scales by v_mfma_scale_f32_32x32x64_f8f6f4
// (Qops / Qsc: operands and scale dwords of the query rows; Krec: the K records in natural key order; see launch_mx_group); the
// accumulator layout is that of the 16-bit products, and dP, dS and dQ are computed as before (dO, dS are 16-bit values).
// NW waves of 32 query rows each share the K / V tiles: 4, or 8 for the passes of a large problem (half the
// tile copies per query row).
struct DqArgs {
    const uint16_t *Qb, *Kb, *Vb, *dOb;
    const float2* rowstat; const float* bound_part; uint16_t* dQ;
    int L, Lp, Hq, G, NHq; float c /* log2e/sqrt(d) */, rs /* 1/sqrt(d) */;
    const unsigned char* Qops; const uint32_t* Qsc; const unsigned char* Krec;
};
template <int D, bool CAUSAL, bool MXS, int NW>
__device__ __forceinline__ void bwd_dq_body(const DqArgs& A, int bh, int qt)
{
    constexpr int DS = D / 16, MB = D / 32, KCH = D / 8, KLD = KCH / NW, QT = 32 * NW /* query rows of a workgroup */;
    constexpr int KSM = D / 64, KREC = mx_ktrain_rec_bytes(D);
    // 32-key blocks of a tile whose S and dP are computed at a time.  One, where that brings the registers down to those of three
    // wavefronts per SIMD (d = 64; both blocks of d = 64 in MX fit as they are): with two, every wavefront waits for its own chains
    // of products and exponentials.  2 x 16/4 heads, L = 3001, d = 64 causal, training step 312 -> 290 us, MX 266.6 -> 263.5 us; 12 heads,
    // L = 2000, where there are no three workgroups per compute unit, 127 us as before.
    constexpr int KH = D == 64 && !MXS ? 1 : 2;
    extern __shared__ __align__(256) unsigned char smem_raw[];
    DqSmem<D, MXS>& sm = *reinterpret_cast<DqSmem<D, MXS>*>(smem_raw);
    const uint16_t *__restrict__ Qb = A.Qb, *__restrict__ Kb = A.Kb, *__restrict__ Vb = A.Vb, *__restrict__ dOb = A.dOb;
    const float2* __restrict__ rowstat = A.rowstat;
    const float* __restrict__ bound_part = A.bound_part;
    uint16_t* __restrict__ dQ = A.dQ;
    const unsigned char *__restrict__ Qops = A.Qops, *__restrict__ Krec = A.Krec;
    const uint32_t* __restrict__ Qsc = A.Qsc;
    const int L = A.L, Lp = A.Lp, Hq = A.Hq, G = A.G, NHq = A.NHq;
    const float c = A.c, rs = A.rs;

    const int b = bh / Hq, h = bh % Hq;
    const int bhkv = b * (Hq / G) + h / G;
    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);        // scalar: LDS destinations and branches use it
    const int q_row = qt * QT + wave * 32 + ln;
    const bool wave_live = NW == 4 || qt * QT + wave * 32 < Lp;      // a wave past the padded rows takes part in the copies and barriers only
    const int q_ld = wave_live ? q_row : ln;         // row its loads read instead

    uint4v qreg[MXS ? 1 : DS], doreg[DS], qop[MXS ? KSM : 1];
    uint32_t qs = 0u;
    {
        const size_t off = ((size_t)bh * Lp + q_ld) * D + 8 * hf;
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
            if constexpr (!MXS) qreg[ds] = *reinterpret_cast<const uint4v*>(Qb + off + 16 * ds);
            doreg[ds] = *reinterpret_cast<const uint4v*>(dOb + off + 16 * ds);
        }
        if constexpr (MXS) {
            const size_t grp = (size_t)bh * (Lp / 32) + ((q_ld - ln) >> 5);
#pragma unroll
            for (int ks = 0; ks < KSM; ++ks) qop[ks] = *reinterpret_cast<const uint4v*>(Qops + ((grp * KSM + ks) * 64 + lane) * 16);
            qs = Qsc[grp * 64 + lane];
        }
    }
    const float2 st_ = rowstat[(size_t)bh * Lp + q_ld];
    // FOLD (see dq_row_scale): -2^k D_i is what the accumulators of dP start from, and 1 / sqrt(d) goes into the exponent of P, so that dS is one
    // multiplication (32 of 112 vector instructions of a tile, which add to the time of
    // its 48 products: the same tree otherwise, in turn, 4 x 32/8 heads, L = 4096 causal 2922 -> 2884 us, 40 heads, L = 75600 418.7 ->
    // 416.3 ms, MX 4 x 8/2 heads, L = 3124 759 -> 749 us; MX of d = 128 under a causal mask lost, 2 x 16/4 heads, L = 3001 428.0 -> 429.7 us;
    // d = 64 gains there, 265.8 -> 260.0 us, and without a mask, 2 x 24 heads, L = 3000 633 -> 618 us).
    constexpr bool FOLD = !(MXS && CAUSAL && D == 128);
    float ds_scale, do_scale;
    dq_row_scale<FOLD>(doreg, bound_of(bound_part, NHq, 0, bhkv), st_.y, rs, ds_scale, do_scale);
    const float Ls = FOLD ? dq_row_exponent<D>(st_.x, ds_scale, do_scale) : st_.x;
    const float rs_s = rs * ds_scale, Dq_s = st_.y * rs_s;            // (not FOLD) D_i / sqrt(d), scaled
    floatx16 dp0;                                                    // what dP starts from: -2^k D_i in every register
#pragma unroll
    for (int i = 0; i < 16; ++i) dp0[i] = FOLD ? -st_.y * do_scale : 0.0f;

    const int nkt_all = (L + 63) / 64;
    const int nkt = CAUSAL ? min((qt + 1) * (QT / 64), nkt_all) : nkt_all;
    const int wave_qmax = qt * QT + wave * 32 + 31;

    // direct-to-LDS tile loads: wave-uniform tile base + this lane's byte offset inside the tile
    uint32_t kv_ld[KLD];
#pragma unroll
    for (int i = 0; i < KLD; ++i) {
        const int slot = 64 * (wave * KLD + i) + lane, r = slot / KCH, pc = slot % KCH;
        kv_ld[i] = 2u * (uint32_t)(r * D + 8 * swz<KCH>(r, pc));
    }
    const uint16_t* k_head = Kb + (size_t)bhkv * Lp * D;
    const uint16_t* v_head = Vb + (size_t)bhkv * Lp * D;
    const unsigned char* k_recs = MXS ? Krec + (size_t)bhkv * (Lp / 64) * KREC : nullptr;
    auto issue_tile = [&](int buf, int jt) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < KLD; ++i) {
            async_copy16(k_head + (size_t)jt * (64 * D), kv_ld[i], &sm.k[buf][512 * (wave * KLD + i)]);
            async_copy16(v_head + (size_t)jt * (64 * D), kv_ld[i], &sm.v[buf][512 * (wave * KLD + i)]);
        }
        if constexpr (MXS) {
            for (int i = wave; i < KREC / 1024; i += NW)
                async_copy16(k_recs + (size_t)jt * KREC, (uint32_t)(i * 1024 + lane * 16), &sm.krec[buf][i * 1024]);
        }
    };

    // LDS element offsets (buffer 0).  Row blocks of 32 (kb) and key steps of 16 (ks) add
    // compile-time constants: they do not change a row's swizzle key.
    //   koff[ds]    16-byte operand reads of K and V rows: row ln, d-slots 16*ds + 8*hf
    //   toff[mb][v] transpose reads of K^T: lane r of a group of 16 points at key 4*hf + r/4 + 8*v,
    //               columns 32*mb + 16*grp + 4*(r%4); the lane receives column 32*mb + ln of 4 keys
    const int tr_r = lane & 15, tr_grp = (lane >> 4) & 1;
    // (LDS byte addresses inside buffer 0 of the K tile, as integers: with the buffer a compile-time constant in the loop
    //  below, every read is this register plus an immediate)
    const uint32_t k0_ad = lds_addr_of(&sm.k[0][0]);
    uint32_t koff[DS], toff[MB][2];
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) koff[ds] = k0_ad + 2u * (uint32_t)((ln * KCH + swz<KCH>(ln, 2 * ds + hf)) * 8);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int v = 0; v < 2; ++v)
            toff[mb][v] = k0_ad + 2u * (uint32_t)swz_elem<KCH>(4 * hf + (tr_r >> 2) + 8 * v, 32 * mb + 16 * tr_grp + 4 * (tr_r & 3));
    // (opaque: the addition of the base of LDS, which is zero, is otherwise left for every tile, eight instructions)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) asm volatile("" : "+v"(toff[mb][0]), "+v"(toff[mb][1]));
    constexpr uint32_t kTileB = 64 * D * 2, kVfromK = 2 * kTileB;      // bytes of a tile buffer; sm.v[b] lies kVfromK after sm.k[b]

    floatx16 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[mb][i] = 0.0f;

    issue_tile(0, 0);
    // Q, dO and the row scalars must have arrived BEFORE the loop: a load still pending at loop entry
    // makes the compiler wait for all vector-memory traffic at the first product of every iteration,
    // i.e. for the tile prefetch it has just issued.
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) {
        if constexpr (!MXS) asm volatile("" : "+v"(qreg[ds]));
        asm volatile("" : "+v"(doreg[ds]));
    }
    if constexpr (MXS) {
#pragma unroll
        for (int ks = 0; ks < KSM; ++ks) asm volatile("" : "+v"(qop[ks]));
        asm volatile("" : "+v"(qs));
    }
    asm volatile("" :: "v"(Ls));
    // (opaque: sixteen equal values would otherwise be one register, copied sixteen times in front of every chain of products)
    if constexpr (FOLD) {
#pragma unroll
        for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(dp0[i]));
    } else asm volatile("" :: "v"(rs_s), "v"(Dq_s));
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // one key tile; BUF = j mod 2 at compile time
    auto tile = [&](auto buf_tag, int j) __attribute__((always_inline)) {
        constexpr int BUF = decltype(buf_tag)::value;
        const int k0 = j * 64;
        if (j + 1 < nkt) issue_tile(BUF ^ 1, j + 1);
        const bool active = (!CAUSAL || k0 <= wave_qmax) && wave_live;
        if (active) {
#pragma unroll
            for (int h0 = 0; h0 < 2; h0 += KH) {
            floatx16 s[KH], dp[KH];
            if constexpr (MXS) {
                // S^T from the codes (2 * D/64 products), then dP^T = V^F dO^T: 2*DS steps, step i: ds = i/2, kb = i%2
                const uint32_t rec = lds_addr_of(&sm.krec[BUF][0]);
                const uint32_t ksc = *(const __attribute__((address_space(3))) uint32_t*)(uintptr_t)(rec + 2 * KSM * 1024 + lane * 4);
                uint4v a[2][KSM];
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int ks = 0; ks < KSM; ++ks) a[kb][ks] = lds_read16_at(rec + (uint32_t)(((kb * KSM + ks) * 64 + lane) * 16));
                const floatx16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp4_opnd(a[0][0]), fp4_opnd(qop[0]), zero, 4, 4, 0, ksc, 0, qs);
                s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp4_opnd(a[1][0]), fp4_opnd(qop[0]), zero, 4, 4, KSM, ksc, 0, qs);
                if constexpr (KSM == 2) {
                    s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp4_opnd(a[0][1]), fp4_opnd(qop[1]), s[0], 4, 4, 1, ksc, 1, qs);
                    s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp4_opnd(a[1][1]), fp4_opnd(qop[1]), s[1], 4, 4, 3, ksc, 1, qs);
                }
                mfma_scale_settle(s[0], s[1]);
                constexpr int NST = 2 * DS, RING = 6;
                auto opnd = [&](int i) __attribute__((always_inline)) -> uint4v {
                    return lds_read16_at(koff[i >> 1] + (uint32_t)(BUF * kTileB + kVfromK + (i & 1) * (32 * D * 2)));
                };
                uint4v ring[RING];
#pragma unroll
                for (int i = 0; i < RING; ++i) ring[i] = opnd(i);
#pragma unroll
                for (int i = 0; i < NST; ++i) {
                    const uint4v av = ring[i % RING];
                    if (i + RING < NST) ring[i % RING] = opnd(i + RING);
                    dp[i & 1] = mfma_bf16(av, doreg[i >> 1], i < 2 ? dp0 : dp[i & 1]);
                }
            } else
            {   // S^T = K^F Q^F^T and dP^T = V^F dO^T: 2*KH*DS steps, step i: ds = i/(2*KH), kb = (i/2)%KH, K or V = i%2
                constexpr int NST = 2 * KH * DS, RING = D == 128 ? 5 : 6;      // (six operands of d = 128 do not fit beside dp0)
                auto opnd = [&](int i) __attribute__((always_inline)) -> uint4v {
                    return lds_read16_at(koff[i / (2 * KH)] + (uint32_t)(BUF * kTileB + (i & 1) * kVfromK + (h0 + (i >> 1) % KH) * (32 * D * 2)));
                };
                uint4v ring[RING];
#pragma unroll
                for (int i = 0; i < RING; ++i) ring[i] = opnd(i);
#pragma unroll
                for (int kb = 0; kb < KH; ++kb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) s[kb][i] = 0.0f;
#pragma unroll
                for (int i = 0; i < NST; ++i) {
                    const uint4v a = ring[i % RING];
                    if (i + RING < NST) ring[i % RING] = opnd(i + RING);
                    const int kb = (i >> 1) % KH, ds = i / (2 * KH);
                    if (i & 1) dp[kb] = mfma_bf16(a, doreg[ds], ds == 0 ? dp0 : dp[kb]);
                    else       s[kb] = mfma_f16(a, qreg[ds], s[kb]);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, RING, 0);
#pragma unroll
                for (int i = 0; i < NST; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    if (i + RING < NST) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
            }
            // masked keys (beyond L, or after the query): S = -inf so that P = 0
            const bool need_mask = (k0 + 64 > L) || (CAUSAL && k0 + 63 > qt * QT + wave * 32);
            if (__builtin_expect(need_mask, 0)) {
                const int klim = CAUSAL ? min(L - 1, q_row) : L - 1;
#pragma unroll
                for (int kb = 0; kb < KH; ++kb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int key = k0 + 32 * (h0 + kb) + 8 * (i >> 2) + 4 * hf + (i & 3);
                        if (key > klim) s[kb][i] = -INFINITY;
                    }
            }
            // dQ^T += K^F^T dS^T, 16 keys per step; the K^T operands of a step are read (transposed)
            // before that step's dS is computed, so their latency hides behind the VALU work
#pragma unroll
            for (int ks = 2 * h0; ks < 2 * (h0 + KH); ++ks) {
                const int kb = (ks >> 1) - h0, g = ks & 1;
                uint4v at[MB];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    at[mb] = join(lds_read_tr16_at(toff[mb][0] + (uint32_t)(BUF * kTileB + ks * (16 * D * 2))),
                                  lds_read_tr16_at(toff[mb][1] + (uint32_t)(BUF * kTileB + ks * (16 * D * 2))));
                uint4v bds;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r0 = 8 * g + 2 * i;
                    const float p0 = __builtin_amdgcn_exp2f(fmaf(s[kb][r0], c, -Ls));           // P = exp(S - L_i) (FOLD: / sqrt(d))
                    const float p1 = __builtin_amdgcn_exp2f(fmaf(s[kb][r0 + 1], c, -Ls));
                    // dS = P (dP - D_i)/sqrt(d), times 2^k, to fp16
                    if constexpr (FOLD) bds[i] = pack_f16x2(p0 * dp[kb][r0], p1 * dp[kb][r0 + 1]);
                    else bds[i] = pack_f16x2(p0 * fmaf(dp[kb][r0], rs_s, -Dq_s), p1 * fmaf(dp[kb][r0 + 1], rs_s, -Dq_s));
                }
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[mb] = mfma_f16(at[mb], bds, acc[mb]);
            }
            }
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    };
    for (int j = 0; j < nkt; j += 2) {
        tile(std::integral_constant<int, 0>{}, j);
        if (j + 1 < nkt) tile(std::integral_constant<int, 1>{}, j + 1);
    }

    if (q_row < L && wave_live) {
        const size_t row = (size_t)bh * L + q_row;
        const float un = 1.0f / ds_scale;                            // exact: a power of two
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint2v w;
                w[0] = pack_bf16x2(acc[mb][4 * t] * un, acc[mb][4 * t + 1] * un);
                w[1] = pack_bf16x2(acc[mb][4 * t + 2] * un, acc[mb][4 * t + 3] * un);
                *reinterpret_cast<uint2v*>(dQ + row * D + 32 * mb + 8 * t + 4 * hf) = w;
            }
    }
}

template <int D, bool CAUSAL, bool MXS, int NW = 4>
__global__ __launch_bounds__(64 * NW, NW == 4 ? (D == 64 ? 3 : 2) : 1) void bwd_dq_kernel(DqArgs A)
{
    const int nqt = (A.Lp + 32 * NW - 1) / (32 * NW);      // (Lp is a multiple of 128: with 8 waves the last workgroup may own only 128 rows)
    int bh, qt;
    head_tile_of_block(blockIdx.x, A.NHq, nqt, bh, qt);
    bwd_dq_body<D, CAUSAL, MXS, NW>(A, bh, CAUSAL ? nqt - 1 - qt : qt);
}

static DqArgs dq_args(const void* qb, const void* kb, const void* vb, const void* dob, const float* rowstat, const float* bound_part,
                      int B, int Hq, int Hkv, int L, int D, void* dq, const MxScoreOps* mx)
{
    const float rs = 1.0f / sqrtf((float)D);
    return DqArgs{(const uint16_t*)qb, (const uint16_t*)kb, (const uint16_t*)vb, (const uint16_t*)dob, (const float2*)rowstat, bound_part,
                  (uint16_t*)dq, L, round_up(L, kRowPad), Hq, Hq / Hkv, B * Hq, 1.4426950408889634f * rs, rs,
                  (const unsigned char*)(mx ? mx->qops : nullptr), (const uint32_t*)(mx ? mx->qsc : nullptr),
                  (const unsigned char*)(mx ? mx->krec : nullptr)};
}

template <int D, bool CAUSAL, bool MXS, int NW>
static int launch_dq_v(const void* qb, const void* kb, const void* vb, const void* dob,
                       const float* rowstat, const float* bound_part, int B, int Hq, int Hkv, int L, void* dq, hipStream_t st,
                       const MxScoreOps* mx)
{
    const size_t smem = sizeof(DqSmem<D, MXS>);
    auto kern = bwd_dq_kernel<D, CAUSAL, MXS, NW>;
    static unsigned long long lds_set = 0;          // one per instantiation
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)smem, lds_set)) return -1;
    const DqArgs A = dq_args(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, D, dq, mx);
    hipLaunchKernelGGL(kern, dim3((unsigned)(B * Hq * ((A.Lp + 32 * NW - 1) / (32 * NW)))), dim3(64 * NW), smem, st, A);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Eight waves per workgroup for a separate pass (plan.hpp says which problems run those) whose problem still leaves every compute
// unit two such workgroups to balance with, and, under a causal mask, whose sequences are long enough for the 256 rows at the diagonal,
// where part of the workgroup idles, not to matter (llm32k_gqa: 1.5 % faster with eight; llm4k_gqa: 2 - 8 % slower; the plan leaves
// no shorter causal problem here but the ablation with the unquantized P); or when a test forces them; four otherwise.  d = 64: four, of
// which three share a compute unit (bwd_plan).
static bool wide_workgroups(int D, bool causal, long long groups_of_256, int Lp)
{
    const int forced = __atomic_load_n(&g_bwd_waves, __ATOMIC_RELAXED);
    if (forced != 0) return forced == 8;
    return D == 128 && groups_of_256 >= 2LL * device_cu_count() && (!causal || Lp >= 16384);
}

template <int D, bool CAUSAL, bool MXS>
static int launch_dq_t(const void* qb, const void* kb, const void* vb, const void* dob,
                       const float* rowstat, const float* bound_part, int B, int Hq, int Hkv, int L, void* dq, hipStream_t st,
                       const MxScoreOps* mx)
{
    if (wide_workgroups(D, CAUSAL, (long long)B * Hq * ((round_up(L, kRowPad) + 255) / 256), round_up(L, kRowPad)))
        return launch_dq_v<D, CAUSAL, MXS, 8>(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, dq, st, mx);
    return launch_dq_v<D, CAUSAL, MXS, 4>(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, dq, st, mx);
}

int launch_bwd_dq(const void* qb, const void* kb, const void* vb, const void* dob,
                  const float* rowstat, const float* bound_part,
                  int B, int Hq, int Hkv, int L, int D, bool causal, void* dq, hipStream_t st, const MxScoreOps* mx)
{
    if (mx && (!mx->qops || !mx->qsc || !mx->krec)) return -1;
#define AQ_DQ(DD, C) (mx ? launch_dq_t<DD, C, true>(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, dq, st, mx) \
                         : launch_dq_t<DD, C, false>(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, dq, st, nullptr))
    if (D == 128) return causal ? AQ_DQ(128, true) : AQ_DQ(128, false);
    if (D == 64)  return causal ? AQ_DQ(64, true) : AQ_DQ(64, false);
#undef AQ_DQ
    return -1;
}

// ------------------------------------------------------------------ dK/dV pass
// A workgroup of NW waves owns 32 NW keys of one kv head (32 per wave, held in registers as MFMA A
// operands) and walks over the query rows of every query head of the group in tiles of 32.  NW = 4
// everywhere except the passes of a large problem (any format of P except the ablation), which run NW = 8: every
// Q / dO tile a workgroup fetches then serves twice the keys, which halves the pass's read traffic.
// The per-wave [query][key] staging tiles (32 queries x 32 keys, 16-bit values, rows of 64 bytes).  By the bank-conflict
// counter the LDS takes an 8-byte store from 16 lanes per cycle on 32 banks of 4 bytes and serves an 8-byte (transposing)
// read to 32 lanes per cycle on 64 banks.  A store instruction writes one 8-byte chunk of 16 consecutive queries per cycle,
// a read fetches the whole rows of four consecutive queries.  The rows of four consecutive queries (a group) are therefore
// contiguous, 256 bytes: a read touches every bank once.  For the stores every group is followed by 16 bytes of padding
// (the next group starts four banks further) and in the third and fourth row of a group neighbouring chunks are swapped:
// with the row's own 64 bytes = 16 banks that puts the 16 queries of a cycle on 16 different bank pairs.  (Rows padded
// to 72 bytes instead made every read collide once: 6 % of the pass's LDS cycles.)
constexpr int kTGroupB = 4 * 64 + 16;  // bytes of a group of four queries
constexpr int kTTileB = 8 * kTGroupB;  // bytes of a tile

template <int D, bool MXS, int NW>
struct DkvSmem {
    uint16_t q[2][32 * D];           // Q^F rows [query][d], fp16, swizzled
    uint16_t g[2][32 * D];           // dO rows  [query][d], bf16, swizzled
    uint16_t t[NW][2][kTTileB / 2];    // per wave: P^F (bf16) and dS (fp16, scaled) as [query][key]
    float rmax[NW][32];              // two-level P: per wave, the largest P of every query row over the wave's 32 keys
    unsigned char qrec[MXS ? 2 : 1][MXS ? (D / 64) * 1024 + 256 : 16];      // MX: Q operands of the FP4 instruction of a tile and their scale dwords
};

struct DkvArgs {
    const uint16_t *Qb, *Kb, *Vb, *dOb;
    const float2* rowstat; const float* bound_part;
    uint16_t *dK, *dV; unsigned long long* tile_counts;
    int L, Lp, Hq, G, NHq, NHkv; float c, rs;
    float* pdump /* COUNT only, may be null: P^F of query rows [dump_row0, dump_row0 + 128), [B*Hq][128][L] */; int dump_row0;
    const unsigned char* Qops; const uint32_t* Qsc;      // PQ == 2 (MX) only: the scores come from the
    const unsigned char* Kops; const uint32_t* Ksc;      // codes, see bwd_dq_body
    int splits, split_iters; float* part;                // SPLIT only: see bwd_joint_kernel
};
// SPLIT: only the query tiles piece * split_iters .. of the workgroup's key tile; where that is not all of them, the sums go to
// `part` as fp32 for dkdv_reduce_kernel instead of to dK and dV.
template <int D, bool CAUSAL, bool COUNT /* measurement / test variant: count tiles, dump P^F */,
          int PQ /* phi(P): 0 none (ablation: dV from the fp32 P), 1 NVFP4, 2 MX, 3 NVFP4 after the two-level row factor */,
          int NW /* waves, 32 keys each */, bool SPLIT>
__device__ __forceinline__ void bwd_dkdv_body(const DkvArgs& A, int bhkv, int kt_, int piece)
{
    constexpr bool MXS = PQ == 2;
    constexpr int KSM = D / 64, QREC = KSM * 1024 + 256;
    constexpr int DS = D / 16, NB = D / 32, KCH = D / 8;
    constexpr int NWL = (32 * KCH) / 64;             // 1 KiB wave-loads per tile of 32 rows
    constexpr int PER_WAVE = NWL >= NW ? NWL / NW : 1;
    extern __shared__ __align__(256) unsigned char smem_raw[];   // XORs of address bits 5..7 below commute with adding this base
    DkvSmem<D, MXS, NW>& sm = *reinterpret_cast<DkvSmem<D, MXS, NW>*>(smem_raw);

    const uint16_t *__restrict__ Qb = A.Qb, *__restrict__ Kb = A.Kb, *__restrict__ Vb = A.Vb, *__restrict__ dOb = A.dOb;
    const float2* __restrict__ rowstat = A.rowstat;
    const float* __restrict__ bound_part = A.bound_part;
    uint16_t *__restrict__ dK = A.dK, *__restrict__ dV = A.dV;
    unsigned long long* __restrict__ tile_counts = A.tile_counts;
    float* __restrict__ pdump = A.pdump;
    const unsigned char *__restrict__ Qops = A.Qops, *__restrict__ Kops = A.Kops;
    const uint32_t *__restrict__ Qsc = A.Qsc, *__restrict__ Ksc = A.Ksc;
    const int L = A.L, Lp = A.Lp, Hq = A.Hq, G = A.G, NHq = A.NHq, dump_row0 = A.dump_row0;
    const float c = A.c, rs = A.rs;

    constexpr int KT = 32 * NW;                      // keys of a workgroup
    const int Hkv = Hq / G;
    const int b = bhkv / Hkv, hk = bhkv % Hkv;
    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);        // scalar: LDS destinations and branches use it
    const int key0_w = kt_ * KT + wave * 32;        // this wave's first key
    const bool wave_live = NW == 4 || key0_w < Lp;  // a wave past the padded rows takes part in the copies and barriers only

    // K^F, V^F rows of this lane's key: A operands (row = key, d-slots 16*ds + 8*hf)
    uint4v kreg[MXS ? 1 : DS], vreg[DS], kop[MXS ? KSM : 1];
    uint32_t ksc = 0u;
    {
        const size_t off = ((size_t)bhkv * Lp + (wave_live ? key0_w : 0) + ln) * D + 8 * hf;
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
            if constexpr (!MXS) kreg[ds] = *reinterpret_cast<const uint4v*>(Kb + off + 16 * ds);
            vreg[ds] = *reinterpret_cast<const uint4v*>(Vb + off + 16 * ds);
        }
        if constexpr (MXS) {
            const size_t grp = (size_t)bhkv * (Lp / 32) + ((wave_live ? key0_w : 0) >> 5);
#pragma unroll
            for (int ks = 0; ks < KSM; ++ks) kop[ks] = *reinterpret_cast<const uint4v*>(Kops + ((grp * KSM + ks) * 64 + lane) * 16);
            ksc = Ksc[grp * 64 + lane];
        }
    }

    floatx16 dk[NB], dv[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int i = 0; i < 16; ++i) { dk[nb][i] = 0.0f; dv[nb][i] = 0.0f; }

    // query tiles of 32 rows, query heads of the group one after another; under a causal mask
    // only rows >= the workgroup's first key matter
    const int nq32 = (L + 31) / 32;
    const int qt_first = CAUSAL ? (kt_ * KT) / 32 : 0;
    const int per_head = nq32 - qt_first;
    int niter = per_head > 0 ? per_head * G : 0;
    int first = 0;                                   // the first of this workgroup's query tiles
    bool whole = true;
    if constexpr (SPLIT) {
        const int pieces = (niter + A.split_iters - 1) / A.split_iters;
        if (piece >= pieces) return;                 // (workgroup-uniform; no barrier passed yet)
        whole = pieces == 1;
        first = piece * niter / pieces;
        niter = (piece + 1) * niter / pieces - first;
    }
    const size_t bh0 = (size_t)b * Hq + hk * G;      // first query head of the group

    // dS goes to fp16 after multiplication by ds_scale = 2^k, one k for the kv head, from the bound
    // (max_i |dO_i| max_j |V^F_j| + max_i |D_i|) / sqrt(d) >= |dS_ij| over the query heads of the group
    float ds_scale;
    {
        // (the heads are joined lane by lane, four loads on their way at a time, and the lanes once for all of them)
        const float* p = bound_part + (size_t)bhkv * kBoundParts + (tid & 63);
        const float *p1 = bound_part + ((size_t)NHq + bh0) * kBoundParts + (tid & 63), *p2 = p1 + (size_t)NHq * kBoundParts;
        float vmax = *p, domax = 0.0f, dmax = 0.0f;
        for (int g0 = 0; g0 < G; g0 += 4) {
            float a[4], e[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { const size_t o = (size_t)min(g0 + i, G - 1) * kBoundParts; a[i] = p1[o]; e[i] = p2[o]; }
#pragma unroll
            for (int i = 0; i < 4; ++i) { domax = fmaxf(domax, a[i]); dmax = fmaxf(dmax, e[i]); }
        }
        vmax = lanes_max<32, 1>(vmax); domax = lanes_max<32, 1>(domax); dmax = lanes_max<32, 1>(dmax);
        ds_scale = ds_scale_for(domax * vmax * rs + dmax);
    }
    const float rs_s = rs * ds_scale;

    // direct-to-LDS loads: this wave's chunk slots and their (row, swizzled chunk)
    const bool loader = NWL >= NW || wave < NWL;
    uint32_t slot_off[PER_WAVE];                     // this lane's byte offset inside a tile's source rows
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
        const int slot = 64 * (wave * PER_WAVE + i) + lane;
        slot_off[i] = 2u * (uint32_t)((slot / KCH) * D + 8 * swz<KCH>(slot / KCH, slot % KCH));
    }
    // (head, tile) walk without divisions: state of the NEXT tile to load and of the current tile
    int ld_g = SPLIT ? first / per_head : 0, ld_t = SPLIT ? first % per_head : 0;      // next tile to issue: head index in group, tile in head
    int cur_g = ld_g, cur_t = ld_t;
    auto issue_next = [&](int buf) __attribute__((always_inline)) {
        const size_t row0 = (bh0 + ld_g) * Lp + (size_t)(qt_first + ld_t) * 32;
        if (loader) {
#pragma unroll
            for (int i = 0; i < PER_WAVE; ++i) {
                async_copy16(Qb + row0 * D, slot_off[i], &sm.q[buf][512 * (wave * PER_WAVE + i)]);
                async_copy16(dOb + row0 * D, slot_off[i], &sm.g[buf][512 * (wave * PER_WAVE + i)]);
            }
        }
        if constexpr (MXS) {      // the tile's Q operands (KSM wave copies of 1 KiB) and their 64 scale dwords
            const size_t grp = (bh0 + ld_g) * (Lp / 32) + (size_t)(qt_first + ld_t);
            if (wave < KSM) async_copy16(Qops + grp * (KSM * 1024), (uint32_t)(wave * 1024 + lane * 16), &sm.qrec[buf][wave * 1024]);
            if (wave == 3 && lane < 16) async_copy16(Qsc + grp * 64, (uint32_t)(lane * 16), &sm.qrec[buf][KSM * 1024]);
        }
        if (++ld_t == per_head) { ld_t = 0; ++ld_g; }
    };

    // LDS byte offsets.  A row of a tile is D*2 bytes = KCH 16-byte chunks and chunk c of row r sits
    // at chunk c ^ key(r), so an offset is (per-lane constant) XOR (compile-time constant):
    //   operand reads of Q / dO rows (row ln, d-slots 16*ds + 8*hf):   a_rd ^ (ds << 5)
    //   transpose reads of Q / dO columns (lane r of a group of 16 points at query
    //   8*hf + r/4 + 4*v, columns 32*nb + 16*grp + 4*(r%4)):           g_rd[v] ^ (nb << 6)
    // 16 more rows, the other buffer and the dO tile are constant byte distances.
    constexpr int kRowB = 2 * D, kBufB = 32 * kRowB, kGB = 2 * kBufB;
    const int tr_r = lane & 15, tr_grp = (lane >> 4) & 1;
    const int a_rd = 2 * swz_elem<KCH>(ln, 8 * hf);
    int g_rd[2];
#pragma unroll
    for (int v = 0; v < 2; ++v) g_rd[v] = 2 * swz_elem<KCH>(8 * hf + (tr_r >> 2) + 4 * v, 16 * tr_grp + 4 * (tr_r & 3));
    // staging tiles of this wave, as LDS byte addresses (integers: pointer arithmetic on the dynamic LDS symbol costs an
    // add per access): this lane's writes and its transpose reads; the dS tile lies kTB bytes after the P^F tile
    constexpr int kTB = kTTileB;
    const uint32_t t_base = lds_addr_of(&sm.t[wave][0][0]);
    // writes: query ln, chunk hf + 2 t4 (keys 4 hf + 8 t4 .. + 3; t4 = 0..3 at compile time); reads: query 8 hf + tr_r/4 +
    // 16 ks + 4 s (group 2 hf + 4 ks + s), chunk 4 tr_grp + tr_r%4; the swap of neighbouring chunks flips the lane's part
    const uint32_t tw_ad = t_base + (uint32_t)(kTGroupB * (ln >> 2) + 64 * (ln & 3) + 8 * (hf ^ ((ln >> 1) & 1)));
    const uint32_t ta_ad = t_base + (uint32_t)(kTGroupB * (2 * hf) + 64 * (tr_r >> 2) + 32 * tr_grp + 8 * ((tr_r & 3) ^ ((tr_r >> 3) & 1)));
    const int lds0 = (int)lds_addr_of(smem_raw);

    // {L_i log2(e), D_i / sqrt(d)} of this lane's query row of the next tile
    float2 st_n = make_float2(0.0f, 0.0f);
    if (niter > 0) { issue_next(0); st_n = rowstat[(bh0 + cur_g) * Lp + (size_t)(qt_first + cur_t) * 32 + ln]; }
    // every load of the prologue must have arrived before the loop (see the dQ pass)
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) {
        if constexpr (!MXS) asm volatile("" : "+v"(kreg[ds]));
        asm volatile("" : "+v"(vreg[ds]));
    }
    if constexpr (MXS) {
#pragma unroll
        for (int ks = 0; ks < KSM; ++ks) asm volatile("" : "+v"(kop[ks]));
        asm volatile("" : "+v"(ksc));
    }
    asm volatile("" : "+v"(st_n.x), "+v"(st_n.y));
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    unsigned n_tiles = 0, n_pf_tiles = 0;            // measurement only (wave-uniform)
    for (int it = 0; it < niter; ++it) {
        const int buf = it & 1;
        const int q0 = (qt_first + cur_t) * 32;
        const float Ls = st_n.x, Dq_s = st_n.y * rs_s;
        // next tile: start its copy and fetch its row scalars now, they are needed one iteration later
        int nx_g = cur_g, nx_t = cur_t + 1;
        if (nx_t == per_head) { nx_t = 0; ++nx_g; }
        if (it + 1 < niter) {
            issue_next(buf ^ 1);
            st_n = rowstat[(bh0 + nx_g) * Lp + (size_t)(qt_first + nx_t) * 32 + ln];
        }
        // wave-uniform.  With the two-level P every wave takes part in every tile: the exchange of the row maxima below
        // contains a workgroup barrier, and a wave whose keys all lie after the tile's queries computes P = 0 throughout
        // (which costs the first four query tiles of a workgroup some idle products and nothing else).
        const bool active = PQ == 3 || ((!CAUSAL || q0 + 31 >= key0_w) && wave_live);
        if (active) {
            // Q^F tile of this iteration (dO is kGB further).  The per-lane offsets are made opaque once
            // per iteration: otherwise the compiler hoists every (offset ^ constant) out of the loop and
            // pays for it with a dozen registers that this kernel does not have.
            int a_it = a_rd + buf * kBufB + lds0, g_it0 = g_rd[0] + buf * kBufB + lds0, g_it1 = g_rd[1] + buf * kBufB + lds0;
            asm volatile("" : "+v"(a_it), "+v"(g_it0), "+v"(g_it1));
            floatx16 s, dp;
            if constexpr (MXS) {
                // S^T from the codes (D/64 products), then dP^T = V^F dO^T over the dO tile (DS steps)
                const uint32_t rec = lds_addr_of(&sm.qrec[buf][0]);
                const uint32_t qsl = *(const __attribute__((address_space(3))) uint32_t*)(uintptr_t)(rec + KSM * 1024 + lane * 4);
                uint4v bq4[KSM];
#pragma unroll
                for (int ks = 0; ks < KSM; ++ks) bq4[ks] = lds_read16_at(rec + (uint32_t)((ks * 64 + lane) * 16));
                const floatx16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                s = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp4_opnd(kop[0]), fp4_opnd(bq4[0]), zero, 4, 4, 0, ksc, 0, qsl);
                if constexpr (KSM == 2)
                    s = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp4_opnd(kop[1]), fp4_opnd(bq4[1]), s, 4, 4, 1, ksc, 1, qsl);
                mfma_scale_settle(s);
                constexpr int RING = 3;
                auto opnd = [&](int i) __attribute__((always_inline)) -> uint4v {
                    return lds_read16_at((uint32_t)((a_it ^ (i << 5)) + kGB));
                };
                uint4v ring[RING];
#pragma unroll
                for (int i = 0; i < RING; ++i) ring[i] = opnd(i);
#pragma unroll
                for (int i = 0; i < 16; ++i) dp[i] = 0.0f;
#pragma unroll
                for (int i = 0; i < DS; ++i) {
                    const uint4v bq = ring[i % RING];
                    if (i + RING < DS) ring[i % RING] = opnd(i + RING);
                    dp = mfma_bf16(vreg[i], bq, dp);
                }
            } else
            {   // S^T = K^F Q^F^T, dP^T = V^F dO^T: 2*DS steps, step i: ds = i/2, Q or dO = i%2
                // (the two-level variant carries the exchanged row maximum and its LDS slot on top: its ring is one shorter)
                constexpr int NST = 2 * DS, RING = PQ == 3 ? 2 : 3;
                auto opnd = [&](int i) __attribute__((always_inline)) -> uint4v {
                    return lds_read16_at((uint32_t)((a_it ^ ((i >> 1) << 5)) + (i & 1) * kGB));
                };
                uint4v ring[RING];
#pragma unroll
                for (int i = 0; i < RING; ++i) ring[i] = opnd(i);
#pragma unroll
                for (int i = 0; i < 16; ++i) { s[i] = 0.0f; dp[i] = 0.0f; }
#pragma unroll
                for (int i = 0; i < NST; ++i) {
                    const uint4v bq = ring[i % RING];
                    if (i + RING < NST) ring[i % RING] = opnd(i + RING);
                    if (i & 1) dp = mfma_bf16(vreg[i >> 1], bq, dp);
                    else       s = mfma_f16(kreg[i >> 1], bq, s);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, RING, 0);
#pragma unroll
                for (int i = 0; i < NST; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    if (i + RING < NST) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
            }
            // masked keys (beyond L, or after the query): S = -inf so that P = 0
            const bool need_mask = (key0_w + 32 > L) || (CAUSAL && key0_w + 31 > q0);
            if (__builtin_expect(need_mask, 0)) {
                const int klim = CAUSAL ? min(L - 1, q0 + ln) : L - 1;
// (SPLIT: half of the wave taken afresh, as in the epilogue: no register holds it from one masked tile to the next)
                int hf_m = hf;
                if constexpr (SPLIT) {
                    uint32_t lane_m = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
                    asm volatile("" : "+v"(lane_m));
                    hf_m = (int)lane_m >> 5;
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int key = key0_w + 8 * (i >> 2) + 4 * hf_m + (i & 3);
                    if (key > klim) s[i] = -INFINITY;
                }
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], c, -Ls));    // P = exp(S - L_i)
            // block scales of phi(P): one per 16 keys = registers 8*gq .. 8*gq+7 of both halves
            constexpr bool PQUANT = PQ != 0;
            float sc[2], inv[2], gmax[2] = {0.0f, 0.0f};
            bool nz = false;
            auto group_maxima = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int gq = 0; gq < 2; ++gq) gmax[gq] = nvfp4_group_max(s, gq);
            };
            if constexpr (PQ == 2) {
                // MX format: this wave's 32 keys are one block with a power-of-two scale
                float a4[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) a4[t] = fmaxf(fmaxf(s[t], s[4 + t]), fmaxf(s[8 + t], s[12 + t]));
                const float amax = xhalf_max(fmaxf(fmaxf(a4[0], a4[1]), fmaxf(a4[2], a4[3])));
                const uint32_t byte = e8m0_of_amax(amax);
                sc[0] = sc[1] = e8m0_as_f32(byte);
                nz = amax > 0.0f;
            } else if constexpr (PQ == 1) {
                // Is any block scale of this tile non-zero?  The scales themselves are only needed where the answer is yes (below).
                group_maxima();
                nz = nvfp4_scale_nonzero(fmaxf(gmax[0], gmax[1]));
            }
            // Two-level quantization of P (PQ == 3): the row factor belongs to an aligned group of 64 keys, the tile row
            // of the forward, i.e. to this wave's 32 keys and those of its neighbour (waves 0|1 and 2|3 of the
            // workgroup).  The two waves exchange their partial row maxima through LDS.
            float pair_max = 0.0f;
            if constexpr (PQ == 3) {
                group_maxima();
                const float own = xhalf_max(fmaxf(gmax[0], gmax[1]));
                // rmax[w][row] sits 128 w + 4 row bytes into a 256-byte aligned array: the neighbour's slot is address ^ 128
                const uint32_t rm_ad = lds_addr_of(&sm.rmax[0][0]) + 128u * (uint32_t)wave + 4u * (uint32_t)ln;
                *(__attribute__((address_space(3))) float*)(uintptr_t)rm_ad = own;      // both half-waves hold the same value
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                pair_max = fmaxf(own, *(const __attribute__((address_space(3))) float*)(uintptr_t)(rm_ad ^ 128u));
            }
            // block scales of phi(P): one per 16 keys = registers 8*gq .. 8*gq+7 of both halves (NVFP4, with or without
            // the row factor of the two-level form)
            auto nvfp4_scales = [&]() __attribute__((always_inline)) {
                if constexpr (PQ == 1) {
                    nvfp4_pair_scales(gmax, sc, inv);
                    return true;
                }
                // Two-level quantization of P (PQ == 3): the row of the aligned 64-key group is divided by s1, the
                // smallest power of two with 2688 s1 >= max(row maximum of the group, 2^-24), before the NVFP4 blocks
                const float base = fmaxf(pair_max, 5.9604644775390625e-08f);
                const uint32_t e1 = ((__float_as_uint(base) + 0x0057FFFFu) >> 23) - 11u;      // 2688 = 1.3125 * 2^11
                const float s1 = __uint_as_float(e1 << 23), inv1 = __uint_as_float((254u - e1) << 23);
                bool any = false;
#pragma unroll
                for (int gq = 0; gq < 2; ++gq) {
                    const float s2 = rne_e4m3_grid_of_product(xhalf_max(gmax[gq]) * inv1, 1.0f / 6.0f);
                    // P^F = (s1 s2) * code and the code is RNE(P / (s1 s2)): from here on the product of the two levels
                    // stands in for the block scale (a power of two times an E4M3 value: still exact in bf16)
                    sc[gq] = s2 * s1;
                    inv[gq] = s2 > 0.0f ? __builtin_amdgcn_rcpf(s2) * inv1 : 0.0f;
                    any = any || s2 > 0.0f;
                }
                return any;
            };
            if constexpr (PQ == 3) nz = nvfp4_scales();      // after the row factor a tile is almost never all zero
            // If every block scale of this 32x32 tile rounded to 0 (max P <= 6 * 2^-10: the usual case for long rows),
            // P^F is identically 0: quantizing it, staging it and the dV products are skipped.  Wave-uniform, exact.
            const bool with_pf = PQUANT && __builtin_amdgcn_ballot_w64(nz) != 0;
            if constexpr (COUNT) { ++n_tiles; if (with_pf) ++n_pf_tiles; }
            // P^F = phi^-1(phi(P)) as bf16, staged as [query][key] before dS is: both tiles are then in LDS when the
            // products start, and the dV products of a tile that has them follow its dK products in one stream (a wave
            // that quantized, staged and multiplied P^F only after its dK products kept the other three waiting at the
            // tile barrier for the whole of that dependent chain).
            if (with_pf) {
                if constexpr (PQ == 1) nvfp4_scales();
                if constexpr (PQUANT) {
#pragma unroll
                    for (int t4 = 0; t4 < 4; ++t4) {
                        const int r0 = 4 * t4, gq = t4 >> 1;
                        uint2v wp;
                        if constexpr (PQ == 2) {      // the conversions divide and multiply by a power of two themselves (117 -> 68 vector instructions)
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                const uint32_t codes = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(any_register(), s[r0 + 2 * u], s[r0 + 2 * u + 1], sc[gq], 0);
                                wp[u] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, sc[gq], 0));
                            }
                        } else wp = nvfp4_pf_quad(s, r0, sc[gq], inv[gq]);
                        lds_write8_at(tw_ad + (uint32_t)(16 * t4), wp);
                        if constexpr (COUNT) {
                            const int qr = q0 + ln;      // registers r0 .. r0 + 3: keys key0_w + 8 t4 + 4 hf + e of query row qr
                            if (pdump && qr >= dump_row0 && qr < dump_row0 + 128 && qr < L) {
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    const int key = key0_w + 8 * t4 + 4 * hf + e;
                                    if (key < L) pdump[((size_t)(bh0 + cur_g) * 128 + (qr - dump_row0)) * L + key] = e & 1 ? bf16_hi_f32(wp[e >> 1]) : bf16_lo_f32(wp[e >> 1]);
                                }
                            }
                        }
                    }
                }
            }
            // dS = P (dP - D_i)/sqrt(d) from the fp32 P, scaled, as fp16, staged as [query][key]
#pragma unroll
            for (int t4 = 0; t4 < 4; ++t4) {                           // 4 consecutive keys per store
                const int r0 = 4 * t4;
                float dsv[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) dsv[e] = s[r0 + e] * fmaf(dp[r0 + e], rs_s, -Dq_s);
                uint2v wh;
                wh[0] = pack_f16x2(dsv[0], dsv[1]); wh[1] = pack_f16x2(dsv[2], dsv[3]);
                // registers r0..r0+3 <-> keys 8*(r0>>2) + 4*hf + 0..3 of this wave's 32 keys
                lds_write8_at(tw_ad + (uint32_t)(kTB + 16 * t4), wh);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // dK += dS^T Q^F (steps 0 .. NSTEP-1) and dV += P^F^T dO (steps NSTEP .. 2 NSTEP-1), NSTEP = 2*NB steps each:
            // step j of a product covers queries 16*(j/NB) .. +15 (contraction slots 0-3: queries 16*ks + 8*hf + 0..3,
            // slots 4-7: the next four) and columns 32*(j%NB) .. +31.  The operands of a step are read while the step
            // before it multiplies.
            constexpr int NSTEP = 2 * NB;
            auto rd_b = [&](int j, int extra) __attribute__((always_inline)) -> uint4v {
                const int nb = j % NB, ks = j / NB;
                return join(lds_read_tr16_at((uint32_t)((g_it0 ^ (nb << 6)) + ks * (16 * kRowB) + extra)),
                            lds_read_tr16_at((uint32_t)((g_it1 ^ (nb << 6)) + ks * (16 * kRowB) + extra)));
            };
            auto rd_t = [&](int tb /* 0: P^F tile, kTB: dS tile */, int ks) __attribute__((always_inline)) -> uint4v {
                const uint32_t ta = ta_ad + (uint32_t)(tb + ks * (4 * kTGroupB));       // 16 rows = 4 groups further
                return join(lds_read_tr16_at(ta), lds_read_tr16_at(ta + kTGroupB));
            };
            // steps [FIRST, LAST) of the stream
            auto products = [&](auto first_tag, auto last_tag) __attribute__((always_inline)) {
                constexpr int FIRST = decltype(first_tag)::value, LAST = decltype(last_tag)::value;
                auto a_of = [&](int st) __attribute__((always_inline)) -> uint4v { return rd_t(st < NSTEP ? kTB : 0, (st % NSTEP) / NB); };
                auto b_of = [&](int st) __attribute__((always_inline)) -> uint4v { return rd_b(st % NSTEP, st < NSTEP ? 0 : kGB); };
                uint4v a = a_of(FIRST), b[2];
                b[FIRST & 1] = b_of(FIRST);
#pragma unroll
                for (int st = FIRST; st < LAST; ++st) {
                    const int nb = st % NB;
                    const bool new_a = st + 1 < LAST && (st + 1) % NB == 0;
                    if (st + 1 < LAST) b[(st + 1) & 1] = b_of(st + 1);
                    uint4v a_n;
                    if (new_a) a_n = a_of(st + 1);
                    if (st < NSTEP) dk[nb] = mfma_f16(a, b[st & 1], dk[nb]);
                    else            dv[nb] = mfma_bf16(a, b[st & 1], dv[nb]);
                    if (new_a) a = a_n;
                }
                __builtin_amdgcn_sched_group_barrier(0x100, 2 + 2, 0);
#pragma unroll
                for (int st = FIRST; st < LAST; ++st) {
                    if (st + 1 < LAST) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    if (st + 1 < LAST && (st + 1) % NB == 0) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                }
            };
            typedef std::integral_constant<int, 0> I0;
            typedef std::integral_constant<int, NSTEP> I1;
            typedef std::integral_constant<int, 2 * NSTEP> I2;
            if constexpr (PQUANT) {
                // (two branches, each with its whole stream, would let the dV operand reads start under the dK products; the
                //  compiler then shuffles the 256 accumulator registers between the branches and spills)
                products(I0{}, I1{});
                if (with_pf) products(I1{}, I2{});
            } else {
                // Ablation (Sec. 3.2, "no fake quantization of P in the backward"): dV from the fp32 P itself, which enters
                // its product in two passes as a bf16 hi + lo pair
                products(I0{}, I1{});
#pragma unroll
                for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
                    for (int t4 = 0; t4 < 4; ++t4) {
                        const int r0 = 4 * t4;
                        float pf[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float hi = __uint_as_float((uint32_t)f32_to_bf16_rne(s[r0 + e]) << 16);
                            pf[e] = pass == 0 ? hi : s[r0 + e] - hi;
                        }
                        uint2v wp;
                        wp[0] = pack_bf16x2(pf[0], pf[1]); wp[1] = pack_bf16x2(pf[2], pf[3]);
                        lds_write8_at(tw_ad + (uint32_t)(16 * t4), wp);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    products(I1{}, I2{});
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
        cur_g = nx_g; cur_t = nx_t;
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        asm volatile("" : "+v"(st_n.x), "+v"(st_n.y));     // the next tile's row scalars are consumed here, not earlier
    }

    if (COUNT && lane == 0 && tile_counts) {
        atomicAdd(&tile_counts[0], (unsigned long long)n_tiles);
        atomicAdd(&tile_counts[1], (unsigned long long)n_pf_tiles);
    }

    // accumulators: row = key 8*(i>>2) + 4*hf + (i&3) of the wave, column d = 32*nb + ln
    // (SPLIT: the lane number is taken afresh; what the second kind of store needs of it would otherwise lie in scratch during the loop)
    uint32_t lane_o = (uint32_t)lane;
    if constexpr (SPLIT) {
        lane_o = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(lane_o));
    }
    const int ln_o = (int)lane_o & 31, hf_o = (int)lane_o >> 5;
    if constexpr (SPLIT) {
        if (!whole) {
            // four accumulators (keys 8 t4 + 4 hf .. + 3) at a time, as they lie in the lanes: 1 KiB per wave and store
            floatx4* dst = reinterpret_cast<floatx4*>(A.part) + (((size_t)bhkv * (Lp / KT) + kt_) * A.splits + piece) * (2 * NB * 4 * NW * 64) + wave * 64 + lane_o;
            const float un = rs / rs_s;              // 1 / ds_scale, exact: a power of two
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int t4 = 0; t4 < 4; ++t4) {
                    floatx4 wk, wv;
#pragma unroll
                    for (int e = 0; e < 4; ++e) { wk[e] = dk[nb][4 * t4 + e] * un; wv[e] = dv[nb][4 * t4 + e]; }
                    dst[(size_t)(nb * 4 + t4) * (NW * 64)] = wk;
                    dst[(size_t)((NB + nb) * 4 + t4) * (NW * 64)] = wv;
                }
            return;
        }
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int key = key0_w + 8 * (i >> 2) + 4 * hf_o + (i & 3);
            if (key < L) {
                const size_t o = ((size_t)bhkv * L + key) * D + 32 * nb + ln_o;
                dK[o] = f32_to_bf16_rne(dk[nb][i] * (rs / rs_s));            // / ds_scale, exact: a power of two
                dV[o] = f32_to_bf16_rne(dv[nb][i]);
            }
        }
}

template <int D, bool CAUSAL, bool COUNT, int PQ, int NW = 4>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void bwd_dkdv_kernel(DkvArgs A)
{
    const int nkt = (A.Lp + 32 * NW - 1) / (32 * NW);      // (Lp is a multiple of 128: with 8 waves the last workgroup may own only 128 keys)
    int bhkv, kt;
    head_tile_of_block(blockIdx.x, A.NHkv, nkt, bhkv, kt);    // key tiles in increasing order: under a causal mask the first see the most queries
    bwd_dkdv_body<D, CAUSAL, COUNT, PQ, NW, false>(A, bhkv, kt, 0);
}

static DkvArgs dkv_args(const void* qb, const void* kb, const void* vb, const void* dob, const float* rowstat, const float* bound_part,
                        int B, int Hq, int Hkv, int L, int D, void* dk, void* dv, const MxScoreOps* mx)
{
    const float rs = 1.0f / sqrtf((float)D);
    return DkvArgs{(const uint16_t*)qb, (const uint16_t*)kb, (const uint16_t*)vb, (const uint16_t*)dob, (const float2*)rowstat, bound_part,
                   (uint16_t*)dk, (uint16_t*)dv, nullptr, L, round_up(L, kRowPad), Hq, Hq / Hkv, B * Hq, B * Hkv, 1.4426950408889634f * rs, rs,
                   nullptr, 0, (const unsigned char*)(mx ? mx->qops : nullptr), (const uint32_t*)(mx ? mx->qsc : nullptr),
                   (const unsigned char*)(mx ? mx->kops : nullptr), (const uint32_t*)(mx ? mx->ksc : nullptr), 1, 0, nullptr};
}

template <int D, bool CAUSAL, bool COUNT, int PQ, int NW>
static int launch_dkdv_v(const void* qb, const void* kb, const void* vb, const void* dob,
                         const float* rowstat, const float* bound_part,
                         int B, int Hq, int Hkv, int L, void* dk, void* dv, unsigned long long* tile_counts,
                         hipStream_t st, float* p_dump, int dump_row0, const MxScoreOps* mx)
{
    const size_t smem = sizeof(DkvSmem<D, PQ == 2, NW>);
    auto kern = bwd_dkdv_kernel<D, CAUSAL, COUNT, PQ, NW>;
    static unsigned long long lds_set = 0;          // one per instantiation
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)smem, lds_set)) return -1;
    DkvArgs A = dkv_args(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, D, dk, dv, mx);
    A.tile_counts = tile_counts; A.pdump = p_dump; A.dump_row0 = dump_row0;
    hipLaunchKernelGGL(kern, dim3((unsigned)(B * Hkv * ((A.Lp + 32 * NW - 1) / (32 * NW)))), dim3(64 * NW), smem, st, A);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int D, bool CAUSAL>
static int launch_dkdv_t(const void* qb, const void* kb, const void* vb, const void* dob,
                         const float* rowstat, const float* bound_part,
                         int B, int Hq, int Hkv, int L, void* dk, void* dv, unsigned long long* tile_counts,
                         int p_quant, hipStream_t st, float* p_dump, int dump_row0, const MxScoreOps* mx)
{
    if (p_quant < 0 || p_quant > 3) return -1;
    if (p_quant == 2 && !(mx && mx->qops && mx->qsc && mx->kops && mx->ksc)) return -1;
    if (p_quant != 1) { if (p_dump) return -1; tile_counts = nullptr; }
#define AQ_DKV(COUNT, PQ, NW) launch_dkdv_v<D, CAUSAL, COUNT, PQ, NW>(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, dk, dv, \
                                                                       tile_counts, st, p_dump, dump_row0, mx)
    if (tile_counts || p_dump) return AQ_DKV(true, 1, 4);       // the counting / dumping variant
    if (p_quant == 0) return AQ_DKV(false, 0, 4);               // the ablation
    if (wide_workgroups(D, CAUSAL, (long long)B * Hkv * ((round_up(L, kRowPad) + 255) / 256), round_up(L, kRowPad)))
        return p_quant == 1 ? AQ_DKV(false, 1, 8) : p_quant == 2 ? AQ_DKV(false, 2, 8) : AQ_DKV(false, 3, 8);
    return p_quant == 1 ? AQ_DKV(false, 1, 4) : p_quant == 2 ? AQ_DKV(false, 2, 4) : AQ_DKV(false, 3, 4);
#undef AQ_DKV
}

int launch_bwd_dkdv(const void* qb, const void* kb, const void* vb, const void* dob,
                    const float* rowstat, const float* bound_part,
                    int B, int Hq, int Hkv, int L, int D, bool causal, void* dk, void* dv,
                    unsigned long long* tile_counts, int p_quant, hipStream_t st, float* p_dump, int dump_row0, const MxScoreOps* mx)
{
    if (D == 128) return causal ? launch_dkdv_t<128, true>(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, dk, dv, tile_counts, p_quant, st, p_dump, dump_row0, mx)
                                : launch_dkdv_t<128, false>(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, dk, dv, tile_counts, p_quant, st, p_dump, dump_row0, mx);
    if (D == 64)  return causal ? launch_dkdv_t<64, true>(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, dk, dv, tile_counts, p_quant, st, p_dump, dump_row0, mx)
                                : launch_dkdv_t<64, false>(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, dk, dv, tile_counts, p_quant, st, p_dump, dump_row0, mx);
    return -1;
}

// ------------------------------------------------------------------ both passes in one launch
// A problem that gives the chip few workgroups, or a last round that is mostly empty, runs both passes side by side (four-wave
// workgroups of either kind), and where even that leaves compute units idle, or a causal mask leaves one with a tile that is
// several times the average, the query tiles of a key tile are shared by several workgroups ("pieces" of about split_iters query
// tiles), whose fp32 sums dkdv_reduce_kernel adds in order.  The arithmetic of a tile and the order inside a piece are those of
// bwd_dkdv_kernel.  The dK/dV pieces come first, the dQ tiles fill in behind them (alternating the two kinds was 0 - 30 % slower),
// or the other way round where a dQ tile is the longer piece.  Measured, backward call, passes one after another -> joint
// without pieces -> as planned (plan.hpp): 2 x 16/4 heads, L = 3001 causal 617 -> 518 -> 292 us (MX 683 -> 596 -> 328 us);
// 8/2 heads, L = 8192 causal 1264 -> 1139 -> 475 us; 12 heads, L = 1560 120 -> 91 -> 82 us; 4 x 32/8 heads, L = 4096 causal
// 2.09 -> 1.85 ms (no pieces); 12 heads, L = 6240 833 -> 698 us (no pieces).
// The pieces of a kv head's key tiles under a causal mask, in the order in which they are handed out: the first piece of every tile, then the second of
// those that have one (the first tiles), and so on; without a mask all tiles have all pieces.  A lane counts the tiles that have piece number s0 + lane.
// Workgroups go to the XCDs in turn and, inside an XCD, to its four shader engines (eight compute units each) in turn, and one whose turn it is waits for room in
// its own engine while others have some.  So every four workgroups in a row of an XCD should take the same time.  Tile after tile with room for the largest number of
// pieces, four here, the fourth engine got the last pieces, shorter or empty, and stood idle: 384 workgroups at once instead of 512.  With this order,
// the joint launch: 2 x 16/4 heads, L = 3001 causal 304 -> 251 us (MX 288 -> 236 us); 2 x 32/8 heads 552 -> 474 us; 16/4 heads, L = 6000 520 -> 428 us.
__device__ __forceinline__ void piece_of_rank(int rank, const DkvArgs& K, int nt, int& kt, int& piece)
{
    const int lane = threadIdx.x & 63, nq32 = (K.L + 31) / 32;
    int base = 0, p = 0;
    for (int s0 = 0; s0 < K.splits; s0 += 64) {
        // (tile kt has (nq32 - 4 kt) G query tiles)
        const int more = nq32 - 1 - (int)((unsigned)(s0 + lane) * (unsigned)K.split_iters / (unsigned)K.G);
        int sum = more < 0 ? 0 : min(more / 4 + 1, nt);
#pragma unroll
        for (int d = 1; d < 64; d *= 2) { const int x = __shfl_up(sum, d); if (lane >= d) sum += x; }
        const unsigned long long past = __builtin_amdgcn_ballot_w64(rank < base + sum);
        if (past) {
            const int f = __builtin_ctzll(past);
            if (f > 0) base += __builtin_amdgcn_readlane(sum, f - 1);
            p = s0 + f;
            break;
        }
        base += __builtin_amdgcn_readlane(sum, 63);
    }
    kt = rank - base; piece = p;
}

template <int D, bool CAUSAL, int PQ, bool COUNT = false /* the measurement variant of bwd_dkdv_body */>
__global__ __launch_bounds__(256, D == 64 ? 3 : 2) void bwd_joint_kernel(DqArgs Q, DkvArgs K, int n_dkdv, int n_dq, int pieces /* of a kv head */, bool dq_first)
{
    const int nt = K.Lp / 128;
    int block = blockIdx.x;
    const bool dkdv = dq_first ? block >= n_dq : block < n_dkdv;
    if (dkdv == dq_first) block -= dq_first ? n_dq : n_dkdv;
    // Under a causal mask the longest tiles of all heads first (32 heads, L = 4096: 3 - 5 %), but head after head on long sequences,
    // where the heads an XCD works on would no longer share its L2 (4 x 32/8 heads, L = 8192: 7.0 against 7.4 ms in MX).
    const bool by_length = CAUSAL && K.Lp < 8192;
    auto place = [&](int heads, int per_head, int& head, int& rank) __attribute__((always_inline)) {
        if (by_length) {
            const bool pinned = (heads & 7) == 0;
            const int hx = pinned ? heads >> 3 : heads, i = pinned ? block >> 3 : block;
            head = pinned ? (block & 7) + 8 * (i % hx) : i % hx;
            rank = i / hx;
        } else head_tile_of_block(block, heads, per_head, head, rank);
    };
    int head, rank;
    if (dkdv) {
        if (block >= K.NHkv * pieces) return;                   // (n_dkdv and n_dq are rounded up to whole rounds of the XCDs)
        place(K.NHkv, pieces, head, rank);
        int piece = 0;
        if (K.splits > 1) {
            if constexpr (CAUSAL) piece_of_rank(rank, K, nt, rank, piece);
            else { piece = rank / nt; rank %= nt; }
        }
        bwd_dkdv_body<D, CAUSAL, COUNT, PQ, 4, true>(K, head, rank, piece);
    } else {
        if (block >= Q.NHq * nt) return;
        place(Q.NHq, nt, head, rank);
        bwd_dq_body<D, CAUSAL, PQ == 2, 4>(Q, head, CAUSAL ? nt - 1 - rank : rank);
    }
}

// dK and dV of the key tiles whose query tiles several workgroups shared: their fp32 sums added in order.  A workgroup takes 32
// columns of dK or dV of one key tile.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(256) void dkdv_reduce_kernel(const float* __restrict__ part, uint16_t* __restrict__ dK, uint16_t* __restrict__ dV,
                                                          int L, int Lp, int G, int splits, int split_iters)
{
    constexpr int NB = D / 32;
    const int nt = Lp / 128, tile = blockIdx.x / (2 * NB), col = blockIdx.x % (2 * NB);
    const int bhkv = tile / nt, kt = tile % nt;
    const int niter = ((L + 31) / 32 - (CAUSAL ? kt * 4 : 0)) * G, np = (niter + split_iters - 1) / split_iters;
    if (np < 2) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, ln = lane & 31, hf = lane >> 5;
    const floatx4* src = reinterpret_cast<const floatx4*>(part) + (size_t)tile * splits * (2 * NB * 4 * 256) + (size_t)col * (4 * 256) + threadIdx.x;
    floatx4 sum[4];
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4) sum[t4] = src[t4 * 256];
    for (int p = 1; p < np; ++p) {
        src += 2 * NB * 4 * 256;
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
            const floatx4 x = src[t4 * 256];
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[t4][e] += x[e];
        }
    }
    uint16_t* out = col < NB ? dK : dV;
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int key = kt * 128 + wave * 32 + 8 * t4 + 4 * hf + e;
            if (key < L) out[((size_t)bhkv * L + key) * D + 32 * (col % NB) + ln] = f32_to_bf16_rne(sum[t4][e]);
        }
}

// ------------------------------------------------------------------ few rows
// Both passes for problems that leave most compute units idle (few_rows), NVFP4 (the scores of the MX form and the row factor of the two-level form have not been
// written for it: their backwards of few rows take the joint launch).  What bounds those is the chain of one workgroup, tile after tile; here a
// workgroup owns 32 keys (or 32 query rows), its four waves take four query tiles (key tiles) at a time, wave w tile 4 n + w for S, dP, P^F and
// dS, and then one block of 32 columns of dK and of dV (of dQ) for the products of all four, whose P^F and dS they find in LDS: a chain is a quarter as
// long, and every sum has the order, so every result the bits, of the kernels above.  Two barriers per four tiles; one workgroup per compute unit,
// whose waves have the registers of two.  V^F of a dQ tile goes straight to registers: nobody else reads it, and the LDS has no room for two rounds of it.
// Joint launch -> this, with the preparing launch: d = 64: 2 heads, L = 256 16.3 -> 12.0 us, L = 700 27.4 -> 17.8 us; 4 heads, L = 1000 30.3 -> 21.6 us;
// 12 heads, L = 200 17.0 -> 13.2 us; one head, L = 2000 58.8 -> 32.4 us; d = 128: 2 heads, L = 700 35.6 -> 23.6 us, 4 heads, L = 1000 38.3 -> 30.4 us, 8 heads,
// L = 700 causal 35.1 -> 26.2 us.
template <int D>
struct FewDkv {
    uint16_t q[2][4][32 * D];            // Q^F tiles of this round and the next [query][d], fp16, swizzled
    uint16_t g[2][4][32 * D];            // dO tiles
    uint16_t t[4][2][kTTileB / 2];       // P^F and dS of the four tiles, as in DkvSmem
    int pf[4];                           // whether tile t has a non-zero P^F
};
template <int D>
struct FewDq {
    uint16_t k[2][4][64 * D];            // K^F tiles of this round and the next [key][d], fp16, swizzled
    uint4v ds[4][4][64];                 // dS of the four tiles as operands of the dQ products: [tile][16 keys][lane]
};

// What this wave has written to LDS is there, what it has read has arrived, and the other waves have got here too (the copies and loads of the next
// round stay on their way).
__device__ __forceinline__ void few_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);                  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

template <int D, bool CAUSAL>
__device__ __forceinline__ void few_dkdv(const DkvArgs& A, int bhkv, int kt /* 32 keys */)
{
    constexpr int DS = D / 16, NB = D / 32, KCH = D / 8, NWL = D / 16 /* 1 KiB copies of a tile */;
    constexpr uint32_t kRowB = 2 * D, kTB = 32 * kRowB, kGB = 8 * kTB;
    extern __shared__ __align__(256) unsigned char smem_raw[];
    FewDkv<D>& sm = *reinterpret_cast<FewDkv<D>*>(smem_raw);
    const int L = A.L, Lp = A.Lp, Hq = A.Hq, G = A.G, Hkv = Hq / G;
    const int b = bhkv / Hkv, hk = bhkv % Hkv;
    const int lane = threadIdx.x & 63, ln = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int key0 = kt * 32;

    uint4v kreg[DS], vreg[DS];                           // A operands: row = key, d-slots 16 ds + 8 hf
    {
        const size_t off = ((size_t)bhkv * Lp + key0 + ln) * D + 8 * hf;
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
            kreg[ds] = *reinterpret_cast<const uint4v*>(A.Kb + off + 16 * ds);
            vreg[ds] = *reinterpret_cast<const uint4v*>(A.Vb + off + 16 * ds);
        }
    }
    // query tiles of 32 rows, query heads of the group one after another; this wave's in round r is number 4 r + wave
    const int qt_first = CAUSAL ? kt : 0, per_head = (L + 31) / 32 - qt_first, niter = per_head * G;
    const size_t bh0 = (size_t)b * Hq + hk * G;
    auto row_of = [&](int it) __attribute__((always_inline)) { return (bh0 + it / per_head) * Lp + (size_t)(qt_first + it % per_head) * 32; };
    uint32_t slot_off[NWL];
#pragma unroll
    for (int i = 0; i < NWL; ++i) {
        const int slot = 64 * i + lane;
        slot_off[i] = 2u * (uint32_t)((slot / KCH) * D + 8 * swz<KCH>(slot / KCH, slot % KCH));
    }
    float2 st_n = make_float2(0.0f, 0.0f);
    auto request = [&](int buf, int it) __attribute__((always_inline)) {
        if (it >= niter) return;
        const size_t row0 = row_of(it);
#pragma unroll
        for (int i = 0; i < NWL; ++i) {
            async_copy16(A.Qb + row0 * D, slot_off[i], &sm.q[buf][wave][512 * i]);
            async_copy16(A.dOb + row0 * D, slot_off[i], &sm.g[buf][wave][512 * i]);
        }
        st_n = A.rowstat[row0 + ln];
    };
    request(0, wave);
    // (the factor of dS: as in bwd_dkdv_body)
    float ds_scale;
    {
        const float* p = A.bound_part + (size_t)bhkv * kBoundParts + lane;
        const float *p1 = A.bound_part + ((size_t)A.NHq + bh0) * kBoundParts + lane, *p2 = p1 + (size_t)A.NHq * kBoundParts;
        float vmax = *p, domax = 0.0f, dmax = 0.0f;
        for (int g = 0; g < G; ++g) { domax = fmaxf(domax, p1[(size_t)g * kBoundParts]); dmax = fmaxf(dmax, p2[(size_t)g * kBoundParts]); }
        vmax = lanes_max<32, 1>(vmax); domax = lanes_max<32, 1>(domax); dmax = lanes_max<32, 1>(dmax);
        ds_scale = ds_scale_for(domax * vmax * A.rs + dmax);
    }
    const float rs_s = A.rs * ds_scale;

    const uint32_t lds0 = lds_addr_of(smem_raw), t0 = lds_addr_of(&sm.t[0][0][0]);
    const int tr_r = lane & 15, tr_grp = (lane >> 4) & 1;
    const uint32_t a_rd = lds0 + 2u * (uint32_t)swz_elem<KCH>(ln, 8 * hf) + (uint32_t)wave * kTB;
    // this wave's block: columns 32 nb .. of dK and dV (d = 64: of dK, waves 0 and 1, or of dV)
    constexpr bool BOTH = NB == 4;
    const int nb = BOTH ? wave : wave & 1;
    const bool do_k = BOTH || wave < 2, do_v = BOTH || wave >= 2;
    uint32_t g_rd[2];
#pragma unroll
    for (int v = 0; v < 2; ++v) g_rd[v] = (lds0 + 2u * (uint32_t)swz_elem<KCH>(8 * hf + (tr_r >> 2) + 4 * v, 16 * tr_grp + 4 * (tr_r & 3))) ^ (uint32_t)(nb << 6);
    const uint32_t tw_ad = t0 + (uint32_t)(wave * 2 * kTTileB + kTGroupB * (ln >> 2) + 64 * (ln & 3) + 8 * (hf ^ ((ln >> 1) & 1)));
    const uint32_t ta_ad = t0 + (uint32_t)(kTGroupB * (2 * hf) + 64 * (tr_r >> 2) + 32 * tr_grp + 8 * ((tr_r & 3) ^ ((tr_r >> 3) & 1)));
    floatx16 dk, dv;
#pragma unroll
    for (int i = 0; i < 16; ++i) { dk[i] = 0.0f; dv[i] = 0.0f; }
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) asm volatile("" : "+v"(kreg[ds]), "+v"(vreg[ds]));
    asm volatile("" : "+v"(st_n.x), "+v"(st_n.y));
    __builtin_amdgcn_s_waitcnt(0);

    for (int r0 = 0, buf = 0; r0 < niter; r0 += 4, buf ^= 1) {
        const int it = r0 + wave, nt = min(niter - r0, 4);
        const float Ls = st_n.x, Dq_s = st_n.y * rs_s;
        request(buf ^ 1, it + 4);
        if (it < niter) {
            const int q0 = (qt_first + it % per_head) * 32;
            const uint32_t a_it = a_rd + (uint32_t)buf * (4 * kTB);
            uint4v qo[DS], go[DS];
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) { qo[ds] = lds_read16_at(a_it ^ (uint32_t)(ds << 5)); go[ds] = lds_read16_at((a_it ^ (uint32_t)(ds << 5)) + kGB); }
            floatx16 s, dp;
#pragma unroll
            for (int i = 0; i < 16; ++i) { s[i] = 0.0f; dp[i] = 0.0f; }
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) { s = mfma_f16(kreg[ds], qo[ds], s); dp = mfma_bf16(vreg[ds], go[ds], dp); }
            if ((key0 + 32 > L) || (CAUSAL && key0 + 31 > q0)) {
                const int klim = CAUSAL ? min(L - 1, q0 + ln) : L - 1;
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (key0 + 8 * (i >> 2) + 4 * hf + (i & 3) > klim) s[i] = -INFINITY;
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], A.c, -Ls));    // P = exp(S - L_i)
            float gmax[2];
#pragma unroll
            for (int gq = 0; gq < 2; ++gq) gmax[gq] = nvfp4_group_max(s, gq);
            const bool with_pf = __builtin_amdgcn_ballot_w64(nvfp4_scale_nonzero(fmaxf(gmax[0], gmax[1]))) != 0;
            if (lane == 0) sm.pf[wave] = with_pf;
            if (with_pf) {
                float sc[2], inv[2];
                nvfp4_pair_scales(gmax, sc, inv);
#pragma unroll
                for (int t4 = 0; t4 < 4; ++t4) lds_write8_at(tw_ad + (uint32_t)(16 * t4), nvfp4_pf_quad(s, 4 * t4, sc[t4 >> 1], inv[t4 >> 1]));
            }
#pragma unroll
            for (int t4 = 0; t4 < 4; ++t4) {
                float dsv[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) dsv[e] = s[4 * t4 + e] * fmaf(dp[4 * t4 + e], rs_s, -Dq_s);
                uint2v wh;
                wh[0] = pack_f16x2(dsv[0], dsv[1]); wh[1] = pack_f16x2(dsv[2], dsv[3]);
                lds_write8_at(tw_ad + (uint32_t)(kTTileB + 16 * t4), wh);
            }
        }
        few_barrier();
        // dK += dS^T Q^F, dV += P^F^T dO, tile after tile (contraction slots as in bwd_dkdv_body)
        auto product = [&](int t, uint32_t staged, uint32_t rows, int ks, uint4v& a, uint4v& bq) __attribute__((always_inline)) {
            const uint32_t ta = ta_ad + (uint32_t)(t * 2 * kTTileB) + staged + (uint32_t)(ks * (4 * kTGroupB)), o = (uint32_t)((buf * 4 + t) * kTB) + rows + (uint32_t)(ks * 16 * kRowB);
            a = join(lds_read_tr16_at(ta), lds_read_tr16_at(ta + kTGroupB));
            bq = join(lds_read_tr16_at(g_rd[0] + o), lds_read_tr16_at(g_rd[1] + o));
        };
        auto tiles = [&](auto full) __attribute__((always_inline)) {
            constexpr bool FULL = decltype(full)::value;
            uint4v a[4][2], bq[4][2];
            if (do_k) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (FULL || t < nt)
#pragma unroll
                        for (int ks = 0; ks < 2; ++ks) product(t, kTTileB, 0u, ks, a[t][ks], bq[t][ks]);
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (FULL || t < nt)
#pragma unroll
                        for (int ks = 0; ks < 2; ++ks) dk = mfma_f16(a[t][ks], bq[t][ks], dk);
            }
            if (do_v) {
                int pf[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) pf[t] = __builtin_amdgcn_readfirstlane(sm.pf[t]);
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if ((FULL || t < nt) && pf[t])
#pragma unroll
                        for (int ks = 0; ks < 2; ++ks) product(t, 0u, kGB, ks, a[t][ks], bq[t][ks]);
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if ((FULL || t < nt) && pf[t])
#pragma unroll
                        for (int ks = 0; ks < 2; ++ks) dv = mfma_bf16(a[t][ks], bq[t][ks], dv);
            }
        };
        if (nt == 4) tiles(std::true_type{}); else tiles(std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0);                   // this wave's tile of the next round is in LDS
        few_barrier();
        asm volatile("" : "+v"(st_n.x), "+v"(st_n.y));
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int key = key0 + 8 * (i >> 2) + 4 * hf + (i & 3);
        if (key < L) {
            const size_t o = ((size_t)bhkv * L + key) * D + 32 * nb + ln;
            if (do_k) A.dK[o] = f32_to_bf16_rne(dk[i] * (A.rs / rs_s));          // / ds_scale, exact: a power of two
            if (do_v) A.dV[o] = f32_to_bf16_rne(dv[i]);
        }
    }
}

template <int D, bool CAUSAL>
__device__ __forceinline__ void few_dq(const DqArgs& A, int bh, int qt /* 32 rows */)
{
    constexpr int DS = D / 16, MB = D / 32, KCH = D / 8, KLD = D / 8 /* 1 KiB copies of a tile */;
    constexpr uint32_t kTB = 64 * D * 2;
    extern __shared__ __align__(256) unsigned char smem_raw[];
    FewDq<D>& sm = *reinterpret_cast<FewDq<D>*>(smem_raw);
    const int L = A.L, Lp = A.Lp, Hq = A.Hq, G = A.G;
    const int b = bh / Hq, h = bh % Hq, bhkv = b * (Hq / G) + h / G;
    const int lane = threadIdx.x & 63, ln = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int row0 = qt * 32, q_row = row0 + ln;
    const int nkt_all = (L + 63) / 64, nkt = CAUSAL ? min((row0 + 31) / 64 + 1, nkt_all) : nkt_all;

    const uint16_t* k_head = A.Kb + (size_t)bhkv * Lp * D;
    const uint16_t* v_lane = A.Vb + ((size_t)bhkv * Lp + ln) * D + 8 * hf;
    uint32_t k_ld[KLD];
#pragma unroll
    for (int i = 0; i < KLD; ++i) {
        const int slot = 64 * i + lane, r = slot / KCH, pc = slot % KCH;
        k_ld[i] = 2u * (uint32_t)(r * D + 8 * swz<KCH>(r, pc));
    }
    uint4v vn[2][DS];                                    // V^F rows of this wave's next tile: nobody else reads them
    auto request = [&](int buf, int j) __attribute__((always_inline)) {
        if (j >= nkt) return;
#pragma unroll
        for (int i = 0; i < KLD; ++i) async_copy16(k_head + (size_t)j * (64 * D), k_ld[i], &sm.k[buf][wave][512 * i]);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) vn[kb][ds] = *reinterpret_cast<const uint4v*>(v_lane + (size_t)(j * 64 + 32 * kb) * D + 16 * ds);
    };
    uint4v qreg[DS], doreg[DS];
    {
        const size_t off = ((size_t)bh * Lp + q_row) * D + 8 * hf;
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) {
            qreg[ds] = *reinterpret_cast<const uint4v*>(A.Qb + off + 16 * ds);
            doreg[ds] = *reinterpret_cast<const uint4v*>(A.dOb + off + 16 * ds);
        }
    }
    const float2 st_ = A.rowstat[(size_t)bh * Lp + q_row];
    const float vmax_part = A.bound_part[(size_t)bhkv * kBoundParts + lane];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) vn[kb][ds] = uint4v{0u, 0u, 0u, 0u};
    request(0, wave);
    float ds_scale, do_scale;
    dq_row_scale<true>(doreg, lanes_max<32, 1>(vmax_part), st_.y, A.rs, ds_scale, do_scale);
    const float Ls = dq_row_exponent<D>(st_.x, ds_scale, do_scale);
    floatx16 dp0, acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) { dp0[i] = -st_.y * do_scale; acc[i] = 0.0f; }

    const uint32_t lds0 = lds_addr_of(smem_raw), ds0 = lds_addr_of(&sm.ds[0][0][0]);
    const int tr_r = lane & 15, tr_grp = (lane >> 4) & 1;
    const int mb = wave & (MB - 1);
    const bool do_q = wave < MB;                         // d = 64: two blocks of dQ
    uint32_t koff[DS], toff[2];
#pragma unroll
    for (int ds = 0; ds < DS; ++ds) koff[ds] = lds0 + (uint32_t)wave * kTB + 2u * (uint32_t)((ln * KCH + swz<KCH>(ln, 2 * ds + hf)) * 8);
#pragma unroll
    for (int v = 0; v < 2; ++v) toff[v] = lds0 + 2u * (uint32_t)swz_elem<KCH>(4 * hf + (tr_r >> 2) + 8 * v, 32 * mb + 16 * tr_grp + 4 * (tr_r & 3));
    __builtin_amdgcn_s_waitcnt(0);

    for (int j0 = 0, buf = 0; j0 < nkt; j0 += 4, buf ^= 1) {
        const int j = j0 + wave, nt = min(nkt - j0, 4);
        uint4v vc[2][DS];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) vc[kb][ds] = vn[kb][ds];
        request(buf ^ 1, j + 4);
        if (j < nkt) {
            const int k0 = j * 64;
            floatx16 s[2], dp[2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) s[kb][i] = 0.0f;
#pragma unroll
            for (int ds = 0; ds < DS; ++ds)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    s[kb] = mfma_f16(lds_read16_at(koff[ds] + (uint32_t)buf * (4 * kTB) + (uint32_t)(kb * 32 * D * 2)), qreg[ds], s[kb]);
                    dp[kb] = mfma_bf16(vc[kb][ds], doreg[ds], ds == 0 ? dp0 : dp[kb]);
                }
            if ((k0 + 64 > L) || (CAUSAL && k0 + 63 > row0)) {
                const int klim = CAUSAL ? min(L - 1, q_row) : L - 1;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (k0 + 32 * kb + 8 * (i >> 2) + 4 * hf + (i & 3) > klim) s[kb][i] = -INFINITY;
            }
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                uint4v bds;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int kb = ks >> 1, r = 8 * (ks & 1) + 2 * i;
                    const float p0 = __builtin_amdgcn_exp2f(fmaf(s[kb][r], A.c, -Ls)), p1 = __builtin_amdgcn_exp2f(fmaf(s[kb][r + 1], A.c, -Ls));
                    bds[i] = pack_f16x2(p0 * dp[kb][r], p1 * dp[kb][r + 1]);
                }
                lds_write16_at(ds0 + (uint32_t)((wave * 4 + ks) * 1024 + 16 * lane), bds);
            }
        }
        few_barrier();
        if (do_q) {
            auto tiles = [&](auto full) __attribute__((always_inline)) {
                constexpr bool FULL = decltype(full)::value;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (FULL || t < nt)
#pragma unroll
                        for (int ks = 0; ks < 4; ++ks) {
                            const uint32_t o = (uint32_t)((buf * 4 + t) * kTB) + (uint32_t)(ks * 16 * D * 2);
                            const uint4v at = join(lds_read_tr16_at(toff[0] + o), lds_read_tr16_at(toff[1] + o));
                            acc = mfma_f16(at, lds_read16_at(ds0 + (uint32_t)((t * 4 + ks) * 1024 + 16 * lane)), acc);
                        }
            };
            if (nt == 4) tiles(std::true_type{}); else tiles(std::false_type{});
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0);                   // this wave's tile of the next round is in LDS
        few_barrier();
    }
    if (q_row < L && do_q) {
        const float un = 1.0f / ds_scale;                // exact: a power of two
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint2v w;
            w[0] = pack_bf16x2(acc[4 * t] * un, acc[4 * t + 1] * un);
            w[1] = pack_bf16x2(acc[4 * t + 2] * un, acc[4 * t + 3] * un);
            *reinterpret_cast<uint2v*>(A.dQ + ((size_t)bh * L + q_row) * D + 32 * mb + 8 * t + 4 * hf) = w;
        }
    }
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, 1) void bwd_few_kernel(DqArgs Q, DkvArgs K)
{
    const int n32 = (K.L + 31) / 32, n_dkdv = K.NHkv * n32;
    int block = blockIdx.x;                              // (under a causal mask the longest first)
    if (block < n_dkdv) few_dkdv<D, CAUSAL>(K, block % K.NHkv, block / K.NHkv);
    else {
        block -= n_dkdv;
        few_dq<D, CAUSAL>(Q, block % Q.NHq, CAUSAL ? n32 - 1 - block / Q.NHq : block / Q.NHq);
    }
}

bool bwd_few_rows(int BHq, int BHkv, int L, bool causal, bool pieces, int cus)
{
    if (__atomic_load_n(&g_bwd_waves, __ATOMIC_RELAXED) != 0) return false;      // (a test forces separate passes)
    return few_rows(BHq, BHkv, L, causal, pieces, cus);
}

int launch_bwd_few(const void* qb, const void* kb, const void* vb, const void* dob, const float* rowstat, const float* bound_part,
                   int B, int Hq, int Hkv, int L, int D, bool causal, void* dq, void* dk, void* dv, hipStream_t st)
{
    const DqArgs Q = dq_args(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, D, dq, nullptr);
    const DkvArgs K = dkv_args(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, D, dk, dv, nullptr);
    auto go = [&](auto kern, size_t smem, unsigned long long& lds_set) -> int {
        if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)smem, lds_set)) return -1;
        hipLaunchKernelGGL(kern, dim3((unsigned)((Q.NHq + K.NHkv) * ((L + 31) / 32))), dim3(256), smem, st, Q, K);
        return hipGetLastError() == hipSuccess ? 0 : -1;
    };
    static unsigned long long lds_set[4] = {0, 0, 0, 0};      // one per instantiation
#define AQ_FEW(DD, C, I) go(bwd_few_kernel<DD, C>, sizeof(FewDkv<DD>) > sizeof(FewDq<DD>) ? sizeof(FewDkv<DD>) : sizeof(FewDq<DD>), lds_set[I])
    if (D == 128) return causal ? AQ_FEW(128, true, 0) : AQ_FEW(128, false, 1);
    if (D == 64)  return causal ? AQ_FEW(64, true, 2) : AQ_FEW(64, false, 3);
#undef AQ_FEW
    return -1;
}

BwdPlan bwd_plan(int BHq, int BHkv, int L, int D, bool causal, int cus)
{
    if (__atomic_load_n(&g_bwd_waves, __ATOMIC_RELAXED) != 0) return BwdPlan{false, 1, 0, 0, false};      // (a test forces separate passes)
    const BwdPlan p = plan_backward(BHq, BHkv, L, D, causal, cus);
    // d = 64: three four-wave workgroups of the joint launch share a compute unit, where an eight-wave one has it to itself (its registers
    // would have to halve).  Training step, separate passes of eight -> joint: 24 heads, L = 8192 2270 -> 1993 us, MX 16 heads 1476 -> 1304 us;
    // 16 heads, L = 32768 causal 11.80 -> 9.50 ms, MX 11.96 -> 9.80 ms.  (Separate passes of four: 1 % behind the joint launch.)
    // Where three lose against two, the launch asks for two (joint_in_pairs).
    if (p.joint || D != 64) return p;
    return BwdPlan{true, 1, (L + 31) / 32 * (BHq / BHkv), 0, false};
}

template <int D, bool CAUSAL, int PQ, bool COUNT = false>
static int launch_joint_t(const DqArgs& Q, DkvArgs K, const BwdPlan& plan, float* part, hipStream_t st)
{
    const size_t dq_lds = sizeof(DqSmem<D, PQ == 2>), dkv_lds = sizeof(DkvSmem<D, PQ == 2, 4>), need = dq_lds > dkv_lds ? dq_lds : dkv_lds;
    constexpr size_t kPairLds = (size_t)64 << 10;   // two fit into the 160 KiB of a compute unit, three do not
    static_assert(D != 64 || (sizeof(DqSmem<D, PQ == 2>) <= kPairLds && sizeof(DkvSmem<D, PQ == 2, 4>) <= kPairLds), "LDS of the joint kernel");
    const size_t smem = joint_in_pairs(plan, Q.NHq, K.NHkv, K.L, D, CAUSAL, device_cu_count()) ? kPairLds : need;
    auto kern = bwd_joint_kernel<D, CAUSAL, PQ, COUNT>;
    static unsigned long long lds_set = 0;          // one per instantiation
    if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)(D == 64 ? kPairLds : need), lds_set)) return -1;
    K.splits = plan.splits; K.split_iters = plan.iters; K.part = part;
    const int nt = K.Lp / 128;
    int pieces = nt * K.splits;
    if (CAUSAL && K.splits > 1) {
        pieces = 0;
        for (int kt = 0; kt < nt; ++kt) pieces += (int)(((unsigned)((K.L + 31) / 32 - 4 * kt) * (unsigned)K.G + (unsigned)K.split_iters - 1) / (unsigned)K.split_iters);
    }
    const int n_dkdv = round_up(K.NHkv * pieces, 8), n_dq = round_up(Q.NHq * nt, 8);
    hipLaunchKernelGGL(kern, dim3((unsigned)(n_dkdv + n_dq)), dim3(256), smem, st, Q, K, n_dkdv, n_dq, pieces, plan.dq_first);
    if (hipGetLastError() != hipSuccess) return -1;
    if (plan.splits > 1)
        hipLaunchKernelGGL((dkdv_reduce_kernel<D, CAUSAL>), dim3((unsigned)(K.NHkv * nt * 2 * (D / 32))), dim3(256), 0, st,
                           part, K.dK, K.dV, K.L, K.Lp, K.G, K.splits, K.split_iters);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_bwd_joint(const void* qb, const void* kb, const void* vb, const void* dob, const float* rowstat, const float* bound_part,
                     int B, int Hq, int Hkv, int L, int D, bool causal, void* dq, void* dk, void* dv, int p_quant,
                     const BwdPlan& plan, float* part, unsigned long long* tile_counts, hipStream_t st, float* p_dump, int dump_row0,
                     const MxScoreOps* mx)
{
    if (p_quant != 1) { if (p_dump) return -1; tile_counts = nullptr; }
    if (p_quant < 1 || p_quant > 3 || (p_quant == 2) != (mx != nullptr) || (plan.splits > 1 && !part)) return -1;
    const DqArgs Q = dq_args(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, D, dq, mx);
    DkvArgs K = dkv_args(qb, kb, vb, dob, rowstat, bound_part, B, Hq, Hkv, L, D, dk, dv, mx);
    K.tile_counts = tile_counts; K.pdump = p_dump; K.dump_row0 = dump_row0;
    const bool count = tile_counts || p_dump;
#define AQ_J(DD, C) (count ? launch_joint_t<DD, C, 1, true>(Q, K, plan, part, st) : p_quant == 1 ? launch_joint_t<DD, C, 1>(Q, K, plan, part, st) : p_quant == 2 ? launch_joint_t<DD, C, 2>(Q, K, plan, part, st) \
                                                                                   : launch_joint_t<DD, C, 3>(Q, K, plan, part, st))
    if (D == 128) return causal ? AQ_J(128, true) : AQ_J(128, false);
    if (D == 64)  return causal ? AQ_J(64, true) : AQ_J(64, false);
#undef AQ_J
    return -1;
}

}  // namespace aq
