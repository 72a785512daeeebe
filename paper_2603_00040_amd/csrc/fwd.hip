// Fused forward of Attn-QAT on gfx950: Alg. 1 (inference) and Alg. 2 (training).
//
// Work split: a workgroup of 8 waves owns 256 query rows of one head; each wave owns 32
// of them.  Key tiles of B_k = 64 keys are visited in increasing order; K and V^T tiles
// are copied global->LDS directly (global_load_lds, double buffered, in the order of the
// matrix instruction's operands) and shared by the eight waves.  Waves 0-3 and waves 4-7 run half an iteration apart
// (vector phase / matrix phase, separated by barriers).  Problems that do not fill the chip with
// such workgroups run four waves and 128 rows (fwd_narrow_kernel, chosen by narrow_workgroups):
// the same arithmetic in the same order, one barrier per tile, two workgroups per compute unit;
// and the smallest four waves that share 32 rows (fwd_split_kernel, chosen by split_key_tiles).
//
// MFMA shapes (v_mfma_f32_32x32x16_f16, fp32 accumulate).  All operands are the
// dequantized NVFP4 values s*c, which fp16 represents exactly, so the products are those
// of Eq. 4 (BF16MM on fake-quantized operands == FP4MM of Eq. 3).
//   S^T[key, query]   = K^F (A, from LDS)   x  Q^F^T (B, registers, made of Q here)
//   O^T[d, query]    += V^F^T (A, from LDS) x  P-tilde^F^T (B, registers)
//   O'^T[d, query]   += V^F^T (same A)      x  P-tilde^T   (B, registers; training only)
// With S transposed, a lane owns ONE query row and 8+8 keys of every aligned group of 16
// keys: the row max, the row sum and the 16-key block max of phi(P-tilde) are register
// reductions plus one exchange between the two 32-lane halves, and the accumulator
// layout of S^T already is the B-operand layout of the P.V products (V^T is stored with
// the matching key permutation, see v_operand_offset).
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "mx_quant.hpp"
#include "nvfp4.hpp"

namespace aq {

template <int D>
struct FwdSmem {
    half_t k[2][64 * D];      // K tile in the order of the S products' operands (k_operand_offset)
    half_t v[2][D * 64];      // V^T tile, in the order of the P V products' (v_operand_offset)
};

// PQ, the format of P-tilde in the P V product: 0 NVFP4, 1 MX, 2 NVFP4 with the two-level row factor,
// 3 bf16 with V left in bf16 as well (the mixed recipe "NVFP4 Q K^T, BF16 P V" of Sec. 2.5; the tile buffer of V^T then
// holds bf16 bit patterns and the P V products are bf16 MFMAs; inference only).
// VARLEN (serving): every sequence b has its own number of keys kv_lens[b] (read here, on the device), the copies of K and V^T
// are laid out for Lkp positions per head, and the L query rows are the LAST L positions of their sequence: under the causal
// mask query i sees keys 0 .. kv_lens[b] - L + i (a chunk of a prefill; needs kv_lens[b] >= L).
// SPLIT (fwd_split_kernel): the four waves share 32 query rows and take four key tiles at a time; see there.
template <int D, bool TRAIN, bool CAUSAL, bool DUMP, int PQ, bool VARLEN, int NW, bool SPLIT = false>
__device__ __forceinline__ void fwd_body(
    const half_t* __restrict__ Qh, const half_t* __restrict__ Kh, const half_t* __restrict__ Vt,
    uint16_t* __restrict__ O, float* __restrict__ lse, float* __restrict__ Ohp,
    int L, int Lp, int Hq, int G, float c /* log2(e)/sqrt(d) */, int dump_row0, float* __restrict__ pdump,
    int Lkp_arg, const int* __restrict__ kv_lens, int B /* batch (VARLEN: sequences) */, int q_copy)
{
    constexpr int KS = SPLIT ? NW : 1;
    constexpr int QT = 32 * NW / KS;       // query rows of a workgroup
    constexpr bool PHASES = NW == 8 && !SPLIT, PAIRED = CAUSAL && PHASES;
    // PQ == 1 (MX): S = Q^F K^F^T comes from the E2M1 codes and E8M0 scales by v_mfma_scale_f32_32x32x64_f8f6f4 (a quarter of
    // the matrix time of the 16-bit products, a quarter of the K bytes through LDS).  Qh then is Q itself in bf16, of which
    // the waves make the operands of that instruction (MxQ), and Kh the K records of mx_ktrain_rec_bytes(D) bytes per key tile.  The accumulator layout is
    // that of the 16-bit products, so everything after the scores is unchanged (O and O' stay 16-bit products: O' needs the
    // un-quantized P-tilde, which is no operand of that instruction).
    constexpr bool MXS = PQ == 1;
    constexpr int KSM = D / 64, KREC = mx_ktrain_rec_bytes(D);
    typedef int int8v __attribute__((ext_vector_type(8)));
    constexpr int DS = D / 16;      // contraction steps of S
    constexpr int MB = D / 32;      // 32-row blocks of O^T
    constexpr int OB = MB >= KS ? MB / KS : 1;      // those of a wave
    constexpr bool BOTH = MB >= KS;                 // a wave has its blocks of O and of O' (else: of either, or of nothing)
    constexpr int KLD = D / 8 / NW; // 1 KiB wave-loads per wave for the K tile
    constexpr int VLD = D / 8 / NW; // ... for the V^T tile
    extern __shared__ __align__(256) unsigned char smem_raw[];
    FwdSmem<D>& sm = *reinterpret_cast<FwdSmem<D>*>(smem_raw);

    // Work items: a tile of 256 query rows of one head.  Without a mask a workgroup takes one.  Under a causal mask tile qt
    // visits 4 qt + 4 key tiles, so a workgroup takes a pair, tile nqt - 1 - p and then tile p: every workgroup then does
    // the same amount of work (no tail of long tiles at the end of a head) and there are half as many workgroups, each of
    // which costs the CU a fixed 20 - 30 us of start-up and wind-down that nothing overlaps at one workgroup per CU.
    // Four waves (128 rows): one tile per workgroup, the longest first under a causal mask.
    const int nqt = SPLIT ? (L + QT - 1) / QT : (Lp + QT - 1) / QT;
    const int per_head = PAIRED ? (nqt + 1) / 2 : nqt;
    int bh, qt0;
    if constexpr (VARLEN && !PHASES) {
        if (!varlen_item(blockIdx.x, kv_lens, B, Hq, G, nqt, bh, qt0)) return;
    } else if (CAUSAL && !PHASES) longest_first(blockIdx.x, B * Hq, per_head, bh, qt0);
    // (The heads from the arguments, or from the grid: the same number, but the longer entry moves the key loop, see fwd_mx_kernel.
    //  Training, eight waves: 4 x 64/8 heads, L = 4096, d = 64 1903 -> 1884 us from the grid, d = 128 even; inference and four waves
    //  are better off without the division: 2 x 12 heads, L = 32760, d = 128 11.31 -> 11.24 ms, 2 heads, L = 256 training step 30.6 -> 30.3 us.)
    else head_tile_of_block(blockIdx.x, TRAIN && PHASES ? gridDim.x / per_head : B * Hq, per_head, bh, qt0);
    const int nitems = (PAIRED && nqt - 1 - qt0 != qt0) ? 2 : 1;
    const int b = bh / Hq, h = bh % Hq;
    const int bhkv = b * (Hq / G) + h / G;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);        // scalar: LDS destinations and branches use it
    const bool late = PHASES && wave >= 4;               // the group that runs one phase behind
    // keys of this sequence, row stride of the K / V^T copies, and how far the causal diagonal is shifted
    const int Lk = VARLEN ? max(1, min(kv_lens[b], Lkp_arg)) : L;
    const int Lkp = VARLEN ? Lkp_arg : Lp;
    const int off = (VARLEN && CAUSAL) ? max(0, Lk - L) : 0;
    const int nkt_all = (Lk + 63) / 64;

    for (int item = 0; item < nitems; ++item) {
    // (the lane number is taken afresh for every item and made opaque: everything formed from it would otherwise be kept
    //  in registers, or rather in scratch, across the key loop for the sake of the second item)
    uint32_t lane_i = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(lane_i));
    const int lane = (int)lane_i, ln = lane & 31, hf = lane >> 5;

    // The copies lie in memory, and so in LDS, in the order of the operands: operand i of a tile is the KiB at 1024 i, of which a
    // lane takes the 16 bytes at 16 lane.  Copies and reads are then one lane offset plus constants (an LDS read's own offset
    // field): rows in LDS, their chunks swizzled against bank conflicts, cost an XOR per read and two offset registers, and the
    // vector pipe is what bounds these kernels.
    const unsigned char* kbase = reinterpret_cast<const unsigned char*>(&sm.k[0][0]);
    const unsigned char* vbase = reinterpret_cast<const unsigned char*>(&sm.v[0][0]);

    const half_t* k_head = Kh + (size_t)bhkv * Lkp * D;      // tiles of 64 keys, 64 D values each
    const half_t* v_head = Vt + (size_t)bhkv * D * Lkp;
    const unsigned char* k_recs = reinterpret_cast<const unsigned char*>(Kh) + (size_t)bhkv * (Lkp / 64) * KREC;
    auto issue_k = [&](int buf, int jt) __attribute__((always_inline)) {
        if constexpr (MXS) {      // a record is KREC / 1024 wave copies of 1 KiB
#pragma unroll
            for (int i = 0; i < (KREC / 1024 + NW - 1) / NW; ++i) {
                const int ch = wave + i * NW;
                if (ch < KREC / 1024)
                    async_copy16(k_recs + (size_t)jt * KREC, (uint32_t)(ch * 1024 + lane * 16), reinterpret_cast<unsigned char*>(&sm.k[buf][0]) + ch * 1024);
            }
        } else {
#pragma unroll
            for (int i = 0; i < KLD; ++i)
                async_copy16(k_head + (size_t)jt * (64 * D) + 512 * (wave * KLD + i), 16u * (uint32_t)lane, &sm.k[buf][512 * (wave * KLD + i)]);
        }
    };
    auto issue_v = [&](int buf, int jt) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < VLD; ++i)
            async_copy16(v_head + (size_t)jt * (64 * D) + 512 * (wave * VLD + i), 16u * (uint32_t)lane, &sm.v[buf][512 * (wave * VLD + i)]);
    };

    const int qt = CAUSAL ? (item == 0 ? nqt - 1 - qt0 : qt0) : qt0;      // (four waves: item is 0)
    const int row0_w = qt * QT + (SPLIT ? 0 : wave * 32);
    const bool has_rows = !PHASES || row0_w < Lp;        // false only in the last tile of a head (Lp is a multiple of 128)
    const int q_row = row0_w + ln;

    // Q^F operand: this lane's query row, d-slots 16*ds + 8*hf .. +7.  phi(Q) is made here, in registers (about 360 vector instructions for a wave's 32 rows,
    // while the first tiles are on their way), with the bits of the preparing launch, which read and wrote all of Q once more: 32 heads of 8 kv heads, L = 777 causal,
    // inference 24.8 -> 21.6 us; 4 x 32/8 heads, L = 4096, training: that launch 66.7 -> 27.9 us, this kernel even.
    // (q_copy: Qh is Q^F in fp16 instead, rows padded to Lp: packed inputs.  SPLIT: the waves share the work, and the rows through LDS.  Q_LDS, the split training kernel at d = 128: it has no registers for them)
    constexpr bool Q_LDS = SPLIT && TRAIN && D == 128 && !MXS;
    const size_t grp = (size_t)bh * (Lp / 32) + ((has_rows ? row0_w : 0) >> 5);      // (MXS) group of 32 rows
    const int q_tid = SPLIT ? (int)threadIdx.x : lane;
    constexpr int DSW = SPLIT ? DS / NW : DS;      // contraction steps of Q^F that this wave makes
    const bool q_phi = TRAIN || VARLEN || DUMP || PQ != 0 || !q_copy;
    uint4v qreg[MXS || Q_LDS ? DSW : DS];
    MxQ<D, SPLIT ? 64 * NW : 64> Q;      // (SPLIT: the four waves share the rows)
    if constexpr (MXS) {
        Q.fetch(Qh, nullptr, bh, has_rows ? row0_w : 0, grp, q_tid, L);
    } else {
        const half_t* qp = Qh + ((size_t)bh * (q_phi ? L : Lp) + min(q_row, L - 1)) * D + 8 * hf + (SPLIT ? 16 * DSW * wave : 0);
#pragma unroll
        for (int i = 0; i < DSW; ++i) qreg[i] = *reinterpret_cast<const uint4v*>(qp + 16 * i);
    }
    auto phi_q = [&]() __attribute__((always_inline)) {
        if (!q_phi) return;
        if constexpr (DSW == 1) { uint4v same = qreg[0]; phi_half_blocks(qreg[0], same); }
        else
#pragma unroll
            for (int i = 0; i + 1 < DSW; i += 2) phi_half_blocks(qreg[i], qreg[i + 1]);
    };
    const int nkt = CAUSAL ? min((qt * QT + QT - 1 + off) / 64 + 1, nkt_all) : nkt_all;     // key tiles this item visits
    const int wave_qmax = row0_w + 31 + off;             // the last key that a row of this wave sees

    floatx16 o[OB], op[TRAIN && BOTH ? OB : 1];
#pragma unroll
    for (int mb = 0; mb < OB; ++mb) {
#pragma unroll
        for (int i = 0; i < 16; ++i) { o[mb][i] = 0.0f; if constexpr (TRAIN && BOTH) op[mb][i] = 0.0f; }
    }
    float m = -INFINITY, lsum = 0.0f;     // lsum: this half-wave's part of l (same alpha in both halves)
    float s1_prev = 1.0f, s1_cur = 1.0f;  // two-level P-tilde: the row factor O is currently expressed in, and this tile's
    floatx16 s[2];                        // S^T of the current tile, then P-tilde
#pragma unroll
    for (int i = 0; i < 16; ++i) { s[0][i] = 0.0f; s[1][i] = 0.0f; }

    // ---- S^T = K^F Q^F^T of one tile.  A wave sustains about one 1 KiB LDS read per 40 cycles and the
    // read latency is ~130 cycles, so the K operands are read RING steps ahead of the MFMA that consumes
    // them (the scheduling groups keep the compiler from sinking them).
    auto scores = [&](int buf) __attribute__((always_inline)) {
        if constexpr (MXS) {
            const uint32_t rec = lds_addr_of(kbase) + (uint32_t)(buf * (int)sizeof(sm.k[0]));
            const uint32_t ksc = *(const __attribute__((address_space(3))) uint32_t*)(uintptr_t)(rec + 2 * KSM * 1024 + lane * 4);
            uint4v a[2][KSM];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int ks = 0; ks < KSM; ++ks) a[kb][ks] = lds_read16_at(rec + (uint32_t)(((kb * KSM + ks) * 64 + lane) * 16));
            auto as8 = [](const uint4v& x) __attribute__((always_inline)) -> int8v {
                int8v r = {(int)x[0], (int)x[1], (int)x[2], (int)x[3], 0, 0, 0, 0};
                return r;
            };
            const floatx16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            // (format codes 4, 4: both operands E2M1; the scale operands are a dword of four bytes and the index of the byte)
            s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[0][0]), as8(Q.op[0]), zero, 4, 4, 0, ksc, 0, Q.sc);
            s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[1][0]), as8(Q.op[0]), zero, 4, 4, KSM, ksc, 0, Q.sc);
            if constexpr (KSM == 2) {
                s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[0][1]), as8(Q.op[1]), s[0], 4, 4, 1, ksc, 1, Q.sc);
                s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(a[1][1]), as8(Q.op[1]), s[1], 4, 4, 3, ksc, 1, Q.sc);
            }
            mfma_scale_settle(s[0], s[1]);
            return;
        }
        const uint32_t k_it = 16u * (uint32_t)lane + (uint32_t)(buf * (int)sizeof(sm.k[0])) + lds_addr_of(kbase);
        auto k_opnd = [&](int i) __attribute__((always_inline)) -> half8 { return __builtin_bit_cast(half8, lds_read16_at(k_it + 1024u * i)); };
        constexpr int NS = 2 * DS, RING = 6;
        half8 ring[RING];
#pragma unroll
        for (int i = 0; i < RING; ++i) ring[i] = k_opnd(i);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[kb][i] = 0.0f;
#pragma unroll
        for (int i = 0; i < NS; ++i) {                  // step i: ds = i / 2, kb = i % 2
            const half8 a = ring[i % RING];
            if (i + RING < NS) ring[i % RING] = k_opnd(i + RING);
            s[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, __builtin_bit_cast(half8, qreg[i >> 1]), s[i & 1], 0, 0, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, RING, 0);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (i + RING < NS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    };

    // ---- SPLIT: LDS holds P-tilde^F and (training) P-tilde of the four tiles as operands of the P V products, 4 KiB each; then per
    // tile the row maxima, alpha, and l's terms.
    constexpr int PT = KS * 4096;                       // bytes of one kind of P
    const uint32_t p_lds = lds_addr_of(smem_raw);
    float* x_max = reinterpret_cast<float*>(smem_raw + (TRAIN ? 2 : 1) * PT);      // [KS][32]
    float* x_alpha = x_max + KS * 32;                   // [KS][32]
    float* x_sum = x_alpha + KS * 32;                   // [KS][64]
    const uint32_t q_lds = lds_addr_of(x_sum + KS * 64) + 16u * (uint32_t)lane;      // Q_LDS: [d / 16] operands of 1 KiB
    float m_next = 0.0f;                                // the running maximum after the four tiles
    int nt = 0;                                         // how many of them there are for these rows
    // K operands of this wave's next tile and V^T operands of its blocks of O for the next four tiles: straight to registers, no
    // other wave reads them
    half8 kr[SPLIT && !MXS ? 2 * DS : 1], vr[SPLIT ? KS : 1][4][OB];
    uint4v kr_mx[SPLIT && MXS ? 2 * KSM : 1];
    uint32_t ksc_mx = 0u;
    // AHEAD (training, d = 128): S of the next four tiles is computed between the P V products, whose accumulators' rescaling (a quarter of the vector
    // instructions: on few keys some row moves its maximum in nearly every tile) then has products beside it instead of waiting for the last ones; its K operands are
    // asked for while P-tilde is quantized, when its registers are free.  1 - 5 % (12 heads, L = 1560 53.7 -> 52.2 us, 15 heads causal 39.9 -> 38.4 us).  Inference, with half
    // the products and rescaling: even to 3 % slower; d = 64: 2 % slower.
    constexpr bool AHEAD = Q_LDS;
    int k_tile = 0; bool k_more = false;                // AHEAD: the tile of those operands, if there is one
    auto load_k = [&](int jt) __attribute__((always_inline)) {
        if constexpr (MXS) {
            const unsigned char* rec = k_recs + (size_t)jt * KREC;
#pragma unroll
            for (int i = 0; i < 2 * KSM; ++i) kr_mx[i] = *reinterpret_cast<const uint4v*>(rec + 1024 * i + 16 * lane);
            ksc_mx = *reinterpret_cast<const uint32_t*>(rec + 2 * KSM * 1024 + 4 * lane);
        } else {
#pragma unroll
            for (int i = 0; i < 2 * DS; ++i) kr[i] = *reinterpret_cast<const half8*>(k_head + (size_t)jt * (64 * D) + 512 * i + 8 * lane);
        }
    };
    // ---- prologue: K(0), V(0), K(1) land, then every wave computes its S of tile 0
    if constexpr (!SPLIT) {
        issue_k(0, 0);
        issue_v(0, 0);
        if (nkt > 1) issue_k(1, 1);
    }
    // The Q registers must have arrived BEFORE the loop: a load still pending at loop entry makes the
    // compiler wait for all vector-memory traffic at the first product of every iteration.
    if constexpr (MXS) {
        if constexpr (!SPLIT) {
            // (phi(Q) through the second V^T buffer and what the K record leaves of the first K buffer: neither has been asked for yet)
            static_assert(NW * kMxQOps<D> <= sizeof(sm.v[1]) && KREC + NW * 256 <= (int)sizeof(sm.k[0]));
            const uint32_t ops = lds_addr_of(vbase) + (uint32_t)sizeof(sm.v[0]) + (uint32_t)(wave * kMxQOps<D>), scs = lds_addr_of(kbase) + (uint32_t)(KREC + wave * 256);
            Q.quantize(nullptr, ops, scs, q_tid);
            mx_q_wave_fence();
            Q.read(Qh, nullptr, grp, lane, ops, scs);
        }
    } else if constexpr (!SPLIT) {
        phi_q();
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) asm volatile("" : "+v"(qreg[ds]));
    }
    if constexpr (!SPLIT) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (has_rows) scores(0);
    }
    if (late) __builtin_amdgcn_s_barrier();              // one phase behind from here on
    if constexpr (!PHASES && !SPLIT) {
        // everyone is past the scores of tile 0: K(2) may take its buffer.  The barrier alone orders nothing: up to six LDS reads of
        // the products behind it were still on their way, and another wave's copy of K(2) could have overtaken them.
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_s_barrier();
    }

    // Two phases per key tile, separated by barriers; waves 0-3 are in the vector phase while waves
    // 4-7 are in the matrix phase and vice versa, so every SIMD holds one wave of each kind:
    //   vector phase j:  mask, online softmax, block scales of phi(P-tilde)         (no MFMA, no LDS)
    //   matrix phase j:  O, O' += V^F^T P(j) with the FP4 round trip of P-tilde in between;  S(j+1)
    // (The MFMAs of one wave run beside the vector instructions of the other; each costs those about 7 cycles of issue.  At full fill the kernel
    // is held by the clock under its load: 2 x 12 heads, L = 32760 11.7 ms on random data, 9.7 ms on zeros; without the raised priority 8 % more.)
    // Tile traffic: K(j+2) and V(j+1) are requested at the start of matrix phase j into the buffers
    // whose last readers (matrix phase j-1 of either group) are two barriers back.
    // SPLIT: what this wave has written to LDS is there, what it has read has arrived, and the other waves have got here too
    auto lds_barrier = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    // ---- vector phase of one key tile: mask, online softmax, block scales of phi(P-tilde)  (no MFMA; LDS only for SPLIT, the tiles' row maxima)
    // (psc[ks]: reciprocal of the scale of group ks, with the scale in element ks / 2 of bsc[ks % 2]; MX: the scale, a power of two)
    auto vector_phase = [&](int j, half2v (&bsc)[2], float (&psc)[4]) __attribute__((always_inline)) {
        const int k0 = j * 64;
        // mask: keys beyond L, and keys after the query when causal
        const bool need_mask = (k0 + 64 > Lk) || (CAUSAL && k0 + 63 > row0_w + off);
        if (__builtin_expect(need_mask, 0)) {
            const int klim = CAUSAL ? min(Lk - 1, q_row + off) : Lk - 1;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int key = k0 + 32 * kb + 8 * (i >> 2) + 4 * hf + (i & 3);
                    if (key > klim) s[kb][i] = -INFINITY;
                }
        }
        // online softmax (Alg. 2: m_new, alpha, P-tilde, l).  Four interleaved chains each: a single
        // chain of 32 dependent max / add instructions would run at the instruction latency.
        // The maxima are taken on S: one per group of 16 keys (registers 8g..8g+7 of both halves), the tile's row
        // maximum from those four.  exp2 of a group's largest score, by the same instructions on the same inputs as
        // that element's P-tilde, then is the group's largest P-tilde, which the block scale of phi needs below.
        float mt, gmax[4], gpair[2];
        if constexpr (PQ == 1) {
            // MX: the blocks are the tile's two halves of 32 keys; block 0's maximum in lanes 0-31, block 1's in lanes 32-63
            float bmax[2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const floatx16& sv = s[kb];
                const float a0 = max_nc(max_nc(sv[0], sv[1]), sv[2]), a1 = max_nc(max_nc(sv[3], sv[4]), sv[5]);
                const float a2 = max_nc(max_nc(sv[6], sv[7]), sv[8]), a3 = max_nc(max_nc(sv[9], sv[10]), sv[11]);
                const float a4 = max_nc(max_nc(sv[12], sv[13]), sv[14]);
                bmax[kb] = max_nc(max_nc(max_nc(max_nc(a0, a1), a2), max_nc(a3, a4)), sv[15]);
            }
            gpair[0] = xhalf_max_pair(bmax[0], bmax[1]);
            mt = xhalf_max(gpair[0]);
        } else if constexpr (PQ == 3) {
            float mp[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) mp[t] = max_nc(s[0][t], s[1][t]);
#pragma unroll
            for (int i = 4; i < 16; ++i) mp[i & 3] = max_nc(max_nc(mp[i & 3], s[0][i]), s[1][i]);
            mt = xhalf_max(max_nc(max_nc(mp[0], mp[1]), max_nc(mp[2], mp[3])));
        } else {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const floatx16& sv = s[ks >> 1];
                const int b0 = 8 * (ks & 1);
                const float a0 = max_nc(max_nc(sv[b0], sv[b0 + 1]), sv[b0 + 2]);
                const float a1 = max_nc(max_nc(sv[b0 + 3], sv[b0 + 4]), sv[b0 + 5]);
                // (SPLIT has no barrier between the products and here: max_raw only beside what was made from the same product)
                if constexpr (SPLIT) gmax[ks] = max_raw(max_nc(max_nc(a0, a1), sv[b0 + 6]), sv[b0 + 7]);
                else gmax[ks] = max_nc(max_nc(a0, a1), max_raw(sv[b0 + 6], sv[b0 + 7]));
            }
            if constexpr (PQ == 0) {
                // groups 0 and 2 in lanes 0-31, groups 1 and 3 in lanes 32-63: one exchange for two groups
                gpair[0] = xhalf_max_pair(gmax[0], gmax[1]);
                gpair[1] = xhalf_max_pair(gmax[2], gmax[3]);
                mt = xhalf_max(max_raw(gpair[0], gpair[1]));
            } else {
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) gmax[ks] = xhalf_max(gmax[ks]);
                mt = max_nc(max_nc(gmax[0], gmax[1]), max_nc(gmax[2], gmax[3]));
            }
        }
        if constexpr (SPLIT) {
            // the tile's row maxima to the waves that have the other tiles; the running maximum before this tile from theirs
            if (hf == 0) x_max[wave * 32 + ln] = mt;
            lds_barrier();
            float xm[KS];
#pragma unroll
            for (int t = 0; t < KS; ++t) xm[t] = x_max[t * 32 + ln];
            m_next = m;
#pragma unroll
            for (int t = 0; t < KS; ++t) {
                if (t < wave) m = max_nc(m, xm[t]);
                if (t < nt) m_next = max_nc(m_next, xm[t]);
            }
        }
        const float mnew = max_raw(m, mt);                  // (both come out of vector instructions)
        const float alpha = __builtin_amdgcn_exp2f((m - mnew) * c);
        const float ms = mnew * c;
        m = mnew;
        float rp[4];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                s[kb][i] = __builtin_amdgcn_exp2f(fmaf(s[kb][i], c, -ms));
                if (kb == 0 && i < 4) rp[i] = s[kb][i];
                else                  rp[i & 3] += s[kb][i];
            }
        if constexpr (SPLIT) {
            x_sum[wave * 64 + lane] = (rp[0] + rp[1]) + (rp[2] + rp[3]);
            if (hf == 0) x_alpha[wave * 32 + ln] = alpha;
        } else
        lsum = lsum * alpha + ((rp[0] + rp[1]) + (rp[2] + rp[3]));          // un-quantized P-tilde
        // (pinned: the compiler otherwise sinks the additions to the end of the tile and keeps P-tilde alive beside the next S)
        if constexpr (!PHASES && !SPLIT) asm volatile("" : "+v"(lsum));
        // rescale: exact no-op unless some row of this wave moved its maximum (rare after the
        // first tiles), so it lives on the cold path
        float inv1 = 1.0f;
        if constexpr (SPLIT) {
            // (O and O' are rescaled by the waves that hold them)
        } else if constexpr (PQ == 2) {
            // Two-level quantization of P-tilde (Sec. 2.1): the row of this tile is divided by s1, the smallest power
            // of two with 2688 s1 >= max(row maximum, 2^-24), before the NVFP4 blocks.  The row maximum is exp2 of the
            // tile's largest score, the same instructions on the same inputs as that element's P-tilde.
            // O is kept in units of the current s1 (its products use P-tilde / s1, which fp16 holds exactly whatever
            // the magnitude of the row), so it is re-based on every tile; O' only needs alpha.
            const float base = fmaxf(__builtin_amdgcn_exp2f(fmaf(mt, c, -ms)), 5.9604644775390625e-08f);
            const uint32_t e1 = ((__float_as_uint(base) + 0x0057FFFFu) >> 23) - 11u;      // 2688 = 1.3125 * 2^11
            s1_cur = __uint_as_float(e1 << 23);
            inv1 = __uint_as_float((254u - e1) << 23);
            const float f = alpha * s1_prev * inv1;
            s1_prev = s1_cur;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[mb][i] *= f;
            if constexpr (TRAIN) {
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0, 0)) {
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                        for (int i = 0; i < 16; ++i) op[mb][i] *= alpha;
                }
            }
        } else if (__builtin_expect(__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0, 0)) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) { o[mb][i] *= alpha; if constexpr (TRAIN) op[mb][i] *= alpha; }
        }
        if constexpr (PQ == 3) return;      // bf16 P-tilde has no block scales
        if constexpr (PQ == 1) {
            // MX format: one power-of-two scale per 32 keys = all 16 registers of s[kb] in both halves, formed by one of them
            const uint32_t byte = e8m0_of_amax(__builtin_amdgcn_exp2f(fmaf(gpair[0], c, -ms)));
            const auto sb = __builtin_amdgcn_permlane32_swap(byte << 23, byte << 23, false, false);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) psc[2 * kb] = psc[2 * kb + 1] = __uint_as_float(sb[kb]);
            return;
        }
        // block scales of phi(P-tilde) for the four 16-key groups of the tile (keys of a group =
        // registers 8g..8g+7 of both halves)
        if constexpr (PQ == 0) {
            // A lane forms the scales of two groups, its half's (gpair), and hands them to the other half: two instructions of a kind
            // instead of four, and the exchange of the two scale bytes is one.
            float bm[2], inv[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) bm[t] = __builtin_amdgcn_exp2f(fmaf(gpair[t], c, -ms)) * (1.0f / 6.0f);
            // RNE_E4M3(amax / 6) by the hardware conversion (OCP E4M3, round to nearest even, subnormals kept; two values
            // per instruction) and back: the same values as rne_e4m3_grid in a quarter of the instructions.
            // P-tilde <= 1: no saturation
            typedef short short2v __attribute__((ext_vector_type(2)));
            const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(__builtin_bit_cast(short2v, any_register()), bm[0], bm[1], 1.0f, false));
            // reciprocals.  A scale of 0: P^F is 0 whatever the codes are (the dequantization multiplies by the scale), so
            // any finite factor serves; 512 = 1 / (smallest non-zero scale) keeps the quotients finite.
            inv[0] = fminf(__builtin_amdgcn_rcpf(__builtin_amdgcn_cvt_scalef32_f32_fp8(w, 1.0f, 0)), 512.0f);
            inv[1] = fminf(__builtin_amdgcn_rcpf(__builtin_amdgcn_cvt_scalef32_f32_fp8(w, 1.0f, 1)), 512.0f);
            const auto wb = __builtin_amdgcn_permlane32_swap(w, w, false, false);
#pragma unroll
            for (int g = 0; g < 2; ++g)                  // (g: which half formed them)
                bsc[g] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(wb[g], 1.0f, false);      // (an E4M3 scale is an fp16 number)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const auto ib = __builtin_amdgcn_permlane32_swap(__float_as_uint(inv[t]), __float_as_uint(inv[t]), false, false);
                psc[2 * t] = __uint_as_float(ib[0]); psc[2 * t + 1] = __uint_as_float(ib[1]);
            }
        } else {
            // (two-level: the block maxima of P-tilde / s1 are at most 2688 (1 + 2^-23), whose sixth rounds to 448, the largest scale)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const float sc = rne_e4m3_grid_of_product(__builtin_amdgcn_exp2f(fmaf(gmax[ks], c, -ms)) * inv1, 1.0f / 6.0f);
                bsc[ks & 1][ks >> 1] = (half_t)sc;
                psc[ks] = fminf(__builtin_amdgcn_rcpf(sc), 512.0f) * inv1;
            }
        }
    };
    // ---- matrix phase of one key tile: O, O' += V^F^T P with the FP4 round trip of P-tilde in between
    auto matrix_phase = [&](int j, const half2v (&bsc)[2], const float (&psc)[4]) __attribute__((always_inline)) {
        const int k0 = j * 64;
        (void)k0;
        // per 16 keys: phi^-1(phi(P-tilde)), then O^T += V^F^T P-tilde^F^T and O'^T += V^F^T P-tilde^T
        // (an LDS address as an integer: pointer arithmetic on the dynamic LDS symbol costs an add per read)
        const uint32_t v_it = 16u * (uint32_t)lane + (uint32_t)((j & 1) * (int)sizeof(sm.v[0])) + lds_addr_of(vbase);
        struct QState { uint32_t c01, c23; };
        float pfv[DUMP ? 8 : 1];
        // the FP4 round trip of one group of 16 keys, cut into four parts of a few instructions
        auto q_part = [&](int ks, int part, QState& st, uint4v& bq, uint4v& bu) __attribute__((always_inline)) {
            const int b0 = 8 * (ks & 1);
            const floatx16& sv = s[ks >> 1];
            if constexpr (PQ == 3) {
                // bf16 P-tilde: one rounding (nearest even), no codes and no scales
                if (part == 0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) bq[i] = pack_bf16x2_cvt(sv[b0 + 2 * i], sv[b0 + 2 * i + 1]);
                    if constexpr (DUMP) {
                        if (q_row >= dump_row0 && q_row < dump_row0 + 128 && q_row < L) {
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const int key = k0 + 32 * (ks >> 1) + 16 * (ks & 1) + 8 * (i >> 2) + 4 * hf + (i & 3);
                                if (key < L)
                                    pdump[((size_t)bh * 128 + (q_row - dump_row0)) * L + key] =
                                        __uint_as_float((i & 1) ? (bq[i >> 1] & 0xFFFF0000u) : (bq[i >> 1] << 16));
                            }
                        }
                    }
                }
                return;
            }
            // (MX: the conversions themselves divide and multiply by a power of two.  With the blocks' maxima taken on S, about 100 vector instructions
            //  less per tile; with the backward's share 2 x 16/4 heads, L = 3001 causal, training step 426 -> 404 us)
            const float inv = MXS ? 1.0f : psc[ks], cs = MXS ? psc[ks] : 1.0f;
            auto quo = [&](int e) __attribute__((always_inline)) { return MXS ? sv[b0 + e] : sv[b0 + e] * inv; };
            if (part == 0) {
                // (the conversion replaces one byte of its first operand; bytes 2 and 3 of the code registers are never read)
                st.c01 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(any_register(), quo(0), quo(1), cs, 0);
                st.c23 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(any_register(), quo(4), quo(5), cs, 0);
            } else if (part == 1) {
                st.c01 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(st.c01, quo(2), quo(3), cs, 1);
                st.c23 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(st.c23, quo(6), quo(7), cs, 1);
            } else if (part == 2) {
                half2v f[4];
                f[0] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(st.c01, cs, 0);
                f[1] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(st.c01, cs, 1);
                f[2] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(st.c23, cs, 0);
                f[3] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(st.c23, cs, 1);
                uint32_t w[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (!MXS) {
                        const half_t sc = bsc[ks & 1][ks >> 1];
                        f[i] *= half2v{sc, sc};
                    }
                    w[i] = __builtin_bit_cast(uint32_t, f[i]);
                }
                bq[0] = w[0]; bq[1] = w[1]; bq[2] = w[2]; bq[3] = w[3];
                if constexpr (DUMP) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const half2v pr = __builtin_bit_cast(half2v, w[i]);
                        pfv[2 * i] = (float)pr[0]; pfv[2 * i + 1] = (float)pr[1];
                    }
                    if (q_row >= dump_row0 && q_row < dump_row0 + 128 && q_row < L) {
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const int key = k0 + 32 * (ks >> 1) + 16 * (ks & 1) + 8 * (i >> 2) + 4 * hf + (i & 3);
                            if (key < L)
                                pdump[((size_t)bh * 128 + (q_row - dump_row0)) * L + key] = PQ == 2 ? pfv[i] * s1_cur : pfv[i];
                        }
                    }
                }
            } else if constexpr (TRAIN) {
#pragma unroll
                for (int i = 0; i < 4; ++i) bu[i] = pack_f16x2(sv[b0 + 2 * i], sv[b0 + 2 * i + 1]);
            }
        };
        // A wave issues in order: a block of MFMAs followed by a block of vector instructions leaves the
        // vector ALU idle while the MFMAs queue up.  So the parts of step ks+1 follow the products of
        // step ks one by one (scheduling fences keep the compiler from regrouping them); a V^T operand
        // register is reloaded for step ks+1 as soon as its last product of step ks has issued.
        if constexpr (SPLIT) {
            // the whole tile as operands of the P V products, to the waves that have the blocks of O
            const uint32_t dst = p_lds + (uint32_t)(wave * 4096 + 16 * lane);
            QState st;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                uint4v bq, bu;
#pragma unroll
                for (int part = 0; part < 4; ++part) q_part(ks, part, st, bq, bu);
                lds_write16_at(dst + 1024u * ks, bq);
                if constexpr (TRAIN) lds_write16_at(dst + PT + 1024u * ks, bu);
                if constexpr (AHEAD) {
                    if (k_more) {
#pragma unroll
                        for (int i = ks * (DS / 2); i < (ks + 1) * (DS / 2); ++i)
                            kr[i] = *reinterpret_cast<const half8*>(k_head + (size_t)k_tile * (64 * D) + 512 * i + 8 * lane);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            return;
        }
        half8 av[MB];
        uint4v bq[2], bu[2];
        QState st;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            av[mb] = __builtin_bit_cast(half8, lds_read16_at(v_it + 1024u * mb));
#pragma unroll
        for (int part = 0; part < 4; ++part) q_part(0, part, st, bq[0], bu[0]);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int cur = ks & 1, nxt = cur ^ 1;
            const half8 bqh = __builtin_bit_cast(half8, bq[cur]);
            const half8 buh = __builtin_bit_cast(half8, bu[cur]);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                if constexpr (!DUMP) __builtin_amdgcn_sched_barrier(0);
                if constexpr (PQ == 3)
                    o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[mb]), __builtin_bit_cast(bf16x8, bqh), o[mb], 0, 0, 0);
                else
                    o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[mb], bqh, o[mb], 0, 0, 0);
                if constexpr (TRAIN) {
                    if constexpr (!DUMP) __builtin_amdgcn_sched_barrier(0);
                    op[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[mb], buh, op[mb], 0, 0, 0);
                }
                if (ks < 3) {
#pragma unroll
                    for (int part = (4 * mb) / MB; part < (4 * (mb + 1)) / MB; ++part) q_part(ks + 1, part, st, bq[nxt], bu[nxt]);
                    av[mb] = __builtin_bit_cast(half8, lds_read16_at(v_it + 1024u * ((ks + 1) * MB + mb)));
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        };
    // the tile copies of matrix phase j
    auto request_tiles = [&](int j) __attribute__((always_inline)) {
        if (j + 2 < nkt) issue_k(j & 1, j + 2);
        if (j + 1 < nkt) issue_v((j + 1) & 1, j + 1);
    };

    // Under a causal mask the workgroup's first 4 qt + 1 key tiles are visible to every one of its waves (the tile that
    // starts at the workgroup's first row included; rows inside it are masked in the vector phase), and only the last
    // three have waves that skip.  The two kinds of tile get loops of their own: the form with the skipping branch
    // schedules markedly worse (17 % slower on tiles where nobody skips), so it only runs where somebody does.
    // which blocks of O (and O') this wave has: OB of them from ob0 on; fewer blocks than waves: one block of O, or of O', or none
    const int ob0 = !SPLIT ? 0 : BOTH ? wave * OB : wave % MB;
    const bool second = !BOTH && wave >= MB, has_o = BOTH || wave < (TRAIN ? 2 : 1) * MB;
    if constexpr (SPLIT) {
        const half_t* v_lane = v_head + 512 * ob0 + 8 * lane;
        const uint32_t p_src = p_lds + 16u * (uint32_t)lane + (TRAIN && second ? (uint32_t)PT : 0u);
        // V^T operand of this wave's block ob, keys 16 ks .. of tile t of the four from j0 on (beyond the last tile: the last one again,
        // not used)
        auto v_opnd = [&](int j0, int t, int ks, int ob) __attribute__((always_inline)) -> half8 {
            return *reinterpret_cast<const half8*>(v_lane + (size_t)min(j0 + t, nkt - 1) * (64 * D) + 512 * (ks * MB + ob));
        };
        // Four key tiles.  MORE: not the last ones; an operand register is reloaded for the next four right behind its last product
        // (asked for all at once, the 16 KiB of each wave held it up for the time they take to get through the compute unit's
        // cache at 64 bytes per clock).
        // S of a tile of this wave, in KS parts.  RELOAD: the operand registers take those of tile k_next
        constexpr int RQ = 4, SP = 2 * DS / KS;
        half8 qr[Q_LDS ? RQ : 1];
        auto q_opnd = [&](int ds) __attribute__((always_inline)) { return __builtin_bit_cast(half8, lds_read16_at(q_lds + 1024u * ds)); };
        auto s_part = [&](auto reload, int part, int k_next) __attribute__((always_inline)) {
            constexpr bool RELOAD = decltype(reload)::value;
            if (part == 0) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) s[kb][i] = 0.0f;
                if constexpr (Q_LDS) {
#pragma unroll
                    for (int ds = 0; ds < RQ; ++ds) qr[ds] = q_opnd(ds);
                }
            }
#pragma unroll
            for (int i = part * SP; i < (part + 1) * SP; ++i) {
                const int ds = i >> 1;
                s[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kr[MXS ? 0 : i], Q_LDS ? qr[Q_LDS ? ds % RQ : 0] : __builtin_bit_cast(half8, qreg[Q_LDS || MXS ? 0 : ds]), s[i & 1], 0, 0, 0);
                if constexpr (Q_LDS) { if ((i & 1) && ds + RQ < DS) qr[ds % RQ] = q_opnd(ds + RQ); }
                if constexpr (RELOAD) kr[MXS ? 0 : i] = *reinterpret_cast<const half8*>(k_head + (size_t)k_next * (64 * D) + 512 * i + 8 * lane);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto four_tiles = [&](auto more, int j0) __attribute__((always_inline)) {
            constexpr bool MORE = decltype(more)::value;
            const int j = j0 + wave, k_next = min(j + KS, nkt - 1);
            k_tile = k_next; k_more = MORE;
            const bool active = MORE || j < nkt;
            nt = MORE ? KS : nkt - j0;
            if (active) {
                if constexpr (MXS) {
                    auto as8 = [](const uint4v& x) __attribute__((always_inline)) -> int8v {
                        int8v r = {(int)x[0], (int)x[1], (int)x[2], (int)x[3], 0, 0, 0, 0};
                        return r;
                    };
                    const floatx16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                    s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr_mx[0]), as8(Q.op[0]), zero, 4, 4, 0, ksc_mx, 0, Q.sc);
                    s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr_mx[KSM]), as8(Q.op[0]), zero, 4, 4, KSM, ksc_mx, 0, Q.sc);
                    if constexpr (KSM == 2) {
                        s[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr_mx[1]), as8(Q.op[1]), s[0], 4, 4, 1, ksc_mx, 1, Q.sc);
                        s[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as8(kr_mx[3]), as8(Q.op[1]), s[1], 4, 4, 3, ksc_mx, 1, Q.sc);
                    }
                    mfma_scale_settle(s[0], s[1]);
                    if constexpr (MORE) load_k(k_next);
                } else if constexpr (!AHEAD) {
#pragma unroll
                    for (int part = 0; part < KS; ++part) s_part(more, part, k_next);
                }
                half2v bsc[2]; float psc[4];
                vector_phase(j, bsc, psc);
                matrix_phase(j, bsc, psc);
            } else {
                lds_barrier();
                m_next = m;
#pragma unroll
                for (int t = 0; t < KS; ++t) if (t < nt) m_next = max_nc(m_next, x_max[t * 32 + ln]);
            }
            m = m_next;
            lds_barrier();                               // P, alpha and the sums are in LDS
            float al[KS], sm_[KS];
#pragma unroll
            for (int t = 0; t < KS; ++t) { al[t] = x_alpha[t * 32 + ln]; sm_[t] = x_sum[t * 64 + lane]; }
            // operands are read R steps of 16 keys ahead of their products
            constexpr int R = AHEAD ? 2 : 4;
            uint4v rq[R], ru[TRAIN && BOTH ? R : 1];
            auto fetch = [&](int i) __attribute__((always_inline)) {
                rq[i % R] = lds_read16_at(p_src + 1024u * i);
                if constexpr (TRAIN && BOTH) ru[i % R] = lds_read16_at(p_src + (uint32_t)PT + 1024u * i);
            };
            if (has_o) {
#pragma unroll
                for (int i = 0; i < R; ++i) fetch(i);
            }
#pragma unroll
            for (int t = 0; t < KS; ++t) {
                if (MORE || t < nt) {
                    const float alpha = al[t];
                    lsum = lsum * alpha + sm_[t];        // l in tile order
                    if (has_o) {
                        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
                            for (int ob = 0; ob < OB; ++ob)
#pragma unroll
                                for (int i = 0; i < 16; ++i) { o[ob][i] *= alpha; if constexpr (TRAIN && BOTH) op[ob][i] *= alpha; }
                        }
#pragma unroll
                        for (int ks = 0; ks < 4; ++ks) {
                            const int i = 4 * t + ks;
                            const half8 pf = __builtin_bit_cast(half8, rq[i % R]), pu = __builtin_bit_cast(half8, ru[TRAIN && BOTH ? i % R : 0]);
#pragma unroll
                            for (int ob = 0; ob < OB; ++ob) {
                                if constexpr (PQ == 3)
                                    o[ob] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vr[t][ks][ob]), __builtin_bit_cast(bf16x8, pf), o[ob], 0, 0, 0);
                                else
                                    o[ob] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vr[t][ks][ob], pf, o[ob], 0, 0, 0);
                                if constexpr (TRAIN && BOTH) op[ob] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vr[t][ks][ob], pu, op[ob], 0, 0, 0);
                                if constexpr (MORE) vr[t][ks][ob] = v_opnd(j0 + KS, t, ks, ob);
                            }
                            if (i + R < 4 * KS) fetch(i + R);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
                if constexpr (MORE && AHEAD) s_part(std::false_type{}, t, 0);
            }
        };
        load_k(min(wave, nkt - 1));
        if (has_o) {
#pragma unroll
            for (int t = 0; t < KS; ++t)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int ob = 0; ob < OB; ++ob) vr[t][ks][ob] = v_opnd(0, t, ks, ob);
        }
        if constexpr (MXS) {
            // (phi(Q) through the room of P, which is first written behind the barrier of the maxima)
            Q.quantize(nullptr, p_lds, p_lds + kMxQOps<D>, q_tid);
            lds_barrier();
            Q.read(Qh, nullptr, grp, lane, p_lds, p_lds + kMxQOps<D>);
        } else {
            // (Q_LDS: they stay there.  Else through the room of P, as above)
            phi_q();
            const uint32_t q_ops = Q_LDS ? q_lds : p_lds + 16u * (uint32_t)lane;
#pragma unroll
            for (int i = 0; i < DSW; ++i) lds_write16_at(q_ops + 1024u * (uint32_t)(wave * DSW + i), qreg[i]);
            lds_barrier();
            if constexpr (!Q_LDS) {
#pragma unroll
                for (int ds = 0; ds < DS; ++ds) qreg[ds] = lds_read16_at(q_ops + 1024u * ds);
            }
        }
        if constexpr (AHEAD) {
#pragma unroll
            for (int part = 0; part < KS; ++part) s_part(std::false_type{}, part, 0);
        }
        int j0 = 0;
        for (; j0 + KS < nkt; j0 += KS) four_tiles(std::true_type{}, j0);
        four_tiles(std::false_type{}, j0);
    } else if constexpr (PHASES) {
    const int j_all = CAUSAL ? min(nkt, (qt * QT + 31 + off) / 64 + 1) : nkt;
    for (int j = 0; j < j_all; ++j) {
        const int k0 = j * 64;
        half2v bsc[2]; float psc[4];
        if (has_rows) vector_phase(j, bsc, psc);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_s_setprio(1);    // the MFMA stream is the scarce one: it wins issue conflicts
        request_tiles(j);
        if (has_rows) matrix_phase(j, bsc, psc);
        // S of the next tile (its P-tilde predecessor in the same registers has been consumed above)
        if (has_rows && j + 1 < nkt && (!CAUSAL || k0 + 64 <= wave_qmax)) scores((j + 1) & 1);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_s_waitcnt(0);        // this wave's parts of K(j+2) and V(j+1) are in LDS
        __builtin_amdgcn_s_barrier();
    }
    if constexpr (CAUSAL) {
        for (int j = j_all; j < nkt; ++j) {
            const int k0 = j * 64;
            const bool active = has_rows && k0 <= wave_qmax;          // wave-uniform
            // Waves skip the tiles above the diagonal.  The whole tile sits in one branch, with a barrier on
            // either path: written as two branches around a common barrier, the softmax state looks live to
            // the compiler on the skipping path and the kernel spills.
            if (active) {
                half2v bsc[2]; float psc[4];
                vector_phase(j, bsc, psc);
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_s_setprio(1);
                request_tiles(j);
                matrix_phase(j, bsc, psc);
            } else {
                __builtin_amdgcn_s_barrier();
                request_tiles(j);
            }
            if (has_rows && j + 1 < nkt && k0 + 64 <= wave_qmax) scores((j + 1) & 1);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_s_waitcnt(0);
            __builtin_amdgcn_s_barrier();
        }
    }
    if (!late) __builtin_amdgcn_s_barrier();             // pairs with the late group's extra barrier
    } else {
        // Four waves run in step, one barrier per key tile: at the top of tile j every wave is past the scores of tile j (the last
        // reads of the K buffer that K(j+2) goes to) and past the products of tile j-1 (the V^T buffer of V(j+1)).  The second
        // workgroup of the compute unit is what fills the SIMDs while this one waits.
        auto step = [&](int j, bool active, bool next_active) __attribute__((always_inline)) {
            request_tiles(j);
            if (active) {
                half2v bsc[2]; float psc[4];
                vector_phase(j, bsc, psc);
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_setprio(1);
                matrix_phase(j, bsc, psc);
            }
            if (next_active) scores((j + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_s_waitcnt(0);
            __builtin_amdgcn_s_barrier();
        };
        // (the last two tiles under a causal mask are the ones that some waves skip; as above, that form gets its own loop)
        const int j_all = CAUSAL ? min(nkt, (qt * QT + 31 + off) / 64 + 1) : nkt;
        for (int j = 0; j < j_all; ++j) step(j, true, j + 1 < nkt && (!CAUSAL || j * 64 + 64 <= wave_qmax));
        if constexpr (CAUSAL)
            for (int j = j_all; j < nkt; ++j) step(j, j * 64 <= wave_qmax, j + 1 < nkt && j * 64 + 64 <= wave_qmax);
    }

    // ---- epilogue: O /= l, O' /= l, L = m + log l
    const float l = xhalf_sum(lsum);
    const float inv_l = 1.0f / l;
    const float inv_lo = PQ == 2 ? s1_prev * inv_l : inv_l;      // O leaves the units of the last row factor
    if (q_row < L && has_o) {
        const size_t row = (size_t)bh * L + q_row;
#pragma unroll
        for (int mb = 0; mb < OB; ++mb)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int d0 = 32 * (ob0 + mb) + 8 * t + 4 * hf;
                if (!second) {
                    uint2v w;
                    w[0] = pack_bf16x2_rne(o[mb][4 * t] * inv_lo, o[mb][4 * t + 1] * inv_lo);
                    w[1] = pack_bf16x2_rne(o[mb][4 * t + 2] * inv_lo, o[mb][4 * t + 3] * inv_lo);
                    *reinterpret_cast<uint2v*>(O + row * D + d0) = w;
                }
                if (TRAIN && (BOTH || second)) {
                    const floatx16& acc = BOTH ? op[BOTH && TRAIN ? mb : 0] : o[mb];
                    floatx4 f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[e] = acc[4 * t + e] * inv_l;
                    *reinterpret_cast<floatx4*>(Ohp + row * D + d0) = f;
                }
            }
        if (hf == 0 && (!SPLIT || wave == 0)) lse[row] = m * (c * 0.6931471805599453f) + logf(l);   // m is in raw q.k units
    }
    // (a second item may overwrite the tile buffers at once: every wave's last read of them lies before a barrier that
    //  all eight waves have passed by now)
    }
}

#define AQ_FWD_ARGS \
    const half_t* __restrict__ Qh, const half_t* __restrict__ Kh, const half_t* __restrict__ Vt, \
    uint16_t* __restrict__ O, float* __restrict__ lse, float* __restrict__ Ohp, \
    int L, int Lp, int Hq, int G, float c, int dump_row0, float* __restrict__ pdump, \
    int Lkp, const int* __restrict__ kv_lens, int B, int q_copy
template <int D, bool TRAIN, bool CAUSAL, bool DUMP, int PQ, bool VARLEN = false>
__global__ __launch_bounds__(512, 2) void fwd_kernel(AQ_FWD_ARGS)
{
    fwd_body<D, TRAIN, CAUSAL, DUMP, PQ, VARLEN, 8>(Qh, Kh, Vt, O, lse, Ohp, L, Lp, Hq, G, c, dump_row0, pdump, Lkp, kv_lens, B, q_copy);
}
template <int D, bool TRAIN, bool CAUSAL, int PQ, bool VARLEN = false>
__global__ __launch_bounds__(256, 2) void fwd_narrow_kernel(AQ_FWD_ARGS)
{
    fwd_body<D, TRAIN, CAUSAL, false, PQ, VARLEN, 4>(Qh, Kh, Vt, O, lse, Ohp, L, Lp, Hq, G, c, dump_row0, pdump, Lkp, kv_lens, B, q_copy);
}
// Alg. 1 / Alg. 2 where there are too few query rows to fill the chip: a workgroup owns 32 rows, and its four waves take four key
// tiles at a time, wave w tile 4 n + w for S, the softmax and phi(P-tilde), and block w of O (and O') for the P V products of all four.
// What bounds a problem of this size is not a rate but the chain of one wave: 13 tiles in sequence at 1.6 us (infer) or 2.1 us
// (train), half of it waiting, while the other SIMDs idle.  Here a chain is a quarter as long, and its steps shorter: O's rescaling and
// its registers are shared out too.  Nothing of Alg. 1 changes: the running maximum before a tile is the largest of the tiles' row
// maxima, exchanged through LDS between the scores and the softmax, so every P-tilde^F has the bits it has in sequence; P goes
// through LDS as operands of the products (4 KiB per tile); each element of O is added up by one wave in tile order and l from
// the tiles' sums in tile order: all results have the bits of fwd_kernel.
// K and V^T operands go straight to registers: each is read by one wave only (a version with 64 rows per workgroup and tiles in
// LDS spent its time on the LDS ports: 8700 cycles per four tiles and 64 rows, this one 3600 where two workgroups share a compute unit).
// Two barriers per four tiles.  Two workgroups per compute unit.  Measured, four-wave tiles of 128 rows -> this, with the preparing launch:
// d = 128, training: 2 heads, L = 1000 40.3 -> 19.6 us; 8 heads, L = 2000 75.6 -> 48.9 us; 12 heads, L = 2300 causal 84 -> 53 us;
// inference, 32 heads, L = 777 causal 32.8 -> 28.8 us; d = 64, training: 2 heads, L = 256 13.2 -> 10.3 us.
template <int D, bool TRAIN, bool CAUSAL, int PQ, bool VARLEN = false>
__global__ __launch_bounds__(256, 2) void fwd_split_kernel(AQ_FWD_ARGS)
{
    fwd_body<D, TRAIN, CAUSAL, false, PQ, VARLEN, 4, true>(Qh, Kh, Vt, O, lse, Ohp, L, Lp, Hq, G, c, dump_row0, pdump, Lkp, kv_lens, B, q_copy);
}
#undef AQ_FWD_ARGS

// Which of the two workgroup shapes.  The eight-wave one (256 rows, one workgroup per compute unit) makes half the tile copies
// per row and runs its two halves in opposite phases; at equal fill it is 2 - 3 % faster at d = 128.  The four-wave one (128 rows,
// two per compute unit) fills the chip with half the rows and leaves a smaller last round.
// Without a mask all workgroups cost the same and rounds can be counted: a round of eight-wave workgroups costs 100, two four-wave
// ones sharing a unit 102, one alone on its unit 80.  Measured, training forward, eight -> four waves: 12 heads, L = 1560 (84 against
// 156 workgroups) 75 -> 61 us; L = 6240 (300 / 588) 483 -> 435 us; L = 3120 (156 / 300) 122 -> 122 us; 40 heads, L = 1560 (280 / 520)
// 123 -> 125 us; 24 heads, L = 8192 (768 / 1536) 1033 -> 1050 us.
// Under a causal mask an eight-wave workgroup pairs a long with a short tile, so that all cost the same, while four-wave workgroups
// are ordered by length (longest_first) and balance themselves: they win wherever the pairs do not fill whole rounds (64 pairs,
// 32 heads, L = 777: 71 -> 34 us; 192 pairs, L = 3001: 163 -> 127 us; 564 pairs, L = 24000: 2969 -> 2322 us).  Full rounds of long
// pairs are even at 4096 positions (1024 pairs: 804 and 808 us) and 0 - 3 % faster on eight waves from 16384 on; d = 64 runs three
// of the small workgroups per compute unit and always gains (16 heads, L = 32000: 3624 -> 3348 us).
static bool narrow_workgroups(int heads, int Lp, int D, bool causal)
{
    const long long cus = device_cu_count(), n4 = (long long)heads * (Lp / 128);
    const long long per_head = (Lp + 255) / 256, n8 = heads * (causal ? (per_head + 1) / 2 : per_head);
    const long long rounds8 = (n8 + cus - 1) / cus;
    if (causal) return D != 128 || Lp < 4096 || n8 * 100 < rounds8 * cus * 96;
    const long long rest = n4 % (2 * cus);
    return n4 / (2 * cus) * 102 + (rest == 0 ? 0 : rest <= cus ? 80 : 102) < rounds8 * 100;
}

// Whether the key tiles are shared (fwd_split_kernel), for heads x n32 groups of 32 rows: up to a number of groups per compute unit, which was
// measured over 420 shapes (L = 33 - 9000, 1 - 384 heads, 0.9 - 6 groups per unit), each on both kernels.
// All rows of the same length (no mask, or chunks of sequences that are mostly longer than they): two such workgroups share a compute unit, a
// round of 2 per unit costs 40 where narrow_workgroups counts 102 for its own, one more per unit 23, against 80 for the 128-row tiles that leave
// units idle: up to three per unit (training, d = 128: 588 groups 61.7 -> 55.7 us, 752 groups 103.6 -> 87.6 us; 800 groups 46.4 -> 46.6 us; chunks
// of a prefill gain 5 - 120 % up to there), two or less for short rows, where the start of a workgroup is most of it (inference, 144 heads,
// L = 100 21.0 -> 23.6 us; 64 heads, L = 320 25.9 -> 28.0 us).
// Causal: the 128-row tiles wait for their longest chain, these only for a quarter of it: up to six per unit (training, 24 heads, L = 2000 82.9 ->
// 72.4 us; inference, 40 heads, L = 777 37.8 -> 33.8 us, 6 heads, L = 6000 1.5 times), fewer for short rows (inference, 64 heads, L = 256 21.4 -> 18.1 us,
// 96 heads 22.3 -> 23.7 us).
// A group reads K and V for 32 rows instead of 128.  Where the number of heads does not let every head stay on one XCD (spread: a head's groups lie
// on two, four or all eight), the L2s see the K and V of many heads, and with many heads the kernel waits for them: fewer groups (inference, causal,
// 35 heads, L = 1250 53.8 -> 87.8 us, L = 777 36.6 -> 43.7 us; 46 heads, L = 1000 48.8 -> 65.9 us; 44 heads, L = 1000 47.1 -> 49.9 us; but 21 heads, L = 1600 even, 9 heads,
// L = 4000 1.3 times).  Training does twice the work per byte of K and V and loses later (35 heads, L = 1250 64.0 -> 89.7 us, L = 777 43.8 -> 46.6 us).
static bool split_key_tiles(int heads, int n32, bool causal, bool varlen, bool train, bool mx)
{
    const int spread = heads % 8 == 0 ? 0 : heads % 4 == 0 ? 1 : heads % 2 == 0 ? 2 : 3;
    int quarters;                                      // of a group per compute unit
    if (varlen) quarters = n32 < 40 ? 12 : 10;         // (heads stay on their XCD, see varlen_item)
    else if (!causal) {
        if (train) quarters = n32 < 4 ? (mx ? 4 : 12) : n32 == 4 || (n32 > 8 && n32 < 12) ? 8 : 12;
        else quarters = n32 < 4 ? 4 : n32 < 8 ? 8 : n32 < 12 ? (spread ? 4 : 8) : n32 < 16 ? (spread ? 8 : 10) : n32 < 20 ? (spread ? 10 : 12) : n32 < 32 ? (spread ? 8 : 9) : 12;
    } else {
        if (train) quarters = mx && n32 < 4 ? 4 : 4 * min(6, 2 + n32 / 8);
        else quarters = n32 < 4 ? 4 : n32 < 10 ? 8 : n32 < 16 ? 10 : n32 < 32 ? 16 : n32 < 63 ? 20 : 24;
        if (heads > (spread == 0 ? 65535 : spread == 1 ? 28 : spread == 2 ? 22 : 13)) {
            if (train) quarters = min(quarters, spread == 1 ? 24 : mx ? 19 : heads <= (spread == 2 ? 30 : 19) ? 16 : 13);
            else quarters = min(quarters, n32 < 16 ? 8 : n32 < 25 ? 10 : spread == 1 ? (n32 < 32 ? 14 : 18) : spread == 2 && n32 >= 32 && heads <= 30 ? 16 : spread == 2 ? 12 : 13);
        }
    }
    return (long long)heads * n32 * 4 <= (long long)device_cu_count() * quarters;
}
// (P-tilde^F, and P-tilde, of four tiles; row maxima, alpha and two parts of l; Q where it has no registers)
static size_t split_lds_bytes(int D, bool train, int pq) { return (size_t)(train ? 2 : 1) * 4 * 4096 + 4 * 128 * 4 + (train && D == 128 && pq != 1 ? 8192 : 0); }

template <int D, bool TRAIN, bool CAUSAL, bool DUMP, int PQ, bool VARLEN = false>
static int launch_t(const void* qh, const void* kh, const void* vt, int B, int Hq, int Hkv, int L,
                    void* o, float* lse, float* o_hp, int dump_row0, float* p_dump, hipStream_t st,
                    int Lkp = 0, const int* kv_lens = nullptr, bool q_copy = false)
{
    const int Lp = round_up(L, kRowPad);
    const int nqt = (Lp + 255) / 256;
    const int per_head = CAUSAL ? (nqt + 1) / 2 : nqt;         // under a causal mask a workgroup takes a long and a short tile
    const size_t smem = sizeof(FwdSmem<D>);
    const float c = 1.4426950408889634f / sqrtf((float)D);
    auto go = [&](auto kern, unsigned grid, unsigned block, size_t smem, unsigned long long& lds_set) -> int {
        if (!ensure_dynamic_lds(reinterpret_cast<const void*>(kern), (int)smem, lds_set)) return -1;
        hipLaunchKernelGGL(kern, dim3(grid), dim3(block), smem, st,
                           (const half_t*)qh, (const half_t*)kh, (const half_t*)vt, (uint16_t*)o, lse, o_hp,
                           L, Lp, Hq, Hq / Hkv, c, dump_row0, p_dump, Lkp, kv_lens, B, q_copy ? 1 : 0);
        return hipGetLastError() == hipSuccess ? 0 : -1;
    };
    if constexpr (!DUMP && PQ != 2) {
        static unsigned long long lds_set_split = 0;       // one per instantiation
        const int n32 = (L + 31) / 32;
        if (split_key_tiles(B * Hq, n32, CAUSAL, VARLEN, TRAIN, PQ == 1)) {
            const int groups = VARLEN ? round_up(B * Hkv, 8) : B * Hkv;       // (see varlen_item)
            return go(fwd_split_kernel<D, TRAIN, CAUSAL, PQ, VARLEN>, (unsigned)(groups * (Hq / Hkv) * n32), 256, split_lds_bytes(D, TRAIN, PQ), lds_set_split);
        }
    }
    if constexpr (!DUMP) {
        static unsigned long long lds_set_narrow = 0;      // one per instantiation
        if (narrow_workgroups(B * Hq, Lp, D, CAUSAL)) {
            const int groups = VARLEN ? round_up(B * Hkv, 8) : B * Hkv;       // (see varlen_item)
            return go(fwd_narrow_kernel<D, TRAIN, CAUSAL, PQ, VARLEN>, (unsigned)(groups * (Hq / Hkv) * (Lp / 128)), 256, smem, lds_set_narrow);
        }
    }
    static unsigned long long lds_set = 0;          // one per instantiation
    return go(fwd_kernel<D, TRAIN, CAUSAL, DUMP, PQ, VARLEN>, (unsigned)(B * Hq * per_head), 512, smem, lds_set);
}

template <int D, int PQ>
static int launch_d(const void* qh, const void* kh, const void* vt, int B, int Hq, int Hkv, int L,
                    bool causal, bool train, void* o, float* lse, float* o_hp,
                    int dump_row0, float* p_dump, hipStream_t st, bool q_copy)
{
    if (p_dump) {
        return causal ? launch_t<D, false, true, true, PQ>(qh, kh, vt, B, Hq, Hkv, L, o, lse, o_hp, dump_row0, p_dump, st)
                      : launch_t<D, false, false, true, PQ>(qh, kh, vt, B, Hq, Hkv, L, o, lse, o_hp, dump_row0, p_dump, st);
    }
    if constexpr (PQ != 3) {
        if (train) {
            return causal ? launch_t<D, true, true, false, PQ>(qh, kh, vt, B, Hq, Hkv, L, o, lse, o_hp, 0, nullptr, st)
                          : launch_t<D, true, false, false, PQ>(qh, kh, vt, B, Hq, Hkv, L, o, lse, o_hp, 0, nullptr, st);
        }
    }
    return causal ? launch_t<D, false, true, false, PQ>(qh, kh, vt, B, Hq, Hkv, L, o, lse, o_hp, 0, nullptr, st, 0, nullptr, q_copy)
                  : launch_t<D, false, false, false, PQ>(qh, kh, vt, B, Hq, Hkv, L, o, lse, o_hp, 0, nullptr, st, 0, nullptr, q_copy);
}

int launch_fwd(const void* qh, const void* kh, const void* vt,
               int B, int Hq, int Hkv, int L, int D, bool causal, bool train, int p_quant,
               void* o, float* lse, float* o_hp, int dump_row0, float* p_dump, hipStream_t st, bool q_copy)
{
#define AQ_FWD(DD, PQ) launch_d<DD, PQ>(qh, kh, vt, B, Hq, Hkv, L, causal, train, o, lse, o_hp, dump_row0, p_dump, st, q_copy)
    if (p_quant == 3 && train) return -1;           // the bf16 P V recipe has no backward
    if (q_copy && (train || p_quant != 0 || p_dump)) return -1;
    if (D == 128) return p_quant == 1 ? AQ_FWD(128, 1) : p_quant == 2 ? AQ_FWD(128, 2) : p_quant == 3 ? AQ_FWD(128, 3) : AQ_FWD(128, 0);
    if (D == 64)  return p_quant == 1 ? AQ_FWD(64, 1) : p_quant == 2 ? AQ_FWD(64, 2) : p_quant == 3 ? AQ_FWD(64, 3) : AQ_FWD(64, 0);
#undef AQ_FWD
    return -1;
}

// Alg. 1 for sequences of different lengths: the last Lq positions of every sequence as queries, kv_lens[b] keys, K and V^T
// copies laid out for Lkp positions per head (a multiple of 64).
int launch_fwd_varlen(const void* qh, const void* kh, const void* vt, int B, int Hq, int Hkv, int Lq, int Lkp, int D, bool causal,
                      const int* kv_lens, void* o, float* lse, hipStream_t st)
{
    if (!kv_lens || Lkp < 64 || Lkp % 64) return -1;
#define AQ_FWDV(DD, C) launch_t<DD, false, C, false, 0, true>(qh, kh, vt, B, Hq, Hkv, Lq, o, lse, nullptr, 0, nullptr, st, Lkp, kv_lens)
    if (D == 128) return causal ? AQ_FWDV(128, true) : AQ_FWDV(128, false);
    if (D == 64)  return causal ? AQ_FWDV(64, true) : AQ_FWDV(64, false);
#undef AQ_FWDV
    return -1;
}

}  // namespace aq
