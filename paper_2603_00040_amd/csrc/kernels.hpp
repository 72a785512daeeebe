// Host-side launchers of the gfx950 kernels (one translation unit each).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "plan.hpp"

namespace aq {

// Compute units of a whole MI355X: what the size queries plan for.  They ask no device (they have to work on a machine without one,
// and a process that asked for a size may still fork); a call plans for the device it runs on and does with the room it is given.
constexpr int kChipCus = 256;

// phi of x [BH, L, D] bf16 in the public layout (codes, scales, bf16 dequantized copy xf; any may be null).
int launch_quantize(const void* x, int BH, int L, int D, uint8_t* codes, uint8_t* scales, void* xf, hipStream_t st);

// The pages of an NVFP4 KV cache as a source of K or V.
struct PagedSrc {
    const unsigned char* cache; const int* table; const int* kv_lens;
    int max_pages, num_pages, Hkv, which;          // which: 0 the K part, 1 the V part
};

// Everything a forward or a backward prepares, in one launch.  Q and K become fp16 rows (zero padded to Lp = round_up(L, 128)), V
// becomes transposed fp16 (forward; bf16 and unquantized with v_quant = false) or bf16 rows (backward).  From bf16 tensors, or
// from codes and scales (attnqat_quantize's layout; codes[2] != null), or, K and V, from the pages of a cache (ps.cache != null).
// With grad.d_o the statistics of the backward are made as well (Alg. 3, first line): rowstat [BHq, Lp, 2] = {L log2(e), D},
// D = rowsum(dO o O'), zeros in the padding rows; and in bounds, 3 * BHq * kBoundParts floats, partial maxima per head
// that limit |dS|: |V^F_j| (kv heads), |dO_i|, |D_i| / sqrt(d).
constexpr int kBoundParts = 64;
struct GradArgs {
    const uint16_t* d_o; const void* o_acc; bool o_is_bf16; const float* lse; float rs /* 1 / sqrt(d) */;
    float2* rowstat; float* bounds; uint16_t* dob;         // dob: zero-padded copy of dO, or null
};
struct PrepGroup {
    const uint16_t *q, *k, *v;
    const uint8_t *codes[3], *scales[3];
    uint16_t *q_out, *k_out, *v_out;             // q_out: Q^F (backward, packed inputs) or a copy of Q [BHq, L, D] (forward of bf16 Q), null: none; k_out null: K is left out
    const float* k_sub;                          // [BHkv, D]: subtracted from the rows of K before phi (K smoothing)
    int BHq, BHkv, L, Lp, L_kv, Lp_kv, D;
    bool v_quant;
    PagedSrc ps;
    GradArgs grad;
};
int launch_prep_group(const PrepGroup& g, hipStream_t st);

// Token mean of every channel of x [BH, L, D] bf16 -> mean [BH, D] fp32 (fp64 sums in a fixed order).
// scratch: colmean_scratch_bytes() bytes.
size_t colmean_scratch_bytes(int BH, int D);
int launch_colmean(const void* x, int BH, int L, int D, double* scratch, float* mean, hipStream_t st);

// Alg. 1 (train=false) / Alg. 2 (train=true): q is Q itself in bf16, of which the kernels make phi(Q) (no result may lie over it), kh and vt are copies made by
// launch_prep_group.  q_copy (inference, p_quant 0): q is such a copy too.
// p_quant 1 (MX): kh the K records of launch_mx_group (MX_TRAIN, krec), not fp16
// copies: the scores are computed from the codes; vt stays the fp16 copy.
// p_quant: phi(P-tilde) 0 NVFP4; 1 in the MX format (blocks of 32 keys, power-of-two scale); 2 NVFP4 after the
// two-level row factor (every 64-key tile row divided by a power of two that brings its maximum just below 448 * 6).
int launch_fwd(const void* q, const void* kh, const void* vt,
               int B, int Hq, int Hkv, int L, int D, bool causal, bool train, int p_quant,
               void* o, float* lse, float* o_hp, int dump_row0, float* p_dump, hipStream_t st, bool q_copy = false);

// Alg. 1 for sequences of different lengths (serving): queries are the last Lq positions of every sequence, sequence b has
// kv_lens[b] keys (device array), kh / vt are laid out for Lkp positions per kv head.
int launch_fwd_varlen(const void* q, const void* kh, const void* vt, int B, int Hq, int Hkv, int Lq, int Lkp, int D, bool causal,
                      const int* kv_lens, void* o, float* lse, hipStream_t st);

// The NVFP4 KV cache (pages of 128 positions; per kv head K codes, K scales, V codes, V scales in the public layout).
size_t nvfp4_page_bytes(int Hkv, int D);
int launch_kv_page_write(const void* k, const void* v, int Hkv, int n, int D, int pos0,
                         void* cache, int num_pages, const int* page_ids, hipStream_t st);

// Alg. 1 for decode steps over the NVFP4 pages: at most decode_max_rows() query rows per (sequence, kv head), i.e.
// (Hq / Hkv) * Lq of them; q [B*Hkv, (Hq/Hkv)*Lq, D] (the rows of a kv group are neighbours in [B,Hq,Lq,d]); qh: scratch for
// phi(Q), [B*Hkv][128][D] fp16.  ws: decode_ws_bytes() bytes.  spin_limit bounds the polls of a chunk waiting for the row maxima
// of the chunks before it (see decode.hip); if it runs out the int at ws + 4 is set and that result is wrong.
int decode_max_rows();
int decode_halvings(int B, int Hkv, int R, int max_pages, int cus);        // how often the chunks of keys are halved at best; any smaller number works
size_t decode_ws_bytes(int B, int Hkv, int R, int max_pages, int D, int halvings);
int launch_decode(const void* q, void* qh, const void* cache, int num_pages, const int* page_table, int max_pages, const int* kv_lens,
                  int B, int Hq, int Hkv, int Lq, int D, bool causal, void* ws, int halvings, int spin_limit, void* o, float* lse, hipStream_t st);

// The same for a step with few chunks: two launches without a queue (see decode.hip).  ws: decode_direct_ws_bytes() bytes.
bool decode_is_direct(int B, int Hkv, int R, int max_pages, int cus);
size_t decode_direct_ws_bytes(int B, int Hkv, int R, int max_pages);
int launch_decode_direct(const void* q, const void* cache, int num_pages, const int* page_table, int max_pages, const int* kv_lens,
                         int B, int Hq, int Hkv, int Lq, int D, bool causal, void* ws, void* o, float* lse, hipStream_t st);

// The MX format's operand arrays of the scaled FP4 instruction, from which the backward recomputes the scores (launch_mx_group):
// kops / ksc: a wave's 32 keys as the A operand of the dK/dV pass; krec: 64-key records, the A operand of the dQ pass.
struct MxScoreOps { const void *qops, *qsc, *kops, *ksc, *krec; };

// Alg. 3, query-stationary pass: dQ.  qh, kh: fp16 copies; vb, dob: bf16 copies.
int launch_bwd_dq(const void* qb, const void* kb, const void* vb, const void* dob,
                  const float* rowstat, const float* bound_part,
                  int B, int Hq, int Hkv, int L, int D, bool causal, void* dq, hipStream_t st,
                  const MxScoreOps* mx = nullptr /* the MX format: scores from the codes */);

// Alg. 3, key-stationary pass: dK, dV (summed over the query heads of a group).
int launch_bwd_dkdv(const void* qb, const void* kb, const void* vb, const void* dob,
                    const float* rowstat, const float* bound_part,
                    int B, int Hq, int Hkv, int L, int D, bool causal, void* dk, void* dv,
                    unsigned long long* tile_counts /* may be null */,
                    int p_quant /* phi(P): 0 none (ablation), 1 NVFP4, 2 MX, 3 NVFP4 with the two-level row factor */, hipStream_t st,
                    float* p_dump = nullptr /* test hook, p_quant 1 only: P^F of query rows [dump_row0, dump_row0 + 128), [B*Hq][128][L] */,
                    int dump_row0 = 0, const MxScoreOps* mx = nullptr /* p_quant 2: required */);
// Both passes in one launch (plan.joint: problems that do not fill the chip evenly), as planned (plan.hpp); partial sums meet in `part`.
// launch_bwd_dq and launch_bwd_dkdv run what is not joint.
BwdPlan bwd_plan(int BHq, int BHkv, int L, int D, bool causal, int cus);
int launch_bwd_joint(const void* qb, const void* kb, const void* vb, const void* dob, const float* rowstat, const float* bound_part,
                     int B, int Hq, int Hkv, int L, int D, bool causal, void* dq, void* dk, void* dv, int p_quant /* 1, 2 or 3 */,
                     const BwdPlan& plan, float* part, unsigned long long* tile_counts, hipStream_t st, float* p_dump, int dump_row0,
                     const MxScoreOps* mx);
// Both passes of an NVFP4 backward of few rows, with the bits of the others where those share no key tile among workgroups (few_rows in plan.hpp; never
// while set_bwd_waves forces separate passes).
bool bwd_few_rows(int BHq, int BHkv, int L, bool causal, bool pieces, int cus);
int launch_bwd_few(const void* qb, const void* kb, const void* vb, const void* dob, const float* rowstat, const float* bound_part,
                   int B, int Hq, int Hkv, int L, int D, bool causal, void* dq, void* dk, void* dv, hipStream_t st);
// Waves per workgroup of the dQ and dK/dV passes: 0 = chosen per problem (the default), 4 or 8 = forced where that
// variant exists (8: not the ablation and not the counting variant).  Process-wide; for tests.
void set_bwd_waves(int waves);

// ---- MX variant (E2M1, blocks of 32, E8M0 scale; mx.hip, mxprep.hip) ----
// The public quantizer: phi with the blocks along d (axis 0) or along the sequence (axis 1).  x [BH, L, D] bf16; codes, scales,
// optional bf16 xf: see attnqat.h.  fp8: E4M3 elements instead of E2M1 (axis 1 only).
int launch_mx_quant(const void* x, int BH, int L, int D, int axis, bool fp8, unsigned char* codes, unsigned char* scales, void* xf, hipStream_t st);
// Everything that an MX forward or backward prepares, in one launch (null outputs are left out):
//   Q: operands of the scaled MFMA (qops, scale dwords qsc)              [not MX_TRAIN]; fp16 rows q_row    [MX_BWD]; a copy of Q in q_row    [MX_TRAIN]
//   K: the K part of the 64-key kv records kv                            [MX_INFER, MX_INFER_FP8V]
//      records in natural key order krec                                 [MX_TRAIN, MX_BWD]
//      operands kops, ksc as of Q; fp16 rows k_row                       [MX_BWD]
//   V: the V part of the kv records                                      [MX_INFER, MX_INFER_FP8V (E4M3 elements)]
//      transposed fp16 v_out (the layout of launch_prep_group)           [MX_TRAIN]
//      bf16 rows v_out and the bound of |V^F_j| in grad.bounds           [MX_BWD]
//   dO and O': grad, as in launch_prep_group                             [MX_BWD]
//   the block lists of a block-sparse forward: list, list_count from mask [BHq * nb, nb] bytes, nb = Lp / 128   [MX_INFER]
// page_ids (MX_INFER; device int32, one entry per 128 positions): the records go into the pages of a KV cache laid out
// [page][kv head][2 records] instead of one after another; BHkv then is the number of kv heads of ONE sequence.  Records whose
// page id lies outside [0, num_pages) are not written.
enum MxKind { MX_INFER, MX_INFER_FP8V, MX_TRAIN, MX_BWD };
struct MxGroup {
    const uint16_t *q, *k, *v;                   // q null: no Q; k and v null: neither
    unsigned char *qops, *qsc, *kops, *ksc, *krec, *kv;
    uint16_t *q_row, *k_row, *v_out;
    int BHq, BHkv, L, Lp;
    const int* page_ids; int num_pages;
    const unsigned char* mask; int *list, *list_count;
    GradArgs grad;
};
int launch_mx_group(const MxGroup& g, MxKind kind, int D, hipStream_t st);
size_t mx_kv_bytes(int BHkv, int L, int D, bool fp8v);
size_t mx_ktrain_bytes(int BHkv, int L, int D);      // K records of the MX training forward (krec)
size_t mx_qops_bytes(int BHq, int L, int D);
size_t mx_qsc_bytes(int BHq, int L);
// Alg. 1 on the arrays made by launch_mx_group, here and below with Q itself in the place of qops where qsc is null.  fp8pv: P-tilde and V in MXFP8 (mixed recipe).
int launch_fwd_mx(const void* qops, const void* qsc, const void* kv, int B, int Hq, int Hkv, int L, int D, bool causal, bool fp8pv,
                  void* o, float* lse, hipStream_t st);

// The same forward on a paged KV cache: a head has Lq rows, positions kv_lens[b] - lq_inner .. of its sequence, repeated
// Lq / lq_inner times when the query heads of a kv group are packed into one head (then Hq == Hkv).
size_t mx_page_bytes(int D);
int launch_fwd_mx_paged(const void* qops, const void* qsc, const void* cache, int B, int Hq, int Hkv, int Lq, int D, bool causal,
                        const int* page_table, const int* kv_lens, int max_pages, int num_pages, int lq_inner,
                        unsigned char* part /* mx_decode_part_bytes() bytes, or null: one workgroup per head */, void* o, float* lse, hipStream_t st);
constexpr int kMxDecUnits = 2048;                   // most chunks of pages, times heads, of a decode step
constexpr int kMxDecPageHeads = 8192;               // most pages, times heads, whose P the workspace of a decode step has room for
size_t mx_decode_part_bytes(int heads /* B * Hq */, int Lq, int D);      // 0: such a step is not cut into chunks

// Block-sparse forward on contiguous kv records, over the block lists that launch_mx_group made: list [B*Hq*nb, nb] and
// cnt [B*Hq*nb], int32, nb = ceil(L/128).
int launch_fwd_mx_sparse(const void* qops, const void* qsc, const void* kv, int B, int Hq, int Hkv, int L, int D, bool causal,
                         const int* list, const int* cnt, void* o, float* lse, hipStream_t st);

}  // namespace aq
