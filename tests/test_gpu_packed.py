"""The packed-input forms (attnqat_fwd_infer_packed, attnqat_bwd_packed): Alg. 1 and Alg. 3 on the codes and scales that
attnqat_quantize wrote.  The dequantized values are the same numbers the quantizing calls compute themselves, and the
attention kernels are the same, so the bar is bit equality with attnqat_fwd_infer / attnqat_bwd (whose parity with the
oracle the other tests establish)."""
import pytest
import torch

from tests.gpu_util import random_inputs, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("shape", [(2, 4, 2, 300, 128), (1, 3, 1, 333, 64), (1, 2, 2, 1, 128)])
def test_packed_forms_equal_the_quantizing_forms_bit_for_bit(shape, causal):
    import paper_2603_00040_amd as aq
    B, Hq, Hkv, L, d = shape
    x = random_inputs(B, Hq, Hkv, L, d, seed=800 + L, k_chan=4, dist="t3", scale=0.5, tok_mod=50)
    q, k, v, do = (to_dev(x[n]) for n in ("q", "k", "v", "do"))
    packs = [aq.attnqat_quantize(t, want_xf=False)[:2] for t in (q, k, v)]
    o, lse, ohp = aq.attnqat_fwd(q, k, v, causal)
    oi, lsei = aq.attnqat_fwd_infer(q, k, v, causal)
    op, lsep = aq.attnqat_fwd_infer_packed(*packs, causal, d)
    dq, dk, dv = aq.attnqat_bwd(q, k, v, do, lse, ohp, causal)
    dqp, dkp, dvp = aq.attnqat_bwd_packed(*packs, do, lse, ohp, causal)
    torch.cuda.synchronize()
    assert torch.equal(op, oi) and torch.equal(lsep, lsei)
    assert torch.equal(dqp, dq) and torch.equal(dkp, dk) and torch.equal(dvp, dv)


# Packed Q is read as fp16 rows padded to a multiple of 128, bf16 Q from where it is, quantized by the attention kernel: the same bits in its workgroups of 128 rows
# (80 heads, L = 1000), of 256 rows (128 heads, L = 450) and of a long and a short tile of 256 (32 heads, L = 4001, causal)
@pytest.mark.parametrize("shape,causal", [((2, 40, 8, 1000, 128), False), ((2, 40, 8, 1000, 64), True), ((2, 64, 16, 450, 128), False), ((2, 64, 16, 450, 64), False),
                                          ((1, 32, 4, 4001, 128), True)])
def test_packed_forward_equals_the_quantizing_one_in_whole_workgroups(shape, causal):
    import paper_2603_00040_amd as aq
    B, Hq, Hkv, L, d = shape
    x = random_inputs(B, Hq, Hkv, L, d, seed=900 + L, k_chan=4, dist="t3", scale=0.5, tok_mod=50)
    q, k, v = (to_dev(x[n]) for n in "qkv")
    packs = [aq.attnqat_quantize(t, want_xf=False)[:2] for t in (q, k, v)]
    oi, lsei = aq.attnqat_fwd_infer(q, k, v, causal)
    op, lsep = aq.attnqat_fwd_infer_packed(*packs, causal, d)
    o, lse, _ = aq.attnqat_fwd(q, k, v, causal)
    torch.cuda.synchronize()
    assert torch.equal(op, oi) and torch.equal(lsep, lsei)
    assert torch.equal(o, oi) and torch.equal(lse, lsei)


def test_packed_argument_errors():
    import paper_2603_00040_amd as aq
    L_ = aq.lib()
    z = torch.zeros(4096, dtype=torch.uint8, device="cuda")
    o = torch.zeros((1, 1, 64, 128), dtype=torch.bfloat16, device="cuda"); lse = torch.zeros((1, 1, 64), device="cuda")
    ws = torch.empty(aq.workspace_bytes(aq.WS_FWD_INFER, 1, 1, 1, 64, 128), dtype=torch.uint8, device="cuda")
    p = z.data_ptr()
    f = lambda **kw: L_.attnqat_fwd_infer_packed(kw.get("qc", p), p, p, p, p, p, 1, 1, 1, 64, kw.get("d", 128), 0, 0, o.data_ptr(), lse.data_ptr(),
                                                 ws.data_ptr(), kw.get("wsb", ws.numel()), None)
    assert f() == aq.OK
    assert f(qc=None) == aq.EINVAL and f(qc=p + 4) == aq.EINVAL        # codes are read 8 bytes at a time
    assert f(d=96) == aq.ESHAPE and f(wsb=16) == aq.EWORKSPACE
    torch.cuda.synchronize()
