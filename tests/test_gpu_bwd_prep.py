"""dO is read by the backward's attention passes as it is where its rows need no padding and its address suits the 16-byte copies
to LDS, and from a copy otherwise: the results do not depend on which."""
import pytest
import torch

from tests.gpu_util import random_inputs, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,L,d,causal", [(1, 2, 2, 256, 64, False), (1, 4, 2, 384, 128, True), (2, 2, 1, 129, 128, False)])
def test_address_of_do_does_not_matter(B, Hq, Hkv, L, d, causal):
    import paper_2603_00040_amd as aq
    x = random_inputs(B, Hq, Hkv, L, d, seed=L)
    q, k, v, do = (to_dev(x[n]) for n in ("q", "k", "v", "do"))
    odd = torch.empty(do.numel() + 4, dtype=do.dtype, device="cuda")[4:].view(do.shape)      # 8 bytes off
    odd.copy_(do)
    assert do.data_ptr() % 16 == 0 and odd.data_ptr() % 16 == 8
    for fwd, bwd in ((aq.attnqat_fwd, aq.attnqat_bwd), (aq.attnqat_fwd_mx, aq.attnqat_bwd_mx)):
        _, lse, ohp = fwd(q, k, v, causal)
        a, b = bwd(q, k, v, do, lse, ohp, causal), bwd(q, k, v, odd, lse, ohp, causal)
        assert all(torch.equal(s, t) for s, t in zip(a, b))
