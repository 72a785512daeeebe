"""The joint backward under a causal mask where the query tiles of a key tile are shared out in pieces: every piece is computed once, whatever the number of
pieces of a tile."""
import pytest
import torch

from tests.gpu_util import random_inputs, to_dev

pytestmark = pytest.mark.gpu


# more than 64 pieces in the first key tile (groups of lanes count them), tiles with four pieces to one, a last tile of a few rows, two kv heads per XCD, heads that are
# no multiple of the XCDs
@pytest.mark.parametrize("mx", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,L,d", [(1, 64, 1, 512, 128), (1, 64, 1, 600, 64), (2, 16, 4, 1601, 128), (1, 32, 16, 1300, 128), (1, 12, 3, 2050, 64)])
def test_equals_separate_passes(B, Hq, Hkv, L, d, mx):
    import paper_2603_00040_amd as aq
    fwd, bwd = (aq.attnqat_fwd_mx, aq.attnqat_bwd_mx) if mx else (aq.attnqat_fwd, aq.attnqat_bwd)
    x = random_inputs(B, Hq, Hkv, L, d, seed=L + d, k_chan=4)
    q, k, v, do = (to_dev(x[n]) for n in ("q", "k", "v", "do"))
    _, lse, ohp = fwd(q, k, v, True)
    got = bwd(q, k, v, do, lse, ohp, True)
    aq.debug_bwd_waves(4)
    try:
        want = bwd(q, k, v, do, lse, ohp, True)
    finally:
        aq.debug_bwd_waves(0)
    assert torch.equal(got[0], want[0])
    for a, b in zip(got[1:], want[1:]):
        a, b = a.float(), b.float()
        # the same fp32 terms in another grouping, both rounded to bf16: an element moves by one bf16 step (2^-8 of it) at most, beside fp32 errors of the sums
        # (a few thousand terms, 2^-24 of the largest partial sum each); a missing or doubled piece moves whole columns by their own size
        assert float((a - b).norm() / b.norm()) < 2.0 ** -8
        n = b.norm(dim=-1)
        assert float(((a - b).norm(dim=-1) / (n + 1e-3 * n.max())).max()) < 2.0 ** -4
