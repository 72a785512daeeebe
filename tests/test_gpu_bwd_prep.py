"""dO is read by the backward's attention passes as it is where its rows need no padding and its address suits the 16-byte copies
to LDS and no result is written over it, and from a copy otherwise: the results do not depend on which."""
import numpy as np
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


@pytest.mark.parametrize("Hq,Hkv,L,d,causal", [(2, 2, 256, 64, False), (4, 2, 257, 128, True), (4, 4, 256, 128, True), (8, 8, 4096, 64, True)])
@pytest.mark.parametrize("mx", [False, True])
@pytest.mark.parametrize("waves", [0, 4, 8])
def test_results_written_over_do(Hq, Hkv, L, d, causal, mx, waves):
    """dQ (and with as many kv heads dK, dV) has the shape and type of dO and may take its place, whole or in part."""
    import paper_2603_00040_amd as aq
    x = random_inputs(1, Hq, Hkv, L, d, seed=L)
    q, k, v, do = (to_dev(x[n]) for n in ("q", "k", "v", "do"))
    fwd, bwd = (aq.attnqat_fwd_mx, aq.attnqat_bwd_mx) if mx else (aq.attnqat_fwd, aq.attnqat_bwd)
    _, lse, ohp = fwd(q, k, v, causal)
    aq.debug_bwd_waves(waves)
    try:
        want = bwd(q, k, v, do, lse, ohp, causal)
        for which in range(3 if Hq == Hkv else 1):
            for shift in (0, 8 * d):                    # the result in dO's place, or eight rows behind it
                room = torch.empty(do.numel() + shift, dtype=do.dtype, device="cuda")
                buf, res = room[:do.numel()].view(do.shape).copy_(do), room[shift:].view(do.shape)
                out = [torch.empty_like(t) for t in (q, k, v)]
                out[which] = res
                got = bwd(q, k, v, buf, lse, ohp, causal, out=tuple(out))
                assert all(torch.equal(a, b) for a, b in zip(got, want)), (which, shift)
    finally:
        aq.debug_bwd_waves(0)


def _sum_in_order(x):
    """fp32 sum of the last axis, eight at a time (pairs 0, 2, 1, 3 of them), the groups of eight in a tree whose last level joins neighbours."""
    x = x.astype(np.float32)
    pairs = (x[..., 0::2] + x[..., 1::2]).reshape(*x.shape[:-1], -1, 4)
    s = ((pairs[..., 0] + pairs[..., 2]) + pairs[..., 1]) + pairs[..., 3]
    while s.shape[-1] > 1:
        half = s.shape[-1] // 2
        s = s[..., :half] + s[..., half:]
    return s[..., 0]


@pytest.mark.parametrize("L,d", [(128, 64), (100, 64), (256, 128), (129, 128)])
def test_d_is_summed_in_its_order(L, d):
    """D = rowsum(dO o O') with terms that cancel: its value shows the order of the fp32 sum.  With Q = 0, V = 0, dO = 1 and K = 1 every
    product is exact and dQ_i = -D_i K^F / sqrt(d), up to the roundings of dS to fp16 and of dQ to bf16."""
    import paper_2603_00040_amd as aq
    rng = np.random.default_rng(L + d)
    big = np.exp2(rng.integers(18, 24, size=(L, d // 4))) * (1.0 + rng.integers(0, 2 ** 10, size=(L, d // 4)) / 2.0 ** 10)
    o = rng.permuted(np.concatenate([big, -big, rng.standard_normal((L, d // 2))], axis=1), axis=1).astype(np.float32)
    D = _sum_in_order(o)
    other = o.astype(np.float32).cumsum(axis=1, dtype=np.float32)[:, -1]
    assert (np.abs(other - D) > 0.1 * np.abs(D)).sum() > L // 8          # another order would be seen
    one = torch.ones((1, 1, L, d), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((1, 1, L), float(np.log(L)), device="cuda")
    zero = torch.zeros_like(one)
    for bwd in (aq.attnqat_bwd, aq.attnqat_bwd_mx):
        dq = bwd(zero, one, zero, one, lse, torch.from_numpy(o)[None, None].cuda(), False)[0][0, 0].float().cpu().numpy()
        factor = dq[np.abs(D).argmax(), 0] / D[np.abs(D).argmax()]
        # one rounding to fp16 and one to bf16 on either side of the comparison
        assert (np.abs(dq - factor * D[:, None]) <= 2.0 * (2.0 ** -9 + 2.0 ** -11 + 1e-4) * np.abs(factor * D[:, None])).all(), bwd.__name__
