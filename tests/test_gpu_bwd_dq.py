"""dQ, whose accumulators of dP start from -D and whose exponentials carry the power of two of dS, element by element against float64
with a bound made of the roundings on the way; and the range of dS of a group whose query heads differ in magnitude."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _inputs(Hq, Hkv, L, d, offset, spread, seed):
    g = torch.Generator().manual_seed(seed)
    mk = lambda H: torch.randn(1, H, L, d, generator=g)  # noqa: E731
    q, k, v, do = mk(Hq), mk(Hkv), mk(Hkv) + offset, mk(Hq)
    do = do * torch.exp2(torch.linspace(-spread, spread, L)[torch.randperm(L, generator=g)])[None, None, :, None]
    return [x.to(torch.bfloat16).cuda() for x in (q, k, v, do)]


# tiles of 64 keys in blocks of 32, workgroups of 128 rows: one row, below, at and above the edges; dP and D that nearly cancel (V with a
# large common part) and rows of dO over 110 powers of two (the clamp of the factor of dS at 2^60 among them)
@pytest.mark.parametrize("Hq,Hkv,L,d,causal", [(1, 1, 1, 64, False), (2, 1, 31, 64, True), (2, 2, 97, 64, False), (2, 1, 129, 64, True), (1, 1, 193, 64, False),
                                               (2, 1, 33, 128, True), (2, 2, 160, 128, False), (2, 1, 257, 128, True)])
@pytest.mark.parametrize("offset,spread", [(0.0, 0.0), (96.0, 0.0), (0.0, 55.0)])
@pytest.mark.parametrize("waves", [0, 8])
def test_dq_within_its_roundings(Hq, Hkv, L, d, causal, offset, spread, waves):
    import paper_2603_00040_amd as aq
    q, k, v, do = _inputs(Hq, Hkv, L, d, offset, spread, seed=L + d)
    _, lse, ohp = aq.attnqat_fwd(q, k, v, causal)
    aq.debug_bwd_waves(waves)
    try:
        dq = aq.attnqat_bwd(q, k, v, do, lse, ohp, causal)[0].double().cpu()
    finally:
        aq.debug_bwd_waves(0)
    rep = lambda x: x.double().cpu().repeat_interleave(Hq // x.shape[1], 1)  # noqa: E731
    qf, kf, vf = (rep(aq.attnqat_quantize(x)[2]) for x in (q, k, v))
    do, lse, ohp = do.double().cpu(), lse.double().cpu()[..., None], ohp.double().cpu()
    rs, u = d ** -0.5, 2.0 ** -24
    s = qf @ kf.transpose(2, 3) * rs
    if causal:
        s = s.masked_fill(torch.ones(L, L, dtype=torch.bool).triu(1), -float("inf"))
    p = torch.exp(s - lse)
    dp, D = do @ vf.transpose(2, 3), (do * ohp).sum(3, keepdim=True)
    ds = p * (dp - D) * rs
    want = ds @ kf
    # sums of d products in fp32 (dP with -D in front, and D itself); the exponent (its terms, and the 60 of the factor at most) and exp2;
    # dS to fp16 (half of its smallest step is 2^-25, of a bound on |dS| scaled to 2^14.5 at least, or scaled by 2^60); the sum over the
    # keys in fp32; bf16
    mag = do.abs() @ vf.abs().transpose(2, 3) + (do * ohp).abs().sum(3, keepdim=True)
    s0 = s.masked_fill(s.isinf(), 0.0)
    arg = (d * u * (qf.abs() @ kf.abs().transpose(2, 3)) * rs + 4 * u * (s0.abs() + lse.abs() + 60.0)) * 1.5 + 4 * u
    bound = do.norm(dim=3, keepdim=True) * vf.norm(dim=3).amax(2)[..., None, None] * rs + D.abs() * rs
    err = p * rs * (d + 4) * u * mag + ds.abs() * (arg + 2.0 ** -11) + torch.where(p > 0, (bound * 2.0 ** -39).clamp_min(2.0 ** -85), 0.0)
    tol = (err + L * u * ds.abs()) @ kf.abs()
    assert bool(((dq - want).abs() <= 1.01 * tol + 2.0 ** -8 * want.abs() + 1e-37).all())


@pytest.mark.parametrize("mx", [False, True])
@pytest.mark.parametrize("Hq,Hkv,L,d,causal", [(4, 1, 513, 128, True), (2, 2, 300, 128, False), (2, 1, 640, 64, True), (2, 2, 97, 64, False)])
def test_gradients_scale_exactly_with_dO(Hq, Hkv, L, d, causal, mx):
    """Everything between dO and the gradients is linear in dO and rounds relative to its size: dO times a power of two gives the same
    gradients times that power, bit for bit, as long as nothing leaves the normal range (the gradients of 2^-40 dO lie above 2^-100)."""
    import paper_2603_00040_amd as aq
    q, k, v, do = _inputs(Hq, Hkv, L, d, 0.0, 0.0, seed=L)
    fwd, bwd = (aq.attnqat_fwd_mx, aq.attnqat_bwd_mx) if mx else (aq.attnqat_fwd, aq.attnqat_bwd)
    _, lse, ohp = fwd(q, k, v, causal)
    one = bwd(q, k, v, do, lse, ohp, causal)
    for e in (-40, -17, 20):
        got = bwd(q, k, v, do * 2.0 ** e, lse, ohp, causal)
        for name, a, b in zip(("dQ", "dK", "dV"), got, one):
            assert torch.equal(a, b * 2.0 ** e), (name, e, float((a.double() - b.double() * 2.0 ** e).norm() / (b.double() * 2.0 ** e).norm()))


def test_dq_where_the_factor_of_ds_would_overflow_dO():
    """V^F all but zero and dO large: dS is tiny, its factor 2^60 and dO beyond the range that dO times that has in bf16."""
    import paper_2603_00040_amd as aq
    for d, causal in ((64, True), (128, False)):
        q, k, v, do = _inputs(2, 1, 130, d, 0.0, 0.0, seed=d)
        v.zero_()
        do *= 2.0 ** 90
        _, lse, ohp = aq.attnqat_fwd(q, k, v, causal)
        dq, dk, dv = aq.attnqat_bwd(q, k, v, do, lse, ohp, causal)
        assert not bool(dq.any()) and not bool(dk.any()) and bool(torch.isfinite(dv.float()).all())


@pytest.mark.parametrize("head", [0, 4, 7])
def test_factor_of_ds_covers_every_head_of_a_group(head):
    """dS of a kv head is scaled by the largest of its eight query heads, whichever that is: fp16 would overflow otherwise."""
    import paper_2603_00040_amd as aq
    q, k, v, do = _inputs(8, 1, 140, 64, 0.0, 0.0, seed=head)
    do[:, head] *= 2.0 ** 24
    _, lse, ohp = aq.attnqat_fwd(q, k, v, False)
    dk = aq.attnqat_bwd(q, k, v, do, lse, ohp, False)[1].double()
    one = aq.attnqat_bwd(q[:, head:head + 1].contiguous(), k, v, do[:, head:head + 1].contiguous(), lse[:, head:head + 1].contiguous(),
                         ohp[:, head:head + 1].contiguous(), False)[1].double()
    # the other heads add 2^-24 of it (their own size, 1, against 2^24; seven of them, their dS rounded to steps of 2^-39 of the bound)
    assert bool(torch.isfinite(dk).all()) and float((dk - one).norm()) <= 2.0 ** -7 * float(one.norm())


@pytest.mark.parametrize("H,L,causal", [(32, 4096, False), (4, 32700, True)])
@pytest.mark.parametrize("mx", [False, True])
def test_large_problems_of_d64_run_both_passes_in_one_launch(H, L, causal, mx):
    """Shapes whose eight-wave workgroups fill the chip evenly: at d = 64 one launch of four-wave workgroups, the bits of the separate passes."""
    import paper_2603_00040_amd as aq
    g = torch.Generator(device="cuda").manual_seed(L)
    q, k, v, do = (torch.randn(1, H, L, 64, generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
    fwd, bwd = (aq.attnqat_fwd_mx, aq.attnqat_bwd_mx) if mx else (aq.attnqat_fwd, aq.attnqat_bwd)
    _, lse, ohp = fwd(q, k, v, causal)
    got = bwd(q, k, v, do, lse, ohp, causal)
    for waves in (4, 8):
        aq.debug_bwd_waves(waves)
        try:
            want = bwd(q, k, v, do, lse, ohp, causal)
        finally:
            aq.debug_bwd_waves(0)
        assert all(torch.equal(a, b) for a, b in zip(got, want))
