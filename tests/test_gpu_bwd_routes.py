"""Backwards on either side of the rule for few rows: the kernel that the shape is for is the one that runs (the marks of the timing interface), and it gives the
results of the two passes one after another."""
import pytest
import torch

from tests.gpu_util import random_inputs, to_dev

pytestmark = pytest.mark.gpu

# (B, Hq, Hkv, L, d, causal).  The four waves of a workgroup share 32 rows: groups up to one per compute unit, two under a mask; four tiles at a time, below, at
# and above whole rounds of them; several query heads to a kv head
FEW = [(1, 2, 2, 256, 64, False), (1, 1, 1, 1, 128, True), (1, 8, 1, 129, 64, False), (1, 8, 8, 480, 64, False), (1, 4, 4, 1000, 128, False), (1, 8, 8, 999, 128, True),
       (1, 4, 2, 300, 128, False), (1, 1, 1, 3900, 64, True)]
# heads of their own whose key tiles are cut: dQ tiles first, under a mask and without one, and last; a last tile of a few rows
CUT = [(1, 2, 2, 4200, 128, True), (1, 4, 4, 3000, 64, False), (2, 3, 3, 1409, 128, False), (1, 2, 2, 6001, 64, True), (1, 12, 12, 1560, 128, False)]
# cut, but small: no room for partial sums is asked for
SPARE = [(1, 2, 2, 256, 64, False), (1, 4, 4, 384, 64, False), (1, 2, 1, 512, 64, True), (1, 1, 1, 600, 128, False), (1, 8, 1, 512, 64, False)]


def _inputs(aq, B, Hq, Hkv, L, d, causal, fwd):
    x = random_inputs(B, Hq, Hkv, L, d, seed=L + Hq + d, k_chan=4)
    q, k, v, do = (to_dev(x[n]) for n in ("q", "k", "v", "do"))
    _, lse, ohp = fwd(q, k, v, causal)
    return q, k, v, do, lse, ohp


def _marks(aq, run):
    aq.profile_enable(True)
    try:
        out = run()
        torch.cuda.synchronize()
        return out, [n for n, _ in aq.profile_read()]
    finally:
        aq.profile_enable(False)


def _separate(aq, run):
    aq.debug_bwd_waves(4)
    try:
        return run()
    finally:
        aq.debug_bwd_waves(0)


@pytest.mark.parametrize("B,Hq,Hkv,L,d,causal", FEW)
def test_few_rows(B, Hq, Hkv, L, d, causal):
    import paper_2603_00040_amd as aq
    args = _inputs(aq, B, Hq, Hkv, L, d, causal, aq.attnqat_fwd)
    got, marks = _marks(aq, lambda: aq.attnqat_bwd(*args, causal))
    assert marks == ["prep_qkvdo", "bwd_few"], marks
    want, marks = _marks(aq, lambda: _separate(aq, lambda: aq.attnqat_bwd(*args, causal)))
    assert marks == ["prep_qkvdo", "bwd_dq", "bwd_dkdv"], marks
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("B,Hq,Hkv,L,d,causal", CUT)
def test_cut_key_tiles_of_heads_of_their_own(B, Hq, Hkv, L, d, causal):
    import paper_2603_00040_amd as aq
    args = _inputs(aq, B, Hq, Hkv, L, d, causal, aq.attnqat_fwd)
    got, marks = _marks(aq, lambda: aq.attnqat_bwd(*args, causal))
    assert marks == ["prep_qkvdo", "bwd_joint"], marks
    assert all(torch.equal(a, b) for a, b in zip(got, aq.attnqat_bwd(*args, causal)))
    want = _separate(aq, lambda: aq.attnqat_bwd(*args, causal))
    assert torch.equal(got[0], want[0])
    for a, r in zip(got[1:], want[1:]):
        # the same fp32 terms added in another grouping (errors of 2^-24 times the sum of their magnitudes, here at most some
        # hundred times the largest result), then one rounding to bf16 each: apart by at most one spacing
        a, r = a.float(), r.float()
        assert bool(((a - r).abs() <= 2.0 ** -7 * r.abs() + 1e-4 * r.abs().max()).all())
    # no room for the partial sums: the order of the separate passes
    nq, nk, Lp = B * Hq, B * Hkv, (L + 127) // 128 * 128
    align = lambda n: (n + 255) // 256 * 256  # noqa: E731
    small = torch.empty(2 * (nq + nk) * Lp * d * 2 + align(nq * Lp * 8) + align(3 * nq * 64 * 4) + align(nk * 32 * d * 8) + align(nk * d * 4),
                        dtype=torch.uint8, device="cuda")
    assert small.numel() < aq.workspace_bytes(aq.WS_BWD, B, Hq, Hkv, L, d)
    assert all(torch.equal(a, b) for a, b in zip(aq.attnqat_bwd(*args, causal, workspace=small), want))


@pytest.mark.parametrize("B,Hq,Hkv,L,d,causal", SPARE)
@pytest.mark.parametrize("mx", [False, True])
def test_bits_of_the_joint_launch_do_not_depend_on_spare_room(B, Hq, Hkv, L, d, causal, mx):
    """MX and two-level backwards keep the joint launch where an NVFP4 one has few rows: below the size from which room for partial sums is asked for they
    run unsplit in any workspace, with the bits of the separate passes."""
    import paper_2603_00040_amd as aq
    if mx:
        args, which, bwd = _inputs(aq, B, Hq, Hkv, L, d, causal, aq.attnqat_fwd_mx), aq.WS_BWD_MX, lambda *a, **kw: aq.attnqat_bwd_mx(*a, causal, **kw)
    else:
        args = _inputs(aq, B, Hq, Hkv, L, d, causal, lambda q, k, v, c: aq.attnqat_fwd_opt(q, k, v, c, aq.OPT_TWO_LEVEL_P))
        which, bwd = aq.WS_BWD, lambda *a, **kw: aq.attnqat_bwd_opt(*a, causal, aq.OPT_TWO_LEVEL_P, **kw)
    size = aq.workspace_bytes(which, B, Hq, Hkv, L, d)
    assert size < 2 << 20
    run = lambda n: bwd(*args, workspace=torch.empty(n, dtype=torch.uint8, device="cuda"))  # noqa: E731
    want = _separate(aq, lambda: run(size))
    for spare in (0, 256, 64 << 20):
        got, marks = _marks(aq, lambda: run(size + spare))
        assert marks == ["prep_qkvdo", "bwd_joint"], marks
        assert all(torch.equal(a, b) for a, b in zip(got, want)), spare
