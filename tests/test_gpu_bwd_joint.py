"""The backward as one launch of both passes, several workgroups sharing the query tiles of a key tile, against the two passes one
after another (their parity with the oracle is tested elsewhere)."""
import pytest
import torch

from tests.gpu_util import random_inputs, to_dev

pytestmark = pytest.mark.gpu


# tiles of 32 queries and 128 keys: below, at and above their edges; one head with many keys (dQ tiles first), few kv heads with
# many query heads (pieces span heads), whole rounds of the compute units' slots and more.  (NVFP4 with few rows takes another kernel, four of these shapes among
# them: they are the joint launch's in MX; tests/test_gpu_bwd_routes.py has NVFP4 shapes that are its own)
@pytest.mark.parametrize("B,Hq,Hkv,L,d,causal", [(1, 1, 1, 1, 64, True), (1, 2, 1, 33, 128, True), (1, 8, 1, 129, 64, False), (1, 32, 8, 777, 128, True),
                                                 (1, 12, 12, 1560, 128, False), (1, 1, 1, 4200, 128, True), (2, 16, 2, 1000, 64, True), (1, 40, 40, 1664, 64, True)])
@pytest.mark.parametrize("mx", [False, True])
def test_joint_equals_separate_passes(B, Hq, Hkv, L, d, causal, mx):
    import paper_2603_00040_amd as aq
    x = random_inputs(B, Hq, Hkv, L, d, seed=L + Hq)
    q, k, v, do = (to_dev(x[n]) for n in ("q", "k", "v", "do"))
    fwd, bwd, which = (aq.attnqat_fwd_mx, aq.attnqat_bwd_mx, aq.WS_BWD_MX) if mx else (aq.attnqat_fwd, aq.attnqat_bwd, aq.WS_BWD)
    _, lse, ohp = fwd(q, k, v, causal)
    size = aq.workspace_bytes(which, B, Hq, Hkv, L, d)
    large = torch.empty(size + (256 << 20), dtype=torch.uint8, device="cuda")
    dq, dk, dv = bwd(q, k, v, do, lse, ohp, causal, workspace=large)
    again = bwd(q, k, v, do, lse, ohp, causal, workspace=large)
    assert all(torch.equal(a, b) for a, b in zip((dq, dk, dv), again))
    aq.debug_bwd_waves(4)
    try:
        rq, rk, rv = bwd(q, k, v, do, lse, ohp, causal)
    finally:
        aq.debug_bwd_waves(0)
    assert torch.equal(dq, rq)
    for a, r in ((dk, rk), (dv, rv)):
        # the same fp32 terms added in another grouping (errors of 2^-24 times the sum of their magnitudes, here at most some
        # hundred times the largest result), then one rounding to bf16 each: apart by at most one spacing
        a, r = a.float(), r.float()
        assert bool(((a - r).abs() <= 2.0 ** -7 * r.abs() + 1e-4 * r.abs().max()).all())
    # a workspace without room for the partial sums: one workgroup per key tile, the order of the separate passes
    if mx:
        return
    nq, nk, Lp = B * Hq, B * Hkv, (L + 127) // 128 * 128
    align = lambda n: (n + 255) // 256 * 256  # noqa: E731
    small = torch.empty(2 * (nq + nk) * Lp * d * 2 + align(nq * Lp * 8) + align(3 * nq * 64 * 4) + align(nk * 32 * d * 8) + align(nk * d * 4),
                        dtype=torch.uint8, device="cuda")
    got = bwd(q, k, v, do, lse, ohp, causal, workspace=small)
    assert all(torch.equal(a, b) for a, b in zip(got, (rq, rk, rv)))


@pytest.mark.parametrize("B,Hq,Hkv,L,d,causal", [(1, 2, 2, 256, 64, False), (1, 4, 4, 384, 64, False), (1, 2, 1, 512, 64, True), (1, 1, 1, 600, 128, False),
                                                 (1, 4, 2, 1100, 128, True)])
def test_bits_do_not_depend_on_spare_room(B, Hq, Hkv, L, d, causal):
    """Whether a key tile's query tiles are shared follows from the shape: every workspace from the size asked for on gives the same bits
    (the first four ask for no partial sums, the last one does; the first four have few rows and so no partial sums in any workspace, which
    tests/test_gpu_bwd_routes.py has for the joint launch)."""
    import paper_2603_00040_amd as aq
    x = random_inputs(B, Hq, Hkv, L, d, seed=L)
    q, k, v, do = (to_dev(x[n]) for n in ("q", "k", "v", "do"))
    lse, ohp = torch.full((B, Hq, L), float(torch.tensor(L).log()), device="cuda"), torch.zeros((B, Hq, L, d), device="cuda")
    size = aq.workspace_bytes(aq.WS_BWD, B, Hq, Hkv, L, d)
    run = lambda n: aq.attnqat_bwd(q, k, v, do, lse, ohp, causal, workspace=torch.empty(n, dtype=torch.uint8, device="cuda"))  # noqa: E731
    want = run(size)
    for spare in (256, 64 << 20):
        assert all(torch.equal(a, b) for a, b in zip(run(size + spare), want))


# whole key tiles, a few more than compute units: two workgroups per unit instead of three (257 - 384 tiles; causal from 2048 positions on);
# and next to both limits
@pytest.mark.parametrize("mx", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,L,causal", [(4, 48, 12, 700, False), (2, 32, 16, 1025, False), (4, 48, 12, 1025, False), (2, 34, 17, 2050, True), (2, 36, 18, 2050, True)])
def test_whole_key_tiles_equal_separate_passes(B, Hq, Hkv, L, causal, mx):
    import paper_2603_00040_amd as aq
    x = random_inputs(B, Hq, Hkv, L, 64, seed=L + Hq)
    q, k, v, do = (to_dev(x[n]) for n in ("q", "k", "v", "do"))
    fwd, bwd = (aq.attnqat_fwd_mx, aq.attnqat_bwd_mx) if mx else (aq.attnqat_fwd, aq.attnqat_bwd)
    _, lse, ohp = fwd(q, k, v, causal)
    got = bwd(q, k, v, do, lse, ohp, causal)
    aq.debug_bwd_waves(4)
    try:
        want = bwd(q, k, v, do, lse, ohp, causal)
    finally:
        aq.debug_bwd_waves(0)
    assert all(torch.equal(a, b) for a, b in zip(got, want))
