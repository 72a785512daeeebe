"""Block scales of P^F in the backward where the largest P of a block is a tie of the E4M3 grid times 6, and next to one: RNE of the unrounded product of P
with the fp32 number 1/6, in every kernel that forms them, with and without the row factor of the two-level form."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SIXTH = np.float64(np.float32(1.0 / 6.0))
E2M1 = np.array([0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0])


def _rne_e4m3(x):
    """x >= 0 (fp64) to the E4M3 grid (subnormal spacing 2^-9 below 2^-6), ties to even; no saturation."""
    spacing = np.exp2(np.maximum(np.floor(np.log2(np.maximum(x, 2.0 ** -40))), -6.0) - 3.0)
    return np.rint(x / spacing) * spacing


def _row_factor(p):
    """Two-level form: the smallest power of two s1 with 2688 s1 >= P (every key of a row has the same P here)."""
    s1 = np.exp2(np.floor(np.log2(p / 2688.0)))
    return np.where(2688.0 * s1 >= p, s1, 2.0 * s1)


def _lse_near_ties(two_level):
    """Rows' lse (fp32) whose P = exp(-lse) lies at a tie or within 16 steps of lse from one."""
    if two_level:        # P / s1 / 6 lies in (224, 448]: spacing 16, then 32
        ties = [(2 * m + 1) * 8.0 for m in range(14, 16)] + [(2 * m + 1) * 16.0 for m in range(8, 14)]
        values = [6.0 * t * 2.0 ** e for t in ties for e in range(-20, -10) if 6.0 * t * 2.0 ** e <= 1.0]
    else:                # subnormal scales, the binades up to 1/6
        ties = [(2 * m + 1) * 2.0 ** -10 for m in range(8)] + [(1 + (2 * m + 1) / 16) * 2.0 ** e for e in range(-6, -2) for m in range(8)]
        values = [6.0 * t for t in ties if 6.0 * t <= 1.0]
    out = []
    for v in values:
        c = np.float32(-np.log(v))
        step = np.spacing(np.abs(c))
        out += [np.float32(c + i * step) for i in range(-16, 17)]
    return np.array(out, np.float32)


@pytest.mark.parametrize("two_level", [False, True])
@pytest.mark.parametrize("heads,d,waves", [(24, 128, 0), (40, 64, 0), (48, 128, 0), (96, 64, 0), (24, 128, 4), (24, 128, 8), (48, 64, 4)])
def test_scales_at_ties(heads, d, waves, two_level):
    import paper_2603_00040_amd as aq
    # K = 0: S = 0 and P = exp2(-lse log2 e) for every key.  Row i of a head has dO = e_i, so column i of dV is P^F of that row, exact in bf16.
    L = d
    rng = np.random.default_rng(d + heads)
    lse_h = rng.permutation(np.resize(_lse_near_ties(two_level), heads * L)).reshape(1, heads, L)
    lse = torch.from_numpy(lse_h.copy()).cuda()
    zero = torch.zeros((1, heads, L, d), dtype=torch.bfloat16, device="cuda")
    v, do = torch.ones_like(zero), torch.eye(L, d, dtype=torch.bfloat16, device="cuda").expand(1, heads, L, d).contiguous()
    ohp = torch.zeros((1, heads, L, d), dtype=torch.float32, device="cuda")
    aq.debug_bwd_waves(waves)
    try:
        got = (aq.attnqat_bwd_opt(zero, zero, v, do, lse, ohp, False, aq.OPT_TWO_LEVEL_P) if two_level else aq.attnqat_bwd(zero, zero, v, do, lse, ohp, False))[2]
    finally:
        aq.debug_bwd_waves(0)
    p32 = torch.exp2(-(lse * np.float32(1.4426950408889634)))
    got = got[0].double().cpu().numpy().transpose(0, 2, 1)                    # [head, row, key]
    p = p32[0].double().cpu().numpy()
    s1 = _row_factor(p) if two_level else np.ones_like(p)
    s = _rne_e4m3(p / s1 * SIXTH) * s1
    once = _rne_e4m3(np.float64(np.float32(p / s1 * SIXTH))) * s1                    # the product rounded to fp32 first
    # codes: P / s to the E2M1 grid; where that is itself within 2^-20 of a boundary, either neighbour (P times an approximate reciprocal is rounded)
    q = p / np.where(s > 0, s, 1.0)
    lo, hi = (E2M1[np.abs(E2M1[None, None] - (q * (1 + e))[..., None]).argmin(-1)] for e in (-2.0 ** -20, 2.0 ** -20))
    if not two_level:
        # a tile of 32 rows whose products, rounded to fp32, are all at most 2^-10 has no P^F at all
        tile = (np.float32(p * SIXTH) > np.float32(2.0 ** -10)).reshape(heads, L // 32, 32).any(-1).repeat(32, -1)
        s = np.where(tile, s, 0.0)
    ok = (got == (s * lo)[..., None]) | (got == (s * hi)[..., None])
    assert ok.all(), (int((~ok).any(-1).sum()), p[(~ok).any(-1)][:4], (got / s1[..., None])[(~ok).any(-1)][:4, 0])
    # rows whose scale depends on that the product is not rounded first are among them
    assert (once != s)[s > 0].sum() >= 4
