"""The forward for few query rows (four waves share 32 rows and four key tiles): chosen by the number of 32-row groups, so heads computed
alone take it and the same heads among many others do not.  Rows do not depend on each other and both forms add up in the same
order, so the two have to agree bit for bit (their parity with the oracle is tested elsewhere).  Lengths around its edges: 32 rows,
64 keys, four tiles."""
import pytest
import torch

from tests.gpu_util import random_inputs, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 31, 33, 64, 65, 192, 255, 257, 330, 1025])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_few_rows_equal_many(L, d, causal):
    import paper_2603_00040_amd as aq
    H = 6 * 256 // ((L + 31) // 32) + 1                            # more groups than any rule takes
    x = random_inputs(1, 8, 8, L, d, seed=L, k_chan=2)
    few = [to_dev(x[n]) for n in ("q", "k", "v")]
    many = [t.repeat(1, (H + 7) // 8, 1, 1) for t in few]
    for f in (aq.attnqat_fwd, aq.attnqat_fwd_mx, aq.attnqat_fwd_infer, aq.attnqat_fwd_infer_bf16pv):
        for a, b in zip(f(*few, causal), f(*many, causal)):
            assert torch.isfinite(a.float()).all() and torch.equal(a, b[:, :8]) and torch.equal(a, b[:, -8:]), f.__name__


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Lq,d", [(33, 64), (70, 128)])
def test_short_chunks_of_long_sequences(Lq, d, causal):
    """A chunk of a paged prefill alone and among copies of itself."""
    import paper_2603_00040_amd as aq
    Hq, Hkv, n, B = 4, 4, 900, 70
    pages = (n + 127) // 128
    x = random_inputs(1, Hkv, Hkv, n, d, seed=3)
    cache = torch.zeros(pages * aq.kv_cache_page_bytes_nvfp4(Hkv, d), dtype=torch.uint8, device="cuda")
    table = torch.arange(pages, dtype=torch.int32, device="cuda").flip(0)[None].contiguous()
    aq.attnqat_kv_cache_write(to_dev(x["k"]), to_dev(x["v"]), cache, table[0].contiguous(), 0, pages)
    q = to_dev(random_inputs(1, Hq, Hkv, Lq, d, seed=4)["q"])
    for kv in (n, 129, 100):
        lens = torch.tensor([kv], dtype=torch.int32, device="cuda")
        o, lse = aq.attnqat_fwd_infer_paged(q, cache, pages, table, lens, Hkv, causal)
        ob, lb = aq.attnqat_fwd_infer_paged(q.repeat(B * 3, 1, 1, 1), cache, pages, table.repeat(B * 3, 1), lens.repeat(B * 3), Hkv, causal)
        assert all(torch.equal(o[0], ob[i]) and torch.equal(lse[0], lb[i]) for i in (0, B, 3 * B - 1)), kv


@pytest.mark.parametrize("L", [1, 33, 64, 65, 255, 257, 330, 1025])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_few_rows_equal_many_mx(L, d, causal):
    import paper_2603_00040_amd as aq
    H, nb = 6 * 256 // ((L + 31) // 32) + 1, (L + 127) // 128      # more groups than any rule takes
    x = random_inputs(1, 8, 8, L, d, seed=L, k_chan=2)
    few = [to_dev(x[n]) for n in ("q", "k", "v")]
    many = [t.repeat(1, (H + 7) // 8, 1, 1) for t in few]
    mask = (torch.rand((1, 8, nb, nb), generator=torch.Generator().manual_seed(L)) < 0.5).to(torch.uint8).cuda()      # (rows without keys, blocks above the diagonal)
    for f in (aq.attnqat_fwd_infer_mx, aq.attnqat_fwd_infer_mx_fp8pv,
              lambda *a: aq.attnqat_fwd_infer_mx_sparse(*a, mask.repeat(1, a[0].shape[1] // 8, 1, 1))):
        for a, b in zip(f(*few, causal), f(*many, causal)):
            assert not torch.isnan(a.float()).any() and torch.equal(a, b[:, :8]) and torch.equal(a, b[:, -8:])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Hq,Hkv,Lq,d", [(4, 4, 33, 64), (8, 2, 30, 128), (4, 2, 70, 128)])
def test_short_chunks_of_long_sequences_mx(Hq, Hkv, Lq, d, causal):
    """A chunk of a paged prefill alone and among copies of itself; grouped heads that share a tile (4 heads of 30 positions)."""
    import paper_2603_00040_amd as aq
    n, B = 900, 210
    pages = (n + 127) // 128
    x = random_inputs(1, Hkv, Hkv, n, d, seed=3)
    cache = torch.zeros(pages * aq.kv_cache_page_bytes(Hkv, d), dtype=torch.uint8, device="cuda")
    table = torch.arange(pages, dtype=torch.int32, device="cuda").flip(0)[None].contiguous()
    aq.attnqat_kv_cache_write_mx(to_dev(x["k"]), to_dev(x["v"]), cache, table[0].contiguous(), pages)
    q = to_dev(random_inputs(1, Hq, Hkv, Lq, d, seed=4)["q"])
    for kv in (n, 129, 100):
        lens = torch.tensor([kv], dtype=torch.int32, device="cuda")
        o, lse = aq.attnqat_fwd_infer_mx_paged(q, cache, pages, table, lens, Hkv, causal)
        ob, lb = aq.attnqat_fwd_infer_mx_paged(q.repeat(B, 1, 1, 1), cache, pages, table.repeat(B, 1), lens.repeat(B), Hkv, causal)
        assert all(torch.equal(o[0], ob[i]) and torch.equal(lse[0], lb[i]) for i in (0, B // 2, B - 1)), kv
