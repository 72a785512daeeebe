"""Calls whose output lies over their Q, against the same call with an output of its own.  MX inference, block-sparse and paged: the attention kernel
quantizes Q itself, or takes operands that the preparing launch made: two ways to the same bits.  NVFP4 and MX training: the kernel reads Q, or a copy of it
(its phi(Q) is held against packed inputs, and against the oracle, elsewhere)."""
import pytest
import torch

from tests.gpu_util import random_inputs, to_dev

pytestmark = pytest.mark.gpu

# (B, Hq, Hkv, L): rows beyond the last whole group of 32 and of 128, one row, several heads of a kv head; the last one takes the
# workgroups of 128 rows
SHAPES = [(1, 2, 2, 1), (1, 4, 2, 33), (2, 4, 1, 130), (1, 2, 2, 257), (2, 40, 8, 1000)]


def _both(run, q):
    """run(q, o) with an output of its own, then with the output over Q."""
    own = run(q, torch.empty_like(q))
    over = q.clone()
    return own, run(over, over)


def _same(a, b):
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,L", SHAPES)
@pytest.mark.parametrize("kind", ["mx", "mx_fp8pv", "mx_sparse", "mx_train", "nvfp4", "nvfp4_train"])
def test_forward(kind, B, Hq, Hkv, L, d, causal):
    import paper_2603_00040_amd as aq
    x = random_inputs(B, Hq, Hkv, L, d, seed=L + d, k_chan=4)
    q, k, v = (to_dev(x[n]) for n in "qkv")

    def run(q, o):
        lse = torch.empty((B, Hq, L), dtype=torch.float32, device="cuda")
        if kind in ("mx_train", "nvfp4_train"):
            return (aq.attnqat_fwd_mx if kind == "mx_train" else aq.attnqat_fwd)(q, k, v, causal, out=(o, lse, torch.empty((B, Hq, L, d), dtype=torch.float32, device="cuda")))
        if kind == "mx_sparse":
            nb = (L + 127) // 128
            mask = torch.ones((B, Hq, nb, nb), dtype=torch.uint8, device="cuda")
            mask[..., ::2, 1::3] = 0
            return aq.attnqat_fwd_infer_mx_sparse(q, k, v, causal, mask, out=(o, lse))
        return {"nvfp4": aq.attnqat_fwd_infer, "mx": aq.attnqat_fwd_infer_mx, "mx_fp8pv": aq.attnqat_fwd_infer_mx_fp8pv}[kind](q, k, v, causal, out=(o, lse))
    _same(*_both(run, q))


# a step of decoding walked and in parts (one and more rows per head), a chunk of a prefill
@pytest.mark.parametrize("B,Hq,Hkv,Lq,n", [(1, 4, 1, 1, 3000), (40, 2, 2, 1, 260), (2, 8, 2, 5, 700), (2, 4, 2, 77, 300)])
@pytest.mark.parametrize("d", [64, 128])
def test_paged(B, Hq, Hkv, Lq, n, d):
    import paper_2603_00040_amd as aq
    x = random_inputs(B, Hq, Hkv, n, d, seed=n + d, k_chan=4)
    pages = (n + 127) // 128
    cache = torch.zeros(B * pages * aq.kv_cache_page_bytes(Hkv, d), dtype=torch.uint8, device="cuda")
    table = torch.arange(B * pages, dtype=torch.int32, device="cuda").flip(0).reshape(B, pages).contiguous()
    k, v = to_dev(x["k"]), to_dev(x["v"])
    for b in range(B):
        aq.attnqat_kv_cache_write_mx(k[b:b + 1], v[b:b + 1], cache, table[b])
    q = to_dev(x["q"])[:, :, n - Lq:].contiguous()
    lens = torch.full((B,), n, dtype=torch.int32, device="cuda")

    def run(q, o):
        lse = torch.empty((B, Hq, Lq), dtype=torch.float32, device="cuda")
        return aq.attnqat_fwd_infer_mx_paged(q, cache, B * pages, table, lens, Hkv, True, out=(o, lse))
    _same(*_both(run, q))


# NVFP4: a prompt's last positions over the pages of a cache, rows of one length and of several
@pytest.mark.parametrize("B,Hq,Hkv,Lq,n", [(2, 4, 2, 77, 300), (1, 40, 8, 1000, 1000)])
@pytest.mark.parametrize("d", [64, 128])
def test_paged_nvfp4(B, Hq, Hkv, Lq, n, d):
    import paper_2603_00040_amd as aq
    x = random_inputs(B, Hq, Hkv, n, d, seed=n + d, k_chan=4)
    pages = (n + 127) // 128
    cache = torch.zeros(B * pages * aq.kv_cache_page_bytes_nvfp4(Hkv, d), dtype=torch.uint8, device="cuda")
    table = torch.arange(B * pages, dtype=torch.int32, device="cuda").flip(0).reshape(B, pages).contiguous()
    k, v = to_dev(x["k"]), to_dev(x["v"])
    for b in range(B):
        aq.attnqat_kv_cache_write(k[b:b + 1], v[b:b + 1], cache, table[b])
    q = to_dev(x["q"])[:, :, n - Lq:].contiguous()
    lens = torch.tensor([n, n - 60][:B], dtype=torch.int32, device="cuda")

    def run(q, o):
        lse = torch.empty((B, Hq, Lq), dtype=torch.float32, device="cuda")
        return aq.attnqat_fwd_infer_paged(q, cache, B * pages, table, lens, Hkv, True, out=(o, lse))
    _same(*_both(run, q))
