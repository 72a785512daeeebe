"""The workgroup shapes of the forward (eight waves = 256 query rows, four waves = 128, four waves that share 32 rows) and the order in
which the four-wave workgroups take their tiles: the dispatch picks by the size of the whole problem, rows do not depend on each other,
so heads and sequences computed together and alone have to agree bit for bit (the parity of either with the oracle is tested elsewhere)."""
import pytest
import torch

from tests.gpu_util import random_inputs, to_dev

pytestmark = pytest.mark.gpu


# One head alone always shares its key tiles (at most three groups of 32 rows per compute unit).  Together: without a mask 257 - 512 tiles of
# 128 rows run on eight waves, one row per head and tiles that would leave a small second round on four; under a causal mask eight waves
# are taken from 4096 positions on when the pairs of tiles fill whole rounds of the compute units (8 heads x 32 pairs), four otherwise.
@pytest.mark.parametrize("H,L,d,causal", [(130, 256, 64, False), (160, 129, 128, False), (150, 255, 128, False), (88, 300, 64, False), (8, 16384, 128, True),
                                          (800, 1, 128, False), (200, 257, 128, False), (72, 511, 128, True), (50, 1025, 64, True)])
def test_heads_together_equal_heads_alone(H, L, d, causal):
    import paper_2603_00040_amd as aq
    x = random_inputs(1, H, H, L, d, seed=H + L, k_chan=2)
    q, k, v = (to_dev(x[n]) for n in ("q", "k", "v"))
    o, lse, ohp = aq.attnqat_fwd(q, k, v, causal)
    om, lm, _ = aq.attnqat_fwd_mx(q, k, v, causal)
    for h in (0, H // 2, H - 1):
        part = tuple(t[:, h:h + 1].contiguous() for t in (q, k, v))
        o1, l1, p1 = aq.attnqat_fwd(*part, causal)
        assert torch.equal(o[:, h:h + 1], o1) and torch.equal(lse[:, h:h + 1], l1) and torch.equal(ohp[:, h:h + 1], p1), h
        o1, l1, _ = aq.attnqat_fwd_mx(*part, causal)
        assert torch.equal(om[:, h:h + 1], o1) and torch.equal(lm[:, h:h + 1], l1), h


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,Lq,d", [(20, 6, 3, 200, 64), (22, 8, 8, 130, 128), (100, 4, 2, 40, 64), (3, 32, 8, 300, 128)])
def test_sequences_together_equal_sequences_alone(B, Hq, Hkv, Lq, d, causal):
    """Prefill chunks of sequences of very different lengths over the paged NVFP4 cache (sorted by length on the device up to 64
    sequences, in their own order beyond).  Together on 128 rows per workgroup, alone with shared key tiles."""
    import paper_2603_00040_amd as aq
    g = torch.Generator().manual_seed(B)
    lens = torch.randint(Lq, 1500 if B < 20 else 500, (B,), generator=g)
    lens[B // 2] = lens[0]                                         # a tie
    pages = [(int(n) + 127) // 128 for n in lens]
    num_pages, max_pages = sum(pages), max(pages)
    cache = torch.zeros(num_pages * aq.kv_cache_page_bytes_nvfp4(Hkv, d), dtype=torch.uint8, device="cuda")
    perm = torch.randperm(num_pages, generator=g).to(torch.int32)
    table = torch.zeros((B, max_pages), dtype=torch.int32)
    at = 0
    for b in range(B):
        table[b, :pages[b]] = perm[at:at + pages[b]]
        at += pages[b]
        x = random_inputs(1, Hkv, Hkv, int(lens[b]), d, seed=31 + b)
        aq.attnqat_kv_cache_write(to_dev(x["k"]), to_dev(x["v"]), cache, table[b, :pages[b]].cuda(), 0, num_pages)
    table, lens = table.cuda(), lens.to(torch.int32).cuda()
    q = to_dev(random_inputs(B, Hq, Hkv, Lq, d, seed=7)["q"])
    o, lse = aq.attnqat_fwd_infer_paged(q, cache, num_pages, table, lens, Hkv, causal)
    for b in sorted({0, 1, B // 2, B - 1}):
        o1, l1 = aq.attnqat_fwd_infer_paged(q[b:b + 1].contiguous(), cache, num_pages, table[b:b + 1].contiguous(), lens[b:b + 1].contiguous(), Hkv, causal)
        assert torch.equal(o[b:b + 1], o1) and torch.equal(lse[b:b + 1], l1), b


def test_long_prefill_chunk_equals_its_parts():
    """A chunk of 4096 positions under the causal mask runs on eight waves (2 sequences x 16 heads x 8 pairs of tiles are a whole round of
    the compute units), its parts of 1000 - 2048 positions on four: rows do not depend on each other.  Lengths with and without keys in
    front of the chunk."""
    import paper_2603_00040_amd as aq
    Hq, Hkv, d, Lq, lens = 16, 4, 128, 4096, (5000, 4096)
    pages = [(n + 127) // 128 for n in lens]
    num_pages, max_pages = sum(pages), max(pages)
    cache = torch.zeros(num_pages * aq.kv_cache_page_bytes_nvfp4(Hkv, d), dtype=torch.uint8, device="cuda")
    table, at = torch.zeros((len(lens), max_pages), dtype=torch.int32, device="cuda"), 0
    for b, n in enumerate(lens):
        table[b, :pages[b]] = torch.arange(at, at + pages[b], dtype=torch.int32, device="cuda").flip(0)
        at += pages[b]
        x = random_inputs(1, Hkv, Hkv, n, d, seed=5 + b)
        aq.attnqat_kv_cache_write(to_dev(x["k"]), to_dev(x["v"]), cache, table[b, :pages[b]].contiguous(), 0, num_pages)
    q = to_dev(random_inputs(len(lens), Hq, Hkv, Lq, d, seed=7)["q"])
    kl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    o, lse = aq.attnqat_fwd_infer_paged(q, cache, num_pages, table, kl, Hkv, True)
    for lo, hi in ((0, 1000), (1000, 2048), (2048, 4096)):
        part, pl = aq.attnqat_fwd_infer_paged(q[:, :, lo:hi].contiguous(), cache, num_pages, table, kl - (Lq - hi), Hkv, True)
        assert torch.equal(o[:, :, lo:hi], part) and torch.equal(lse[:, :, lo:hi], pl), (lo, hi)
