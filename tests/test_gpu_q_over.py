"""Forwards whose results lie over their Q, all of it or a part: the bits of a call with results of their own, in as many launches, eagerly and replayed from a
graph."""
import ctypes

import pytest
import torch

from tests.gpu_util import random_inputs, to_dev

pytestmark = pytest.mark.gpu

KINDS = ["nvfp4", "nvfp4_train", "two_level", "smooth_k", "bf16pv", "mx", "mx_fp8pv", "mx_train"]
# (a few rows: the waves share a workgroup's 32; workgroups of 128 rows; of 256.  Lengths that are no multiple of 64)
SHAPES = [(1, 4, 2, 77, 128), (2, 3, 1, 130, 64), (2, 40, 8, 1000, 128)]


def _calls(aq, kind, k, v, causal, ws):
    """run(q, o, lse, o_hp) of one kind."""
    opt = {"two_level": aq.OPT_TWO_LEVEL_P, "smooth_k": aq.OPT_SMOOTH_K}

    def run(q, o, lse, ohp):
        if kind in opt:
            aq.attnqat_fwd_opt(q, k, v, causal, opt[kind], train=True, workspace=ws, out=(o, lse, ohp))
        elif kind.endswith("_train"):
            (aq.attnqat_fwd_mx if kind == "mx_train" else aq.attnqat_fwd)(q, k, v, causal, workspace=ws, out=(o, lse, ohp))
        else:
            f = {"nvfp4": aq.attnqat_fwd_infer, "bf16pv": aq.attnqat_fwd_infer_bf16pv, "mx": aq.attnqat_fwd_infer_mx, "mx_fp8pv": aq.attnqat_fwd_infer_mx_fp8pv}[kind]
            f(q, k, v, causal, workspace=ws, out=(o, lse))
    return run


def _layouts(B, Hq, L, d, train):
    """(name, q, o, lse, o_hp) as views of one buffer each: nothing over Q, O over Q, O over a part of it, L over Q, O' over Q."""
    rows = B * Hq * L
    nq, nl = rows * d * 2, rows * 4
    pad = lambda n: (n + 255) // 256 * 256  # noqa: E731
    for name, at in (("apart", {}), ("o", {"o": 0}), ("o_part", {"o": 64 * d * 2}), ("lse", {"lse": 0}), ("lse_end", {"lse": nq - nl}), ("o_hp", {"o_hp": 0}), ("o_hp_end", {"o_hp": -nq})):
        if "o_hp" in at and not train:
            continue
        base = pad(2 * nq)
        off, end = {"q": base}, base + pad(2 * nq)
        for t, n in (("o", nq), ("lse", nl), ("o_hp", 2 * nq)):
            if t in at:
                off[t] = base + at[t]
            else:
                off[t], end = end, end + pad(n)
        end += pad(2 * nq)
        buf = torch.empty(end, dtype=torch.uint8, device="cuda")
        view = lambda t, n, dt, shape: buf[off[t]:off[t] + n].view(dt).view(shape)  # noqa: E731
        yield (name, view("q", nq, torch.bfloat16, (B, Hq, L, d)), view("o", nq, torch.bfloat16, (B, Hq, L, d)), view("lse", nl, torch.float32, (B, Hq, L)),
               view("o_hp", 2 * nq, torch.float32, (B, Hq, L, d)))


def _nodes(graph):
    n = ctypes.c_size_t(0)
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


def _check(run, src, layouts, outs):
    """outs(o, lse, o_hp): the results to compare."""
    want = launches = None
    side = torch.cuda.Stream()
    for name, q, *res in layouts:
        q.copy_(src)
        with torch.cuda.stream(side):
            side.wait_stream(torch.cuda.current_stream())
            run(q, *res)
        side.synchronize()
        got = [t.clone() for t in outs(*res)]
        if want is None:
            want = got
        assert all(torch.equal(a, b) for a, b in zip(got, want)), name
        g = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(g, stream=side):
            run(q, *res)
        n = _nodes(g)
        launches = launches or n
        assert n == launches, (name, n, launches)
        g.instantiate()
        for _ in range(3):
            q.copy_(src)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(outs(*res), want)), name


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,L,d", SHAPES)
@pytest.mark.parametrize("kind", KINDS)
def test_forward(kind, B, Hq, Hkv, L, d, causal):
    import paper_2603_00040_amd as aq
    x = random_inputs(B, Hq, Hkv, L, d, seed=L + d, k_chan=4)
    src, k, v = (to_dev(x[n]) for n in "qkv")
    train = kind in ("nvfp4_train", "mx_train", "two_level", "smooth_k")
    ws = torch.empty(max(aq.workspace_bytes(w, B, Hq, Hkv, L, d) for w in (aq.WS_FWD, aq.WS_FWD_MX, aq.WS_FWD_INFER_MX, aq.WS_FWD_INFER_MX_FP8PV)), dtype=torch.uint8, device="cuda")
    _check(_calls(aq, kind, k, v, causal, ws), src, _layouts(B, Hq, L, d, train), lambda o, lse, ohp: (o, lse, ohp) if train else (o, lse))


@pytest.mark.parametrize("B,Hq,Hkv,Lq,n,d", [(2, 4, 2, 77, 300, 128), (1, 40, 8, 1000, 1000, 64)])
def test_paged_nvfp4(B, Hq, Hkv, Lq, n, d):
    import paper_2603_00040_amd as aq
    x = random_inputs(B, Hq, Hkv, n, d, seed=n + d, k_chan=4)
    pages = (n + 127) // 128
    cache = torch.zeros(B * pages * aq.kv_cache_page_bytes_nvfp4(Hkv, d), dtype=torch.uint8, device="cuda")
    table = torch.arange(B * pages, dtype=torch.int32, device="cuda").flip(0).reshape(B, pages).contiguous()
    k, v = to_dev(x["k"]), to_dev(x["v"])
    for b in range(B):
        aq.attnqat_kv_cache_write(k[b:b + 1], v[b:b + 1], cache, table[b])
    src = to_dev(x["q"])[:, :, n - Lq:].contiguous()
    lens = torch.tensor([n, n - 60][:B], dtype=torch.int32, device="cuda")
    ws = torch.empty(aq.lib().attnqat_paged_workspace_bytes(B, Hq, Hkv, Lq, pages, d), dtype=torch.uint8, device="cuda")

    def run(q, o, lse, _):
        aq.attnqat_fwd_infer_paged(q, cache, B * pages, table, lens, Hkv, True, workspace=ws, out=(o, lse))
    _check(run, src, _layouts(B, Hq, Lq, d, False), lambda o, lse, _: (o, lse))
