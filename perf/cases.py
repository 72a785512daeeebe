"""The work that is timed to see whether the framework got faster: one pass of each case goes through the public entry
points of ``paper_2603_00040_amd`` as a training step, an inference call or a serving step does.

Kinds of case
  train    Alg. 2 and Alg. 3: forward, then backward (``attnqat_fwd``/``attnqat_bwd`` or their MX forms)
  infer    Alg. 1 on bf16 tensors: NVFP4, NVFP4 with BF16 P V, MX, MX with FP8 P V
  sparse   Alg. 1 (MX) under a mask of 128 x 128 blocks
  prefill  a chunk of new positions of every sequence: appended to the paged KV cache, then attended to
  decode   one or a few new positions of every sequence against the paged KV cache; ``append`` writes them first

As ``bench.py`` does, the program keeps its workspace and its output tensors from step to step.
"""
import math

import torch

import paper_2603_00040_amd as aq

DEV = "cuda"
PAGE = 128                        # positions per page of the KV cache


def listed():
    attn = lambda name, kind, fmt, B, Hq, Hkv, L, d, causal, dist: {  # noqa: E731
        "name": name, "kind": kind, "fmt": fmt, "B": B, "Hq": Hq, "Hkv": Hkv, "L": L, "d": d, "causal": causal, "dist": dist}
    serve = lambda name, kind, fmt, B, Hq, Hkv, d, Lq, kv_min, kv_max, append: {  # noqa: E731
        "name": name, "kind": kind, "fmt": fmt, "B": B, "Hq": Hq, "Hkv": Hkv, "d": d, "Lq": Lq, "kv_min": kv_min, "kv_max": kv_max, "append": append}
    return [
        # the smallest benchmark configuration (tiny_ref): a step of a toy or unit-test size model, launches and latency
        attn("train_tiny", "train", "nvfp4", 1, 2, 2, 256, 64, False, "normal"),
        # one latent frame of the 480p video model (30 x 52 tokens, 12 heads): fine-tuning on stills, sequence ragged
        attn("train_frame", "train", "nvfp4", 1, 12, 12, 1560, 128, False, "t3"),
        # the grouped-query language model at 4k (llm4k_gqa): an ordinary training step of one layer
        attn("train_llm4k", "train", "nvfp4", 4, 32, 8, 4096, 128, True, "k_outliers"),
        # the same in the MX format on an odd length: a packed batch is seldom a multiple of a tile
        attn("train_llm_mx", "train", "mx", 2, 16, 4, 3001, 128, True, "k_outliers"),
        # the 720p video model (dit720p_train, the default of bench.py): the largest step
        attn("train_dit720p", "train", "nvfp4", 1, 40, 40, 75600, 128, False, "t3"),
        # a user's prompt before its first token: one short sequence, grouped-query heads
        attn("infer_prompt", "infer", "nvfp4", 1, 32, 8, 777, 128, True, "k_outliers"),
        # the 480p video model sampling with guidance (dit480p_infer), in the paper's format and on the FP4 instruction
        attn("infer_dit480p", "infer", "nvfp4", 2, 12, 12, 32760, 128, False, "t3"),
        attn("infer_dit480p_mx", "infer", "mx", 2, 12, 12, 32760, 128, False, "t3"),
        # block-sparse attention over a long prompt, a quarter of the lower triangle kept
        dict(attn("sparse_llm8k", "sparse", "mx", 1, 32, 8, 8192, 128, True, "k_outliers"), keep=0.25),
        # serving: a decode step of 32 sequences of 4k - 16k keys (bench.py --paged-lq 1)
        serve("decode_batch32", "decode", "nvfp4", 32, 32, 8, 128, 1, 4096, 16384, False),
        # ... of one user with a conversation of about 3000 tokens: append the position, attend
        serve("decode_single", "decode", "nvfp4", 1, 32, 8, 128, 1, 3000, 3000, True),
        # ... and a 512-position chunk of the prompts of eight sequences of 2k - 16k keys
        serve("prefill_chunk", "prefill", "nvfp4", 8, 32, 8, 128, 512, 2048, 16384, True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same kinds: sizes spread over the logarithm of their range, most of them no multiple of anything;
    no attention call of more than a fifth of train_dit720p's pairs, no cache of more than decode_batch32's."""
    kind = rng.choice(["train", "train", "infer", "infer", "sparse", "decode", "decode", "prefill"])
    d = rng.choice([64, 128, 128])
    G = rng.choice([1, 1, 2, 4, 8])
    Hkv = rng.choice([1, 2, 3, 4, 8, 12]) if G > 1 else rng.choice([1, 2, 4, 12, 24, 40])
    if kind in ("train", "infer", "sparse"):
        B = rng.choice([1, 1, 2, 4])
        cap = math.sqrt(0.2 * 40 * 75600.0 ** 2 / (B * G * Hkv))
        L = _log_int(rng, 160, min(cap, 8192 if kind == "sparse" else 75600))
        c = {"kind": kind, "B": B, "Hq": G * Hkv, "Hkv": Hkv, "L": L, "d": d, "causal": rng.random() < 0.5 or kind == "sparse",
             "dist": rng.choice(["normal", "t3", "k_outliers"])}
        c["fmt"] = {"train": rng.choice(["nvfp4", "nvfp4", "mx"]), "infer": rng.choice(["nvfp4", "nvfp4", "bf16pv", "mx", "mx_fp8pv"]), "sparse": "mx"}[kind]
        if kind == "sparse":
            c["keep"] = round(rng.uniform(0.1, 0.6), 2)
        return c
    c = {"kind": kind, "fmt": rng.choice(["nvfp4", "nvfp4", "mx"]), "Hq": G * Hkv, "Hkv": Hkv, "d": d}
    if kind == "decode":
        c["B"] = _log_int(rng, 1, 64)
        c["Lq"] = rng.choice([1, 1, 1, 2, max(1, 16 // G)])
        c["append"] = c["fmt"] == "nvfp4" and c["B"] <= 4        # (the MX cache grows by whole pages)
    else:
        c["B"] = _log_int(rng, 1, 12)
        c["Lq"] = _log_int(rng, 48, 2048)
        c["append"] = c["fmt"] == "nvfp4"
    top = max(1024, min(16384, int(32 * 10240 * 8 / (c["B"] * Hkv))))
    a, b = sorted(_log_int(rng, 256, top) for _ in range(2))
    c["kv_min"], c["kv_max"] = max(a, c["Lq"]), max(b, c["Lq"])
    return c


# ---------------------------------------------------------------------------------------------------------- inputs
def _normal(shape, g):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)


def _tensor(shape, dist, what, g, outlier_tokens=None):
    """bf16 values as the benchmark's workloads draw them.  normal: N(0,1).  t3: 0.5 Student-t with 3 degrees of freedom, 1 % of
    the tokens x10 in Q, K and V.  k_outliers: N(0,1), four channels of every K head x20."""
    out = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    B, H, L, d = shape
    for b in range(B):
        for h in range(H):
            x = _normal((L, d), g)
            if dist == "t3":
                x = 0.5 * x / (_normal((3, L, d), g).square().sum(0) / 3.0).sqrt()
                if outlier_tokens is not None and what != "do":
                    x = torch.where(outlier_tokens[:, None], 10.0 * x, x)
            elif dist == "k_outliers" and what == "k":
                x[:, torch.randperm(d, generator=g, device=DEV)[:4]] *= 20.0
            out[b, h] = x.to(torch.bfloat16)
    return out


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _prepare_attention(c, g):
    B, Hq, Hkv, L, d = c["B"], c["Hq"], c["Hkv"], c["L"], c["d"]
    tok = torch.rand(L, generator=g, device=DEV) < 0.01 if c["dist"] == "t3" else None
    s = {n: _tensor((B, Hkv if n in ("k", "v") else Hq, L, d), c["dist"], n, g, tok) for n in ("q", "k", "v")}
    o = torch.empty_like(s["q"])
    lse = torch.empty((B, Hq, L), dtype=torch.float32, device=DEV)
    which = {"nvfp4": aq.WS_FWD_INFER, "bf16pv": aq.WS_FWD_INFER, "mx": aq.WS_FWD_INFER_MX, "mx_fp8pv": aq.WS_FWD_INFER_MX_FP8PV}[c["fmt"]]
    size = lambda w: aq.workspace_bytes(w, B, Hq, Hkv, L, d)  # noqa: E731
    if c["kind"] == "train":
        s["do"] = _tensor((B, Hq, L, d), c["dist"], "do", g)
        s["out_fwd"] = (o, lse, torch.empty((B, Hq, L, d), dtype=torch.float32, device=DEV))
        s["out_bwd"] = tuple(torch.empty_like(s[n]) for n in ("q", "k", "v"))
        mx = c["fmt"] == "mx"
        need = max(size(aq.WS_FWD_MX if mx else aq.WS_FWD), size(aq.WS_BWD_MX if mx else aq.WS_BWD))
    else:
        s["out"] = (o, lse)
        need = size(aq.WS_FWD_INFER_MX_SPARSE if c["kind"] == "sparse" else which)
    if c["kind"] == "sparse":
        nb = (L + 127) // 128
        m = torch.rand((B, Hq, nb, nb), generator=g, device=DEV) < c["keep"]
        m |= torch.eye(nb, dtype=torch.bool, device=DEV)                     # every block of queries keeps its own keys
        if c["causal"]:
            m &= torch.ones((nb, nb), dtype=torch.bool, device=DEV).tril()
        s["mask"] = m.to(torch.uint8)
    s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    return s


def _kv_lens(c, seed):
    """The sequences' lengths: from the seed, between kv_min and kv_max (on the host: the page lists follow from them)."""
    g = torch.Generator()
    g.manual_seed(int(seed))
    return torch.randint(c["kv_min"], c["kv_max"] + 1, (c["B"],), generator=g).tolist()


def _prepare_serving(c, g, seed):
    B, Hq, Hkv, d, Lq = c["B"], c["Hq"], c["Hkv"], c["d"], c["Lq"]
    nv = c["fmt"] == "nvfp4"
    lens = _kv_lens(c, seed)
    pages_of = [(n + PAGE - 1) // PAGE for n in lens]
    max_pages = (c["kv_max"] + PAGE - 1) // PAGE
    num_pages = B * max_pages                                # the pool: enough for B sequences of the longest length
    page_bytes = (aq.kv_cache_page_bytes_nvfp4 if nv else aq.kv_cache_page_bytes)(Hkv, d)
    cache = torch.zeros(num_pages * page_bytes, dtype=torch.uint8, device=DEV)
    perm = torch.randperm(num_pages, generator=g, device=DEV).to(torch.int32)      # pages of a sequence lie anywhere in the cache
    table = torch.zeros((B, max_pages), dtype=torch.int32, device=DEV)
    new, at = [], 0
    for b, n in enumerate(lens):
        ids = perm[at:at + pages_of[b]].contiguous()
        at += pages_of[b]
        table[b, :pages_of[b]] = ids
        k, v = (_tensor((1, Hkv, n, d), "k_outliers", t, g) for t in ("k", "v"))
        if nv:
            aq.attnqat_kv_cache_write(k, v, cache, ids, 0, num_pages)
        else:
            aq.attnqat_kv_cache_write_mx(k, v, cache, ids, num_pages)
        if c["append"]:      # the step's new positions
            new.append(tuple(_tensor((1, Hkv, Lq, d), "k_outliers", t, g) for t in ("k", "v")) + (ids, n - Lq))
    q = _tensor((B, Hq, Lq, d), "normal", "q", g)
    if nv:
        need = aq.lib().attnqat_paged_workspace_bytes(B, Hq, Hkv, Lq, max_pages, d)
    else:
        need = aq.workspace_bytes(aq.WS_FWD_INFER_MX_PAGED, B, Hq, Hkv, Lq, d)
    return {"q": q, "cache": cache, "num_pages": num_pages, "table": table, "lens": torch.tensor(lens, dtype=torch.int32, device=DEV), "new": new,
            "out": (torch.empty_like(q), torch.empty((B, Hq, Lq), dtype=torch.float32, device=DEV)), "ws": torch.empty(need, dtype=torch.uint8, device=DEV)}


def prepare(case, seed):
    g = _generator(seed)
    s = _prepare_attention(case, g) if "L" in case else _prepare_serving(case, g, seed)
    s["case"] = case
    return s


# ------------------------------------------------------------------------------------------------------------ passes
def run(s):
    c = s["case"]
    kind, fmt = c["kind"], c["fmt"]
    if kind == "train":
        fwd, bwd = (aq.attnqat_fwd_mx, aq.attnqat_bwd_mx) if fmt == "mx" else (aq.attnqat_fwd, aq.attnqat_bwd)
        o, lse, o_hp = fwd(s["q"], s["k"], s["v"], c["causal"], workspace=s["ws"], out=s["out_fwd"])
        dq, dk, dv = bwd(s["q"], s["k"], s["v"], s["do"], lse, o_hp, c["causal"], workspace=s["ws"], out=s["out_bwd"])
        return {"o": o, "lse": lse, "o_hp": o_hp, "dq": dq, "dk": dk, "dv": dv}
    if kind == "infer":
        f = {"nvfp4": aq.attnqat_fwd_infer, "bf16pv": aq.attnqat_fwd_infer_bf16pv, "mx": aq.attnqat_fwd_infer_mx, "mx_fp8pv": aq.attnqat_fwd_infer_mx_fp8pv}[fmt]
        return f(s["q"], s["k"], s["v"], c["causal"], workspace=s["ws"], out=s["out"])
    if kind == "sparse":
        return aq.attnqat_fwd_infer_mx_sparse(s["q"], s["k"], s["v"], c["causal"], s["mask"], workspace=s["ws"], out=s["out"])
    for k, v, ids, pos0 in s["new"]:
        aq.attnqat_kv_cache_write(k, v, s["cache"], ids, pos0, s["num_pages"])
    f = aq.attnqat_fwd_infer_paged if fmt == "nvfp4" else aq.attnqat_fwd_infer_mx_paged
    o, lse = f(s["q"], s["cache"], s["num_pages"], s["table"], s["lens"], c["Hkv"], True, workspace=s["ws"], out=s["out"])
    return (o, lse, s["cache"]) if s["new"] else (o, lse)


def work(case):
    """Model operations (4 d per query-key pair forward, 10 d backward, masked pairs not counted) and the bytes of the call's
    inputs and outputs, each once."""
    c = case
    d = c["d"]
    if "L" in c:
        B, Hq, Hkv, L = c["B"], c["Hq"], c["Hkv"], c["L"]
        nq, nk, rows = B * Hq * L * d, B * Hkv * L * d, B * Hq * L
        pairs = B * Hq * (L * (L + 1) / 2 if c["causal"] else float(L) * L)
        if c["kind"] == "sparse":
            nb = (L + 127) // 128
            pairs *= min(1.0, c["keep"] + 2.0 / (nb + 1))        # the kept share and the diagonal
            return {"bytes": 4 * nq + 4 * nk + 4 * rows + B * Hq * nb * nb, "flops": 4 * d * pairs}
        if c["kind"] == "infer":
            return {"bytes": 4 * nq + 4 * nk + 4 * rows, "flops": 4 * d * pairs}
        # q, k, v, do in; o, lse, o_hp, dq, dk, dv out
        return {"bytes": (2 + 2 + 2 + 4 + 2) * nq + (4 + 4) * nk + 4 * rows, "flops": 14 * d * pairs}
    B, Hq, Hkv, Lq = c["B"], c["Hq"], c["Hkv"], c["Lq"]
    keys = B * (c["kv_min"] + c["kv_max"]) / 2.0
    per_key = Hkv * 2 * d * (4.5 if c["fmt"] == "nvfp4" else 4.25) / 8
    rows = B * Hq * Lq
    new = B * Lq * (4 * Hkv * d + per_key) if c["append"] else 0.0
    return {"bytes": keys * per_key + 4 * rows * d + 4 * rows + new, "flops": 4 * d * Hq * Lq * (keys - B * (Lq - 1) / 2.0)}


def tolerance(case):
    """Rounding an output to bf16 costs 1.65e-3 (relative 2-norm) by itself; against the fp64 oracle every bf16 output of these paths
    measures 1.4e-3 to 1.8e-3.  Four times that.  Cache bytes are whole numbers and stay the same."""
    return {"rel": 7e-3}
