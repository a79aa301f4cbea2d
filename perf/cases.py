"""Performance cases: what a program that decodes with this library has it do, over the sizes it is used at.

A case is a dict of plain values.  `kind` names the path:
  decode    one token's fused step over `layers` layer caches (append, score, select, attend), one call
  mixed     the same with whole-cache attention on the first `dense_first` layers
  quantize  the 1-bit copy of a key cache after prefill
  calls     one layer's step as separate calls: append, score, top-k, attention over the selection
  pages     one layer's step with the page-level selector: append, page scores, top-k over pages, expansion, attention
Contexts are `ctx` tokens for every sequence, or spread over [ctx_lo, ctx] where ctx_lo is smaller; the budget is
`budget` tokens, or `budget_pct` per cent of each context where `budget` is 0.
"""
import math

import numpy as np
import torch

from paper_2508_08256_amd import binding as B

D = 128
_BASE = dict(kind="decode", batch=1, n_q_heads=8, n_kv_heads=8, ctx_lo=4096, ctx=4096, dtype="f16", group=32, layers=1,
             budget=0, budget_pct=11.0, block_tokens=0, index_list=False, dense_first=0, page_tokens=16, page_mode=0)


def _case(name, **kw):
    c = dict(_BASE, name=name, **kw)
    c["ctx_lo"] = kw.get("ctx_lo", c["ctx"])
    return c


def listed():
    return [
        # the smallest call: one layer of a small model at a short context, where launches and latency are everything
        _case("decode-4k", ctx=4096, budget=512),
        # one 32-head multi-head layer at 32k tokens, 11 % budget: the headline workload
        _case("decode-32k", n_q_heads=32, n_kv_heads=32, ctx=32768, budget=3604),
        # one grouped-query layer, four sequences at 128k tokens: scoring is half of the step
        _case("decode-128k-gqa", batch=4, n_q_heads=32, ctx=131072, budget=4096, dtype="bf16"),
        # the top of the budget sweep at 64k tokens: the gather dominates
        _case("decode-64k-wide", n_q_heads=32, n_kv_heads=32, ctx=65536, budget=16384),
        # a serving batch of 16 ragged long sequences, several layers per call
        _case("decode-ragged", batch=16, n_q_heads=32, ctx_lo=8192, ctx=65536, dtype="bf16", layers=4),
        # a serving batch of 8 ragged short sequences on paged K / V rows, a whole 16-layer stack per call
        _case("decode-chat-paged", batch=8, n_q_heads=32, ctx_lo=1000, ctx=8000, dtype="bf16", layers=16,
              block_tokens=64),
        # odd sizes, larger quantization groups and the index list as a second output
        _case("decode-list-g128", batch=2, n_q_heads=24, ctx=20011, group=128, index_list=True, layers=2),
        # the deployment policy: full attention in the first two layers, the selective step in the others
        _case("mixed-32k", n_q_heads=32, ctx=32768, dtype="bf16", layers=8, dense_first=2),
        # after prefill: the packed copy of one 32-head layer's keys
        _case("quantize-32k", kind="quantize", n_q_heads=32, n_kv_heads=32, ctx=32768),
        # the same for a ragged batch with larger groups
        _case("quantize-ragged-g128", kind="quantize", batch=4, n_q_heads=32, ctx_lo=3001, ctx=24001, dtype="bf16",
              group=128),
        # the step as separate calls, as a program that wants the scores and the selection makes them
        _case("calls-64k", kind="calls", n_q_heads=32, ctx=65001, dtype="bf16"),
        # the page-level selector on the headline shape
        _case("pages-32k", kind="pages", n_q_heads=32, n_kv_heads=32, ctx=32768, budget=3604),
    ]


def draw(rng):
    most = max(work(c)["bytes"] for c in listed())
    while True:
        kind = rng.choice(["decode"] * 6 + ["mixed", "quantize", "quantize", "calls", "pages"])
        n_q, n_kv = rng.choice([(8, 8), (16, 8), (24, 8), (32, 8), (64, 8), (28, 4), (32, 32), (32, 32)])
        ctx = int(math.exp(rng.uniform(math.log(1000), math.log(131072))))
        c = dict(_BASE, kind=kind, n_q_heads=n_q, n_kv_heads=n_kv, ctx=ctx, dtype=rng.choice(["f16", "bf16"]),
                 batch=int(math.exp(rng.uniform(0, math.log(16.99)))))
        c["ctx_lo"] = max(1, int(ctx * rng.choice([1.0, 1.0, 0.5, 0.125])))
        c["group"] = 32 if kind == "pages" else rng.choice([32, 32, 32, 64, 128])
        if kind in ("decode", "mixed"):
            c["layers"] = int(math.exp(rng.uniform(0, math.log(16.99))))
            c["index_list"] = kind == "decode" and rng.random() < 0.2
            if rng.random() < 0.25:
                c["block_tokens"] = rng.choice([64, 128, 256])
                c["group"] = min(c["group"], c["block_tokens"])
        if kind == "mixed":
            c["layers"] = max(3, c["layers"])
            c["dense_first"] = min(2, c["layers"] // 2)
        if rng.random() < 0.4:
            c["budget"] = min(16384, max(64, int(ctx * math.exp(rng.uniform(math.log(0.02), math.log(0.4))))))
            if c["ctx_lo"] < 2 * c["budget"]:
                c["ctx_lo"] = ctx
        else:
            c["budget_pct"] = round(rng.uniform(5.0, 25.0), 1)
        if kind == "pages":
            c["page_tokens"] = rng.choice([16, 16, 32])
            c["page_mode"] = rng.choice([0, 1])
        units = c["batch"] * n_kv
        if work(c)["bytes"] <= most and units * (ctx + 64) * c["layers"] * 512 <= 20e9:
            return c


def _shape(case):
    """Contexts, budgets and row capacity; a ragged batch's contexts are part of the case, not of its inputs."""
    b, lo, hi = case["batch"], case["ctx_lo"], case["ctx"]
    lens = np.full(b, hi, np.int64)
    if lo < hi and b > 1:
        lens[:-1] = np.random.default_rng(hi).integers(lo, hi + 1, size=b - 1)
    pct = case["budget_pct"]
    buds = np.full(b, case["budget"], np.int64) if case["budget"] else np.maximum(1, np.rint(pct / 100 * lens)).astype(np.int64)
    buds = np.minimum(buds, lens)
    gran = max(64, case["group"], case["block_tokens"], 64 * case["page_tokens"] if case["kind"] == "pages" else 0)
    return lens, buds, -(-(hi + 1) // gran) * gran


def work(case):
    lens, buds, _ = _shape(case)
    n_kv, kind = case["n_kv_heads"], case["kind"]
    rep = case["n_q_heads"] // n_kv
    heads = case["batch"] * case["n_q_heads"]
    packed = 16 + 512 // case["group"]          # code word and (s, z) per cached token and unit
    if kind == "quantize":
        return {"bytes": int(n_kv * lens.sum() * (2 * D + packed)), "flops": int(n_kv * lens.sum() * 3 * D)}
    n = lens + 1
    qo = heads * (2 * D + 4 * D)
    attend = int(n_kv * buds.sum())
    if kind == "pages":
        pages = -(-n // case["page_tokens"])
        return {"bytes": int(n_kv * pages.sum() * 4 * D + attend * 4 * D + qo),
                "flops": int(n_kv * rep * (pages.sum() * 4 * D) + attend * rep * 4 * D)}
    bits = int(n_kv * n.sum() * packed)
    sel = {"bytes": bits + attend * 4 * D + qo, "flops": int(n_kv * n.sum() * 2 * D + attend * rep * 4 * D)}
    if kind == "calls":
        # the scores and the index list are results here
        return {"bytes": sel["bytes"] + int(4 * n_kv * n.sum()) + 4 * attend, "flops": sel["flops"]}
    dense = {"bytes": int(n_kv * n.sum() * 4 * D + qo), "flops": int(n_kv * n.sum() * rep * 4 * D)}
    nd = case["dense_first"]
    return {k: (case["layers"] - nd) * sel[k] + nd * dense[k] for k in sel}


def tolerance(case):
    # Bits, scales and bounds are defined exactly.
    if case["kind"] == "quantize":
        return "exact"
    # Against the same path in 64 bits (selection and softmax both): rel 3e-7 to 9e-7, max up to 5e-6 over single- and
    # multi-head shapes, both types, and the same tokens selected everywhere; about four times that.  The share of
    # whole values is for a tie of two scores at the budget's edge, which moves the rest of one unit's list by a place.
    return {"rel": 4e-6, "max": 2.5e-5, "differ": 1e-3}


def _rows(gen, k, v, lens_u, scale, q):
    """Fill one layer's keys and values: N(0, 1) with outlier channels; 64 tokens per unit point along the query."""
    units, max_ctx, _ = k.shape
    per = max(1, (1 << 27) // (max_ctx * D))
    for u in range(0, units, per):
        e = min(units, u + per)
        kf = torch.randn((e - u, max_ctx, D), generator=gen, device="cuda") * scale[u:e, None, :]
        at = (torch.rand((e - u, 64), generator=gen, device="cuda") * lens_u[u:e, None]).long()[:, :, None].expand(-1, -1, D)
        qs = q[u:e].sum(dim=1)
        qs = qs / qs.norm(dim=-1, keepdim=True)
        kf.scatter_(1, at, 0.8 * math.sqrt(D) * qs[:, None, :] + 0.2 * kf.gather(1, at))
        k[u:e] = kf
        v[u:e] = torch.randn((e - u, max_ctx, D), generator=gen, device="cuda")


def prepare(case, seed):
    """A program in the middle of decoding: quantized layer caches, the step's queries and new rows, output buffers
    and the workspace it keeps."""
    kind, b, n_q, n_kv, NL = case["kind"], case["batch"], case["n_q_heads"], case["n_kv_heads"], case["layers"]
    lens, buds, max_ctx = _shape(case)
    dtype, code = (torch.float16, B.F16) if case["dtype"] == "f16" else (torch.bfloat16, B.BF16)
    cfg = B.make_config(b, n_q, n_kv, max_ctx, code, group_size=case["group"])
    units, rep = cfg.units, cfg.n_rep
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    i32 = lambda a: torch.as_tensor(np.asarray(a, np.int32), device="cuda")  # noqa: E731
    seq_lens = i32(lens)
    lens_u = seq_lens.repeat_interleave(n_kv).float()
    caches, qs, kns, vns = [], [], [], []
    bt = case["block_tokens"]
    per_seq = max_ctx // bt if bt else 0
    K = torch.empty((NL, b * per_seq, n_kv, bt, D) if bt else (NL, units, max_ctx, D), dtype=dtype, device="cuda")
    V = torch.empty_like(K)
    for layer in range(NL):
        scale = torch.ones((n_kv, D), device="cuda")
        if case["dtype"] == "bf16":
            scale = torch.exp(0.5 * torch.randn((n_kv, D), generator=gen, device="cuda"))
        scale.scatter_(1, torch.rand((n_kv, D), generator=gen, device="cuda").topk(4, dim=1).indices, 8.0)
        scale = scale.repeat(b, 1)
        q = torch.randn((units, rep, D), generator=gen, device="cuda")
        table = None
        if bt:
            k, v = (torch.empty((units, max_ctx, D), dtype=dtype, device="cuda") for _ in range(2))
            _rows(gen, k, v, lens_u, scale, q)
            perm = torch.randperm(b * per_seq, generator=gen, device="cuda")
            table = perm.to(torch.int32).view(b, per_seq).contiguous()
            for pool, rows in ((K, k), (V, v)):
                blocks = rows.view(b, n_kv, per_seq, bt, D).permute(0, 2, 1, 3, 4).reshape(b * per_seq, n_kv, bt, D)
                pool[layer][perm] = blocks
        else:
            _rows(gen, K[layer], V[layer], lens_u, scale, q)
        kns.append((torch.randn((units, D), generator=gen, device="cuda") * scale).to(dtype))
        vns.append(torch.randn((units, D), generator=gen, device="cuda").to(dtype))
        qs.append(q.to(dtype).view(b, n_q, D))
        c = B.DeviceCache(cfg, K[layer], V[layer], seq_lens, table)
        if kind != "quantize":
            B.quantize_keys(cfg, c)
        caches.append(c)
    mb = int(buds.max())
    s = {"case": case, "cfg": cfg, "caches": caches, "K": K, "V": V, "q": torch.stack(qs), "k_new": torch.stack(kns),
         "v_new": torch.stack(vns), "seq_lens": seq_lens, "budgets": i32(buds), "mb": mb}
    if kind == "quantize":
        return s
    s["out"] = torch.zeros((NL, b, n_q, D), dtype=torch.float32, device="cuda")
    s["idx"] = s["cnt"] = None
    if case["index_list"] or kind in ("mixed", "calls", "pages"):
        s["idx"] = torch.zeros((NL, units, mb), dtype=torch.int32, device="cuda")
        s["cnt"] = torch.zeros((NL, units), dtype=torch.int32, device="cuda")
    s["ws"] = B.make_workspace(cfg, max_ctx if kind == "mixed" else mb)
    if kind == "mixed":
        s["dense"] = [l < case["dense_first"] for l in range(NL)]
        s["idx"] = s["cnt"] = None
    if kind == "calls":
        s["scores"] = torch.zeros((units, max_ctx), dtype=torch.float32, device="cuda")
    if kind == "pages":
        P = case["page_tokens"]
        n_pages = max_ctx // P
        s["pcfg"] = B.make_config(b, n_q, n_kv, n_pages, code)
        s["meta"] = torch.zeros(B.page_meta_bytes(cfg, P) // 4, dtype=torch.int32, device="cuda")
        B.page_minmax(cfg, caches[0], P, s["meta"])
        pb = np.maximum(1, buds // P)
        s["max_pages"] = int(pb.max())
        s["page_budgets"], s["page_lens"] = i32(pb), i32(-(-(lens + 1) // P))
        s["pscores"] = torch.zeros((units, n_pages), dtype=torch.float32, device="cuda")
        s["pidx"] = torch.zeros((units, s["max_pages"]), dtype=torch.int32, device="cuda")
        s["pcnt"] = torch.zeros((units,), dtype=torch.int32, device="cuda")
        mb = s["mb"] = s["max_pages"] * P
        s["idx"] = torch.zeros((1, units, mb), dtype=torch.int32, device="cuda")
        s["ws"] = B.make_workspace(cfg, mb)
    return s


def _packed(s):
    return [(c.kbits, c.kmeta, c.kabsmax) for c in s["caches"]]


def _state(s):  # what an append updates
    return s["K"], s["V"], _packed(s)


def run(s):
    case, cfg, caches, kind = s["case"], s["cfg"], s["caches"], s["case"]["kind"]
    if kind == "quantize":
        B.quantize_keys(cfg, caches[0])
        return _packed(s)
    if kind == "decode":
        B.decode_step(cfg, caches, s["q"], s["k_new"], s["v_new"], s["budgets"], s["mb"], s["out"], s["idx"], s["cnt"],
                      s["ws"])
        return s["out"], s["idx"], s["cnt"], _state(s)
    if kind == "mixed":
        B.decode_step_mixed(cfg, caches, s["dense"], s["q"], s["k_new"], s["v_new"], s["budgets"], s["mb"], s["out"],
                            s["idx"], s["cnt"], s["ws"])
        return s["out"], _state(s)
    c, q, idx, cnt, out = caches[0], s["q"][0], s["idx"][0], s["cnt"][0], s["out"][0]
    B.append_key(cfg, c, s["k_new"][0], s["v_new"][0])
    if kind == "calls":
        B.score(cfg, c, q, 1, s["scores"])
        B.topk_ws(cfg, s["scores"], s["seq_lens"], 1, s["budgets"], s["mb"], idx, cnt, s["ws"])
        B.sparse_attn(cfg, c, q, idx, cnt, s["mb"], out, s["ws"])
        return out, s["scores"], idx, cnt, _state(s)
    P = case["page_tokens"]
    B.page_append(cfg, s["seq_lens"], P, s["k_new"][0], s["meta"])
    B.page_score(cfg, s["meta"], P, s["seq_lens"], 1, q, case["page_mode"], s["pscores"])
    B.topk(s["pcfg"], s["pscores"], s["page_lens"], 0, s["page_budgets"], s["max_pages"], s["pidx"], s["pcnt"])
    B.expand_pages(cfg, s["pidx"], s["pcnt"], s["max_pages"], s["seq_lens"], 1, P, idx, cnt, s["mb"])
    B.sparse_attn(cfg, c, q, idx, cnt, s["mb"], out, s["ws"])
    return out, s["pscores"], idx, cnt, s["meta"], _state(s)
