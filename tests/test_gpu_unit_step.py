"""The step of short contexts, one workgroup per unit, against the two-kernel form of the same call (which the other tests
compare with the oracle) and, where layers share a launch, against single-layer calls; its attention against float64.

The same selection, scores, appended rows and packed caches, bit for bit.  Outputs by their 2-norm: a softmax over N(0, 1) rows at
logits of N(0, 1) is an average, its rounding errors a random walk over the wavefronts' and tiles' sums: under 1e-6 of the output's norm
against float64 (logits: test_gpu_gqa_gather), so 2e-6 there and twice that between two forms.  A lost or repeated row of 1500 would be
3e-2, probabilities rounded to 16 bits 1e-3.  Only with zero queries, where the average of 1500 rows is 40 times smaller than a row, are
the sums' own errors larger beside it: 1500 additions of up to |v| sqrt(1500), sqrt(1500) * 2^-24 * sqrt(1500) / 1500 = 6e-8 of |v|, or
2.4e-6 of the output."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2508_08256_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu
F16, BF16 = 0, 1

CASES = {
    # batch, query heads, kv heads, contexts, budgets, dtype, capacity, block tokens, group, append
    "group_edges": (8, 8, 8, [0, 1, 31, 32, 33, 63, 64, 65], [1, 1, 5, 32, 40, 7, 65, 20], F16, 192, 0, 32, True),
    "ranges": (5, 10, 5, [1022, 1023, 1024, 2047, 3071], [100, 1, 1024, 500, 300], BF16, 3136, 0, 32, True),
    "own_16_waves": (4, 12, 4, [4095, 4096, 4097, 4200], [400, 1100, 700, 4], F16, 4224, 0, 32, True),
    "g64": (3, 16, 4, [127, 128, 2300], [10, 129, 0], BF16, 2304, 64, 64, True),
    "g128": (3, 10, 2, [127, 1400, 2303], [30, 100, 300], F16, 2304, 128, 128, True),
    "g256_full": (4, 18, 3, [255, 256, 600, 768], [30, 100, 300, 200], BF16, 768, 256, 256, True),
    "no_append": (2, 7, 1, [900, 0], [100, 5], F16, 960, 0, 32, False),
    "ragged_8_waves": (36, 64, 8, list(range(300, 5700, 150)), [33 + i for i in range(36)], BF16, 5760, 64, 32, True),
    "own_8_waves": (66, 32, 8, [2048 + 29 * i for i in range(66)], [200] * 66, F16, 4096, 0, 32, True),
    "ties": (2, 4, 4, [3000, 1500], [700, 1500], F16, 3072, 0, 32, True),   # zero queries: every score in one bin
    "tie_edge": (1, 3, 3, [600], [100], BF16, 640, 0, 32, True),
    # 16 wavefronts, LDS far past 64 KiB; 8 wavefronts, a thread owns 32 tokens
    "long_16_waves": (32, 32, 8, [11775 - 61 * i for i in range(32)], [1200 - i for i in range(32)], BF16, 11776, 64, 32, True),
    "long_16_waves_1_head": (25, 4, 4, [6271 - 40 * i for i in range(25)], [500] * 25, F16, 6272, 0, 32, True),
    "long_16_waves_8_heads": (20, 64, 8, [7935 - 101 * i for i in range(20)], [800] * 20, BF16, 7936, 0, 64, True),
    "own_32": (33, 32, 8, [10001 - 83 * i for i in range(33)], [1100] * 33, F16, 10048, 0, 32, True),
    "own_32_2_heads": (64, 16, 8, [9000 - 41 * i for i in range(64)], [600] * 64, BF16, 9024, 0, 32, True),
}


def _off(got, want):
    """The largest distance of a unit's outputs over their 2-norm."""
    want = want.double()
    norm = want.flatten(-2).norm(dim=-1)
    d = (got.double() - want).flatten(-2).norm(dim=-1)
    assert torch.equal(d[norm == 0], norm[norm == 0])  # empty selections: zeros
    return float((d / norm.clamp(min=1e-30)).max())


def _case(name):
    batch, hq, hkv, lens, buds, dtype, cap, bt, group, append = CASES[name]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(len(name))
    td = torch.float16 if dtype == F16 else torch.bfloat16
    cfg = B.make_config(batch, hq, hkv, cap, dtype, group_size=group)
    table, shape = None, (cfg.units, cap, 128)
    if bt:
        table = torch.randperm(batch * (cap // bt), generator=gen, device="cuda").to(torch.int32).view(batch, -1).contiguous()
        shape = (table.numel(), hkv, bt, 128)
    k, v = (torch.randn(shape, generator=gen, device="cuda").to(td) for _ in range(2))
    if name == "tie_edge":
        k[:] = k[:, :1]  # the same row everywhere: equal scores go to the lower index
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device="cuda")  # noqa: E731
    q = torch.randn((1, batch, hq, 128), generator=gen, device="cuda").to(td)
    if name == "ties":
        q.zero_()
    new = [torch.randn((1, cfg.units, 128), generator=gen, device="cuda").to(td) if append else None for _ in range(2)]
    return cfg, k, v, i32(lens), table, q, new, i32(buds), max(buds)


def _scores_end(cfg, mb):
    at = int(B.lib().fier_workspace_scores_offset(ctypes.byref(cfg), mb)) + 4 * cfg.units * cfg.max_ctx
    return -(-at // 256) * 256


def _run(case, phases=None):
    cfg, k, v, lens, table, q, new, buds, mb = case
    cache = B.DeviceCache(cfg, k.clone(), v.clone(), lens, table)
    B.quantize_keys(cfg, cache)
    ws = B.make_workspace(cfg, mb, 1)
    bounds = ws[_scores_end(cfg, mb):][:512 * cfg.units]  # of the appended groups: the score kernel leaves them here
    bounds[:] = 0x5A
    out = torch.full((1, cfg.batch, cfg.n_q_heads, 128), float("nan"), device="cuda")
    idx = torch.full((1, cfg.units, mb), -1, dtype=torch.int32, device="cuda")
    cnt = torch.full((1, cfg.units), -1, dtype=torch.int32, device="cuda")
    args = (cfg, [cache], q, new[0], new[1], buds, mb, out, idx, cnt, ws)
    if phases:
        for p in phases:
            B.decode_step_phase(*args, p)
    else:
        B.decode_step(*args)
    scores = B.workspace_scores(cfg, mb, ws).clone()
    for u in range(cfg.units):
        scores[u, min(int(lens[u // cfg.n_kv_heads]) + (new[0] is not None), cfg.max_ctx):] = 0
    zero = ws[:cfg.units * 64].view(torch.int32).view(-1, 16)[:, :4]
    assert not zero.any()  # the counters
    assert not ws[cfg.units * 64:cfg.units * (64 + 2048)].view(torch.int32).any()  # the histograms
    assert bool((bounds == 0x5A).all()) == (phases is None or new[0] is None)  # a call took one launch
    return out, idx, cnt, [scores, cache.k, cache.v, cache.kbits, cache.kmeta, cache.kabsmax]


@pytest.mark.parametrize("name", CASES)
def test_unit_step_equals_the_two_kernel_form(name):
    case = _case(name)
    want = _run(case, (1, 2 + 32, 3 + 32))
    for phases in (None, (1, 2, 3)):
        got = _run(case, phases)
        assert torch.equal(got[2], want[2]) and torch.equal(got[1], want[1]), name
        assert torch.isfinite(got[0]).all() and _off(got[0].view(-1, 1, 128), want[0].view(-1, 1, 128)) <= (1e-5 if name == "ties" else 4e-6), name
        for a, b in zip(got[3], want[3]):
            assert torch.equal(a, b)


@pytest.mark.parametrize("layers", [3, 17])
def test_unit_step_of_several_layers(layers):
    """Ragged sequences, more workgroups than are resident: the longest go first."""
    rng = np.random.default_rng(layers)
    batch, hq, hkv, cap = 23, 32, 8, 2112
    lens = torch.tensor(rng.integers(0, cap + 1, batch), dtype=torch.int32, device="cuda")
    buds = (lens // 9 + 1).int()
    cfg, mb = B.make_config(batch, hq, hkv, cap, BF16), int(buds.max())
    gen = torch.Generator(device="cuda")
    gen.manual_seed(layers)
    normal = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    rows = [(normal(cfg.units, cap, 128), normal(cfg.units, cap, 128)) for _ in range(layers)]
    q, kn, vn = normal(layers, batch, hq, 128), normal(layers, cfg.units, 128), normal(layers, cfg.units, 128)
    res = []
    for one_by_one in (False, True):
        caches = [B.DeviceCache(cfg, k.clone(), v.clone(), lens) for k, v in rows]
        for c in caches:
            B.quantize_keys(cfg, c)
        out = torch.full((layers, batch, hq, 128), float("nan"), device="cuda")
        idx = torch.full((layers, cfg.units, mb), -1, dtype=torch.int32, device="cuda")
        cnt = torch.zeros((layers, cfg.units), dtype=torch.int32, device="cuda")
        ws = B.make_workspace(cfg, mb, 1)
        for l in [slice(i, i + 1) for i in range(layers)] if one_by_one else [slice(0, layers)]:
            B.decode_step(cfg, caches[l], q[l], kn[l], vn[l], buds, mb, out[l], idx[l], cnt[l], ws)
        res.append((out, idx, cnt, [t for c in caches for t in (c.k, c.v, c.kbits, c.kmeta, c.kabsmax)]))
    (o, i, n, s), (o1, i1, n1, s1) = res
    assert torch.equal(i, i1) and torch.equal(n, n1) and _off(o.view(-1, 1, 128), o1.view(-1, 1, 128)) <= 4e-6
    assert all(torch.equal(a, b) for a, b in zip(s, s1))


@pytest.mark.parametrize("dtype", [F16, BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("n_rep", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("waves", [16, 8])
def test_unit_step_attends_over_the_listed_rows(waves, n_rep, dtype):
    """Selections of up to two rounds of the workgroup's tiles (8 rows a wavefront with one or two heads, else 16), and one row less
    or more, against a float64 softmax over the rows of the index list."""
    tile = waves * (8 if n_rep <= 2 else 16)
    counts = [0, 1, 7, 8, 9, 15, 16, 17, tile - 1, tile, tile + 1, 2 * tile - 1, 2 * tile, 2 * tile + 1]
    hkv, ctx = (1, 640) if waves == 16 else (24, 640)  # 8 wavefronts: more than 256 workgroups
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_rep)
    td = torch.float16 if dtype == F16 else torch.bfloat16
    cfg, mb = B.make_config(len(counts), n_rep * hkv, hkv, ctx, dtype), max(counts)
    normal = lambda *s: torch.randn(s, generator=gen, device="cuda").to(td)  # noqa: E731
    k, v, q = normal(cfg.units, ctx, 128), normal(cfg.units, ctx, 128), normal(1, len(counts), n_rep * hkv, 128)
    new = [normal(1, cfg.units, 128) for _ in range(2)]
    lens, buds = (torch.tensor(x, dtype=torch.int32, device="cuda") for x in ([ctx - 1 - i for i in range(len(counts))], counts))
    out, idx, cnt, (_, k1, v1, *_) = _run((cfg, k, v, lens, None, q, new, buds, mb))
    assert cnt[0].tolist() == [c for c in counts for _ in range(hkv)]
    s = torch.matmul(q.view(cfg.units, n_rep, 128).double(), k1.double().transpose(1, 2).contiguous()) * float(cfg.sm_scale)
    listed = torch.zeros((cfg.units, ctx + 1), dtype=torch.bool, device="cuda")
    listed.scatter_(1, torch.where(idx[0] < 0, ctx, idx[0]).long(), True)
    p = torch.softmax(s.masked_fill(~listed[:, None, :ctx], -1e30), -1) * (cnt[0] > 0)[:, None, None]
    want = torch.matmul(p, v1.double())
    assert _off(out.view(cfg.units, n_rep, 128), want) <= 2e-6
