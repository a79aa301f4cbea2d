"""The step of short contexts, one workgroup per unit, against the two-kernel form of the same call (which the other tests
compare with the oracle) and, where layers share a launch, against single-layer calls.

The same selection, scores, appended rows and packed caches, bit for bit; outputs up to the order of at most 2500 binary32
terms of |v| below about 5, some of which pass through three 16-bit parts that hold all 24 bits: 2500 * 2^-24 * 5 < 1e-3, far
above what is seen."""
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
}


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
        assert torch.isfinite(got[0]).all() and float((got[0] - want[0]).abs().max()) <= 1e-3
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
    assert torch.equal(i, i1) and torch.equal(n, n1) and float((o - o1).abs().max()) <= 1e-3
    assert all(torch.equal(a, b) for a, b in zip(s, s1))
