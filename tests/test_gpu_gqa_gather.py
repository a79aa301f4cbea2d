"""The matrix-core gather (three to eight query heads per kv head) at the edges of its 16-row tiles and 64-row rounds,
against float64: fier_sparse_attn over lists of those lengths, fier_dense_attn over prefixes of those lengths.

Tolerance: a logit is a sum of 128 products in binary32, its error at most 128 * 2^-24 * sum |q_i k_i| * scale, for N(0, 1)
rows below 128 * 6e-8 * 0.64 * 128 / 11.3 = 5.6e-5 in the worst case and about 1/40 of that as a random walk; weights and
output inherit it relatively.  2e-6 of the output's 2-norm leaves room over what is seen (under 5e-7) and is three orders
below what probabilities rounded to the 16-bit type would give."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2508_08256_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu
CTX, D = 320, 128
COUNTS = [1, 3, 15, 16, 17, 63, 64, 65, 127, 128, 129, 193, 256, 257, 319, 320]


def _inputs(n_rep, dtype):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(100 + n_rep)
    b = len(COUNTS)
    cfg = B.make_config(b, n_rep, 1, CTX, B.F16 if dtype == torch.float16 else B.BF16)
    k, v = (torch.randn((b, CTX, D), generator=gen, device="cuda").to(dtype) for _ in range(2))
    q = (2.0 * torch.randn((b, n_rep, D), generator=gen, device="cuda")).to(dtype)
    lens = torch.tensor(COUNTS, dtype=torch.int32, device="cuda")
    idx = torch.stack([torch.randperm(CTX, generator=gen, device="cuda") for _ in range(b)]).to(torch.int32)
    return cfg, k, v, q, lens, idx


def _exact(cfg, k, v, q, rows):
    out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    for u, r in enumerate(rows):
        s = (q[u].double()[:, None, :] * k[u][r].double()[None]).sum(-1) * float(cfg.sm_scale)
        p = torch.softmax(s, dim=-1)
        out[u] = (p[:, :, None] * v[u][r].double()[None]).sum(1)
    return out


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("n_rep", [3, 4, 5, 6, 7, 8])
def test_gather_at_tile_edges(n_rep, dtype):
    cfg, k, v, q, lens, idx = _inputs(n_rep, dtype)
    cache = B.DeviceCache(cfg, k, v, lens)
    ws = B.make_workspace(cfg, CTX, 1)
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    for rows in (None, [idx[u, :c].long() for u, c in enumerate(COUNTS)]):
        if rows is None:
            B.dense_attn(cfg, cache, q, 0, out, ws)
            rows = [torch.arange(c, device="cuda") for c in COUNTS]
        else:
            B.sparse_attn(cfg, cache, q, idx, lens, CTX, out, ws)
        want = _exact(cfg, k, v, q, rows)
        rel = ((out.double() - want).flatten(1).norm(dim=1) / want.flatten(1).norm(dim=1)).cpu().numpy()
        assert rel.max() <= 2e-6, (n_rep, COUNTS[int(rel.argmax())], rel)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("n_rep", [3, 5, 6, 8])
def test_weights_far_below_the_largest(n_rep, dtype):
    """A row of weight 1 with V = 0 and 63 rows of weights 2^-1 .. 2^-45 (q k = the base-2 logit): all that comes out is theirs.
    bf16: their binary32 values, the scale's rounding times 45.  fp16: to 2^-39 of the largest weight per row, 2^-38 from six heads on."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_rep)
    cfg = B.make_config(45, n_rep, 1, 64, B.F16 if dtype == torch.float16 else B.BF16)
    cfg.sm_scale = 0.6931471805599453
    k, q = (torch.zeros(s, dtype=dtype, device="cuda") for s in ((45, 64, D), (45, n_rep, D)))
    q[:, :, 0] = 1
    k[:, 1:, 0] = -torch.arange(1, 46, device="cuda", dtype=dtype)[:, None]
    v = torch.randn((45, 64, D), generator=gen, device="cuda").to(dtype)
    v[:, 0] = 0
    lens = torch.full((45,), 64, dtype=torch.int32, device="cuda")
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    B.dense_attn(cfg, B.DeviceCache(cfg, k, v, lens), q, 0, out, B.make_workspace(cfg, 64, 1))
    p = torch.softmax(k[:, :, 0].double() * float(cfg.sm_scale), -1)
    want, size = ((p[:, :, None] * x.double()).sum(1)[:, None] for x in (v, v.abs()))
    part = (2.0 ** -39 if n_rep <= 5 else 2.0 ** -38) if dtype == torch.float16 else 0.0
    bound = 1e-5 * size + 63 * part * v.abs().double().amax(1)[:, None]
    assert bool(((out.double() - want).abs() <= bound).all())
