"""Attention whose scaled logits are far beyond the integers binary32 holds exactly, against a float64 softmax: one row (or
two equal ones) takes all the weight, so every path has to return that row of V (their mean), whatever the logit rounds to.

Finite inputs of ordinary kinds reach this: 16-bit keys and queries of a few thousand in every channel, or a softmax scale
that makes the step a hard maximum.  Tolerance: the winner leads by far more than the rounding of a logit, so its weight is 1
(or exactly 1/2) and the others' 0: the output is V in binary32, up to the sums of the two parts of a tie."""
import pytest

torch = pytest.importorskip("torch")

from paper_2508_08256_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu
CTX, LENS, D = 640, [1, 17, 64, 65, 300, 639], 128


def _inputs(n_rep, dtype, size):
    """size: of every channel of the queries and of the winning rows."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_rep)
    b = len(LENS)
    normal = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    k, v = normal(b, CTX, D), normal(b, CTX, D).to(dtype)
    wins = [[0], [16], [3, 40], [64], [5, 290], [600]]
    near = lambda *s: size * (1 + 0.01 * torch.rand(s, generator=gen, device="cuda"))  # noqa: E731
    for u, rows in enumerate(wins):
        k[u, rows] = near(D)
    return k.to(dtype), v, near(b, n_rep, D).to(dtype)


def _paths(cfg, k, v, q, lens):
    """(name, output) of every path that attends over rows [0, lens), the steps over a selection of them."""
    b, mb = cfg.batch, 96
    ws = B.make_workspace(cfg, cfg.max_ctx, 1)
    cache = lambda: B.DeviceCache(cfg, k.clone(), v.clone(), lens)  # noqa: E731
    empty = lambda: torch.full(q.shape, float("nan"), device="cuda")  # noqa: E731
    out = empty()
    B.dense_attn(cfg, cache(), q, 0, out, ws)
    yield "dense", out
    out, idx = empty(), torch.arange(CTX - 1, -1, -1, device="cuda", dtype=torch.int32)
    idx = torch.stack([torch.roll(idx, int(n) - CTX) for n in lens]).contiguous()  # n - 1, ..., 0 first
    B.sparse_attn(cfg, cache(), q, idx, lens, CTX, out, ws)
    yield "sparse", out
    budgets = torch.full((b,), mb, dtype=torch.int32, device="cuda")
    for name, phases in (("step", None), ("two kernels", (1, 2 + 32)), ("merged late", (1, 2 + 16)), ("three kernels", (1, 2 + 64, 3 + 64))):
        out, c, w = empty(), cache(), B.make_workspace(cfg, mb, 1)
        B.quantize_keys(cfg, c)
        args = (cfg, [c], q[None], None, None, budgets, mb, out[None], None, None, w)
        for p in phases or ():
            B.decode_step_phase(*args, p)
        if not phases:
            B.decode_step(*args)
        yield name, out


def _check(n_rep, dtype, size, sm_scale=None):
    k, v, q = _inputs(n_rep, dtype, size)
    cfg = B.make_config(len(LENS), n_rep, 1, CTX, B.F16 if dtype == torch.float16 else B.BF16)
    if sm_scale is not None:
        cfg.sm_scale = sm_scale
    lens = torch.tensor(LENS, dtype=torch.int32, device="cuda")
    want = torch.zeros(q.shape, dtype=torch.float64)
    for u, n in enumerate(LENS):
        s = q[u].double().cpu() @ k[u, :n].double().cpu().T * float(cfg.sm_scale)
        want[u] = torch.softmax(s, -1) @ v[u, :n].double().cpu()
    bad = []
    for name, out in _paths(cfg, k, v, q, lens):
        err = (out.double().cpu() - want).abs().amax(dim=(1, 2))
        if not (err <= 1e-6).all():
            bad.append((name, err.tolist()))
    assert not bad, bad


@pytest.mark.parametrize("n_rep", range(1, 9))
@pytest.mark.parametrize("dtype,size", [(torch.float16, s) for s in (100.0, 1900.0, 3000.0, 4000.0, 60000.0)] +
                         [(torch.bfloat16, s) for s in (1900.0, 20000.0, 30000.0, 1e9, 1e15)], ids=str)
def test_a_row_of_large_entries_takes_all(n_rep, dtype, size):
    _check(n_rep, dtype, size)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=str)
@pytest.mark.parametrize("n_rep", [1, 3, 5, 8])
def test_a_large_scale_is_a_hard_maximum(n_rep, dtype):
    _check(n_rep, dtype, 3.0, 1e6)
    _check(n_rep, dtype, 3.0, 1e20)
