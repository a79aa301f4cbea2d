"""fier_quantize_keys where its decision threshold, its wavefront exchanges and its work split can go wrong: bit-exact."""
import numpy as np
import pytest
import torch

from paper_2508_08256_amd import binding as B
from paper_2508_08256_amd import synth

pytestmark = pytest.mark.gpu

F16, BF16 = synth.F16, synth.BF16


def _words(kind, rng, shape, dtype):
    """uint16 words of finite values."""
    top = 0x7BFF if dtype == F16 else 0x7F7F
    sign = (rng.integers(0, 2, shape) << 15).astype(np.uint16)
    if kind == "any":          # every finite bit pattern, subnormals and the largest included
        return rng.integers(0, top + 1, shape).astype(np.uint16) | sign
    if kind == "near":         # a channel's values within a few steps of each other: ranges of a few ulps, midpoints hit
        base = rng.integers(8, top - 8, shape[:1] + (1,) + shape[2:])
        return (base + rng.integers(-3, 4, shape)).astype(np.uint16) | sign[:, :1, :]
    if kind == "zero-mid":     # +-m at the ends, +-0 and values far below m's last place around the midpoint at 0
        m = rng.integers(1, top + 1, shape[:1] + (1,) + shape[2:])
        pick = rng.integers(0, 6, shape)
        small = np.where(pick < 2, 0, rng.integers(0, 1 << 15, shape) % (m + 1) // np.where(pick == 2, 1, 1 << rng.integers(1, 15, shape)))
        w = np.where(pick == 5, m, small).astype(np.uint16) | sign
        w[:, ::16, :] = m.astype(np.uint16)
        w[:, 1::16, :] = m.astype(np.uint16) | 0x8000
        return w
    assert kind == "constant"
    return np.broadcast_to(_words("any", rng, shape[:1] + (1,) + shape[2:], dtype), shape).copy()


def _check(oracle, batch, heads, lens, max_ctx, dtype, g, kind, bt=0):
    import gpu_util

    rng = np.random.default_rng(hash((max_ctx, dtype, g, len(kind))) % 1000)
    wl = synth.make_workload("edges", 3, batch, heads, heads, lens, [1] * batch, dtype, max_ctx=max_ctx, plant=False)
    wl.K[:] = _words(kind, rng, wl.K.shape, dtype)
    dw = gpu_util.PagedWorkload(wl, bt, g) if bt else gpu_util.DeviceWorkload(wl, g)
    B.quantize_keys(dw.cfg, dw.cache)
    torch.cuda.synchronize()
    L = wl.unit_lens
    bits_o, s_o, z_o = oracle.quantize(wl.K, L, g, dtype, 8)
    bits, s, z = dw.cache.unpack()
    amax = dw.cache.kabsmax.cpu().numpy().reshape(wl.units, 128)
    for u in range(wl.units):
        n = int(L[u])
        ng = -(-n // g)
        assert np.array_equal(s[u, :ng], s_o[u, :ng]) and np.array_equal(z[u, :ng], z_o[u, :ng])
        bad = np.argwhere(bits[u, :n] != bits_o[u, :n])
        assert len(bad) == 0, (kind, u, bad[:4], len(bad))
        assert np.all(bits[u, n:-(-n // 64) * 64] == 0)
        zf, sf = oracle.to_f32(z_o[u, :ng], dtype), oracle.to_f32(s_o[u, :ng], dtype)
        with np.errstate(over="ignore"):  # the upper level of a range held at the top of the format
            want = np.maximum(np.abs(zf), np.abs(zf + sf)).max(axis=0) if ng else np.zeros(128, np.float32)
        assert np.array_equal(amax[u], want.astype(np.float32))


@pytest.mark.parametrize("kind", ["any", "near", "zero-mid", "constant"])
@pytest.mark.parametrize("g", [32, 64, 128, 256])
@pytest.mark.parametrize("dtype", [F16, BF16])
def test_thresholds_and_partial_groups(oracle, dtype, g, kind):
    """Lengths one short of, at and one past a group, a pair block and a workgroup's share, an empty and a one-token
    sequence; values that put the decision threshold everywhere a 16-bit format can have it."""
    lens = [0, 1, 31, 33, 63, 64, 65, g - 1, g, g + 1, 256, 257, 511, 1023, 1024]
    _check(oracle, len(lens), 1, lens, 1024, dtype, g, kind)


@pytest.mark.parametrize("dtype,g,bt", [(F16, 32, 64), (BF16, 128, 128), (BF16, 256, 256)])
def test_paged_rows(oracle, dtype, g, bt):
    _check(oracle, 3, 2, [700, 256, 1], 768, dtype, g, "any", bt)


@pytest.mark.parametrize("dtype,g", [(F16, 32), (BF16, 64), (BF16, 128)])
def test_two_blocks_per_wavefront(oracle, dtype, g):
    """8224 pair blocks: the size from which a wavefront takes two of them in turn (four: the full-size tests)."""
    _check(oracle, 2, 8, [32896, 20000], 32896, dtype, g, "any")


@pytest.mark.parametrize("g", [32, 64, 128, 256])
@pytest.mark.parametrize("dtype", [F16, BF16])
@pytest.mark.parametrize("fused", [False, True])
def test_append_at_every_chunk_edge(dtype, g, fused):
    """The row joins an empty cache, a group's first, middle and last 32-token chunk, a fresh group: afterwards rows and
    packed cache are those of a bulk quantization of the longer prefix, in the append call and in the fused step."""
    import gpu_util

    lens = sorted({0, 1, 31, 32, 33, 63, 64, 95, 96, 127, 128, 159, 160, 191, 192, 223, 224, 255, 256, 300, g - 1, g, 511})
    rng = np.random.default_rng(g + dtype)
    wl = synth.make_workload("app", 5, len(lens), 2, 1, lens, [min(20, n + 1) for n in lens], dtype, max_ctx=512, plant=False)
    wl.K[:] = _words("any" if not fused else "near", rng, wl.K.shape, dtype)
    dw, ref = gpu_util.DeviceWorkload(wl, g), gpu_util.DeviceWorkload(wl, g)
    B.quantize_keys(dw.cfg, dw.cache)
    if fused:
        out = torch.zeros((1, wl.units, 2, 128), dtype=torch.float32, device="cuda")
        B.decode_step(dw.cfg, [dw.cache], dw.q[None].contiguous(), dw.k_new[None].contiguous(),
                      dw.v_new[None].contiguous(), dw.budgets, 20, out, None, None, dw.workspace(20))
    else:
        B.append_key(dw.cfg, dw.cache, dw.k_new, dw.v_new)
    for u, n in enumerate(lens):
        ref.K[u, n] = ref.k_new.reshape(wl.units, 128)[u]
        ref.V[u, n] = ref.v_new.reshape(wl.units, 128)[u]
    ref.seq_lens.add_(1)
    B.quantize_keys(ref.cfg, ref.cache)
    torch.cuda.synchronize()
    assert torch.equal(dw.K.view(torch.int16), ref.K.view(torch.int16))
    assert torch.equal(dw.V.view(torch.int16), ref.V.view(torch.int16))
    a, b = dw.cache.unpack(), ref.cache.unpack()
    for u, n in enumerate(lens):
        m, ng = -(-(n + 1) // 64) * 64, -(-(n + 1) // g)
        assert np.array_equal(a[0][u, :m], b[0][u, :m]), (u, n)
        assert np.array_equal(a[1][u, :ng], b[1][u, :ng]) and np.array_equal(a[2][u, :ng], b[2][u, :ng]), (u, n)


def test_short_sequences_in_a_large_capacity_use_the_whole_chip():
    """1000 tokens per unit take about as long in 65536 rows of capacity as in 1024: the few workgroups that have work
    must not meet on one XCD (measured: 1.7 times as long; 11 times where they did)."""
    batch, heads, bt = 64, 8, 1024
    k = torch.randn((batch, heads, bt, 128), device="cuda").half()
    lens = torch.full((batch,), 1000, dtype=torch.int32, device="cuda")
    best = {}
    for max_ctx in (1024, 65536):
        cfg = B.make_config(batch, heads, heads, max_ctx, F16)
        table = torch.zeros((batch, max_ctx // bt), dtype=torch.int32, device="cuda")
        table[:, 0] = torch.arange(batch, dtype=torch.int32, device="cuda")
        cache = B.DeviceCache(cfg, k, k.clone(), lens, table)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(5):
            e0.record()
            for _ in range(10):
                B.quantize_keys(cfg, cache)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        best[max_ctx] = min(times)
    assert best[65536] < 4 * best[1024], best
