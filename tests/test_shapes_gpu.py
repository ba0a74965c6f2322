"""Parity of the bf16 workgroup shapes of 256 rows ("oct", head dim >= 72),
192 rows ("six", head dim <= 72) and 32 or 64 rows ("strip"), forced with XDIT_ATTN_TILE, at the edges of their
query and key tiles, and of the shapes the library picks by itself on both
sides of one workgroup per CU, against the fp64 oracle on sampled rows."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2411_01738_amd as xd
from paper_2411_01738_amd.inputs import random_io, sample_rows
from tests.gpu_util import attention_kernels, bf16_kernel, check_lse, check_out, to_gpu, to_np, torch_mod

pytestmark = pytest.mark.gpu

FORCED = [("oct", 72), ("oct", 128), ("six", 64), ("six", 72), ("strip", 64), ("strip", 72), ("strip", 128)]


def _chunk(torch, orc, B, H, d, nq, nk, what, rows=None, shape=None):
    q, k, v = (random_io((B, n, H, d), "bf16", 5000 + n + i) for i, n in enumerate((nq, nk, nk)))
    out = torch.full((B, nq, H, d), float("nan"), device="cuda", dtype=torch.bfloat16)
    lse = torch.full((B, H, nq), float("nan"), device="cuda", dtype=torch.float32)
    g = [to_gpu(x, "bf16") for x in (q, k, v)]
    names = attention_kernels(lambda: xd.xdit_chunk_attn(*g, out, lse))
    assert shape is None or names == [bf16_kernel(shape, d)]
    rows = np.arange(nq) if rows is None else rows
    ro, rl = orc.attention(q[:, rows].copy(), k, v)
    check_out(to_np(out)[:, rows], ro, "bf16", what)
    check_lse(lse.cpu().numpy()[:, :, rows], rl, "bf16", what + " lse")


@pytest.mark.parametrize("shape,d", FORCED)
def test_chunk_edges(shape, d, monkeypatch):
    torch, orc = torch_mod(), oracle.get()
    monkeypatch.setenv("XDIT_ATTN_TILE", shape)
    rows = {"oct": 256, "six": 192, "strip": 64 if d == 128 else 32}[shape]
    for nq, nk in [(1, 1), (rows - 1, 63), (rows, 64), (rows + 1, 65), (2 * rows + 33, 645), (40, 0), (97, 130)]:
        print(f"[shape] {shape} d={d} {nq} x {nk}", flush=True)
        _chunk(torch, orc, 1, 2, d, nq, nk, f"{shape} d={d} {nq} x {nk}", shape=shape)


@pytest.mark.parametrize("shape,d", FORCED)
def test_patch_and_ring(shape, d, monkeypatch):
    """Two fresh ranges off the tile edges with queries of their own, the
    buffer bit for bit; then a ring of two chunks cut inside a tile."""
    torch, orc = torch_mod(), oracle.get()
    monkeypatch.setenv("XDIT_ATTN_TILE", shape)
    B, H, N, nq = 2, 2, 433, 270
    ranges = [(37, 150), (300, 71)]
    F = sum(n for _, n in ranges)
    q = random_io((B, nq, H, d), "bf16", 1)
    kv = np.ascontiguousarray(random_io((2, B, N, H, d), "bf16", 2))
    fk, fv = random_io((B, F, H, d), "bf16", 3), random_io((B, F, H, d), "bf16", 4)
    kvg = to_gpu(kv, "bf16")
    out = torch.full((B, nq, H, d), float("nan"), device="cuda", dtype=torch.bfloat16)
    lse = torch.full((B, H, nq), float("nan"), device="cuda", dtype=torch.float32)
    xd.xdit_patch_attn_ranges(to_gpu(q, "bf16"), kvg, ranges, to_gpu(fk, "bf16"), to_gpu(fv, "bf16"), out, lse)
    base = 0
    for o, n in ranges:
        kv[0][:, o:o + n], kv[1][:, o:o + n] = fk[:, base:base + n], fv[:, base:base + n]
        base += n
    assert np.array_equal(to_np(kvg), kv)
    ro, rl = orc.attention(q, kv[0].copy(), kv[1].copy())
    check_out(to_np(out), ro, "bf16", f"{shape} patch d={d}")
    check_lse(lse.cpu().numpy(), rl, "bf16", f"{shape} patch lse d={d}")
    out.fill_(float("nan"))
    lse.fill_(float("-inf"))
    for a, b in ((0, 201), (201, N)):
        xd.xdit_chunk_attn_accum(to_gpu(q, "bf16"), to_gpu(kv[0][:, a:b], "bf16"), to_gpu(kv[1][:, a:b], "bf16"), out, lse)
    check_out(to_np(out), ro, "bf16", f"{shape} ring d={d}")
    check_lse(lse.cpu().numpy(), rl, "bf16", f"{shape} ring lse d={d}")


@pytest.mark.parametrize("d,H,nq,nk,shape", [
    (64, 43, 769, 1300, "six"), (72, 43, 850, 1300, "six"), (64, 8, 1024, 700, "strip"), (64, 8, 1025, 700, "narrow"),
    (64, 43, 700, 200, "quad"), (72, 43, 1400, 2600, "quad"),
    (72, 42, 1400, 2600, "oct"), (128, 42, 1400, 2600, "oct"),  # 252 tiles of 256 rows: one round
    (128, 43, 1400, 2600, "quad"),                              # 258: two
    (128, 43, 1300, 2600, "quad"), (128, 64, 510, 200, "quad"), (128, 64, 510, 300, "wide"), (128, 65, 510, 300, "quad"),
    (128, 64, 256, 300, "strip"), (128, 65, 256, 300, "wide")])
def test_picked(d, H, nq, nk, shape):
    """The library's own choice: 32- or 64-row tiles up to one workgroup per
    CU, 8 waves of 64 or 128 rows up to there, then 192-row and 256-row tiles
    where they take fewer rounds than the 128-row ones of 4 waves."""
    torch, orc = torch_mod(), oracle.get()
    print(f"[picked] d={d} H={H} {nq} x {nk}", flush=True)
    rows = sample_rows(nq, 97, [127, 128, 191, 192, 255, 256])
    _chunk(torch, orc, 1, H, d, nq, nk, f"d={d} H={H} {nq} x {nk}", rows, shape)


@pytest.mark.parametrize("form,H,nq,nk,splits,shape", [
    # 64-row tiles fit the CUs
    ("chunk", 24, 17, 1, 1, "quad"), ("chunk", 24, 17, 160, 1, "quad"), ("chunk", 24, 17, 161, 1, "strip"),
    ("chunk", 24, 64, 96, 1, "quad"), ("chunk", 24, 64, 97, 1, "strip"), ("chunk", 24, 100, 64, 1, "strip"),
    ("ring", 24, 128, 32, 1, "quad"), ("ring", 24, 128, 33, 1, "strip"), ("ring", 24, 64, 160, 1, "quad"),
    ("patch", 24, 64, 96, 1, "quad"), ("patch", 24, 64, 97, 1, "strip"), ("patch", 24, 128, 32, 1, "strip"),
    # they do not, 128-row tiles do
    ("chunk", 24, 1000, 160, 1, "quad"), ("chunk", 24, 1000, 192, 1, "wide"), ("chunk", 24, 1000, 224, 1, "quad"),
    ("chunk", 24, 1000, 225, 1, "wide"), ("ring", 24, 1000, 192, 1, "wide"), ("patch", 24, 1000, 192, 1, "quad"),
    ("patch", 24, 1000, 225, 1, "wide"),
    # one tile per head
    ("chunk", 192, 65, 512, 1, "quad"), ("chunk", 192, 65, 513, 1, "wide"), ("chunk", 191, 65, 512, 1, "wide"),
    ("chunk", 225, 65, 700, 1, "quad"),
    # split calls
    ("chunk", 24, 100, 448, 2, "quad"), ("chunk", 24, 100, 514, 2, "wide"), ("chunk", 15, 128, 528, 16, "wide"),
    ("chunk", 3, 78, 228, 6, "quad"), ("chunk", 24, 64, 6144, 10, "quad"), ("chunk", 12, 43, 6164, 16, "quad"),
    ("ring", 12, 43, 8500, 16, "wide"), ("patch", 24, 100, 384, 2, "quad")])
def test_short_sweeps_at_128(form, H, nq, nk, splits, shape):
    """Head dim 128, no more workgroups than CUs: 4-wave workgroups where the
    8-wave ones' merge, or the reads of K/V, cost more than they gain."""
    torch, orc, d = torch_mod(), oracle.get(), 128
    print(f"[short] {form} H={H} {nq} x {nk} in {splits}", flush=True)
    q, k, v = (random_io((1, n, H, d), "bf16", 70 + n + i) for i, n in enumerate((nq, nk, nk)))
    qg, kg, vg = (to_gpu(x, "bf16") for x in (q, k, v))
    out = torch.full_like(qg, float("nan"))
    lse = torch.full((1, H, nq), float("-inf"), device="cuda")  # ring: an empty state
    ws = torch.empty(xd.split_workspace_bytes(qg, nk, splits), device="cuda", dtype=torch.uint8) if splits > 1 else None
    if form == "patch":
        a, n = nk // 3, nk // 2
        kv = torch.stack([kg, vg])
        fresh = kv[:, :, a:a + n].clone()
        kv[:, :, a:a + n] = 0
        f = lambda: xd.xdit_patch_attn_split(qg, kv, [(a, n)], fresh[0], fresh[1], out, lse, splits, ws)
    else:
        g = xd.xdit_chunk_attn_accum_split if form == "ring" else xd.xdit_chunk_attn_split
        f = lambda: g(qg, kg, vg, out, lse, splits, ws)
    assert attention_kernels(f) == [bf16_kernel(shape, d, patch=form == "patch", parts=splits > 1)]
    if form == "patch":
        assert torch.equal(kv[0], kg) and torch.equal(kv[1], vg)
    rows, heads = sample_rows(nq, 23, [0, nq - 1]), slice(0, 2)
    ro, rl = orc.attention(q[:, rows, heads].copy(), k[:, :, heads].copy(), v[:, :, heads].copy())
    check_out(to_np(out)[:, rows, heads], ro, "bf16", shape)
    check_lse(lse.cpu().numpy()[:, heads, rows], rl, "bf16", shape + " lse")
