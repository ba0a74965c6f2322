"""float32 attention at each number of key splits the dispatch chooses (1, 2,
4 and 8 waves per query block, by the counts of queries and keys), ragged in
queries and keys: chunk with LSE, ring step, and a patch step whose two fresh
ranges straddle tile edges, against the fp64 oracle within the float32 bars
of gpu_util (2^-24 relative per product and sum, over a few thousand terms)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2411_01738_amd as xd
from paper_2411_01738_amd.inputs import random_io
from tests.gpu_util import check_lse, check_out, to_gpu, to_np, torch_mod

pytestmark = pytest.mark.gpu

# (queries, keys): one tile (1 split), two (2), five with a ragged end (4; at
# the last tile some waves have no keys), many (8)
SHAPES = [(33, 31), (129, 50), (70, 133), (40, 1505)]


@pytest.mark.parametrize("d", [64, 72, 128])
@pytest.mark.parametrize("nq,nk", SHAPES)
def test_f32_splits(nq, nk, d):
    torch = torch_mod()
    orc = oracle.get()
    B, H = 2, 3
    print(f"[f32] {nq} x {nk}, d = {d}", flush=True)
    q, k, v = (random_io((B, n, H, d), "f32", 9000 + n + d + i) for i, n in enumerate((nq, nk, nk)))
    qg, kg, vg = (to_gpu(x, "f32") for x in (q, k, v))
    out = torch.full((B, nq, H, d), float("nan"), device="cuda")
    lse = torch.full((B, H, nq), float("nan"), device="cuda")
    xd.xdit_chunk_attn(qg, kg, vg, out, lse)
    ro, rl = orc.attention(q, k, v)
    check_out(to_np(out), ro, "f32", "chunk")
    check_lse(lse.cpu().numpy(), rl, "f32", "chunk lse")
    # ring of two chunks, the cut inside a tile
    cut = nk // 2 + 1
    out.fill_(float("nan"))
    lse.fill_(float("-inf"))
    for a, b in ((0, cut), (cut, nk)):
        xd.xdit_chunk_attn_accum(qg, kg[:, a:b].contiguous(), vg[:, a:b].contiguous(), out, lse)
    check_out(to_np(out), ro, "f32", "ring")
    check_lse(lse.cpu().numpy(), rl, "f32", "ring lse")
    # patch step: ranges [1, 1 + n0) and [o1, nk), edges off the tiles'
    n0, o1 = nk // 3, nk - nk // 4
    ranges = [(1, n0), (o1, nk - o1)]
    F = sum(n for _, n in ranges)
    kv = np.ascontiguousarray(np.stack([k, v]))
    fk, fv = (random_io((B, F, H, d), "f32", 9500 + d + i) for i in range(2))
    kvg = to_gpu(kv, "f32")
    out.fill_(float("nan"))
    xd.xdit_patch_attn_ranges(qg, kvg, ranges, to_gpu(fk, "f32"), to_gpu(fv, "f32"), out, lse)
    base = 0
    for o, n in ranges:
        kv[0][:, o:o + n], kv[1][:, o:o + n] = fk[:, base:base + n], fv[:, base:base + n]
        base += n
    assert np.array_equal(to_np(kvg), kv)
    ro, rl = orc.attention(q, kv[0].copy(), kv[1].copy())
    check_out(to_np(out), ro, "f32", "patch")
    check_lse(lse.cpu().numpy(), rl, "f32", "patch lse")
