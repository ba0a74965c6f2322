"""float32 attention at each number of key splits the dispatch chooses (1, 2,
4 and, at head dims 64 and 72, 8 waves per query block, by the counts of
queries and keys), ragged in queries and keys, the kernel that ran read from a
profile: chunk with LSE, ring step, and a patch step whose two fresh
ranges straddle tile edges, against the fp64 oracle within the float32 bars
of gpu_util (2^-24 relative per product and sum, over a few thousand terms)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2411_01738_amd as xd
from paper_2411_01738_amd.inputs import random_io
from tests.gpu_util import attention_kernels, check_lse, check_out, to_gpu, to_np, torch_mod

pytestmark = pytest.mark.gpu

# (queries, keys, splits of the chunk, splits of the ring's two): one tile;
# two; three; five with a ragged end (at the last tile some waves have no
# keys); many; so many that 8 splits are ahead, the last tile of the whole
# sweep with keys for one wave of eight, of the ring's with five
SHAPES = [(33, 31, 1, 1), (129, 50, 2, 1), (129, 90, 4, 2), (70, 133, 4, 4), (40, 1505, 4, 4), (40, 4885, 8, 8)]


def _kernel(d, splits, patch=False):
    """The name of the kernel of that many splits; 4 are the most at 128."""
    ks = min(splits, 4 if d == 128 else 8)
    return f"attn_f32_kernel<{d}, {max(1, 4 // ks)}, {ks}, {str(patch).lower()}>"


@pytest.mark.parametrize("d", [64, 72, 128])
@pytest.mark.parametrize("nq,nk,chunk,ring", SHAPES)
def test_f32_splits(nq, nk, chunk, ring, d):
    torch = torch_mod()
    orc = oracle.get()
    B, H = 2, 3
    print(f"[f32] {nq} x {nk}, d = {d}", flush=True)
    q, k, v = (random_io((B, n, H, d), "f32", 9000 + n + d + i) for i, n in enumerate((nq, nk, nk)))
    qg, kg, vg = (to_gpu(x, "f32") for x in (q, k, v))
    out = torch.full((B, nq, H, d), float("nan"), device="cuda")
    lse = torch.full((B, H, nq), float("nan"), device="cuda")
    assert attention_kernels(lambda: xd.xdit_chunk_attn(qg, kg, vg, out, lse)) == [_kernel(d, chunk)]
    ro, rl = orc.attention(q, k, v)
    check_out(to_np(out), ro, "f32", "chunk")
    check_lse(lse.cpu().numpy(), rl, "f32", "chunk lse")
    # ring of two chunks, the cut inside a tile
    cut = nk // 2 + 1
    out.fill_(float("nan"))
    lse.fill_(float("-inf"))
    for a, b in ((0, cut), (cut, nk)):
        ka, va = kg[:, a:b].contiguous(), vg[:, a:b].contiguous()
        assert attention_kernels(lambda: xd.xdit_chunk_attn_accum(qg, ka, va, out, lse)) == [_kernel(d, ring)]
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
    fkg, fvg = to_gpu(fk, "f32"), to_gpu(fv, "f32")
    names = attention_kernels(lambda: xd.xdit_patch_attn_ranges(qg, kvg, ranges, fkg, fvg, out, lse))
    assert names == [_kernel(d, chunk, patch=True)]
    base = 0
    for o, n in ranges:
        kv[0][:, o:o + n], kv[1][:, o:o + n] = fk[:, base:base + n], fv[:, base:base + n]
        base += n
    assert np.array_equal(to_np(kvg), kv)
    ro, rl = orc.attention(q, kv[0].copy(), kv[1].copy())
    check_out(to_np(out), ro, "f32", "patch")
    check_lse(lse.cpu().numpy(), rl, "f32", "patch lse")
