"""GPU parity of the HIP path against the fp64 oracle, element by element, at
sizes the oracle finishes in seconds that span several tiles and ragged
tails, plus the edge cases.  Every call goes through the C ABI."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2411_01738_amd as xd
from paper_2411_01738_amd.inputs import WORKLOADS, generate, random_io
from tests.gpu_util import TOL, check_lse, check_out, tdtype, to_gpu, to_np, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def orc():
    return oracle.get()


@pytest.fixture(scope="module")
def torch():
    return torch_mod()


@pytest.fixture(params=["auto", "wide", "narrow", "quad"])
def tile_shape(request, monkeypatch):
    """Workgroup shape of unsplit launches of the bf16 kernel: 128 query rows x
    2 key splits ("wide"), 64 x 4 ("narrow", head dims up to 72), 4 waves of
    128 rows ("quad"), or the library's own choice, which is also what
    "narrow" gives at d = 128."""
    if request.param == "auto":
        monkeypatch.delenv("XDIT_ATTN_TILE", raising=False)
    else:
        monkeypatch.setenv("XDIT_ATTN_TILE", request.param)
    return request.param


def _empty_out(torch, B, Nq, H, d, dtype):
    # NaN-filled so that rows the kernel fails to write are caught
    return torch.full((B, Nq, H, d), float("nan"), device="cuda", dtype=tdtype(dtype))


def _lse_buf(torch, B, H, Nq):
    return torch.full((B, H, Nq), float("nan"), device="cuda", dtype=torch.float32)


# ---------------------------------------------------------------------------
# chunk attention (O and LSE)
# ---------------------------------------------------------------------------
CHUNK_CASES = [
    # dtype, B, Nq, Nk, H, d
    ("bf16", 2, 200, 333, 3, 64),
    ("bf16", 1, 130, 257, 2, 72),
    ("bf16", 2, 129, 190, 2, 128),
    ("bf16", 1, 1, 1, 1, 64),
    ("bf16", 1, 5, 64, 1, 72),
    ("bf16", 1, 128, 128, 1, 128),
    # K/V tile counts 3..22, whole and ragged (tiles of 128 keys in the
    # 8-wave shapes at d <= 72, 64 in the 4-wave one at d = 64, 32 at
    # d = 128), so that every way the tile loop can end is taken
    ("bf16", 1, 40, 384, 1, 64),
    ("bf16", 1, 100, 512, 2, 64),
    ("bf16", 1, 70, 645, 2, 72),
    ("bf16", 2, 33, 896, 2, 72),
    ("bf16", 1, 64, 700, 1, 128),
    ("f32", 1, 256, 256, 2, 64),
    ("f32", 2, 70, 97, 3, 72),
    ("f32", 1, 65, 33, 2, 128),
]


@pytest.mark.parametrize("dtype,B,Nq,Nk,H,d", CHUNK_CASES)
def test_chunk_attn(orc, torch, tile_shape, dtype, B, Nq, Nk, H, d):
    seed = B * 1000003 + Nq * 101 + Nk * 7 + d
    q = random_io((B, Nq, H, d), dtype, seed)
    k = random_io((B, Nk, H, d), dtype, seed + 1)
    v = random_io((B, Nk, H, d), dtype, seed + 2)
    ref_o, ref_l = orc.attention(q, k, v)
    out = _empty_out(torch, B, Nq, H, d, dtype)
    lse = _lse_buf(torch, B, H, Nq)
    xd.xdit_chunk_attn(to_gpu(q, dtype), to_gpu(k, dtype), to_gpu(v, dtype), out, lse)
    torch.cuda.synchronize()
    check_out(to_np(out), ref_o, dtype, "chunk out")
    check_lse(to_np(lse), ref_l, dtype, "chunk lse")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 72, 128])
def test_chunk_empty_kv(torch, tile_shape, dtype, d):
    B, Nq, H = 1, 70, 2
    q = to_gpu(random_io((B, Nq, H, d), dtype, 5), dtype)
    e = torch.zeros((B, 0, H, d), device="cuda", dtype=tdtype(dtype))
    out = _empty_out(torch, B, Nq, H, d, dtype)
    lse = _lse_buf(torch, B, H, Nq)
    xd.xdit_chunk_attn(q, e, e, out, lse)
    torch.cuda.synchronize()
    assert torch.all(out == 0).item()
    assert torch.all(torch.isneginf(lse)).item()


def test_chunk_empty_q_is_noop(torch):
    q = torch.zeros((1, 0, 2, 64), device="cuda", dtype=torch.bfloat16)
    k = to_gpu(random_io((1, 10, 2, 64), "bf16", 3), "bf16")
    out = torch.zeros((1, 0, 2, 64), device="cuda", dtype=torch.bfloat16)
    xd.xdit_chunk_attn(q, k, k.clone(), out, None)
    torch.cuda.synchronize()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_chunk_of_more_workgroups_than_one_grid_holds(torch, dtype):
    """17.6 million (batch, head) pairs of one query: more than 2^32 threads
    in all.  With one key the output is V's row and the LSE the score."""
    B, H, d = 1100, 16000, 64
    r = lambda: torch.randn(B, 1, H, d, device="cuda").to(tdtype(dtype))
    q, k, v = r(), r(), r()
    out = torch.full_like(v, float("nan"))
    lse = _lse_buf(torch, B, H, 1)
    xd.xdit_chunk_attn(q, k, v, out, lse)
    assert torch.equal(out, v)
    ref = (q[:, 0].float() * k[:, 0].float()).sum(-1) / d ** 0.5
    err = ((lse[:, :, 0] - ref).abs() / ref.abs().clamp(min=1)).max().item()
    assert err <= TOL[dtype]["lse_rel"]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_patch_of_more_workgroups_than_one_grid_holds(torch, dtype):
    """The same for a patch step: every batch's fresh rows, buffer and output
    are found in each of the launches (524 batches in the first)."""
    B, H, d = 1100, 16000, 64
    r = lambda *s: torch.randn(*s, device="cuda", dtype=torch.float32).to(tdtype(dtype))
    q, fk, fv = r(B, 1, H, d), r(B, 1, H, d), r(B, 1, H, d)
    kv = r(2, B, 2, H, d)
    old = kv[:, :, 0].clone()
    out = torch.full_like(q, float("nan"))
    xd.xdit_patch_attn(q, kv, 1, 1, fk, fv, out)
    assert torch.equal(kv[:, :, 0], old)
    assert torch.equal(kv[0, :, 1:], fk) and torch.equal(kv[1, :, 1:], fv)
    assert not out.isnan().any()
    for b in (0, 523, 524, 1047, 1048, 1099):
        k, v = kv[0, b].double(), kv[1, b].double()
        w = torch.softmax((q[b].double() * k).sum(-1) / d ** 0.5, dim=0)
        # two keys, |v| up to 5.5: the rounding of the weights and of the
        # output, 2^-9 each in bf16, comes to 2 * 2^-9 * 5.5 = 2.2e-2 at most
        check_out(to_np(out[b, 0]), (w[..., None] * v).sum(0).cpu().numpy(), dtype, f"batch {b}", scale=1.5)


@pytest.mark.parametrize("d", [64, 72, 128])
def test_constant_values_give_constant_output(torch, d):
    """Softmax rows sum to one: V rows all equal c gives O = c (up to the bf16
    rounding of c itself, which is exact here)."""
    B, Nq, Nk, H = 1, 150, 300, 2
    q = to_gpu(random_io((B, Nq, H, d), "bf16", 8), "bf16")
    k = to_gpu(random_io((B, Nk, H, d), "bf16", 9), "bf16")
    crow = random_io((B, 1, H, d), "bf16", 10)
    v = to_gpu(np.broadcast_to(crow, (B, Nk, H, d)).copy(), "bf16")
    out = _empty_out(torch, B, Nq, H, d, "bf16")
    xd.xdit_chunk_attn(q, k, v, out, None)
    torch.cuda.synchronize()
    c = np.broadcast_to(crow, (B, Nq, H, d))
    err = np.abs(to_np(out) - c)
    # O = c * sum(bf16(p)) / sum(p), then rounded to bf16: two relative
    # roundings of at most 2^-9 each
    assert np.all(err <= 2 * 2.0 ** -9 * np.abs(c) * 1.01 + 1e-7), err.max()


def _extreme_inputs(kind: str, dtype: str, B: int, Nq: int, Nk: int, H: int, d: int, seed: int):
    """Score distributions that drive the online softmax's reference max:
    "peaked": q, k ~ N(0, 6^2), scores spread over hundreds of log2 units, so
      nearly one-hot rows and rescales in the first tiles;
    "rising": every query along one direction u and key j = (j / Nk) 30 u +
      noise, so each row's max grows along the whole sweep (a rescale in
      most tiles, early weights underflowing to zero);
    "negative": keys pointing against the queries, every score near -300
      (nats), so the reference sits far below zero throughout."""
    from paper_2411_01738_amd.inputs import to_io

    rng = np.random.Generator(np.random.PCG64(seed))
    v = random_io((B, Nk, H, d), dtype, seed + 1)
    if kind == "peaked":
        return random_io((B, Nq, H, d), dtype, seed + 2, 6.0), random_io((B, Nk, H, d), dtype, seed + 3, 6.0), v
    u = rng.standard_normal((1, 1, H, d)).astype(np.float32)
    u /= np.linalg.norm(u, axis=-1, keepdims=True)
    q = u * np.float32(3.0 * np.sqrt(d)) + 0.3 * rng.standard_normal((B, Nq, H, d)).astype(np.float32)
    noise = 0.3 * rng.standard_normal((B, Nk, H, d)).astype(np.float32)
    if kind == "rising":
        k = (np.arange(Nk, dtype=np.float32) / Nk * 30.0)[None, :, None, None] * u + noise
    else:
        k = -100.0 * u + noise
    return to_io(q, dtype), to_io(k.astype(np.float32), dtype), v


def _f32_row_bars(q, k, v) -> np.ndarray:
    """Float32 I/O, per output row [B, Nq, H]: the max-abs bar widened by the
    float32 rounding of the row's scores.  A score s_ij computed as a float32
    dot product of length d carries an error of about sqrt(d) |s_ij| 2^-24
    (rounding errors of the partial sums, which grow to |s_ij| sqrt(d) in raw
    units, add up like a random walk); a score error moves the output by
    sum_j p_ij ds_ij (v_j - o_i), so row i moves by at most
      E_i = sqrt(d) 2^-24 max_j |s_ij| * max_c sum_j p_ij |v_jc - o_ic|,
    with p and o the exact softmax weights and output.  The bar is
    max(1e-5, E_i): E_i takes the random-walk estimate at the row's largest
    score, which overestimates it for the keys that carry the weight; a
    sequential float32 evaluation without fused multiply-adds (more rounding
    than the kernel's) reaches at most 0.9 E_i on the peaked and rising
    inputs.  Where every score of a row shares most of its rounding (the
    "negative" inputs, all scores near -300), the common part cancels in the
    softmax and the bar is loose."""
    d = q.shape[-1]
    q64, k64, v64 = (np.asarray(x, np.float64) for x in (q, k, v))
    s = np.einsum("bihc,bjhc->bhij", q64, k64) / np.sqrt(d)
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    o = np.einsum("bhij,bjhc->bhic", p, v64)
    vj = v64.transpose(0, 2, 1, 3)  # b, h, j, c
    spread = np.stack([np.einsum("hij,hijc->hic", p[b], np.abs(vj[b][:, None] - o[b][:, :, None]))
                       for b in range(p.shape[0])]).max(-1)  # b, h, i
    E = np.sqrt(d) * 2.0 ** -24 * np.abs(s).max(-1) * spread
    return np.maximum(1e-5, E).transpose(0, 2, 1)


@pytest.mark.parametrize("kind", ["peaked", "rising", "negative"])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 72), ("bf16", 128), ("f32", 72)])
def test_chunk_softmax_extremes(orc, torch, tile_shape, kind, dtype, d):
    """Online softmax against the oracle where scores are far from N(0, 1):
    the reference max is raised often, late, or sits far below zero."""
    B, Nq, Nk, H = 1, 140, 1100, 2
    q, k, v = _extreme_inputs(kind, dtype, B, Nq, Nk, H, d, 500 + d)
    ref_o, ref_l = orc.attention(q, k, v)
    out = _empty_out(torch, B, Nq, H, d, dtype)
    lse = _lse_buf(torch, B, H, Nq)
    xd.xdit_chunk_attn(to_gpu(q, dtype), to_gpu(k, dtype), to_gpu(v, dtype), out, lse)
    torch.cuda.synchronize()
    if dtype == "f32":
        err = np.abs(to_np(out).astype(np.float64) - ref_o).max(-1)  # b, i, h
        bars = _f32_row_bars(q, k, v)
        assert np.all(np.isfinite(err)), f"{kind}: non-finite GPU output"
        worst = float((err / bars).max())
        print(f"{kind} d={d}: max err {err.max():.3e}, worst err/bar {worst:.3f}")
        assert worst <= 1.0, f"{kind} out: a row exceeds its float32 bar (worst err/bar {worst:.3f})"
    else:
        check_out(to_np(out), ref_o, dtype, f"{kind} out")
    check_lse(to_np(lse), ref_l, dtype, f"{kind} lse")


@pytest.mark.parametrize("kind", ["peaked", "rising"])
def test_patch_softmax_extremes(orc, torch, kind):
    """The patch step on the same distributions (fresh rows in the middle of
    the sweep, buffer rows around them)."""
    B, N, H, d, off, ln = 1, 1100, 2, 72, 400, 300
    q_all, k, v = _extreme_inputs(kind, "bf16", B, N, N, H, d, 900)
    stale_k = random_io((B, N, H, d), "bf16", 901)
    stale_v = random_io((B, N, H, d), "bf16", 902)
    kv = np.ascontiguousarray(np.stack([stale_k, stale_v]))
    kv[0][:, :off] = k[:, :off]
    kv[0][:, off + ln:] = k[:, off + ln:]
    kv[1][:, :off] = v[:, :off]
    kv[1][:, off + ln:] = v[:, off + ln:]
    q = q_all[:, off:off + ln].copy()
    fk, fv = k[:, off:off + ln].copy(), v[:, off:off + ln].copy()
    ref_o, _ = orc.patch(q, kv.copy(), off, fk, fv)
    kv_g = to_gpu(kv, "bf16")
    out = _empty_out(torch, B, ln, H, d, "bf16")
    xd.xdit_patch_attn(to_gpu(q, "bf16"), kv_g, off, ln, to_gpu(fk, "bf16"), to_gpu(fv, "bf16"), out)
    torch.cuda.synchronize()
    check_out(to_np(out), ref_o, "bf16", f"{kind} patch out")
    assert np.array_equal(to_np(kv_g), np.concatenate([k[None], v[None]]).astype(np.float32)), \
        "buffer after the step differs from the fresh K/V"


# ---------------------------------------------------------------------------
# LSE merge
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 72), ("bf16", 128), ("f32", 64),
                                     ("f32", 128)])
def test_chunks_then_merge_equal_full(orc, torch, tile_shape, dtype, d):
    B, Nq, Nk, H = 2, 150, 500, 2
    q = random_io((B, Nq, H, d), dtype, 20 + d)
    k = random_io((B, Nk, H, d), dtype, 21 + d)
    v = random_io((B, Nk, H, d), dtype, 22 + d)
    ref_o, ref_l = orc.attention(q, k, v)
    bounds = [(0, 64), (64, 64), (64, 200), (200, 201), (201, 500)]  # uneven, with an empty chunk
    qg = to_gpu(q, dtype)
    outs, lses = [], []
    for s, e in bounds:
        o = _empty_out(torch, B, Nq, H, d, dtype)
        l = _lse_buf(torch, B, H, Nq)
        xd.xdit_chunk_attn(qg, to_gpu(k[:, s:e], dtype), to_gpu(v[:, s:e], dtype), o, l)
        outs.append(o)
        lses.append(l)
    out = _empty_out(torch, B, Nq, H, d, dtype)
    lse = _lse_buf(torch, B, H, Nq)
    xd.xdit_lse_merge(outs, lses, len(outs), out, lse)
    torch.cuda.synchronize()
    check_out(to_np(out), ref_o, dtype, "merged out vs full")
    check_lse(to_np(lse), ref_l, dtype, "merged lse vs full")
    # merge alone: the oracle merges the GPU's own partials
    mo, ml = orc.merge([to_np(o) for o in outs], [to_np(l) for l in lses])
    check_out(to_np(out), mo, dtype, "merge vs oracle merge")
    check_lse(to_np(lse), ml, dtype, "merge lse vs oracle merge")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 8, 9, 17, 64])
def test_merge_many_partials(orc, torch, dtype, n):
    """Every partial count the library compiles a form for (2, 3, 4, 6, 8),
    counts that take the general form (5; above one group of in-flight loads,
    9 and 17; the most one call accepts, 64); a third of the partials empty."""
    B, Nq, H, d = 1, 45, 3, 72
    outs, lses, outs_np, lses_np = [], [], [], []
    for r in range(n):
        o = random_io((B, Nq, H, d), dtype, 600 + r)
        l = (random_io((B, H, Nq), "f32", 700 + r) * 3).astype(np.float32)
        if r % 3 == 1:
            l[:] = -np.inf
        outs_np.append(o)
        lses_np.append(l)
        outs.append(to_gpu(o, dtype))
        lses.append(torch.from_numpy(l).cuda())
    out = _empty_out(torch, B, Nq, H, d, dtype)
    lse = _lse_buf(torch, B, H, Nq)
    xd.xdit_lse_merge(outs, lses, n, out, lse)
    torch.cuda.synchronize()
    mo, ml = orc.merge(outs_np, lses_np)
    check_out(to_np(out), mo, dtype, f"merge of {n}")
    check_lse(to_np(lse), ml, dtype, f"merge lse of {n}")


def test_merge_single_partial_is_copy(torch):
    B, Nq, H, d = 1, 77, 3, 72
    o = to_gpu(random_io((B, Nq, H, d), "bf16", 30), "bf16")
    l = torch.from_numpy(random_io((B, H, Nq), "f32", 31)).cuda()
    out = _empty_out(torch, B, Nq, H, d, "bf16")
    lse = _lse_buf(torch, B, H, Nq)
    xd.xdit_lse_merge([o], [l], 1, out, lse)
    torch.cuda.synchronize()
    assert torch.equal(out, o)
    assert torch.equal(lse, l)


def test_merge_in_place_and_all_empty(torch):
    B, Nq, H, d = 1, 40, 2, 64
    parts = [to_gpu(random_io((B, Nq, H, d), "bf16", 40 + r), "bf16") for r in range(3)]
    ninf = [torch.full((B, H, Nq), float("-inf"), device="cuda") for _ in range(3)]
    out = _empty_out(torch, B, Nq, H, d, "bf16")
    lse = _lse_buf(torch, B, H, Nq)
    xd.xdit_lse_merge(parts, ninf, 3, out, lse)
    torch.cuda.synchronize()
    assert torch.all(out == 0).item() and torch.all(torch.isneginf(lse)).item()
    # in place into partial 0, partial 1 empty
    lses = [torch.zeros((B, H, Nq), device="cuda"), ninf[1], torch.zeros((B, H, Nq), device="cuda")]
    expect = ((parts[0].float() + parts[2].float()) / 2).to(torch.bfloat16)
    xd.xdit_lse_merge(parts, lses, 3, parts[0], None)
    torch.cuda.synchronize()
    assert torch.equal(parts[0], expect)


# ---------------------------------------------------------------------------
# PipeFusion patch step
# ---------------------------------------------------------------------------
PATCH_CASES = [
    # dtype, B, N, H, d, patches (offset, length) applied in order
    ("bf16", 2, 300, 2, 64, [(37, 150), (0, 37), (187, 113)]),
    ("bf16", 1, 257, 3, 72, [(0, 64), (64, 129), (193, 64)]),
    ("bf16", 1, 200, 2, 128, [(100, 100), (0, 100)]),
    ("f32", 1, 256, 2, 64, [(0, 64), (64, 64), (128, 64), (192, 64)]),
    ("f32", 2, 150, 2, 72, [(50, 33), (83, 67)]),
    ("f32", 1, 97, 2, 128, [(1, 95)]),
]


@pytest.mark.parametrize("dtype,B,N,H,d,patches", PATCH_CASES)
def test_patch_steps_sequential(orc, torch, tile_shape, dtype, B, N, H, d, patches):
    seed = 7000 + N + d
    q = random_io((B, N, H, d), dtype, seed)
    kf = random_io((B, N, H, d), dtype, seed + 1)
    vf = random_io((B, N, H, d), dtype, seed + 2)
    ks = random_io((B, N, H, d), dtype, seed + 3)
    vs = random_io((B, N, H, d), dtype, seed + 4)
    kv_ref = np.ascontiguousarray(np.stack([ks, vs]))
    kv = to_gpu(kv_ref, dtype)
    for off, ln in patches:
        sl = slice(off, off + ln)
        ref_o, _ = orc.patch(q[:, sl].copy(), kv_ref, off, kf[:, sl].copy(), vf[:, sl].copy())
        out = _empty_out(torch, B, ln, H, d, dtype)
        xd.xdit_patch_attn(to_gpu(q[:, sl], dtype), kv, off, ln, to_gpu(kf[:, sl], dtype),
                           to_gpu(vf[:, sl], dtype), out)
        torch.cuda.synchronize()
        check_out(to_np(out), ref_o, dtype, f"patch ({off},{ln}) out")
        assert np.array_equal(to_np(kv), kv_ref), f"patch ({off},{ln}): buffer not bit-exact"


def test_patch_reads_fresh_rows_not_the_buffer(orc, torch, tile_shape):
    """The own slice of the buffer holds NaN before the step: every workgroup
    must take those rows from the fresh K/V, never from the buffer."""
    B, N, H, d, off, ln = 1, 256, 2, 64, 64, 128
    q = random_io((B, ln, H, d), "bf16", 50)
    kf = random_io((B, ln, H, d), "bf16", 51)
    vf = random_io((B, ln, H, d), "bf16", 52)
    kv_ref = np.stack([random_io((B, N, H, d), "bf16", 53), random_io((B, N, H, d), "bf16", 54)])
    kv_ref = np.ascontiguousarray(kv_ref)
    poisoned = kv_ref.copy()
    poisoned[:, :, off:off + ln] = np.nan
    kv = to_gpu(poisoned, "bf16")
    ref_o, _ = orc.patch(q, kv_ref, off, kf, vf)
    out = _empty_out(torch, B, ln, H, d, "bf16")
    xd.xdit_patch_attn(to_gpu(q, "bf16"), kv, off, ln, to_gpu(kf, "bf16"), to_gpu(vf, "bf16"), out)
    torch.cuda.synchronize()
    check_out(to_np(out), ref_o, "bf16", "poisoned-slice patch out")
    assert np.array_equal(to_np(kv), kv_ref)


def test_patch_idempotent_and_empty(torch):
    B, N, H, d = 1, 192, 2, 72
    kv0 = np.ascontiguousarray(np.stack([random_io((B, N, H, d), "bf16", 60),
                                         random_io((B, N, H, d), "bf16", 61)]))
    kv = to_gpu(kv0, "bf16")
    q = to_gpu(random_io((B, 64, H, d), "bf16", 62), "bf16")
    fk = to_gpu(random_io((B, 64, H, d), "bf16", 63), "bf16")
    fv = to_gpu(random_io((B, 64, H, d), "bf16", 64), "bf16")
    o1 = _empty_out(torch, B, 64, H, d, "bf16")
    o2 = _empty_out(torch, B, 64, H, d, "bf16")
    xd.xdit_patch_attn(q, kv, 64, 64, fk, fv, o1)
    snap = kv.clone()
    xd.xdit_patch_attn(q, kv, 64, 64, fk, fv, o2)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(kv, snap)
    e = torch.zeros((B, 0, H, d), device="cuda", dtype=torch.bfloat16)
    xd.xdit_patch_attn(e, kv, N, 0, e, e, e)
    torch.cuda.synchronize()
    assert torch.equal(kv, snap)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_kv_update_exact(torch, dtype):
    B, N, H, d = 2, 333, 3, 72
    kv0 = np.ascontiguousarray(np.stack([random_io((B, N, H, d), dtype, 70),
                                         random_io((B, N, H, d), dtype, 71)]))
    kv = to_gpu(kv0, dtype)
    off, ln = 101, 77
    fk = random_io((B, ln, H, d), dtype, 72)
    fv = random_io((B, ln, H, d), dtype, 73)
    xd.xdit_kv_update(kv, off, ln, to_gpu(fk, dtype), to_gpu(fv, dtype))
    torch.cuda.synchronize()
    exp = kv0.copy()
    exp[0, :, off:off + ln] = fk
    exp[1, :, off:off + ln] = fv
    assert np.array_equal(to_np(kv), exp)


def test_patch_all_fresh_equals_chunk_attention(torch):
    """A patch step over an all-fresh buffer is plain attention of the patch's
    queries; the GPU's two entry points agree bit for bit."""
    w = WORKLOADS["tiny"]
    t = generate(w)
    kv = to_gpu(np.ascontiguousarray(np.stack([t.k_fresh, t.v_fresh])), "f32")
    k, v = to_gpu(t.k_fresh, "f32"), to_gpu(t.v_fresh, "f32")
    for off, ln in w.patches():
        q = to_gpu(t.q[:, off:off + ln], "f32")
        o1 = _empty_out(torch, w.B, ln, w.H, w.d, "f32")
        o2 = _empty_out(torch, w.B, ln, w.H, w.d, "f32")
        xd.xdit_patch_attn(q, kv, off, ln, k[:, off:off + ln].contiguous(),
                           v[:, off:off + ln].contiguous(), o1)
        xd.xdit_chunk_attn(q, k, v, o2, None)
        torch.cuda.synchronize()
        assert torch.equal(o1, o2)


# ---------------------------------------------------------------------------
# General patch step: several fresh ranges, queries of their own
# ---------------------------------------------------------------------------
RANGE_CASES = [
    # dtype, B, N, H, d, fresh ranges
    ("bf16", 2, 300, 2, 64, [(0, 80), (240, 60)]),     # patch 0 + the text rows after the image
    ("bf16", 1, 400, 2, 72, [(100, 60), (250, 50)]),   # both ranges straddle 128-row tiles
    ("bf16", 1, 333, 2, 128, [(0, 200), (300, 33)]),
    ("bf16", 1, 520, 2, 64, [(384, 136), (0, 256)]),   # range order differs from row order
    ("f32", 1, 200, 2, 64, [(10, 50), (150, 50)]),
    ("f32", 2, 150, 2, 72, [(0, 40), (120, 30)]),
    ("f32", 1, 97, 2, 128, [(0, 32), (64, 33)]),
]


def _range_rows(ranges):
    return np.concatenate([np.arange(o, o + n) for o, n in ranges]).astype(np.int64)


@pytest.mark.parametrize("dtype,B,N,H,d,ranges", RANGE_CASES)
def test_patch_ranges_in_context(orc, torch, tile_shape, dtype, B, N, H, d, ranges):
    """Patch 0 carrying the text rows: the queries are the rows of both
    ranges; then the remaining image patches run as single-range steps."""
    seed = 8000 + N + d
    q = random_io((B, N, H, d), dtype, seed)
    kf = random_io((B, N, H, d), dtype, seed + 1)
    vf = random_io((B, N, H, d), dtype, seed + 2)
    kv_ref = np.ascontiguousarray(np.stack([random_io((B, N, H, d), dtype, seed + 3),
                                            random_io((B, N, H, d), dtype, seed + 4)]))
    kv = to_gpu(kv_ref, dtype)
    rows = _range_rows(ranges)
    qs, fks, fvs = q[:, rows].copy(), kf[:, rows].copy(), vf[:, rows].copy()
    ref_o, ref_l = orc.patch_ranges(qs, kv_ref, ranges, fks, fvs)
    out = _empty_out(torch, B, len(rows), H, d, dtype)
    lse = torch.full((B, H, len(rows)), float("nan"), device="cuda", dtype=torch.float32)
    xd.xdit_patch_attn_ranges(to_gpu(qs, dtype), kv, ranges, to_gpu(fks, dtype),
                              to_gpu(fvs, dtype), out, lse)
    torch.cuda.synchronize()
    check_out(to_np(out), ref_o, dtype, f"ranges {ranges} out")
    check_lse(lse.cpu().numpy(), ref_l, dtype, f"ranges {ranges} lse")
    assert np.array_equal(to_np(kv), kv_ref), f"ranges {ranges}: buffer not bit-exact"
    # a later single-range step sees the fresh text rows
    off, ln = ranges[0][0] + ranges[0][1], 40
    if off + ln <= N and not any(o < off + ln and off < o + n for o, n in ranges):
        sl = slice(off, off + ln)
        ref_o2, _ = orc.patch(q[:, sl].copy(), kv_ref, off, kf[:, sl].copy(), vf[:, sl].copy())
        out2 = _empty_out(torch, B, ln, H, d, dtype)
        xd.xdit_patch_attn(to_gpu(q[:, sl], dtype), kv, off, ln, to_gpu(kf[:, sl], dtype),
                           to_gpu(vf[:, sl], dtype), out2)
        torch.cuda.synchronize()
        check_out(to_np(out2), ref_o2, dtype, "step after the in-context patch")
        assert np.array_equal(to_np(kv), kv_ref)


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 72), ("bf16", 128), ("f32", 72)])
def test_patch_ranges_sp_shards(orc, torch, tile_shape, dtype, d):
    """Hybrid SP x PipeFusion at one GPU's share: each of sp ranks stores the
    same gathered fresh K/V and attends with its own query shard; the buffers
    end identical and the shards' outputs assemble the unsharded step."""
    B, N, H, off, ln, sp = 1, 384, 2, 96, 192, 4
    seed = 9000 + d
    q = random_io((B, ln, H, d), dtype, seed)
    fk = random_io((B, ln, H, d), dtype, seed + 1)
    fv = random_io((B, ln, H, d), dtype, seed + 2)
    kv0 = np.ascontiguousarray(np.stack([random_io((B, N, H, d), dtype, seed + 3),
                                         random_io((B, N, H, d), dtype, seed + 4)]))
    kv_ref = kv0.copy()
    ref_o, ref_l = orc.patch_ranges(q, kv_ref, [(off, ln)], fk, fv)
    outs, lses, bufs = [], [], []
    for r in range(sp):
        sh = slice(r * ln // sp, (r + 1) * ln // sp)
        kv = to_gpu(kv0, dtype)
        n = sh.stop - sh.start
        out = _empty_out(torch, B, n, H, d, dtype)
        lse = torch.empty((B, H, n), device="cuda", dtype=torch.float32)
        xd.xdit_patch_attn_ranges(to_gpu(q[:, sh], dtype), kv, [(off, ln)], to_gpu(fk, dtype),
                                  to_gpu(fv, dtype), out, lse)
        torch.cuda.synchronize()
        outs.append(to_np(out))
        lses.append(lse.cpu().numpy())
        bufs.append(to_np(kv))
    for b in bufs:
        assert np.array_equal(b, kv_ref), "an SP rank's buffer differs"
    check_out(np.concatenate(outs, axis=1), ref_o, dtype, "sharded queries out")
    check_lse(np.concatenate(lses, axis=2), ref_l, dtype, "sharded queries lse")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_patch_ranges_update_only_and_no_fresh_rows(orc, torch, dtype):
    """q_len = 0 only stores the fresh rows; no fresh rows is plain attention
    over the buffer as it stands."""
    B, N, H, d = 2, 200, 2, 64
    kv0 = np.ascontiguousarray(np.stack([random_io((B, N, H, d), dtype, 95),
                                         random_io((B, N, H, d), dtype, 96)]))
    ranges = [(150, 50), (10, 30)]
    fk = random_io((B, 80, H, d), dtype, 97)
    fv = random_io((B, 80, H, d), dtype, 98)
    kv = to_gpu(kv0, dtype)
    e = torch.zeros((B, 0, H, d), device="cuda", dtype=tdtype(dtype))
    xd.xdit_patch_attn_ranges(e, kv, ranges, to_gpu(fk, dtype), to_gpu(fv, dtype), e)
    torch.cuda.synchronize()
    exp = kv0.copy()
    orc.patch_ranges(np.zeros((B, 0, H, d), np.float32), exp, ranges, fk, fv)
    assert np.array_equal(to_np(kv), exp)
    q = random_io((B, 70, H, d), dtype, 99)
    out = _empty_out(torch, B, 70, H, d, dtype)
    lse = torch.empty((B, H, 70), device="cuda", dtype=torch.float32)
    xd.xdit_patch_attn_ranges(to_gpu(q, dtype), kv, [], e, e, out, lse)
    torch.cuda.synchronize()
    ref_o, ref_l = orc.attention(q, exp[0], exp[1])
    check_out(to_np(out), ref_o, dtype, "no fresh rows out")
    check_lse(lse.cpu().numpy(), ref_l, dtype, "no fresh rows lse")
    assert np.array_equal(to_np(kv), exp)


def test_patch_ranges_single_equals_patch_attn(torch):
    """One range with the patch's own queries is xdit_patch_attn, bit for bit."""
    B, N, H, d, off, ln = 2, 300, 2, 72, 70, 150
    q = to_gpu(random_io((B, ln, H, d), "bf16", 41), "bf16")
    fk = to_gpu(random_io((B, ln, H, d), "bf16", 42), "bf16")
    fv = to_gpu(random_io((B, ln, H, d), "bf16", 43), "bf16")
    kv0 = np.ascontiguousarray(np.stack([random_io((B, N, H, d), "bf16", 44),
                                         random_io((B, N, H, d), "bf16", 45)]))
    kv1, kv2 = to_gpu(kv0, "bf16"), to_gpu(kv0, "bf16")
    o1 = _empty_out(torch, B, ln, H, d, "bf16")
    o2 = _empty_out(torch, B, ln, H, d, "bf16")
    xd.xdit_patch_attn(q, kv1, off, ln, fk, fv, o1)
    xd.xdit_patch_attn_ranges(q, kv2, [(off, ln)], fk, fv, o2)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(kv1, kv2)


# ---------------------------------------------------------------------------
# Ring step with the merge fused in
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 72), ("bf16", 128), ("f32", 64),
                                     ("f32", 128)])
def test_ring_accum_equals_full(orc, torch, tile_shape, dtype, d):
    """Chunks merged one by one into a running (out, lse) that starts empty
    (lse = -inf, out NaN) give attention over the whole sequence; an empty
    chunk leaves the running state bit for bit."""
    B, Nq, H, Nk = 2, 130, 2, 357
    chunks = [(0, 100), (100, 200), (200, 200), (200, 357)]
    q = random_io((B, Nq, H, d), dtype, 300 + d)
    k = random_io((B, Nk, H, d), dtype, 301 + d)
    v = random_io((B, Nk, H, d), dtype, 302 + d)
    qg = to_gpu(q, dtype)
    out = _empty_out(torch, B, Nq, H, d, dtype)
    lse = torch.full((B, H, Nq), float("-inf"), device="cuda", dtype=torch.float32)
    for s, e in chunks:
        before = (out.clone(), lse.clone())
        xd.xdit_chunk_attn_accum(qg, to_gpu(k[:, s:e], dtype), to_gpu(v[:, s:e], dtype), out, lse)
        torch.cuda.synchronize()
        if s == e:
            assert torch.equal(out, before[0]) and torch.equal(lse, before[1]), "empty chunk changed the state"
    ref_o, ref_l = orc.attention(q, k, v)
    check_out(to_np(out), ref_o, dtype, "ring accumulation out")
    check_lse(lse.cpu().numpy(), ref_l, dtype, "ring accumulation lse")


def test_ring_accum_continues_chunk_attn(orc, torch):
    """A ring may start from xdit_chunk_attn's output for its first chunk."""
    B, Nq, H, d = 1, 200, 3, 72
    q = random_io((B, Nq, H, d), "bf16", 310)
    k = random_io((B, 600, H, d), "bf16", 311)
    v = random_io((B, 600, H, d), "bf16", 312)
    qg = to_gpu(q, "bf16")
    out = _empty_out(torch, B, Nq, H, d, "bf16")
    lse = torch.empty((B, H, Nq), device="cuda", dtype=torch.float32)
    xd.xdit_chunk_attn(qg, to_gpu(k[:, :256], "bf16"), to_gpu(v[:, :256], "bf16"), out, lse)
    xd.xdit_chunk_attn_accum(qg, to_gpu(k[:, 256:], "bf16"), to_gpu(v[:, 256:], "bf16"), out, lse)
    torch.cuda.synchronize()
    ref_o, ref_l = orc.attention(q, k, v)
    check_out(to_np(out), ref_o, "bf16", "chunk then accum out")
    check_lse(lse.cpu().numpy(), ref_l, "bf16", "chunk then accum lse")


# ---------------------------------------------------------------------------
# Key-split forms
# ---------------------------------------------------------------------------
def _workspace(torch, nbytes):
    return torch.empty(max(nbytes, 1), device="cuda", dtype=torch.uint8)


@pytest.mark.parametrize("d,splits,Nk", [(64, 2, 1000), (72, 3, 777), (128, 4, 600), (64, 16, 700),
                                         (72, 0, 2000), (128, 0, 1300)])
def test_chunk_split(orc, torch, d, splits, Nk):
    """Split sweeps merged by log-sum-exp equal attention over all keys; 16
    splits over fewer tiles leave some parts empty."""
    B, Nq, H = 1, 200, 3
    q = random_io((B, Nq, H, d), "bf16", 400 + d)
    k = random_io((B, Nk, H, d), "bf16", 401 + d)
    v = random_io((B, Nk, H, d), "bf16", 402 + d)
    qg = to_gpu(q, "bf16")
    ws = _workspace(torch, xd.split_workspace_bytes(qg, Nk, splits))
    out = _empty_out(torch, B, Nq, H, d, "bf16")
    lse = torch.empty((B, H, Nq), device="cuda", dtype=torch.float32)
    xd.xdit_chunk_attn_split(qg, to_gpu(k, "bf16"), to_gpu(v, "bf16"), out, lse, splits, ws)
    torch.cuda.synchronize()
    ref_o, ref_l = orc.attention(q, k, v)
    check_out(to_np(out), ref_o, "bf16", f"split {splits} out")
    check_lse(lse.cpu().numpy(), ref_l, "bf16", f"split {splits} lse")


@pytest.mark.parametrize("splits", [2, 4, 0])
def test_patch_split(orc, torch, splits):
    """The key-split patch step stores the fresh rows once and equals the
    oracle's ranged step (in-context form: patch 0 plus the text rows)."""
    B, N, H, d = 2, 900, 2, 64
    ranges = [(0, 160), (800, 100)]
    q = random_io((B, N, H, d), "bf16", 410)
    kf = random_io((B, N, H, d), "bf16", 411)
    vf = random_io((B, N, H, d), "bf16", 412)
    kv_ref = np.ascontiguousarray(np.stack([random_io((B, N, H, d), "bf16", 413),
                                            random_io((B, N, H, d), "bf16", 414)]))
    kv = to_gpu(kv_ref, "bf16")
    rows = _range_rows(ranges)
    qs, fks, fvs = q[:, rows].copy(), kf[:, rows].copy(), vf[:, rows].copy()
    ref_o, ref_l = orc.patch_ranges(qs, kv_ref, ranges, fks, fvs)
    qg = to_gpu(qs, "bf16")
    ws = _workspace(torch, xd.split_workspace_bytes(qg, N, splits))
    out = _empty_out(torch, B, len(rows), H, d, "bf16")
    lse = torch.empty((B, H, len(rows)), device="cuda", dtype=torch.float32)
    xd.xdit_patch_attn_split(qg, kv, ranges, to_gpu(fks, "bf16"), to_gpu(fvs, "bf16"), out, lse,
                             splits, ws)
    torch.cuda.synchronize()
    check_out(to_np(out), ref_o, "bf16", f"patch split {splits} out")
    check_lse(lse.cpu().numpy(), ref_l, "bf16", f"patch split {splits} lse")
    assert np.array_equal(to_np(kv), kv_ref), "split patch: buffer not bit-exact"


# Balanced partition: the whole launch cut into one contiguous range of
# (query tile, K/V tile) units per CU (256 ranges), so ranges cross query
# tiles and a sweep is cut among several workgroups whose partials the fix-up
# merges.  Query-tile counts do not divide 256.
BALANCED_CASES = [
    # B, Nq, Nk, H, d
    (2, 640, 1600, 3, 64),    # 30 query tiles x 13 K/V tiles: ranges of 1-2 tiles
    (1, 500, 700, 9, 128),    # ragged last query tile; 11 tiles of 64 keys
    (2, 700, 1000, 3, 72),    # 36 query tiles x 8 tiles, ragged queries and keys
    (1, 1100, 3000, 4, 64),   # 36 query tiles x 24 tiles: ranges of 3-4 tiles
]


def _slot_bytes(d):
    return 128 * (d + 1) * 4


@pytest.mark.parametrize("B,Nq,Nk,H,d", BALANCED_CASES)
def test_chunk_balanced(orc, torch, monkeypatch, B, Nq, Nk, H, d):
    monkeypatch.setenv("XDIT_PARTITION", "balanced")
    seed = 430 + Nq + d
    q = random_io((B, Nq, H, d), "bf16", seed)
    k = random_io((B, Nk, H, d), "bf16", seed + 1)
    v = random_io((B, Nk, H, d), "bf16", seed + 2)
    qg = to_gpu(q, "bf16")
    need = xd.split_workspace_bytes(qg, Nk, 0)
    assert need == 2 * 256 * _slot_bytes(d), "the balanced partition was not taken"
    ws = _workspace(torch, need)
    out = _empty_out(torch, B, Nq, H, d, "bf16")
    lse = _lse_buf(torch, B, H, Nq)
    xd.xdit_chunk_attn_split(qg, to_gpu(k, "bf16"), to_gpu(v, "bf16"), out, lse, 0, ws)
    torch.cuda.synchronize()
    ref_o, ref_l = orc.attention(q, k, v)
    check_out(to_np(out), ref_o, "bf16", "balanced out")
    check_lse(lse.cpu().numpy(), ref_l, "bf16", "balanced lse")


def test_chunk_whole_rounds_then_cut(orc, torch, monkeypatch):
    """The library's own partition for 272 query tiles (one full round of
    256 CUs and 16 left over): the first 256 sweep whole, each of the 16
    left over is cut into 16 parts, one slot per part."""
    monkeypatch.delenv("XDIT_PARTITION", raising=False)
    B, Nq, Nk, H, d = 1, 2048, 4096, 17, 64
    q = random_io((B, Nq, H, d), "bf16", 450)
    k = random_io((B, Nk, H, d), "bf16", 451)
    v = random_io((B, Nk, H, d), "bf16", 452)
    qg = to_gpu(q, "bf16")
    need = xd.split_workspace_bytes(qg, Nk, 0)
    assert need == 16 * 16 * _slot_bytes(d), "the whole-rounds-then-cut partition was not taken"
    ws = _workspace(torch, need)
    out = _empty_out(torch, B, Nq, H, d, "bf16")
    lse = _lse_buf(torch, B, H, Nq)
    xd.xdit_chunk_attn_split(qg, to_gpu(k, "bf16"), to_gpu(v, "bf16"), out, lse, 0, ws)
    torch.cuda.synchronize()
    ref_o, ref_l = orc.attention(q, k, v)
    check_out(to_np(out), ref_o, "bf16", "whole + cut out")
    check_lse(lse.cpu().numpy(), ref_l, "bf16", "whole + cut lse")


def test_patch_balanced(orc, torch, monkeypatch):
    """Balanced partition of a ranged patch step: the workgroups' unit
    shares together store every fresh row once, bit for bit."""
    monkeypatch.setenv("XDIT_PARTITION", "balanced")
    B, N, H, d = 2, 1500, 3, 72
    ranges = [(0, 300), (1400, 100)]
    q = random_io((B, N, H, d), "bf16", 440)
    kf = random_io((B, N, H, d), "bf16", 441)
    vf = random_io((B, N, H, d), "bf16", 442)
    kv_ref = np.ascontiguousarray(np.stack([random_io((B, N, H, d), "bf16", 443),
                                            random_io((B, N, H, d), "bf16", 444)]))
    kv = to_gpu(kv_ref, "bf16")
    rows = _range_rows(ranges)
    qs, fks, fvs = q[:, rows].copy(), kf[:, rows].copy(), vf[:, rows].copy()
    ref_o, ref_l = orc.patch_ranges(qs, kv_ref, ranges, fks, fvs)
    qg = to_gpu(qs, "bf16")
    need = xd.split_workspace_bytes(qg, N, 0)
    assert need == 2 * 256 * _slot_bytes(d), "the balanced partition was not taken"
    ws = _workspace(torch, need)
    out = _empty_out(torch, B, len(rows), H, d, "bf16")
    lse = _lse_buf(torch, B, H, len(rows))
    xd.xdit_patch_attn_split(qg, kv, ranges, to_gpu(fks, "bf16"), to_gpu(fvs, "bf16"), out, lse, 0, ws)
    torch.cuda.synchronize()
    check_out(to_np(out), ref_o, "bf16", "balanced patch out")
    check_lse(lse.cpu().numpy(), ref_l, "bf16", "balanced patch lse")
    assert np.array_equal(to_np(kv), kv_ref), "balanced patch: buffer not bit-exact"


def test_split_float32_runs_unsplit(orc, torch):
    B, Nq, Nk, H, d = 1, 100, 500, 2, 64
    q = random_io((B, Nq, H, d), "f32", 420)
    k = random_io((B, Nk, H, d), "f32", 421)
    v = random_io((B, Nk, H, d), "f32", 422)
    out = _empty_out(torch, B, Nq, H, d, "f32")
    xd.xdit_chunk_attn_split(to_gpu(q, "f32"), to_gpu(k, "f32"), to_gpu(v, "f32"), out, None, 4, None)
    torch.cuda.synchronize()
    ref_o, _ = orc.attention(q, k, v)
    check_out(to_np(out), ref_o, "f32", "float32 split out")


@pytest.mark.parametrize("d,Nk", [(64, 0), (64, 1), (64, 100), (72, 128), (128, 0), (128, 64)])
@pytest.mark.parametrize("splits", [2, 16, 0])
def test_split_over_one_tile_runs_unsplit(orc, torch, d, Nk, splits):
    """A sweep of one K/V tile or none has nothing to cut: the split call
    needs no workspace and equals the oracle (O = 0, LSE = -inf for no keys)."""
    B, Nq, H = 1, 200, 3
    q = random_io((B, Nq, H, d), "bf16", 460 + d + Nk)
    k = random_io((B, Nk, H, d), "bf16", 461 + d + Nk)
    v = random_io((B, Nk, H, d), "bf16", 462 + d + Nk)
    qg = to_gpu(q, "bf16")
    assert xd.split_workspace_bytes(qg, Nk, splits) == 0
    out = _empty_out(torch, B, Nq, H, d, "bf16")
    lse = _lse_buf(torch, B, H, Nq)
    xd.xdit_chunk_attn_split(qg, to_gpu(k, "bf16"), to_gpu(v, "bf16"), out, lse, splits, None)
    torch.cuda.synchronize()
    ref_o, ref_l = orc.attention(q, k, v)
    check_out(to_np(out), ref_o, "bf16", f"split {splits} over {Nk} keys out")
    check_lse(lse.cpu().numpy(), ref_l, "bf16", f"split {splits} over {Nk} keys lse")


def test_chunk_balanced_one_range_per_query_tile(orc, torch, monkeypatch):
    """Balanced partition of exactly 256 query tiles: each of the 256 ranges
    is one whole sweep, written by its workgroup; no fix-up may touch it."""
    monkeypatch.setenv("XDIT_PARTITION", "balanced")
    B, Nq, Nk, H, d = 1, 2048, 700, 16, 64
    q = random_io((B, Nq, H, d), "bf16", 470)
    k = random_io((B, Nk, H, d), "bf16", 471)
    v = random_io((B, Nk, H, d), "bf16", 472)
    qg = to_gpu(q, "bf16")
    need = xd.split_workspace_bytes(qg, Nk, 0)
    assert need == 256 * _slot_bytes(d), "the balanced partition was not taken"
    # a workspace full of NaN: a fix-up reading a slot nobody wrote would show
    ws = torch.full((need // 4,), float("nan"), device="cuda", dtype=torch.float32)
    out = _empty_out(torch, B, Nq, H, d, "bf16")
    lse = _lse_buf(torch, B, H, Nq)
    xd.xdit_chunk_attn_split(qg, to_gpu(k, "bf16"), to_gpu(v, "bf16"), out, lse, 0, ws)
    torch.cuda.synchronize()
    ref_o, ref_l = orc.attention(q, k, v)
    check_out(to_np(out), ref_o, "bf16", "balanced, one range per tile out")
    check_lse(lse.cpu().numpy(), ref_l, "bf16", "balanced, one range per tile lse")


@pytest.mark.parametrize("d,splits", [(64, 2), (72, 3), (128, 4), (128, 16)])
def test_ring_accum_split_equals_full(orc, torch, d, splits):
    """The ring step's split form: every chunk's cut sweeps are merged by the
    fix-up into the running (out, lse), which starts empty (lse = -inf, out
    NaN); an empty chunk and a one-tile chunk (run unsplit) are in the ring."""
    B, Nq, H, Nk = 2, 200, 2, 1500
    chunks = [(0, 600), (600, 600), (600, 1440), (1440, 1500)]
    q = random_io((B, Nq, H, d), "bf16", 480 + d)
    k = random_io((B, Nk, H, d), "bf16", 481 + d)
    v = random_io((B, Nk, H, d), "bf16", 482 + d)
    qg = to_gpu(q, "bf16")
    ws = _workspace(torch, max(xd.split_workspace_bytes(qg, e - s, splits) for s, e in chunks))
    out = _empty_out(torch, B, Nq, H, d, "bf16")
    lse = torch.full((B, H, Nq), float("-inf"), device="cuda", dtype=torch.float32)
    for s, e in chunks:
        before = (out.clone(), lse.clone())
        xd.xdit_chunk_attn_accum_split(qg, to_gpu(k[:, s:e], "bf16"), to_gpu(v[:, s:e], "bf16"), out, lse,
                                       splits, ws)
        torch.cuda.synchronize()
        if s == e:
            assert torch.equal(out, before[0]) and torch.equal(lse, before[1]), "empty chunk changed the state"
    ref_o, ref_l = orc.attention(q, k, v)
    check_out(to_np(out), ref_o, "bf16", f"ring split {splits} out")
    check_lse(lse.cpu().numpy(), ref_l, "bf16", f"ring split {splits} lse")


def test_ring_accum_library_partition(orc, torch):
    """The ring step where the library cuts: 272 query tiles (a full round of
    256 CUs and 16 left over, each cut in 16 parts) over 4096-key chunks; the
    first chunk by the split chunk step, the others merged into it."""
    B, Nq, H, d = 1, 2048, 17, 64
    chunks = [(0, 4096), (4096, 8192), (8192, 8288)]
    Nk = chunks[-1][1]
    q = random_io((B, Nq, H, d), "bf16", 490)
    k = random_io((B, Nk, H, d), "bf16", 491)
    v = random_io((B, Nk, H, d), "bf16", 492)
    qg = to_gpu(q, "bf16")
    need = xd.split_workspace_bytes(qg, 4096, 0)
    assert need == 16 * 16 * _slot_bytes(d), "the whole-rounds-then-cut partition was not taken"
    ws = _workspace(torch, need)
    out = _empty_out(torch, B, Nq, H, d, "bf16")
    lse = _lse_buf(torch, B, H, Nq)
    for i, (s, e) in enumerate(chunks):
        f = xd.xdit_chunk_attn_split if i == 0 else xd.xdit_chunk_attn_accum_split
        f(qg, to_gpu(k[:, s:e], "bf16"), to_gpu(v[:, s:e], "bf16"), out, lse, 0, ws)
    torch.cuda.synchronize()
    ref_o, ref_l = orc.attention(q, k, v)
    check_out(to_np(out), ref_o, "bf16", "ring, library partition out")
    check_lse(lse.cpu().numpy(), ref_l, "bf16", "ring, library partition lse")
