"""Timing cases of the attention hot path: what a diffusion-transformer
serving program asks of one GPU, through the package's public entry points.

listed() names the fixed cases, draw() makes more over the same ranges,
prepare() builds a case's inputs on the GPU, run() is one pass, work() the
bytes and operations no implementation can do without, exact() the 64-bit
result and tolerance() what the data types allow.

A case's fields: op (see _PREPARE), dtype ("bf16" or "f32"), B, H, d (batch,
heads, head dim), and per op
  patch         N, off, len: rows [off, off + len) of an N-row K/V buffer are
                refreshed and their queries attend over all N rows; the
                N - n_img last rows are text, never stale
  patch_ranges  as patch, with the text rows [N - txt, N) refreshed too and
                their queries appended (in-context conditioning)
  patch_shard   as patch, with only nq query rows of the patch (hybrid
                sequence parallelism), keys split as the library chooses
  chunk         nq queries over nk keys, output and log-sum-exp; split: the
                key-split entry point with the library's choice
  ring          nq queries over `chunks` chunks that share nk keys, each
                merged into the running output
  merge         n partials of nq rows merged
  update        rows [off, off + len) of an N-row buffer refreshed
  stage         C: hidden size; QKV projections, the patch step, output
                projection

Inputs are iid normal, stale K/V differ from fresh ones by N(0, 0.05^2), as
paper_2411_01738_amd.inputs draws them.
"""
from __future__ import annotations

import math

import torch

import paper_2411_01738_amd as xd


def listed():
    return [
        # The smallest call: one patch of the tiny float32 model, all latency.
        dict(name="tiny_patch_f32", op="patch", dtype="f32", B=1, H=2, d=64, N=256, n_img=256, off=64, len=64),
        # A float32 caller's sequence-parallel chunk at Pixart's layer shape.
        dict(name="pixart_chunk_f32", op="chunk", dtype="f32", B=2, H=16, d=72, nq=1024, nk=1024, split=False),
        # K/V received from a peer stored into the SD3 layer's buffer.
        dict(name="sd3_update", op="update", dtype="bf16", B=2, H=24, d=64, N=4429, n_img=4096, off=1536, len=512),
        # Pixart's four sequence-parallel partials merged.
        dict(name="pixart_merge", op="merge", dtype="bf16", B=2, H=16, d=72, nq=1024, n=4),
        # CogVideoX's eight partials merged: the largest merge, 1 GB.
        dict(name="cog_merge", op="merge", dtype="bf16", B=1, H=48, d=64, nq=17776, n=8),
        # Pixart 1024px, one PipeFusion patch step of four (classifier-free-
        # guidance pair): the flagship call.
        dict(name="pixart_patch", op="patch", dtype="bf16", B=2, H=16, d=72, N=4096, n_img=4096, off=1024, len=1024),
        # One chunk of Pixart's sequence-parallel share: a short call.
        dict(name="pixart_chunk", op="chunk", dtype="bf16", B=2, H=16, d=72, nq=1024, nk=1024, split=False),
        # SD3's patch 0 with the 333 text rows travelling along: two fresh
        # ranges, ragged query and key counts.
        dict(name="sd3_text_patch", op="patch_ranges", dtype="bf16", B=2, H=24, d=64, N=4429, n_img=4096, off=0, len=512),
        # PipeFusion with two-way sequence parallelism: half a patch's
        # queries, too few query tiles to fill the GPU.
        dict(name="pixart_shard", op="patch_shard", dtype="bf16", B=2, H=16, d=72, N=4096, n_img=4096, off=2048, len=1024,
             nq=512),
        # CogVideoX, one patch step of sixteen: odd sizes, a long buffer.
        dict(name="cog_patch", op="patch", dtype="bf16", B=1, H=48, d=64, N=17776, n_img=17550, off=3291, len=1097),
        # Flux 2048px over four GPUs, ring form: one GPU's whole share of a
        # layer, the largest case.
        dict(name="flux_ring", op="ring", dtype="bf16", B=1, H=24, d=128, nq=4224, nk=16896, chunks=4),
        # A Pixart stage micro-step: projections around the patch step.
        dict(name="pixart_stage", op="stage", dtype="bf16", B=2, H=16, d=72, N=4096, n_img=4096, off=1024, len=1024, C=1152),
    ]


# (heads, head dim) of the models, whole and split over tensor-parallel ranks
_HEADS = [(16, 72), (8, 72), (24, 64), (12, 64), (48, 64), (6, 64), (24, 128), (12, 128), (3, 128)]
_MOST_FLOPS = {"bf16": 4e11, "f32": 9.6e9}


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges: patches and chunks from a
    few rows to the longest sequences, any offset, any remainder."""
    kind = rng.choice(["patch", "patch", "patch_ranges", "patch_shard", "chunk", "chunk", "chunk", "ring", "merge", "update",
                       "stage", "patch_f32", "chunk_f32"])
    op, f32 = kind.replace("_f32", ""), kind.endswith("_f32")
    H, d = rng.choice(_HEADS)
    B = rng.choice([1, 1, 2])
    c = dict(op=op, dtype="f32" if f32 else "bf16", B=B, H=H, d=d)
    most = _MOST_FLOPS[c["dtype"]]

    def queries(nk, lo=16, hi=18000):
        return max(1, min(_log(rng, lo, hi), int(most / (4.0 * B * H * d * nk))))

    if op == "merge":
        c["n"] = rng.randint(2, 12)
        c["nq"] = min(_log(rng, 64, 18000), int(9e8 / (2.0 * (c["n"] + 1) * B * H * d)))
    elif op in ("chunk", "ring"):
        nk = _log(rng, 64, 4000 if f32 else 18000)
        c["nk"], c["nq"] = nk, queries(nk)
        if op == "chunk":
            c["split"] = rng.random() < 0.5 and not f32
        else:
            c["chunks"] = rng.randint(2, 8)
    else:
        txt = rng.choice([0, 0, rng.randint(64, 512)])
        if op == "patch_ranges":
            txt = max(txt, rng.randint(64, 512))
        img = _log(rng, 256, 2500 if f32 else 17600)
        N = img + txt
        c["N"], c["n_img"] = N, img
        ln = min(img, queries(N, 16, 4500))
        if op == "update":
            ln = min(img, _log(rng, 16, 4500))
        if op == "stage":
            c["C"] = rng.choice([H * d, H * d, 64 * rng.randint(4, 48)])
            ln = min(ln, 2048)
        if op == "patch_shard":
            c["nq"] = max(1, ln // rng.choice([2, 2, 3, 4, 8]))
        c["len"] = ln
        c["off"] = rng.randint(0, img - ln)
    return c


# -- inputs -------------------------------------------------------------------
class _Draws:
    """Normal tensors on the GPU from one seed, in call order."""

    def __init__(self, case, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def f32(self, *shape, scale=1.0):
        return torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32) * scale

    def io(self, *shape, scale=1.0):
        return self.f32(*shape, scale=scale).to(self.dt)


def _empty(case, *shape):
    return torch.empty(shape, device="cuda", dtype=torch.bfloat16 if case["dtype"] == "bf16" else torch.float32)


def _lse(case, nq):
    return torch.empty((case["B"], case["H"], nq), device="cuda", dtype=torch.float32)


def _ranges(case):
    r = [(case["off"], case["len"])]
    if case["op"] == "patch_ranges":
        r.append((case["n_img"], case["N"] - case["n_img"]))
    return r


def _fresh_rows(x, ranges):
    return torch.cat([x[:, o:o + n] for o, n in ranges], dim=1).contiguous()


def _patch_inputs(case, seed):
    """Queries, fresh K/V and the buffer at the start of a diffusion step."""
    D = _Draws(case, seed)
    B, N, H, d = case["B"], case["N"], case["H"], case["d"]
    k, v = D.f32(B, N, H, d), D.f32(B, N, H, d)
    ranges = _ranges(case)
    s = dict(ranges=ranges, fk=_fresh_rows(k, ranges).to(D.dt), fv=_fresh_rows(v, ranges).to(D.dt))
    k[:, :case["n_img"]] += D.f32(B, case["n_img"], H, d, scale=0.05)
    v[:, :case["n_img"]] += D.f32(B, case["n_img"], H, d, scale=0.05)
    s["kv"] = torch.stack([k, v]).to(D.dt)
    s["q"] = D.io(B, case.get("nq", sum(n for _, n in ranges)), H, d)
    return s


def _prepare_patch(case, seed):
    s = _patch_inputs(case, seed)
    s["out"] = torch.empty_like(s["q"])
    return s


def _prepare_patch_ranges(case, seed):
    s = _prepare_patch(case, seed)
    s["lse"] = _lse(case, s["q"].shape[1])
    return s


def _workspace(q, nk):
    n = xd.split_workspace_bytes(q, nk)
    return torch.empty(n, device="cuda", dtype=torch.uint8) if n else None


def _prepare_patch_shard(case, seed):
    s = _prepare_patch(case, seed)
    s["ws"] = _workspace(s["q"], case["N"])
    return s


def _chunk_inputs(case, seed):
    D = _Draws(case, seed)
    B, H, d = case["B"], case["H"], case["d"]
    return dict(q=D.io(B, case["nq"], H, d), k=D.io(B, case["nk"], H, d), v=D.io(B, case["nk"], H, d))


def _prepare_chunk(case, seed):
    s = _chunk_inputs(case, seed)
    s["out"], s["lse"] = torch.empty_like(s["q"]), _lse(case, case["nq"])
    s["ws"] = _workspace(s["q"], case["nk"]) if case["split"] else None
    return s


def _cuts(case):
    n, parts = case["nk"], case["chunks"]
    e = [n * r // parts for r in range(parts + 1)]
    return list(zip(e[:-1], e[1:]))


def _prepare_ring(case, seed):
    s = _prepare_chunk({**case, "split": False}, seed)
    s["chunks"] = [(s["k"][:, a:b].contiguous(), s["v"][:, a:b].contiguous()) for a, b in _cuts(case)]
    del s["k"], s["v"]
    s["ws"] = max((_workspace(s["q"], k.shape[1]) for k, _ in s["chunks"]), key=lambda w: 0 if w is None else w.numel())
    return s


def _merge_inputs(case, seed):
    D = _Draws(case, seed)
    B, H, d, nq, n = case["B"], case["H"], case["d"], case["nq"], case["n"]
    return dict(outs=[D.io(B, nq, H, d, scale=0.1) for _ in range(n)], lses=[7.0 + D.f32(B, H, nq) for _ in range(n)])


def _prepare_merge(case, seed):
    s = _merge_inputs(case, seed)
    s["out"], s["lse"] = torch.empty_like(s["outs"][0]), torch.empty_like(s["lses"][0])
    return s


def _prepare_update(case, seed):
    s = _patch_inputs(case, seed)
    del s["q"]
    return s


def _stage_inputs(case, seed):
    D = _Draws(case, seed)
    B, N, H, d, L, C = case["B"], case["N"], case["H"], case["d"], case["len"], case["C"]
    return dict(kv=D.io(2, B, N, H, d), x=D.io(B, L, C), w=D.io(3, C, H * d, scale=1.0 / math.sqrt(C)),
                wo=D.io(H * d, C, scale=1.0 / math.sqrt(H * d)))


def _prepare_stage(case, seed):
    s = _stage_inputs(case, seed)
    B, H, d, L, C = case["B"], case["H"], case["d"], case["len"], case["C"]
    s.update(off=case["off"], qkv=_empty(case, 3, B, L, H, d), o=_empty(case, B, L, H, d), y=_empty(case, B, L, C))
    return s


_PREPARE = {"patch": _prepare_patch, "patch_ranges": _prepare_patch_ranges, "patch_shard": _prepare_patch_shard,
            "chunk": _prepare_chunk, "ring": _prepare_ring, "merge": _prepare_merge, "update": _prepare_update,
            "stage": _prepare_stage}


def prepare(case, seed):
    s = _PREPARE[case["op"]](case, seed)
    s["op"] = case["op"]
    return s


# -- one pass -----------------------------------------------------------------
def run(s):
    op = s["op"]
    if op == "patch":
        (off, ln), = s["ranges"]
        xd.xdit_patch_attn(s["q"], s["kv"], off, ln, s["fk"], s["fv"], s["out"])
        return s["out"], s["kv"]
    if op == "patch_ranges":
        xd.xdit_patch_attn_ranges(s["q"], s["kv"], s["ranges"], s["fk"], s["fv"], s["out"], s["lse"])
        return s["out"], s["kv"], s["lse"]
    if op == "patch_shard":
        xd.xdit_patch_attn_split(s["q"], s["kv"], s["ranges"], s["fk"], s["fv"], s["out"], None, 0, s["ws"])
        return s["out"], s["kv"]
    if op == "chunk":
        if s["ws"] is not None:
            xd.xdit_chunk_attn_split(s["q"], s["k"], s["v"], s["out"], s["lse"], 0, s["ws"])
        else:
            xd.xdit_chunk_attn(s["q"], s["k"], s["v"], s["out"], s["lse"])
        return s["out"], s["lse"]
    if op == "ring":
        step = xd.xdit_chunk_attn_split  # the first chunk starts the running state
        for k, v in s["chunks"]:
            step(s["q"], k, v, s["out"], s["lse"], 0, s["ws"])
            step = xd.xdit_chunk_attn_accum_split
        return s["out"], s["lse"]
    if op == "merge":
        xd.xdit_lse_merge(s["outs"], s["lses"], len(s["outs"]), s["out"], s["lse"])
        return s["out"], s["lse"]
    if op == "update":
        (off, ln), = s["ranges"]
        xd.xdit_kv_update(s["kv"], off, ln, s["fk"], s["fv"])
        return s["kv"]
    w, (q, k, v) = s["w"], s["qkv"]
    xd.xdit_stage_step(s["x"], w[0], w[1], w[2], s["wo"], s["kv"], s["off"], q, k, v, s["o"], s["y"])
    return s["qkv"], s["o"], s["y"], s["kv"]


# -- accounting ---------------------------------------------------------------
def work(case):
    """Each input read once, each output written once; attention is
    4 B H nq nk d operations, a projection 2 rows C H d."""
    op, B, H, d = case["op"], case["B"], case["H"], case["d"]
    es = 2 if case["dtype"] == "bf16" else 4
    row = B * H * d * es  # one sequence row over the batch and heads
    lse = 4 * B * H
    if op == "merge":
        return {"bytes": (case["n"] + 1) * case["nq"] * (row + lse), "flops": 2.0 * (case["n"] + 1) * B * case["nq"] * H * d}
    if op == "update":
        return {"bytes": 4 * case["len"] * row, "flops": 0}
    if op in ("chunk", "ring"):
        nq, nk = case["nq"], case["nk"]
        return {"bytes": 2 * (nq + nk) * row + nq * lse, "flops": 4.0 * B * H * nq * nk * d}
    fresh = sum(n for _, n in _ranges(case))
    nq = case.get("nq", fresh)
    flops = 4.0 * B * H * nq * case["N"] * d
    # queries and output; stale rows read; fresh rows read and written
    size = 2 * nq * row + 2 * (case["N"] - fresh) * row + 4 * fresh * row
    if op == "patch_ranges":
        size += nq * lse
    if op == "stage":
        L, C = case["len"], case["C"]
        flops += 4 * 2.0 * B * L * C * H * d
        # x and y, the weights, q/k/v/o written, the buffer
        size = 2 * B * L * C * es + 4 * C * H * d * es + 4 * L * row + 2 * (case["N"] - fresh) * row + 2 * fresh * row
    return {"bytes": size, "flops": flops}


def tolerance(case):
    if case["op"] == "update":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 1e-2, "max": 8e-2}


# -- the 64-bit result --------------------------------------------------------
def _attention64(q, k, v):
    """Output [B, nq, H, d] and log-sum-exp [B, H, nq] in 64 bits, one head
    and 2048 query rows at a time."""
    B, nq, H, d = q.shape
    out = torch.empty(q.shape, device=q.device, dtype=torch.float64)
    lse = torch.empty((B, H, nq), device=q.device, dtype=torch.float64)
    for b in range(B):
        for h in range(H):
            kt, vh = k[b, :, h].double().t().contiguous(), v[b, :, h].double()
            for i in range(0, nq, 2048):
                s = torch.matmul(q[b, i:i + 2048, h].double(), kt) / math.sqrt(d)
                lse[b, h, i:i + 2048] = torch.logsumexp(s, dim=1)
                out[b, i:i + 2048, h] = torch.matmul(torch.softmax(s, dim=1), vh)
    return out, lse


def _store(kv, ranges, fk, fv):
    """The 64-bit buffer with the fresh rows in place."""
    kv = kv.double()
    base = 0
    for o, n in ranges:
        kv[0, :, o:o + n] = fk[:, base:base + n].double()
        kv[1, :, o:o + n] = fv[:, base:base + n].double()
        base += n
    return kv


def exact(case, seed):
    op = case["op"]
    if op in ("chunk", "ring"):
        s = _chunk_inputs(case, seed)
        return _attention64(s["q"], s["k"], s["v"])
    if op == "merge":
        s = _merge_inputs(case, seed)
        L = torch.logsumexp(torch.stack([x.double() for x in s["lses"]]), dim=0)
        out = torch.zeros(s["outs"][0].shape, device=L.device, dtype=torch.float64)
        for o, l in zip(s["outs"], s["lses"]):
            out += torch.exp(l.double() - L).transpose(1, 2).unsqueeze(-1) * o.double()
        return out, L
    if op == "stage":
        s = _stage_inputs(case, seed)
        B, L, H, d = case["B"], case["len"], case["H"], case["d"]
        x = s["x"].double()
        qkv = torch.stack([torch.matmul(x, w.double()).view(B, L, H, d) for w in s["w"]])
        kv = _store(s["kv"], _ranges(case), qkv[1], qkv[2])
        o, _ = _attention64(qkv[0], kv[0], kv[1])
        return qkv, o, torch.matmul(o.reshape(B, L, H * d), s["wo"].double()), kv
    s = _patch_inputs(case, seed)
    kv = _store(s["kv"], s["ranges"], s["fk"], s["fv"])
    if op == "update":
        return kv
    out, lse = _attention64(s["q"], kv[0], kv[1])
    return (out, kv, lse) if op == "patch_ranges" else (out, kv)
