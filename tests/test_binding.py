"""The native call path takes only what the checks in Python would pass: a
call it does not take comes back as None, so that the Python path raises what
it always raised; on the GPU it takes the calls it should, and they give the
same bytes by both paths."""
from __future__ import annotations

import pytest

import paper_2411_01738_amd as xd
from paper_2411_01738_amd import XditError


def _binding():
    torch = pytest.importorskip("torch")
    nat = xd._load_native()
    assert nat, "paper_2411_01738_amd/_binding.so is not built"
    return torch, nat


class _Recorder:
    """The native module, with the names and results of its calls."""

    def __init__(self, nat):
        self.nat, self.results = nat, []

    def __getattr__(self, name):
        def call(*args):
            rc = getattr(self.nat, name)(*args)
            self.results.append((name, rc))
            return rc
        return call


def test_declines_host_tensors():
    torch, nat = _binding()
    q = torch.zeros(1, 4, 2, 64)
    kv = torch.zeros(2, 1, 8, 2, 64)
    lse = torch.zeros(1, 2, 4)
    assert nat.chunk(q, q, q, q, lse, False) is None
    assert nat.chunk(None, q, q, q, None, False) is None
    assert nat.chunk_split(q, q, q, q, lse, "2", None, False) is None
    assert nat.patch(q, kv, 0, 4, q, q, q) is None
    assert nat.patch_ranges(q, kv, [(0, 4)], q, q, q, None) is None
    assert nat.patch_split(q, kv, [(0, 4)], q, q, q, None, None, None) is None
    assert nat.merge([q], [lse], 1, q, None) is None
    assert nat.update(kv, 0, 4, q, q) is None
    with pytest.raises(TypeError):
        nat.chunk(q)
    with pytest.raises(XditError, match="must be a GPU tensor"):
        xd.xdit_chunk_attn(q, q, q, q, lse)


@pytest.mark.parametrize("binding", ["missing", "another interpreter's"])
def test_a_binding_that_does_not_load_is_named(monkeypatch, binding):
    """The calls still work, through ctypes, at several times the host time."""
    import sys

    pytest.importorskip("torch")
    if binding == "missing":
        monkeypatch.setitem(sys.modules, "paper_2411_01738_amd._binding", None)
        monkeypatch.delattr(xd, "_binding", raising=False)
    else:
        class Stale:
            def init(self, *a):
                raise ImportError("undefined symbol")
        monkeypatch.setattr(xd, "_binding", Stale(), raising=False)
    monkeypatch.setattr(xd, "_native", None)
    with pytest.warns(RuntimeWarning, match="paper_2411_01738_amd.build"):
        assert not xd._load_native()
    assert xd._native is False


class _GpuTensor:
    """A host tensor that calls itself a GPU tensor: the checks in Python take
    it, and no call may get past them to the library."""

    is_cuda = True

    def __init__(self, x):
        self._x = x

    def __getattr__(self, name):
        return getattr(self._x, name)


@pytest.fixture
def checks_only(monkeypatch):
    """The Python checks alone: no native path, and a library that is never
    to be reached.  Returns a maker of tensors."""
    torch = pytest.importorskip("torch")

    class Library:
        def __getattr__(self, name):
            def launched(*args):
                raise AssertionError(f"{name} was launched")
            return launched

    monkeypatch.setattr(xd, "_native", False)
    monkeypatch.setattr(xd, "lib", lambda: Library())
    monkeypatch.setattr(xd, "_use_current_stream", lambda: None)
    return lambda *s, dt=torch.bfloat16: _GpuTensor(torch.zeros(*s, dtype=dt))


@pytest.mark.parametrize("call", ["ranges", "split"])
def test_patch_forms_check_shapes_and_types(checks_only, call):
    """Sizes that the library cannot see (it takes pointers): a call that
    passes them on would read or write past the tensors."""
    import torch

    t, f32 = checks_only, torch.float32
    B, N, H, d, nq = 1, 8, 2, 64, 6
    f = xd.xdit_patch_attn_ranges if call == "ranges" else xd.xdit_patch_attn_split
    good = dict(q=t(B, nq, H, d), kv_buf=t(2, B, N, H, d), ranges=[(0, 3), (5, 2)], fresh_k=t(B, 5, H, d),
                fresh_v=t(B, 5, H, d), out=t(B, nq, H, d), lse=t(B, H, nq, dt=f32))
    with pytest.raises(AssertionError, match="was launched"):
        f(**good)
    for bad in (dict(out=t(B, nq - 1, H, d)), dict(out=t(B, nq, H, d, dt=f32)), dict(q=t(B, nq, H, 72)),
                dict(q=t(2, nq, H, d)), dict(q=t(B, nq, H, d, dt=f32)), dict(fresh_k=t(B, 4, H, d)),
                dict(fresh_v=t(B, 4, H, d)), dict(fresh_v=t(B, 5, H, d, dt=f32)), dict(kv_buf=t(2, B, N, H, d, dt=f32)),
                dict(lse=t(B, H, nq - 1, dt=f32)), dict(lse=t(B, H, nq)), dict(ranges=[(0, 4), (5, 2)]),
                dict(out=None), dict(fresh_k=None)):
        with pytest.raises(XditError):
            f(**{**good, **bad})
    with pytest.raises(AssertionError, match="was launched"):  # no fresh rows, none given
        f(**{**good, "ranges": [], "fresh_k": None, "fresh_v": None})


def test_merge_checks_the_merged_lse(checks_only):
    """A merged LSE that is short, of another type or of other sizes would be
    written past its end."""
    import torch

    t, f32 = checks_only, torch.float32
    B, Nq, H, d = 1, 6, 2, 64
    outs, lses = [t(B, Nq, H, d)] * 2, [t(B, H, Nq, dt=f32)] * 2
    for lse in (None, t(B, H, Nq, dt=f32)):
        with pytest.raises(AssertionError, match="was launched"):
            xd.xdit_lse_merge(outs, lses, 2, t(B, Nq, H, d), lse)
    for bad in (t(B, H, Nq - 1, dt=f32), t(B, 1, Nq, dt=f32), t(B, H, Nq)):
        with pytest.raises(XditError):
            xd.xdit_lse_merge(outs, lses, 2, t(B, Nq, H, d), bad)


def test_buffer_has_both_planes(checks_only):
    """V's plane starts where K's ends: a buffer of one plane has none."""
    t = checks_only
    B, N, H, d, n = 1, 8, 2, 64, 4
    x = t(B, n, H, d)
    calls = [lambda kv: xd.xdit_patch_attn(x, kv, 0, n, x, x, x), lambda kv: xd.xdit_kv_update(kv, 0, n, x, x),
             lambda kv: xd.xdit_patch_attn_ranges(x, kv, [(0, n)], x, x, x),
             lambda kv: xd.xdit_patch_attn_split(x, kv, [(0, n)], x, x, x),
             lambda kv: xd.xdit_stage_step(t(B, n, 64), *[t(64, H * d)] * 3, t(H * d, 64), kv, 0, x, x, x, x, t(B, n, 64))]
    for call in calls:
        with pytest.raises(AssertionError, match="was launched"):
            call(t(2, B, N, H, d))
        with pytest.raises(XditError):
            call(t(1, B, N, H, d))


@pytest.mark.gpu
def test_native_path_declines_a_buffer_of_one_plane():
    torch, nat = _binding()
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    B, N, H, d, n = 1, 8, 2, 64, 4
    z = lambda *s: torch.zeros(*s, device="cuda", dtype=torch.bfloat16)
    x, o = z(B, n, H, d), z(B, n, H, d)
    kv = z(2, B, N, H, d)[:1]  # the library would find the second plane's memory
    assert nat.patch(x, kv, 0, n, x, x, o) is None
    assert nat.patch_ranges(x, kv, [(0, n)], x, x, o, None) is None
    assert nat.patch_split(x, kv, [(0, n)], x, x, o, None, 1, None) is None
    assert nat.update(kv, 0, n, x, x) is None


@pytest.mark.gpu
def test_both_paths_agree(monkeypatch):
    torch, nat = _binding()
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    g = torch.Generator(device="cuda").manual_seed(3)
    r = lambda *s: torch.randn(*s, device="cuda", generator=g).to(torch.bfloat16)
    B, N, H, d, n = 2, 300, 2, 72, 70
    q, k, v, fk, fv = r(B, n, H, d), r(B, N, H, d), r(B, N, H, d), r(B, n, H, d), r(B, n, H, d)
    kv0 = r(2, B, N, H, d)

    def calls():
        out = []

        def new():
            out.append(torch.zeros_like(q))
            out.append(torch.full((B, H, n), float("-inf"), device="cuda"))
            return out[-2:]

        kv = kv0.clone()
        xd.xdit_chunk_attn(q, k, v, *new())
        xd.xdit_chunk_attn_accum(q, k, v, *new())
        ws = torch.empty(xd.split_workspace_bytes(q, N, 2), device="cuda", dtype=torch.uint8)
        xd.xdit_chunk_attn_split(q, k, v, *new(), 2, ws)
        xd.xdit_chunk_attn_accum_split(q, k, v, *new(), 2, ws)
        xd.xdit_patch_attn(q, kv, 5, n, fk, fv, new()[0])
        xd.xdit_patch_attn_ranges(q, kv, [(5, 30), (200, 40)], fk, fv, *new())
        xd.xdit_patch_attn_split(q, kv, ((5, 30), (200, 40)), fk, fv, *new(), 2, ws)
        xd.xdit_lse_merge([out[0], out[4]], [out[1], out[5]], 2, *new())
        xd.xdit_kv_update(kv, 100, n, fk, fv)
        # and on a stream of its own
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            xd.xdit_chunk_attn(q, k, v, *new())
        torch.cuda.current_stream().wait_stream(s)
        torch.cuda.synchronize()
        return out + [kv]

    rec = _Recorder(nat)
    monkeypatch.setattr(xd, "_native", rec)
    fast = calls()
    assert rec.results == [(name, 0) for name in ("chunk", "chunk", "chunk_split", "chunk_split", "patch", "patch_ranges",
                                                  "patch_split", "merge", "update", "chunk")]
    monkeypatch.setattr(xd, "_native", False)
    for a, b in zip(fast, calls()):
        assert torch.equal(a, b)


@pytest.mark.gpu
def test_rejections_are_the_same(monkeypatch):
    torch, nat = _binding()
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    z = lambda *s, dt=torch.bfloat16: torch.zeros(*s, device="cuda", dtype=dt)
    q, kv, lse = z(1, 4, 2, 64), z(2, 1, 8, 2, 64), z(1, 2, 4, dt=torch.float32)
    # the library's status where the native path passes the call on, None
    # where it leaves the refusal to the checks in Python
    bad = [(None, lambda: xd.xdit_chunk_attn(q, q, z(1, 5, 2, 64), z(1, 4, 2, 64))),
           (-6, lambda: xd.xdit_chunk_attn(q, q, q, q)),                                    # out aliases q
           (None, lambda: xd.xdit_chunk_attn(q.half(), q, q, q)),
           (None, lambda: xd.xdit_chunk_attn(q, q.transpose(1, 2), q, z(1, 4, 2, 64))),
           (None, lambda: xd.xdit_chunk_attn(q, q, q, z(1, 4, 2, 64), lse[:, :, :3])),
           (None, lambda: xd.xdit_chunk_attn_accum(q, q, q, z(1, 4, 2, 64), None)),
           (-4, lambda: xd.xdit_patch_attn(q, kv, 6, 4, q, q, z(1, 4, 2, 64))),             # past the buffer
           (-4, lambda: xd.xdit_patch_attn_ranges(q, kv, [(0, 2), (1, 2)], q, q, z(1, 4, 2, 64))),
           (None, lambda: xd.xdit_patch_attn_ranges(q, kv, [(0, 1), (2, 1), (4, 2)], q, q, z(1, 4, 2, 64))),
           (-4, lambda: xd.xdit_patch_attn_split(q, kv, [(0, 2), (1, 2)], q, q, z(1, 4, 2, 64))),
           (None, lambda: xd.xdit_patch_attn_split(q, kv, [(0, 2)], q, q, z(1, 4, 2, 64))),
           (None, lambda: xd.xdit_patch_attn_split(q, kv, [(0, 4)], q, q, z(1, 3, 2, 64))),
           (None, lambda: xd.xdit_lse_merge([q], [lse], 2, z(1, 4, 2, 64))),
           (None, lambda: xd.xdit_lse_merge([q], [lse], 1, z(1, 4, 2, 64), z(1, 2, 3, dt=torch.float32))),
           (-4, lambda: xd.xdit_kv_update(kv, -1, 4, q, q)),
           (-4, lambda: xd.xdit_chunk_attn_split(q, kv[0], kv[1], z(1, 4, 2, 64), None, 17))]
    codes = []
    rec = _Recorder(nat)
    for native in (rec, False):
        monkeypatch.setattr(xd, "_native", native)
        for _, f in bad:
            with pytest.raises(XditError) as e:
                f()
            codes.append((e.value.code, str(e.value)))
    assert codes[:len(bad)] == codes[len(bad):]
    assert [rc for _, rc in rec.results] == [rc for rc, _ in bad]


@pytest.mark.gpu
def test_declines_one_bad_argument():
    """Arguments that would be taken but for one of another type, shape,
    layout or device.  No call here gets as far as the library."""
    torch, nat = _binding()
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    B, N, H, d, n = 1, 8, 2, 64, 4
    z = lambda *s, dt=torch.bfloat16: torch.zeros(*s, device="cuda", dtype=dt)
    f32 = torch.float32
    x, o, kv, ws = z(B, n, H, d), z(B, n, H, d), z(2, B, N, H, d), z(256, dt=torch.uint8)
    lse = z(B, H, n, dt=f32)
    tensors = [x.cpu(), x.float(), x[:, :3], z(B, n, 1, d), z(B, H, n, d).transpose(1, 2), x[0], None, "x"]
    lses = [lse.cpu(), lse.half(), lse[:, :, :3], z(B, n, H, dt=f32), "lse"]
    forms = {  # entry: (arguments, {position: bad values})
        "chunk": ([x, x, x, o, lse, False], {0: tensors, 2: tensors, 3: tensors, 4: lses}),
        "chunk_split": ([x, x, x, o, lse, 2, ws, False], {1: tensors[4:] + tensors[:2], 4: lses, 5: ["2", None, 2.0, 1 << 40],
                                                          6: [ws.cpu(), "ws"]}),
        "patch": ([x, kv, 0, n, x, x, o], {0: tensors, 1: [kv[:1], kv[0], kv.float(), None], 2: [None, 0.0], 3: [3, 4.0],
                                           5: tensors, 6: tensors}),
        "patch_ranges": ([x, kv, [(0, 1), (3, 3)], x, x, o, lse],
                         {0: tensors, 1: [kv[:1]], 2: [None, [(0, 1)], [(0, 1), [3, 3]], [(0, 1.0), (3, 3)], [(0, 1)] * 3,
                                                       [(0, 1, 2), (3, 3)]], 3: tensors, 4: tensors, 5: tensors, 6: lses}),
        "patch_split": ([x, kv, ((0, 4),), x, x, o, lse, 2, ws], {0: tensors, 1: [kv[:1]], 2: [((0, 3),)], 3: tensors,
                                                                  5: tensors, 6: lses, 7: ["2", None], 8: [ws.cpu()]}),
        "merge": ([[x], [lse], 1, o, lse], {0: [[t] for t in tensors] + [[], (x,)], 1: [[t] for t in lses] + [[None]],
                                            2: [0, 2, 65, None], 3: tensors, 4: lses}),
        "update": ([kv, 0, n, x, x], {0: [kv[:1], kv.float()], 1: [None], 2: [3], 3: tensors, 4: tensors}),
    }
    for name, (args, bad) in forms.items():
        for i, values in bad.items():
            for v in values:
                what = tuple(v.shape) if isinstance(v, torch.Tensor) else v
                assert getattr(nat, name)(*args[:i], v, *args[i + 1:]) is None, f"{name} took argument {i} = {what}"
    # an LSE is needed to merge into
    assert nat.chunk(x, x, x, o, None, True) is None
    assert nat.chunk_split(x, x, x, o, None, 2, ws, True) is None
