"""The native marshalling of ssd.py: where anything is out of the ordinary it answers None and does nothing, so that the
Python path raises what there is to raise; where it takes a call, the results are those of the Python path, bit for bit."""
import ctypes
import os
import subprocess
import sys
import types

import pytest
import torch

from paper_2603_09555_amd import build, ssd

NAMES = ("prefill", "prefill_varlen", "decode_step", "decode_step_layers", "decode_steps_layers", "conv1d_prefill", "conv1d_step")
ARGS = {"prefill": 14, "prefill_varlen": 15, "decode_step": 8, "decode_step_layers": 11, "decode_steps_layers": 11,
        "conv1d_prefill": 6, "conv1d_step": 6}


@pytest.mark.parametrize("name", NAMES)
def test_anything_but_device_tensors_is_left_to_python(name):
    f = getattr(ssd._native, name)
    t = torch.zeros(2, 2, 2, 2)
    assert f() is None
    for arg in (None, 3, "x", t, torch.nn.Parameter(t)):
        assert f(*[arg] * ARGS[name]) is None


def test_errors_are_those_of_the_python_path():
    t = torch.zeros(1, 4, 2, 64)
    with pytest.raises(ValueError, match="x, B and C must share one dtype"):
        ssd.ssd_prefill(t, torch.zeros(1, 4, 2), torch.zeros(2), t.bfloat16(), t, torch.zeros(2), 64)
    with pytest.raises(ValueError, match="inconsistent tensor shapes"):
        ssd.ssd_decode_step(t, t, t, t, t, t, t)
    with pytest.raises(ValueError, match="split must be"):
        ssd.ssd_conv1d_step(torch.zeros(1, 8, 3), torch.zeros(1, 8), torch.zeros(8, 4), split=(4, 5))
    with pytest.raises(ValueError, match="contiguous device tensors"):
        ssd.ssd_prefill(t, torch.zeros(1, 4, 2), torch.zeros(2), t[:, :, :1], t[:, :, :1], torch.zeros(2), 64)


@pytest.mark.parametrize("how", ["missing", "another torch"])
def test_without_the_native_marshalling_everything_is_left_to_python(how):
    """It saves host time and is no more required than that: a box that cannot build it uses the library all the same."""
    plant = {"missing": "None", "another torch": "types.SimpleNamespace(torch_version='1.0')"}[how]
    code = """if True:
        import sys, types, warnings
        sys.modules['paper_2603_09555_amd._ssd_binding'] = %s
        with warnings.catch_warnings(record=True) as w:
            warnings.simplefilter('always')
            from paper_2603_09555_amd import ssd
        assert any('_ssd_binding' in str(v.message) for v in w), w
        import torch
        t = torch.zeros(1, 4, 2, 64)
        try:
            ssd.ssd_prefill(t, torch.zeros(1, 4, 2), torch.zeros(2), t, t, torch.zeros(2), 64)
        except ValueError as e:
            assert 'contiguous device tensors' in str(e), e
        else:
            raise AssertionError('taken')
        """ % plant
    subprocess.run([sys.executable, "-c", code], check=True, cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), timeout=120)


def test_a_binding_of_another_torch_is_built_anew(monkeypatch):
    monkeypatch.setattr(os.path, "getmtime", lambda path: 0.0)   # (no file is newer than another)
    assert not build.needs_build()
    monkeypatch.setattr(build, "torch_version", lambda: "1.0")
    assert build.needs_build()


def _calls(io):
    """(name, arguments as the entry points take them) with given and missing outputs, options and optional tensors"""
    g = torch.Generator(device="cuda").manual_seed(5)
    n = lambda *s, dt=io, k=1.0: torch.randn(s, generator=g, device="cuda").mul_(k).to(dt)   # noqa: E731
    f = torch.float32
    pos = lambda *s: n(*s, dt=f).abs().mul_(0.05)   # noqa: E731
    raw = dict(dt_bias=n(2, dt=f), dt_softplus=True, dt_limit=(1e-3, 1e-1))
    raw_l = dict(raw, dt_bias=n(3, 2, dt=f))
    neg = lambda *s: n(*s, dt=f).abs().neg_()   # noqa: E731
    p = (n(1, 70, 2, 64), pos(1, 70, 2), neg(2), n(1, 70, 1, 16), n(1, 70, 1, 16), n(2, dt=f), 64)
    yield "ssd_prefill", p, {}
    yield "ssd_prefill", p, dict(raw, h0=n(1, 2, 64, 16, dt=f), y=torch.empty_like(p[0]))
    v = tuple(t[0] if i in (0, 1, 3, 4) else t for i, t in enumerate(p[:6])) + (torch.tensor([0, 30, 70], dtype=torch.int32, device="cuda"), 64)
    yield "ssd_prefill_varlen", v, {}
    yield "ssd_prefill_varlen", v, dict(raw, final_state=torch.empty(2, 2, 64, 16, device="cuda"))
    d = (n(2, 2, 64, 16, dt=f), n(2, 2, 64), pos(2, 2), neg(2), n(2, 1, 16), n(2, 1, 16), n(2, dt=f))
    yield "ssd_decode_step", d, {}
    yield "ssd_decode_step", d, dict(y=torch.empty_like(d[1]))
    ly = (n(3, 2, 2, 64, 16, dt=f), n(3, 2, 2, 64), pos(3, 2, 2), neg(3, 2), n(3, 2, 1, 16), n(3, 2, 1, 16), n(3, 2, dt=f))
    yield "ssd_decode_step_layers", ly, {}
    yield "ssd_decode_step_layers", ly, raw_l
    st = (ly[0], n(5, 3, 2, 2, 64), pos(5, 3, 2, 2), ly[3], n(5, 3, 2, 1, 16), n(5, 3, 2, 1, 16), ly[6])
    yield "ssd_decode_steps_layers", st, {}
    yield "ssd_decode_steps_layers", st, raw_l
    u, w = n(2, 9, 24), n(24, 4, dt=f)
    yield "ssd_conv1d_prefill", (u, w), {}
    yield "ssd_conv1d_prefill", (u, w, n(24, dt=f), n(2, 24, 3)), dict(split=(8, 16), activation="none")
    yield "ssd_conv1d_step", (n(2, 24, 3), u[:, 0].contiguous(), w), dict(split=[8, 8, 8])
    yield "ssd_conv1d_step", (n(2, 24, 3), u[:, 0].contiguous(), w, n(24, dt=f)), dict(activation="none")


def _flat(out):
    return [out] if isinstance(out, torch.Tensor) else [t for o in out for t in _flat(o)]


@pytest.mark.gpu
@pytest.mark.parametrize("io", [torch.bfloat16, torch.float32], ids=str)
def test_native_and_python_paths_are_equal(io, monkeypatch):
    clone = lambda v: v.clone() if isinstance(v, torch.Tensor) else v   # noqa: E731
    taken = []
    spy = types.SimpleNamespace(**{k: (lambda *a, k=k: taken.append(getattr(ssd_native, k)(*a)) or taken[-1]) for k in NAMES})
    off = types.SimpleNamespace(**{k: (lambda *a: None) for k in NAMES})
    ssd_native = ssd._native
    for name, args, kw in _calls(io):
        got = []
        for native in (spy, off):
            a, k = [clone(v) for v in args], {q: clone(v) for q, v in kw.items()}
            monkeypatch.setattr(ssd, "_native", native)
            out = getattr(ssd, name)(*a, **k)
            torch.cuda.synchronize()
            if k.get("y") is not None:
                assert (out[0] if isinstance(out, tuple) else out) is k["y"]
            got.append(_flat(out) + [v for v in a if isinstance(v, torch.Tensor)])   # (states updated in place too)
        assert taken.pop() is not None and not taken, name
        assert len(got[0]) == len(got[1]) and all(s.dtype == t.dtype and torch.equal(s, t) for s, t in zip(*got)), name


@pytest.mark.gpu
def test_a_failing_call_raises_its_status():
    z = torch.zeros(1, 4, 3, 64, device="cuda")
    with pytest.raises(ssd.SSDError) as e:   # three heads over two groups
        ssd.ssd_prefill(z, torch.zeros(1, 4, 3, device="cuda"), torch.zeros(3, device="cuda"), torch.zeros(1, 4, 2, 64, device="cuda"),
                        torch.zeros(1, 4, 2, 64, device="cuda"), torch.zeros(3, device="cuda"), 64)
    assert e.value.status == -2


ABI = ("ssd_prefill_workspace_bytes", "ssd_prefill", "ssd_prefill_dt", "ssd_prefill_varlen_workspace_bytes", "ssd_prefill_varlen",
       "ssd_prefill_varlen_dt", "ssd_decode_step", "ssd_decode_step_layers", "ssd_decode_step_layers_dt", "ssd_decode_steps_layers",
       "ssd_decode_steps_layers_dt", "ssd_conv1d_prefill", "ssd_conv1d_step")


@pytest.fixture
def recorded(monkeypatch):
    """The C ABI behind both paths exchanged for functions that note a call and do nothing."""
    calls = []
    stub = lambda name: ctypes.CFUNCTYPE(ctypes.c_int64)(lambda: calls.append(name) or 0)   # noqa: E731  (0: SSD_OK, no workspace)
    stubs = {n: stub(n) for n in ABI}
    init = lambda fs: ssd._native.init([ctypes.cast(f, ctypes.c_void_p).value for f in fs])   # noqa: E731
    init(stubs.values())
    lib = ssd._lib
    monkeypatch.setattr(ssd, "_lib", types.SimpleNamespace(**{n: (lambda *a, n=n: calls.append(n) or 0) for n in ABI}))
    yield calls
    init([getattr(lib, n) for n in ABI])


def _broken(name, args, kw):
    """The call with one tensor changed: another type, the last dimension one short, not dense."""
    names = list(range(len(args))) + list(kw)
    for key in names:
        t = args[key] if isinstance(key, int) else kw[key]
        if not isinstance(t, torch.Tensor):
            continue
        other = {torch.float32: torch.bfloat16, torch.bfloat16: torch.float32, torch.int32: torch.int64}[t.dtype]
        for what, v in (("type", t.to(other)), ("size", t[..., :-1].contiguous()), ("strides", torch.stack([t, t], -1)[..., 0])):
            if t.dim() and v.is_contiguous() and what == "strides":
                continue   # (one value)
            # (calls of their own: a convolution of another type or of fewer taps, without a state; prompts of a smaller head, without a
            # state; fewer packed sequences)
            own = {"ssd_conv1d_prefill": [(0, "type"), (1, "size")] if len(args) == 2 else [],
                   "ssd_prefill": [] if "h0" in kw else [(0, "size")], "ssd_prefill_varlen": [(0, "size"), (6, "size")]}
            if (key, what) in own.get(name, []):
                continue
            a, k = list(args), dict(kw)
            if isinstance(key, int):
                a[key] = v
            else:
                k[key] = v
            yield (key, what), a, k


@pytest.mark.gpu
@pytest.mark.parametrize("io", [torch.bfloat16, torch.float32], ids=str)
def test_every_argument_is_checked_before_a_call(io, recorded):
    """Neither path reaches the C ABI with a tensor of the wrong type, of a size that does not fit, or not dense."""
    outputs = {"ssd_prefill": ("y", "final_state"), "ssd_prefill_varlen": ("y", "final_state"), "ssd_decode_step": ("y",),
               "ssd_decode_step_layers": ("y",), "ssd_decode_steps_layers": ("y",)}
    for name, args, kw in _calls(io):
        f = getattr(ssd, name)
        if name in outputs:
            y, st = torch.empty_like(args[1 if "decode" in name else 0]), torch.empty(2, 2, 64, 16, device="cuda")
            kw = dict(kw, y=y, **({"final_state": st[:1].contiguous() if name == "ssd_prefill" else st} if "final_state" in outputs[name] else {}))
        recorded.clear()
        f(*args, **kw)
        assert recorded, name
        for which, a, k in _broken(name, args, kw):
            recorded.clear()
            try:
                f(*a, **k)
            except ValueError:
                recorded[:] = [c for c in recorded if not c.endswith("workspace_bytes")]   # (host arithmetic)
                assert not recorded, (name, which)
            else:
                pytest.fail("%s took a wrong argument: %s" % (name, which))


@pytest.mark.gpu
def test_larger_outputs_and_other_views_of_the_head_weights_are_taken(recorded):
    """What was taken before: an output with room to spare, A and D of a decode step in any shape."""
    io = torch.bfloat16
    d = [v for n, v, k in _calls(io) if n == "ssd_decode_step"][0]
    y = torch.empty(d[1].numel() + 5, dtype=io, device="cuda")
    for native in (True, False):
        recorded.clear()
        with pytest.MonkeyPatch.context() as m:
            if not native:
                m.setattr(ssd, "_native", types.SimpleNamespace(decode_step=lambda *a: None))
            assert ssd.ssd_decode_step(*d[:3], d[3].view(1, -1), *d[4:6], d[6].view(-1, 1), y=y) is y
        assert recorded == ["ssd_decode_step"]
