"""The native marshalling of ssd.py: where anything is out of the ordinary it answers None and does nothing, so that the
Python path raises what there is to raise; where it takes a call, the results are those of the Python path, bit for bit."""
import types

import pytest
import torch

from paper_2603_09555_amd import ssd

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
