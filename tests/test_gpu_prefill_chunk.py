"""bf16 prefill on the chunk kernels (a workgroup per 64 headdim columns and chunk of 256 tokens) against the oracle, at
the edges of their tiles of 32 tokens, their chunks and the numbers of states folded at a time."""
import numpy as np
import pytest
import torch

from oracle import ssd_oracle
from paper_2603_09555_amd import inputs
from parity import TOL, assert_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ssd():
    from paper_2603_09555_amd import ssd
    yield ssd
    ssd.reset_knobs()


@pytest.fixture(autouse=True)
def _library_choices_restored(ssd):
    ssd.reset_knobs()
    yield
    ssd.reset_knobs()


# batch, tokens, heads, headdim, dstate, groups, chunk argument; initial state; raw step sizes; steps that decay everything
CASES = [((1, 1, 1, 64, 128, 1, 64), False, False, False), ((2, 31, 3, 64, 8, 1, 64), True, False, False),
         ((1, 33, 2, 128, 120, 2, 64), False, True, False), ((1, 255, 5, 64, 128, 1, 256), True, True, True),
         ((3, 256, 2, 64, 64, 1, 100), True, False, False), ((1, 257, 3, 64, 128, 3, 64), True, True, False),
         ((2, 300, 4, 64, 72, 1, 64), False, False, True), ((1, 512, 1, 192, 128, 1, 64), True, False, False),
         ((1, 1025, 2, 64, 128, 1, 64), True, False, False), ((1, 1500, 3, 64, 128, 1, 256), False, True, True),
         ((1, 2100, 1, 64, 40, 1, 64), True, True, False), ((1, 16384, 1, 64, 128, 1, 64), True, False, False)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])) + "-%d%d%d" % c[1:])
def test_chunk_kernels_match_oracle(ssd, case):
    dims, with_h0, raw, steep = case
    cfg = inputs.SSDConfig("t", *dims, "bf16")
    inp = inputs.make_prefill_inputs(cfg, seed=41)
    rng = np.random.default_rng(3)
    if steep:   # (decays up to e^-60 between neighbours, and behind them ordinary tokens)
        inp["dt"] = inp["dt"] * torch.from_numpy(rng.choice([1.0, 40.0], inp["dt"].shape)).float()
    h0 = 0.1 * inputs.make_state(cfg, seed=41) if with_h0 else None
    kw, dt = {}, inp["dt"]
    if raw:
        bias = torch.from_numpy(rng.normal(-4.0, 0.3, cfg.nheads)).float()
        inp["dt"] = torch.from_numpy(rng.normal(0.0, 2.0, inp["dt"].shape)).float()
        kw = dict(dt_bias=bias.cuda(), dt_softplus=True, dt_limit=(1e-3, 0.5))
        dt = ssd_oracle.dt_transform(inp["dt"], bias, True, (1e-3, 0.5))
    ssd.set_knob("chunk", 1)
    sh = ssd.make_shape(*dims, torch.bfloat16)
    assert ssd.prefill_chunks(sh) == (dims[1] + 255) // 256
    print("chunk kernels", case, flush=True)
    dev = {k: v.cuda() for k, v in inp.items()}
    args = [dev[k] for k in ("x", "dt", "A", "B", "C", "D")]
    y, st = ssd.ssd_prefill(*args, cfg.chunk, h0=None if h0 is None else h0.cuda(), **kw)
    torch.cuda.synchronize()
    y_ref, st_ref = ssd_oracle.prefill(inp["x"], dt, inp["A"], inp["B"], inp["C"], inp["D"], h0=h0)
    assert_close(y, y_ref, TOL["bf16"], "y")
    assert_close(st, st_ref, TOL["bf16"], "final state")
    if h0 is not None:   # the state updated in place: the same bits
        # (31 tokens of dstate 8: the workspace has no room for the copy of h0, another kernel runs)
        assert (ssd.prefill_chunks(sh, True) == ssd.prefill_chunks(sh)) == (dims[1] > 31)
        if dims[1] > 31:
            both = h0.cuda()
            y2, st2 = ssd.ssd_prefill(*args, cfg.chunk, h0=both, final_state=both, **kw)
            torch.cuda.synchronize()
            assert torch.equal(y2, y) and torch.equal(st2, st)


def test_where_the_chunk_kernels_are_taken(ssd):
    """Where the launch is about one round of the chip; knobs of the scan kernels ask for those."""
    shape = lambda *d: ssd.make_shape(*d, 128, 1, 256, torch.bfloat16)   # noqa: E731
    assert ssd.prefill_chunks(shape(1, 2048, 24, 64)) == 8
    assert ssd.prefill_chunks(shape(2, 250, 64, 64)) == 1 and ssd.prefill_chunks(shape(1, 250, 129, 64)) == 0
    assert ssd.prefill_chunks(shape(1, 512, 85, 64)) == 2 and ssd.prefill_chunks(shape(1, 512, 86, 64)) == 0
    assert ssd.prefill_chunks(shape(1, 1024, 64, 64)) == 4 and ssd.prefill_chunks(shape(1, 1024, 65, 64)) == 0
    assert ssd.prefill_chunks(shape(1, 4608, 16, 64)) == 18 and ssd.prefill_chunks(shape(1, 4609, 16, 64)) == 0
    assert ssd.prefill_chunks(shape(1, 16384, 80, 64)) == 0
    assert ssd.prefill_chunks(ssd.make_shape(1, 2048, 24, 64, 136, 1, 256, torch.bfloat16)) == 0   # two state slices
    for knob, value in (("seg_blocks", 2), ("seg_chunks", 1), ("scan_heads", 4), ("y_stream", 0), ("fold_max_slots", 0),
                        ("force_generic", 1), ("chunk", 2)):
        ssd.reset_knobs()
        ssd.set_knob(knob, value)
        assert ssd.prefill_chunks(shape(1, 2048, 24, 64)) == 0, knob


def test_chunk_kernels_replayed_from_a_hip_graph(ssd):
    """Two launches and a hand-over through the workspace: every replay follows the inputs it finds."""
    for dims in ((2, 600, 4, 64, 128, 1, 256), (2, 200, 4, 64, 128, 1, 256)):
        cfg = inputs.SSDConfig("t", *dims, "bf16")
        a, b = [{k: v.cuda() for k, v in inputs.make_prefill_inputs(cfg, seed=s).items()} for s in (1, 2)]
        sh = ssd.make_shape(*dims, torch.bfloat16)
        assert ssd.prefill_chunks(sh) > 0
        buf = {k: v.clone() for k, v in a.items()}
        y, st = torch.empty_like(buf["x"]), torch.empty((2, 4, 64, 128), device="cuda")
        ws = torch.empty((ssd.prefill_workspace_bytes(sh),), dtype=torch.uint8, device="cuda")
        call = lambda d, **kw: ssd.ssd_prefill(*[d[k] for k in ("x", "dt", "A", "B", "C", "D")], cfg.chunk, **kw)   # noqa: E731
        want = [[t.clone() for t in call(d)] for d in (a, b)]
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            call(buf, y=y, final_state=st, workspace=ws)
        for i in range(5):
            for k in buf:
                buf[k].copy_((a, b)[i & 1][k])
            ws.fill_(255)   # (nothing is left over from the replay before)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, want[i & 1][0]) and torch.equal(st, want[i & 1][1]), (dims, i)


@pytest.mark.parametrize("tokens", [20, 200, 700])
def test_an_undefined_decay_shows_in_every_row(ssd, tokens):
    """A head whose A is NaN has no defined output, from its first token on; its neighbour is untouched."""
    cfg = inputs.SSDConfig("t", 1, tokens, 2, 64, 128, 1, 256, "bf16")
    dev = {k: v.cuda() for k, v in inputs.make_prefill_inputs(cfg, seed=43).items()}
    ssd.set_knob("chunk", 1)
    assert ssd.prefill_chunks(ssd.make_shape(1, tokens, 2, 64, 128, 1, 256, torch.bfloat16)) > 0
    print("chunk kernels, A undefined", tokens, flush=True)
    call = lambda: ssd.ssd_prefill(*[dev[k] for k in ("x", "dt", "A", "B", "C", "D")], cfg.chunk)   # noqa: E731
    y0, st0 = call()
    dev["A"][0] = float("nan")
    y, st = call()
    torch.cuda.synchronize()
    assert torch.isnan(y[:, :, 0]).all() and torch.isnan(st[:, 0]).all()
    assert torch.equal(y[:, :, 1], y0[:, :, 1]) and torch.equal(st[:, 1], st0[:, 1])


def _classes(a):
    return np.where(np.isnan(a), 3, np.where(np.isposinf(a), 1, np.where(np.isneginf(a), 2, 0)))


@pytest.mark.parametrize("where", ["x", "B", "C", "dt", "h0"])
@pytest.mark.parametrize("same_sign", [False, True])
@pytest.mark.parametrize("tokens, dstate, decay", [(20, 128, 1.0), (256, 64, 1.0), (255, 8, 6.0), (700, 128, 0.02), (700, 72, 1.0), (1100, 128, 5.0)])
def test_infinities_are_what_the_recurrence_makes_of_them(ssd, where, same_sign, tokens, dstate, decay):
    """One infinity among the inputs reaches the outputs that the recurrence lets it reach, of the sign that it has there or
    undefined, however far the weights between the tokens have decayed (2^-decay a token, 256 of them below fp32's range)."""
    H, P = 2, 64
    g = torch.Generator().manual_seed(47)
    draw = lambda *s: (lambda t: t.abs() + 0.25 if same_sign else t)(torch.randn(*s, generator=g))   # noqa: E731
    x, B, C = draw(1, tokens, H, P), draw(1, tokens, 1, dstate), draw(1, tokens, 1, dstate)
    dt = 0.05 * (0.8 + 0.4 * torch.rand(1, tokens, H, generator=g))
    A, D, h0 = torch.full((H,), -decay / 0.05 * float(np.log(2.0))), draw(H), draw(1, H, P, dstate)
    for at in (10, tokens // 2):
        v = [t.clone() for t in (x.bfloat16(), dt, A, B.bfloat16(), C.bfloat16(), D, h0)]
        {"x": v[0][0, at, 0], "B": v[3][0, at, 0], "C": v[4][0, at, 0], "dt": v[1][0, at], "h0": v[6][0, 0, at % P]}[where][
            0 if where == "dt" else 3] = float("inf")
        ssd.set_knob("chunk", 1)
        alias = where == "h0" and tokens > 256
        assert ssd.prefill_chunks(ssd.make_shape(1, tokens, H, P, dstate, 1, 64, torch.bfloat16), alias) == (tokens + 255) // 256
        print("chunk kernels, infinite", where, same_sign, tokens, dstate, decay, at, flush=True)
        dev = [t.cuda() for t in v]
        y, st = ssd.ssd_prefill(*dev[:6], 64, h0=dev[6], final_state=dev[6] if alias else None)
        torch.cuda.synchronize()
        with np.errstate(all="ignore"):
            refs = ssd_oracle.prefill(*[t.float() for t in v[:6]], h0=v[6])
        for got, ref, what in ((y, refs[0], "y"), (st, refs[1], "final state")):
            got = got.double().cpu().numpy()
            assert np.array_equal(_classes(got), _classes(ref)), (what, at)
            ok = np.isfinite(ref)
            assert np.linalg.norm(got[ok] - ref[ok]) <= 2e-2 * np.linalg.norm(ref[ok]), (what, at)
