"""fp32 MFMA prefill in time segments: the state that enters a segment, one contraction over all the tokens before it.
Its edges: quarters of 16 tokens and of more than one set of weights (1024), dstate up to 16 (its own instruction) and
beyond, tokens that decay everything away before, in and behind a quarter."""
import numpy as np
import pytest
import torch

from oracle import ssd_oracle
from paper_2603_09555_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ssd():
    from paper_2603_09555_amd import ssd
    yield ssd
    ssd.reset_knobs()


# batch, tokens, heads, headdim, dstate, groups; segments; raw step sizes; steps that decay everything
CASES = [((1, 65, 2, 32, 8, 1), 2, False, False), ((2, 130, 3, 64, 16, 1), 3, True, False), ((1, 512, 4, 32, 16, 1), 8, False, True),
         ((1, 321, 2, 32, 24, 2), 6, False, False), ((1, 449, 2, 64, 64, 1), 7, True, True), ((2, 200, 2, 32, 96, 1), 4, False, False),
         ((1, 640, 2, 32, 16, 1), 10, False, False), ((1, 640, 2, 32, 32, 1), 10, True, False),   # (eight, nine blocks before a segment)
         ((1, 333, 3, 32, 128, 3), 6, True, False), ((1, 4300, 1, 32, 16, 1), 64, False, False), ((1, 8500, 1, 32, 40, 1), 64, False, True)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])) + "-s%d-%d%d" % c[1:])
def test_state_entering_a_segment(ssd, case):
    dims, segments, raw, steep = case
    cfg = inputs.SSDConfig("t", *dims, 64, "f32")
    inp = inputs.make_prefill_inputs(cfg, seed=51)
    rng = np.random.default_rng(4)
    if steep:
        inp["dt"] = inp["dt"] * torch.from_numpy(rng.choice([1.0, 30.0], inp["dt"].shape, p=[0.98, 0.02])).float()
    h0 = 0.1 * inputs.make_state(cfg, seed=51)
    kw, dt = {}, inp["dt"]
    if raw:
        bias = torch.from_numpy(rng.normal(-4.0, 0.3, cfg.nheads)).float()
        inp["dt"] = torch.from_numpy(rng.normal(0.0, 1.0, inp["dt"].shape)).float()
        kw = dict(dt_bias=bias.cuda(), dt_softplus=True)
        dt = ssd_oracle.dt_transform(inp["dt"], bias, True, None)
    ssd.reset_knobs()
    ssd.set_knob("force_mfma_f32", 1)
    ssd.set_knob("f32_segments", segments)
    print("state entering a segment", case, flush=True)
    dev = {k: v.cuda() for k, v in inp.items()}
    y, st = ssd.ssd_prefill(*[dev[k] for k in ("x", "dt", "A", "B", "C", "D")], 64, h0=h0.cuda(), **kw)
    torch.cuda.synchronize()
    ssd.reset_knobs()
    y_ref, st_ref = ssd_oracle.prefill(inp["x"], dt, inp["A"], inp["B"], inp["C"], inp["D"], h0=h0)
    # 32-bit sums of up to 64 terms a matrix instruction chain at a time, decays from sums of up to 64 steps: 1e-6 of the norm
    for got, ref, what in ((y, y_ref, "y"), (st, st_ref, "final state")):
        err = np.linalg.norm(got.double().cpu().numpy() - ref) / np.linalg.norm(ref)
        print("  %s off by %.2e" % (what, err), flush=True)
        assert err <= 1e-6, (what, err)


@pytest.mark.parametrize("dims, segments", [((577, 2, 32, 8), 16), ((404, 1, 32, 128), 8), ((330, 2, 32, 64), 6)], ids=str)
def test_the_state_is_no_further_off_than_that_of_one_walk(ssd, dims, segments):
    """Over twelve prompts, against 64 bits: a segment's entering state is summed in four chains, with the newest tokens in all of
    them, the walk's in two (two per cent for the luck of single roundings)."""
    tokens, heads, headdim, dstate = dims
    squares = {1: 0.0, segments: 0.0}
    for seed in range(12):
        cfg = inputs.SSDConfig("t", 1, tokens, heads, headdim, dstate, 1, 64, "f32")
        inp = inputs.make_prefill_inputs(cfg, seed=seed)
        _, ref = ssd_oracle.prefill(*[inp[k] for k in ("x", "dt", "A", "B", "C", "D")])
        for s in squares:
            ssd.reset_knobs()
            ssd.set_knob("force_mfma_f32", 1)
            ssd.set_knob("f32_segments", s)
            _, st = ssd.ssd_prefill(*[inp[k].cuda() for k in ("x", "dt", "A", "B", "C", "D")], 64)
            torch.cuda.synchronize()
            squares[s] += float((np.linalg.norm(st.double().cpu().numpy() - ref) / np.linalg.norm(ref)) ** 2)
        ssd.reset_knobs()
    ratio = float(np.sqrt(squares[segments] / squares[1]))
    print("state of %d segments / of one, off from 64 bits: %.3f" % (segments, ratio), flush=True)
    assert ratio <= 1.02


def _classes(a):
    return np.where(np.isnan(a), 3, np.where(np.isposinf(a), 1, np.where(np.isneginf(a), 2, 0)))


@pytest.mark.parametrize("where", ["x", "B", "h0"])
@pytest.mark.parametrize("same_sign", [False, True])
@pytest.mark.parametrize("tokens, headdim, dstate, segments", [(330, 32, 16, 6), (700, 32, 8, 11), (700, 64, 64, 3), (900, 32, 128, 2), (4700, 32, 32, 3)])
def test_infinities_survive_the_way_to_a_segment(ssd, where, same_sign, tokens, headdim, dstate, segments):
    """An infinity in the state stays one while the decay behind it leaves fp32's range (2^-1 a token), as in the recurrence, and
    reaches the outputs of later blocks as what it is there."""
    H = 2
    g = torch.Generator().manual_seed(53)
    draw = lambda *s: (lambda t: t.abs() + 0.25 if same_sign else t)(torch.randn(*s, generator=g))   # noqa: E731
    x, B, C = draw(1, tokens, H, headdim), draw(1, tokens, 1, dstate), draw(1, tokens, 1, dstate)
    dt = 0.05 * (0.8 + 0.4 * torch.rand(1, tokens, H, generator=g))
    A, D, h0 = torch.full((H,), -20.0 * float(np.log(2.0))), draw(H), draw(1, H, headdim, dstate)
    for at in (10, tokens // 4):   # (before the last segment either way)
        v = [t.clone() for t in (x, dt, A, B, C, D, h0)]
        {"x": v[0][0, at, 0], "B": v[3][0, at, 0], "h0": v[6][0, 0, at % headdim]}[where][3] = float("-inf")
        ssd.reset_knobs()
        ssd.set_knob("force_mfma_f32", 1)
        ssd.set_knob("f32_segments", segments)
        print("infinite", where, same_sign, tokens, headdim, dstate, segments, at, flush=True)
        dev = [t.cuda() for t in v]
        y, st = ssd.ssd_prefill(*dev[:6], 64, h0=dev[6])
        torch.cuda.synchronize()
        ssd.reset_knobs()
        with np.errstate(all="ignore"):
            y_ref, st_ref = ssd_oracle.prefill(*v[:6], h0=v[6])
        y, st = y.double().cpu().numpy(), st.double().cpu().numpy()
        assert np.array_equal(_classes(st), _classes(st_ref)), at
        if where != "x" or dstate % 32 == 0:   # (x meets the zeros of padded state columns, and masked scores in its own block)
            later = slice(0 if where == "h0" else (at // 64 + 1) * 64, None)
            assert np.array_equal(_classes(y[:, later]), _classes(y_ref[:, later])), at
        ok = np.isfinite(st_ref)   # (exponents of up to 64 are rounded at 2^-18: 2.6e-6 of a factor)
        assert np.linalg.norm(st[ok] - st_ref[ok]) <= 1e-5 * np.linalg.norm(st_ref[ok])
