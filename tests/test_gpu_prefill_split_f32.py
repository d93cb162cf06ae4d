"""fp32 prefill on split bf16 operands: segments, their states in the workspace or in y, shared single segments."""
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
    return ssd


@pytest.fixture(autouse=True)
def _reset(ssd):
    ssd.reset_knobs()
    yield
    ssd.reset_knobs()


def run(ssd, cfg, inp, h0=None, alias=False, **kw):
    dev = {k: v.cuda() for k, v in inp.items()}
    h = None if h0 is None else h0.cuda()
    y, st = ssd.ssd_prefill(dev["x"], dev["dt"], dev["A"], dev["B"], dev["C"], dev["D"], cfg.chunk, h0=h,
                            final_state=h if alias else None, **kw)
    torch.cuda.synchronize()
    return y, st


def check(ssd, cfg, inp, h0, y, st, what):
    y_ref, st_ref = ssd_oracle.prefill(inp["x"], inp["dt"], inp["A"], inp["B"], inp["C"], inp["D"], h0=h0)
    assert_close(y, y_ref, TOL["f32"], what + " y")
    assert_close(st, st_ref, TOL["f32"], what + " final state")


CASES = [
    # Bt, T, H, P, N, G, L, h0, blocks per segment, workgroups per segment
    (1, 31, 2, 32, 8, 1, 64, False, 1, 1),       # less than a block; dstate padded
    (2, 33, 4, 64, 16, 2, 64, True, 2, 2),       # a block and a token; one segment shared by two
    (1, 300, 5, 64, 128, 1, 64, True, 2, 1),     # ten slices over three workgroups; states in the workspace
    (1, 640, 3, 64, 128, 1, 512, True, 4, 1),    # ... in y (chunks too long for the workspace); segments of 4 blocks
    (2, 500, 6, 96, 72, 3, 1000, False, 5, 1),   # ... in y, dstate 72, slices of one head over two workgroups
    (3, 1000, 4, 32, 40, 2, 100, True, 7, 1),    # uneven segments
    (1, 700, 8, 64, 64, 4, 64, False, 22, 4),    # one segment, four workgroups each
    (1, 256, 2, 32, 96, 1, 64, True, 1, 1),      # as many segments as blocks
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_split_prefill_matches_oracle(ssd, case):
    *dims, with_h0, seg, sub = case
    cfg = inputs.SSDConfig("t", *dims, "f32")
    ssd.set_knob("seg_blocks", seg)
    ssd.set_knob("seg_parts", sub)
    plan = ssd.prefill_plan(ssd.make_shape(*dims, torch.float32))
    print("split fp32", case, plan, flush=True)
    assert plan["path"] == "mfma_f32" and plan["f32_segments"] == 0
    inp = inputs.make_prefill_inputs(cfg, seed=3)
    h0 = inputs.make_state(cfg, seed=3, scale=0.3) if with_h0 else None
    y, st = run(ssd, cfg, inp, h0)
    check(ssd, cfg, inp, h0, y, st, "split")
    y2, st2 = run(ssd, cfg, inp, h0)
    assert torch.equal(y, y2) and torch.equal(st, st2)
    if h0 is not None:   # h0 and final_state in one buffer: the same results
        y3, st3 = run(ssd, cfg, inp, h0, alias=True)
        if plan["segments"] > 1 or plan["parts"] == 1:
            assert torch.equal(y, y3) and torch.equal(st, st3)
        check(ssd, cfg, inp, h0, y3, st3, "aliased")


@pytest.mark.parametrize("seg", [4, 64])
def test_split_prefill_steep_decay_and_step_size_map(ssd, seg):
    cfg = inputs.SSDConfig("t", 2, 600, 4, 64, 128, 1, 256, "f32")
    ssd.set_knob("seg_blocks", seg)
    inp = inputs.make_prefill_inputs(cfg, seed=5)
    inp["dt"] = torch.full_like(inp["dt"], 0.5)
    inp["A"] = torch.tensor([-1.0, -6.0, -12.0, -24.0])
    y, st = run(ssd, cfg, inp)
    check(ssd, cfg, inp, None, y, st, "steep")
    g = torch.Generator().manual_seed(6)
    raw, bias = torch.randn(inp["dt"].shape, generator=g) * 1.5 - 3.0, torch.randn((4,), generator=g) * 0.5
    inp2 = dict(inp, dt=raw)
    y, st = run(ssd, cfg, inp2, dt_bias=bias.cuda(), dt_softplus=True, dt_limit=(1e-3, 0.5))
    inp2["dt"] = torch.from_numpy(ssd_oracle.dt_transform(raw, bias, True, (1e-3, 0.5))).float()
    check(ssd, cfg, inp2, None, y, st, "map")


def test_split_prefill_replayed_from_a_hip_graph(ssd):
    """States between the launches lie in y: replays, with eager work between them, leave what an eager call leaves."""
    cfg = inputs.SSDConfig("t", 1, 1024, 6, 64, 128, 1, 1024, "f32")
    ssd.set_knob("seg_blocks", 8)
    dev = {k: v.cuda() for k, v in inputs.make_prefill_inputs(cfg, seed=9).items()}
    args = [dev[k] for k in ("x", "dt", "A", "B", "C", "D")]
    y_ref, st_ref = ssd.ssd_prefill(*args, cfg.chunk)
    y, st = torch.empty_like(y_ref), torch.empty_like(st_ref)
    ws = torch.empty((ssd.prefill_workspace_bytes(ssd.make_shape(1, 1024, 6, 64, 128, 1, 1024, torch.float32)),),
                     dtype=torch.uint8, device="cuda")
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            ssd.ssd_prefill(*args, cfg.chunk, y=y, final_state=st, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    for _ in range(3):
        y.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, y_ref) and torch.equal(st, st_ref)


@pytest.mark.parametrize("size", [1e2, 1e4, 1e6])
def test_split_prefill_is_exact_behind_steps_of_any_size(ssd, size):
    """Tokens that decay everything away (dt |A| = size) among gentle ones: the decay between the tokens behind them is a
    difference of prefix sums that hold the large step too.  Exponents are good to 2^-26 and each term of an output to a
    handful of roundings of 2^-24: 5e-7 of the terms' magnitudes bounds a head's outputs at a token."""
    H, T = 4, 200
    cfg = inputs.SSDConfig("t", 1, T, H, 64, 128, 1, 64, "f32")
    ssd.set_knob("seg_blocks", 3)
    inp = inputs.make_prefill_inputs(cfg, seed=8)
    inp["D"].zero_()
    for t, h in ((3, 0), (16, 1), (2, 2), (7, 2), (100, 2)):
        inp["dt"][0, t, h] = size / -inp["A"][h]
        inp["x"][0, t, h] /= size   # (its own input would drown what follows)
    print("split fp32 behind a step of", size, flush=True)
    y, st = run(ssd, cfg, inp)
    y_ref, st_ref = ssd_oracle.prefill(inp["x"], inp["dt"], inp["A"], inp["B"], inp["C"], inp["D"])
    mag, _ = ssd_oracle.prefill(inp["x"].abs(), inp["dt"], inp["A"], inp["B"].abs(), inp["C"].abs(), inp["D"])
    err = float((np.linalg.norm(y.cpu().double().numpy() - y_ref, axis=-1) / np.linalg.norm(mag, axis=-1)).max())
    print("  y off by at most %.2e of its terms" % err, flush=True)
    assert err <= 5e-7
    assert_close(st, st_ref, 1e-6, "final state")


@pytest.mark.parametrize("where", ["x", "B", "C", "dt", "h0", "huge x", "huge B and C"])
@pytest.mark.parametrize("seg, sub", [(3, 1), (64, 2)])
def test_split_prefill_keeps_infinities_where_the_recurrence_has_them(ssd, where, seg, sub):
    """An infinity or a NaN reaches exactly the outputs that the recurrence lets it reach, as what it is there; values next
    to the end of fp32's range, and products that leave it, do no harm where the recurrence's stay inside."""
    H, T, P, N = 4, 300, 64, 72
    cfg = inputs.SSDConfig("t", 2, T, H, P, N, 1, 64, "f32")
    ssd.set_knob("seg_blocks", seg)
    ssd.set_knob("seg_parts", sub)
    inp = inputs.make_prefill_inputs(cfg, seed=15)
    inp["dt"] = inp["dt"].clamp(max=0.01)
    h0 = inputs.make_state(cfg, seed=15, scale=0.3)
    if where == "x":
        inp["x"][0, 130, 1, 7] = float("inf")
    elif where == "B":
        inp["B"][1, 70, 0, 5] = float("-inf")
        inp["B"][0, 299, 0, 71] = float("nan")
    elif where == "C":
        inp["C"][0, 33, 0, 40] = float("inf")
    elif where == "dt":
        inp["dt"][1, 36, 2] = float("nan")
    elif where == "h0":
        h0[0, 3, 60, 71] = float("-inf")
    elif where == "huge x":
        inp["x"][0, 40, 2, 9] = 3.4e38
    else:
        inp["B"][0, 100], inp["C"][0, 100] = inp["B"][0, 100] * 1e20, inp["C"][0, 100] * 1e20
        inp["x"][0, 100] = inp["x"][0, 100] * 1e-20
    print("split fp32, out of range:", where, seg, sub, flush=True)
    y, st = run(ssd, cfg, inp, h0)
    with np.errstate(all="ignore"):
        y_ref, st_ref = ssd_oracle.prefill(inp["x"], inp["dt"], inp["A"], inp["B"], inp["C"], inp["D"], h0=h0)
    for got, ref, heads, what in ((y, y_ref, 2, "y"), (st, st_ref, 1, "final state")):
        got = got.cpu().double().numpy()
        for kind in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(kind(got), kind(ref)), (what, kind)
        got, ref = np.moveaxis(got, heads, 0).reshape(H, -1), np.moveaxis(ref, heads, 0).reshape(H, -1)
        for h in range(H):   # (a head at a time: one with huge values would hide the others)
            ok = np.isfinite(ref[h])
            assert np.linalg.norm(got[h][ok] - ref[h][ok]) <= 1e-5 * np.linalg.norm(ref[h][ok]), (what, h)


def errors_against_64_bits(ssd, cfg, inp, h0, knob):
    ssd.reset_knobs()
    ssd.set_knob(*knob)
    got = run(ssd, cfg, inp, h0)
    ref = ssd_oracle.prefill(inp["x"], inp["dt"], inp["A"], inp["B"], inp["C"], inp["D"], h0=h0)
    return [float(np.linalg.norm(g.cpu().double().numpy() - r) / np.linalg.norm(r)) for g, r in zip(got, ref)]


@pytest.mark.parametrize("dims", [(1, 2048, 8, 64, 128, 1, 256), (2, 700, 6, 32, 16, 2, 64), (3, 500, 5, 64, 72, 1, 128)], ids=str)
@pytest.mark.parametrize("with_h0", [False, True])
def test_split_prefill_is_as_accurate_as_the_fp32_matrix_instruction(ssd, dims, with_h0):
    """Against 64 bits, relative 2-norms: at most the error of the kernel that forms its products and sums in the fp32 matrix
    instruction (a tenth more for the luck of single roundings), and 5e-7 -- a part lost anywhere is 1.5e-5."""
    cfg = inputs.SSDConfig("t", *dims, "f32")
    inp = inputs.make_prefill_inputs(cfg, seed=17)
    h0 = inputs.make_state(cfg, seed=17, scale=0.02) if with_h0 else None
    split = errors_against_64_bits(ssd, cfg, inp, h0, ("seg_blocks", 4))
    fp32 = errors_against_64_bits(ssd, cfg, inp, h0, ("force_mfma_f32", 1))
    print("  off by %.2e, state %.2e; fp32 matrix instruction %.2e, %.2e" % (*split, *fp32), flush=True)
    for s, f in zip(split, fp32):
        assert s <= 1.1 * f and s <= 5e-7


def test_split_products_are_fp32_products(ssd):
    """The state of one token is one product per element, of dt x (exact here: dt = 1) and B.  Of it, at most 2^-24 is left
    out, and the sum of the parts' products is cut off once more at 2^-23: three units of 2^-24."""
    H, P, N = 8, 64, 128
    ssd.set_knob("seg_blocks", 1)
    g = torch.Generator().manual_seed(1)
    x, B, C = (torch.randn(s, generator=g) for s in ((4, 1, H, P), (4, 1, 1, N), (4, 1, 1, N)))
    dt, A, D = torch.ones(4, 1, H), -torch.ones(H), torch.zeros(H)
    print("split fp32, one token", flush=True)
    _, st = ssd.ssd_prefill(*[t.cuda() for t in (x, dt, A, B, C, D)], 64)
    torch.cuda.synchronize()
    ref = x.double()[:, 0, :, :, None] * B.double()[:, 0, :, None, :]
    err = float(((st.cpu().double() - ref) / ref).abs().max()) * 2 ** 24
    print("  products off by at most %.2f units of 2^-24" % err, flush=True)
    assert err <= 3.0
