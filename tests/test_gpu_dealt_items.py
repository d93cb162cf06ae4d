"""Packed batches whose scan workgroups are dealt several items (two heads of a list entry each): walks that go from item to
item over any parity of blocks, empty sequences, segments with an entering state, items longer than the 64 blocks whose
factors a wave holds, steep blocks in later items, heads short of a pair, several groups and state slices.  The two-head scan with
an entry to a workgroup is the reference (the same arithmetic: equal bit for bit), the oracle for the values."""
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


def ragged(n, most, seed):
    return [int(v) for v in np.random.default_rng(seed).integers(0, most, n)]


# lengths, heads, dstate, groups, blocks per segment (0: uncut), carried state, steep tokens
CASES = {
    "one item": ([70], 2, 128, 1, 0, False, ()),
    "fewer items than workgroups": (ragged(7, 400, 1), 5, 128, 1, 0, True, ()),
    "two rounds": (ragged(100, 200, 2), 6, 128, 1, 0, False, ()),
    "a round and one": ([64] * 257, 2, 128, 1, 0, True, ()),
    "many rounds": (ragged(300, 140, 3), 8, 64, 2, 0, True, ()),
    "empty ones among them": ([0, 0, 65] * 120 + [0], 3, 128, 1, 0, True, ()),
    "only empty ones but one": ([0] * 300 + [1], 2, 128, 1, 0, True, ()),
    "segments": (ragged(60, 700, 4) + [2000, 1], 12, 128, 1, 3, False, ()),
    "segments, carried": (ragged(90, 500, 5), 7, 128, 1, 2, True, ()),
    "two state slices": (ragged(70, 300, 6), 9, 256, 1, 0, True, ()),
    "two state slices, segments": (ragged(40, 400, 7) + [900], 14, 200, 2, 2, False, ()),
    "longer than 64 blocks": ([4200, 4161] + 130 * [65], 4, 128, 1, 0, False, ()),
    "steep": (ragged(150, 260, 8), 4, 128, 1, 0, True, (5, 3000, 9000, 9070)),
    "steep behind 64 blocks": ([4300] + 140 * [30], 4, 128, 1, 0, False, (4200,)),
}


@pytest.mark.parametrize("name", CASES)
def test_dealt_items_equal_an_entry_each(ssd, name):
    lens, H, N, G, seg, carried, steep = CASES[name]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    cfg = inputs.SSDConfig("t", 1, T, H, 64, N, G, 64, "bf16")
    inp = inputs.make_prefill_inputs(cfg, seed=51)
    for t in steep:
        inp["dt"][:, t:t + 9] *= 60.0
    pk = {k: (v[0] if k in ("x", "dt", "B", "C") else v) for k, v in inp.items()}
    h0 = inputs.make_state(inputs.SSDConfig("h", len(lens), 1, H, 64, N, G, 64, "bf16"), seed=52, scale=0.1) if carried else None
    dev = {k: v.cuda() for k, v in pk.items()}
    out = {}
    for deal in (1, 2):
        ssd.reset_knobs()
        ssd.set_knob("scan_heads", 2)
        ssd.set_knob("seg_blocks", seg or (T + 63) // 64 + 1)
        ssd.set_knob("deal", deal)
        print("dealt items", name, deal, flush=True)
        out[deal] = ssd.ssd_prefill_varlen(*[dev[k] for k in ("x", "dt", "A", "B", "C", "D")], torch.from_numpy(cu).cuda(), cfg.chunk,
                                           h0=None if h0 is None else h0.cuda())
        torch.cuda.synchronize()
    ssd.reset_knobs()
    assert torch.equal(out[1][0], out[2][0]) and torch.equal(out[1][1], out[2][1])
    assert torch.isfinite(out[1][0]).all() and torch.isfinite(out[1][1]).all()
    y_ref, st_ref = ssd_oracle.prefill_varlen(*[pk[k] for k in ("x", "dt", "A", "B", "C", "D")], cu, h0=h0)
    if steep:
        # a steep block leaves outputs of a few large terms of both signs: each within the tolerance of the sum of its terms' sizes
        # (a term is rounded to bf16 three times on its way, 2^-9 each, and y once more)
        ab = {k: v if k in ("dt", "A") else v.abs() for k, v in pk.items()}
        mag = ssd_oracle.prefill_varlen(*[ab[k] for k in ("x", "dt", "A", "B", "C", "D")], cu, h0=None if h0 is None else h0.abs())
        for got, ref, m, what in zip(out[1], (y_ref, st_ref), mag, ("y", "final states")):
            worst = (np.abs(got.float().cpu().numpy().astype(np.float64) - ref) / np.maximum(m, 1e-30)).max()
            assert worst <= TOL["bf16"], (what, worst)
        return
    assert_close(out[1][0], y_ref, TOL["bf16"], "y")
    assert_close(out[1][1], st_ref, TOL["bf16"], "final states")


@pytest.mark.parametrize("H, n", [(34, 30), (3, 230)])
def test_the_library_deals_items_beyond_a_round(ssd, H, n):
    """As it runs by itself: the segment length from the device, changing lengths in one workspace, again and again."""
    T, cfg = 3000, inputs.SSDConfig("t", 1, 3000, H, 64, 128, 1, 64, "bf16")
    inp = inputs.make_prefill_inputs(cfg, seed=53)
    pk = {k: (v[0] if k in ("x", "dt", "B", "C") else v) for k, v in inp.items()}
    dev = {k: v.cuda() for k, v in pk.items()}
    shape = ssd.make_shape(n, T, H, 64, 128, 1, 64, torch.bfloat16)
    ws = torch.empty((int(ssd.raw().ssd_prefill_varlen_workspace_bytes(shape)),), dtype=torch.uint8, device="cuda")
    for seed in (1, 2, 3):
        cuts = np.sort(np.random.default_rng(seed).integers(0, T + 1, n - 1)) if seed < 3 else np.arange(1, n)   # (the last: one long one)
        cu = np.concatenate([[0], cuts, [T]]).astype(np.int32)
        assert ssd.varlen_plan(np.diff(cu), H, 64, 128, 1, 64)["dealt"]
        print("dealt by the library", H, n, seed, flush=True)
        y, st = ssd.ssd_prefill_varlen(*[dev[k] for k in ("x", "dt", "A", "B", "C", "D")], torch.from_numpy(cu).cuda(), cfg.chunk, workspace=ws)
        torch.cuda.synchronize()
        y_ref, st_ref = ssd_oracle.prefill_varlen(*[pk[k] for k in ("x", "dt", "A", "B", "C", "D")], cu)
        assert_close(y, y_ref, TOL["bf16"], "y")
        # (each against its own size: the root mean square of a batch of one-token states says nothing of a long sequence's)
        longest = int(np.argmax(np.diff(cu)))
        others = [q for q in range(n) if q != longest]
        assert_close(st[longest], st_ref[longest], TOL["bf16"], "the longest sequence's state")
        assert_close(st[others], st_ref[others], TOL["bf16"], "the others' states")


@pytest.mark.parametrize("name", ["many rounds", "empty ones among them", "segments, carried", "two state slices", "steep"])
def test_dealt_items_with_the_states_in_place(ssd, name):
    """h0 and final_states in one buffer."""
    lens, H, N, G, seg, carried, steep = CASES[name]
    assert carried
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    inp = inputs.make_prefill_inputs(inputs.SSDConfig("t", 1, T, H, 64, N, G, 64, "bf16"), seed=61)
    for t in steep:
        inp["dt"][:, t:t + 9] *= 60.0
    dev = {k: (v[0] if k in ("x", "dt", "B", "C") else v).cuda() for k, v in inp.items()}
    args = [dev[k] for k in ("x", "dt", "A", "B", "C", "D")] + [torch.from_numpy(cu).cuda(), 64]
    h0 = inputs.make_state(inputs.SSDConfig("h", len(lens), 1, H, 64, N, G, 64, "bf16"), seed=62, scale=0.1).cuda()
    ssd.reset_knobs()
    ssd.set_knob("seg_blocks", seg or (T + 63) // 64 + 1)
    ssd.set_knob("deal", 1)
    print("states in place", name, flush=True)
    y, st = ssd.ssd_prefill_varlen(*args, h0=h0)
    state = h0.clone()
    y2, st2 = ssd.ssd_prefill_varlen(*args, h0=state, final_state=state)
    torch.cuda.synchronize()
    ssd.reset_knobs()
    assert st2.data_ptr() == state.data_ptr()
    assert torch.equal(y, y2) and torch.equal(st, state)


def test_a_captured_dealt_call_follows_the_lengths(ssd):
    """More than a round, the boundaries changed between replays, with eager work and synchronizations in between."""
    T, H, nseq = 3000, 34, 30
    dev = {k: (v[0] if k in ("x", "dt", "B", "C") else v).cuda()
           for k, v in inputs.make_prefill_inputs(inputs.SSDConfig("t", 1, T, H, 64, 128, 1, 64, "bf16"), seed=63).items()}
    args = [dev[k] for k in ("x", "dt", "A", "B", "C", "D")]
    lens = [[100] * 30, [T - 29] + [1] * 29, [0, 900, 1, 700, 0, 3, 64, 65, 128, 500, 100, 39] + [500] + [0] * 17]
    plans = [ssd.varlen_plan(v, H, 64, 128, 1, 64) for v in lens]
    assert all(p["dealt"] and p["chosen"] for p in plans) and len({p["items"] for p in plans}) == 3
    cu = torch.zeros(nseq + 1, dtype=torch.int32, device="cuda")

    def boundaries(v):
        cu.copy_(torch.from_numpy(np.concatenate([[0], np.cumsum(v)]).astype(np.int32)))

    boundaries(lens[0])
    size = int(ssd.raw().ssd_prefill_varlen_workspace_bytes(ssd.make_shape(nseq, T, H, 64, 128, 1, 64, torch.bfloat16)))
    ws = torch.empty((size,), dtype=torch.uint8, device="cuda")
    y, st = torch.empty_like(dev["x"]), torch.empty((nseq, H, 64, 128), device="cuda")
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            ssd.ssd_prefill_varlen(*args, cu, 64, y=y, final_state=st, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    for i in (0, 1, 2, 1, 0):
        boundaries(lens[i])
        y_ref, st_ref = ssd.ssd_prefill_varlen(*args, cu, 64)
        y.fill_(7.0)
        st.fill_(7.0)
        print("captured, lengths", i, flush=True)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, y_ref) and torch.equal(st, st_ref), i


def test_rejected_boundaries_leave_a_dealt_call_nothing_to_do(ssd):
    """Decreasing boundaries: no workgroup has an item, nothing is written; the next call of the same workspace is right."""
    T, H, n = 3000, 34, 30
    dev = {k: (v[0] if k in ("x", "dt", "B", "C") else v).cuda()
           for k, v in inputs.make_prefill_inputs(inputs.SSDConfig("t", 1, T, H, 64, 128, 1, 64, "bf16"), seed=64).items()}
    args = [dev[k] for k in ("x", "dt", "A", "B", "C", "D")]
    good = np.concatenate([[0], np.cumsum([100] * n)]).astype(np.int32)
    bad = good.copy()
    bad[7] = bad[9] + 1
    assert ssd.varlen_plan(np.diff(good), H, 64, 128, 1, 64)["dealt"]
    size = int(ssd.raw().ssd_prefill_varlen_workspace_bytes(ssd.make_shape(n, T, H, 64, 128, 1, 64, torch.bfloat16)))
    ws = torch.empty((size,), dtype=torch.uint8, device="cuda")
    y, st = torch.full_like(dev["x"], 3.0), torch.full((n, H, 64, 128), 5.0, device="cuda")
    print("rejected boundaries", flush=True)
    ssd.ssd_prefill_varlen(*args, torch.from_numpy(bad).cuda(), 64, y=y, final_state=st, workspace=ws)
    torch.cuda.synchronize()
    assert (y == 3.0).all() and (st == 5.0).all()
    y_ref, st_ref = ssd.ssd_prefill_varlen(*args, torch.from_numpy(good).cuda(), 64)
    ssd.ssd_prefill_varlen(*args, torch.from_numpy(good).cuda(), 64, y=y, final_state=st, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(y, y_ref) and torch.equal(st, st_ref)
