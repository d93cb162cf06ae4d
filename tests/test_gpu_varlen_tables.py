"""The tables of a packed batch at the edges of the one-workgroup kernel: around a wave and a workgroup of sequences,
beyond it (two kernels), and lists longer than one trip of its threads."""
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


def lengths(nseq, kind):
    r = np.random.default_rng(nseq)
    if kind == "short":          # empty ones among them
        return r.integers(0, 7, nseq)
    if kind == "mixed":          # some of several segments
        ln = r.integers(0, 40, nseq)
        ln[:: max(1, nseq // 4)] += 700
        return ln
    return np.full(nseq, 64 * 1200 // nseq)   # "blocks": more 64-token blocks than threads


@pytest.mark.parametrize("io", ["bf16", "f32"])   # f32: the generic kernels, whose blocks are chunks
@pytest.mark.parametrize("case", [(1, "mixed"), (63, "mixed"), (64, "mixed"), (65, "mixed"), (1024, "short"), (1025, "short"),
                                  (2, "blocks")], ids=str)
def test_packed_batch_tables(ssd, case, io):
    nseq, kind = case
    lens = lengths(nseq, kind)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, H, P, N, L = int(cu[-1]), 2, 64, 128 if io == "bf16" else 16, 64
    cfg = inputs.SSDConfig("t", 1, T, H, P, N, 1, L, io)
    inp = inputs.make_prefill_inputs(cfg, seed=13)
    pk = {k: (v[0] if k in ("x", "dt", "B", "C") else v) for k, v in inp.items()}
    h0 = inputs.make_state(inputs.SSDConfig("h", nseq, 1, H, P, N, 1, L, io), seed=13, scale=0.1)
    print("packed tables", case, io, "tokens", T, flush=True)
    dev = {k: v.cuda() for k, v in pk.items()}
    y, st = ssd.ssd_prefill_varlen(dev["x"], dev["dt"], dev["A"], dev["B"], dev["C"], dev["D"], torch.from_numpy(cu).cuda(), L,
                                   h0=h0.cuda())
    torch.cuda.synchronize()
    y_ref, st_ref = ssd_oracle.prefill_varlen(pk["x"], pk["dt"], pk["A"], pk["B"], pk["C"], pk["D"], cu, h0=h0)
    assert_close(y, y_ref, TOL[io], "y")
    assert_close(st, st_ref, TOL[io], "final state")


@pytest.mark.parametrize("nseq", [3, 1024, 1025])
def test_rejected_boundaries_write_nothing(ssd, nseq):
    T, H = 2000, 2
    cfg = inputs.SSDConfig("t", 1, T, H, 64, 128, 1, 64, "bf16")
    dev = {k: (v[0] if k in ("x", "dt", "B", "C") else v).cuda() for k, v in inputs.make_prefill_inputs(cfg, seed=1).items()}
    cu = np.linspace(0, T, nseq + 1).astype(np.int32)
    cu[nseq // 2 + 1] = cu[nseq // 2] - 1   # decreasing once
    y, st = torch.full_like(dev["x"], 3.0), torch.full((nseq, H, 64, 128), 5.0, device="cuda")
    ssd.ssd_prefill_varlen(dev["x"], dev["dt"], dev["A"], dev["B"], dev["C"], dev["D"], torch.from_numpy(cu).cuda(), 64, y=y,
                           final_state=st)
    torch.cuda.synchronize()
    assert (y == 3.0).all() and (st == 5.0).all()


@pytest.mark.parametrize("lens", [[4000] + 64 * [1], 40 * [1] + [2500, 0, 1300], [7000] + 1023 * [1], [64, 65, 129, 2000]],
                         ids=lambda v: "%dx" % len(v))
def test_one_long_prompt_among_short_rows(ssd, lens):
    """The segment length is chosen on the device from the lengths: several segments for the long ones."""
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, H, P, N, L = int(cu[-1]), 6, 64, 128, 64
    plan = ssd.varlen_plan(lens, H, P, N, 1, L)
    print("one long prompt among short rows", len(lens), plan, flush=True)
    assert plan["chosen"] and plan["items"] > len(lens)
    pk = {k: (v[0] if k in ("x", "dt", "B", "C") else v)
          for k, v in inputs.make_prefill_inputs(inputs.SSDConfig("t", 1, T, H, P, N, 1, L, "bf16"), seed=14).items()}
    h0 = inputs.make_state(inputs.SSDConfig("h", len(lens), 1, H, P, N, 1, L, "bf16"), seed=14, scale=0.1)
    dev = {k: v.cuda() for k, v in pk.items()}
    y, st = ssd.ssd_prefill_varlen(dev["x"], dev["dt"], dev["A"], dev["B"], dev["C"], dev["D"], torch.from_numpy(cu).cuda(), L,
                                   h0=h0.cuda())
    torch.cuda.synchronize()
    y_ref, st_ref = ssd_oracle.prefill_varlen(pk["x"], pk["dt"], pk["A"], pk["B"], pk["C"], pk["D"], cu, h0=h0)
    assert_close(y, y_ref, TOL["bf16"], "y")
    assert_close(st, st_ref, TOL["bf16"], "final state")


def test_captured_call_follows_the_lengths(ssd):
    """The lengths and the segment length they lead to are the device's: a captured call is right for whatever boundaries its
    tensor holds at a replay, with eager work in between."""
    T, H, nseq = 3000, 4, 12
    dev = {k: (v[0] if k in ("x", "dt", "B", "C") else v).cuda()
           for k, v in inputs.make_prefill_inputs(inputs.SSDConfig("t", 1, T, H, 64, 128, 1, 64, "bf16"), seed=15).items()}
    args = [dev[k] for k in ("x", "dt", "A", "B", "C", "D")]
    lens = [[250] * 12, [T - 11] + [1] * 11, [0, 1400, 1, 700, 0, 3, 64, 65, 128, 500, 100, 39]]
    assert len({ssd.varlen_plan(v, H, 64, 128, 1, 64)["items"] for v in lens}) == 3
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
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, y_ref) and torch.equal(st, st_ref), i
