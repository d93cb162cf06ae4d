"""bf16 prefill with two head slices per workgroup (grids of at most one workgroup per CU) against four: a wave's
arithmetic does not depend on its neighbours, so on the same segments the results are equal bit for bit.  With four
the slots of a group's last workgroup may be without a slice (1, 3, 5 slices per group); with two, those of an odd one."""
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


# batch, tokens, heads, headdim, dstate, groups, chunk; blocks per segment; steps large enough for the steep form
CASES = [((1, 1, 1, 64, 128, 1, 64), 1, False), ((2, 65, 3, 64, 128, 1, 64), 1, False), ((1, 300, 5, 64, 128, 1, 64), 2, False),
         ((1, 640, 6, 64, 64, 2, 128), 3, False), ((2, 333, 2, 128, 256, 2, 64), 2, False), ((1, 500, 5, 64, 128, 1, 64), 3, True),
         ((3, 200, 4, 64, 16, 4, 64), 8, False)]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_two_heads_per_workgroup_equal_four(ssd, case):
    dims, seg_blocks, steep = case
    cfg = inputs.SSDConfig("t", *dims, "bf16")
    inp = inputs.make_prefill_inputs(cfg, seed=31)
    if steep:
        inp["dt"] = inp["dt"] * torch.from_numpy(np.random.default_rng(2).choice([1.0, 40.0], inp["dt"].shape)).float()
    h0 = 0.1 * inputs.make_state(cfg, seed=31)
    dev = {k: v.cuda() for k, v in inp.items()}
    out = {}
    for heads in (2, 4):
        ssd.reset_knobs()
        ssd.set_knob("seg_blocks", seg_blocks)
        ssd.set_knob("scan_heads", heads)
        print("two heads against four", case, heads, flush=True)
        out[heads] = ssd.ssd_prefill(dev["x"], dev["dt"], dev["A"], dev["B"], dev["C"], dev["D"], cfg.chunk, h0=h0.cuda())
        torch.cuda.synchronize()
    ssd.reset_knobs()
    assert torch.equal(out[2][0], out[4][0]) and torch.equal(out[2][1], out[4][1])
    y_ref, st_ref = ssd_oracle.prefill(inp["x"], inp["dt"], inp["A"], inp["B"], inp["C"], inp["D"], h0=h0)
    assert_close(out[2][0], y_ref, TOL["bf16"], "y")
    assert_close(out[2][1], st_ref, TOL["bf16"], "final state")


@pytest.mark.parametrize("heads", [1, 3, 6])
def test_packed_batch_two_heads_per_workgroup_equal_four(ssd, heads):
    lens = [0, 1, 64, 700, 65, 129]
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    cfg = inputs.SSDConfig("t", 1, int(cu[-1]), heads, 64, 128, 1, 64, "bf16")
    inp = {k: (v[0] if k in ("x", "dt", "B", "C") else v) for k, v in inputs.make_prefill_inputs(cfg, seed=32).items()}
    dev = {k: v.cuda() for k, v in inp.items()}
    out = {}
    for n in (2, 4):
        ssd.reset_knobs()
        ssd.set_knob("seg_blocks", 2)
        ssd.set_knob("scan_heads", n)
        print("packed", heads, n, flush=True)
        out[n] = ssd.ssd_prefill_varlen(dev["x"], dev["dt"], dev["A"], dev["B"], dev["C"], dev["D"], cu.cuda(), 64)
        torch.cuda.synchronize()
    ssd.reset_knobs()
    assert torch.equal(out[2][0], out[4][0]) and torch.equal(out[2][1], out[4][1])
    y_ref, st_ref = ssd_oracle.prefill_varlen(inp["x"], inp["dt"], inp["A"], inp["B"], inp["C"], inp["D"], cu.numpy())
    assert_close(out[2][0], y_ref, TOL["bf16"], "y")
    assert_close(out[2][1], st_ref, TOL["bf16"], "final state")
