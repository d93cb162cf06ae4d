"""The step-size map in the prefill kernels: very negative raw values, whose step size is about exp(raw), keep their
relative accuracy."""
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


# A step size's relative error goes into the state as it is.  fp32: at most 2e-7 for the map, and the sums of the state;
# bf16: the bound of every bf16 prefill.
@pytest.mark.parametrize("io, knob, tol", [("f32", ("seg_blocks", 4), 1e-6), ("f32", ("force_mfma_f32", 1), 1e-6),
                                           ("f32", ("force_generic", 1), 1e-6), ("bf16", ("seg_blocks", 0), 2e-2)], ids=str)
def test_small_step_sizes_keep_their_relative_accuracy(ssd, io, knob, tol):
    top = [4.0, -2.0, -6.0, -9.0, -13.0, -17.0, -25.0, -60.0]   # a head each: raw values in [top - 1, top]
    H = len(top)
    cfg = inputs.SSDConfig("t", 2, 200, H, 64, 128, 1, 64, io)
    inp = inputs.make_prefill_inputs(cfg, seed=21)
    g = torch.Generator().manual_seed(22)
    raw = torch.tensor(top) - torch.rand((2, 200, H), generator=g)
    inp["A"] = torch.full((H,), -0.01)
    ssd.reset_knobs()
    ssd.set_knob(*knob)
    print("small step sizes", io, knob, flush=True)
    dev = {k: v.cuda() for k, v in inp.items()}
    _, st = ssd.ssd_prefill(dev["x"], raw.cuda(), dev["A"], dev["B"], dev["C"], dev["D"], cfg.chunk, dt_softplus=True)
    torch.cuda.synchronize()
    ssd.reset_knobs()
    dt = ssd_oracle.dt_transform(raw, None, True, None)
    got = st.cpu().double().numpy()
    for h in range(H):
        one = {k: (v[:, :, h:h + 1] if k == "x" else v[h:h + 1] if k in ("A", "D") else v) for k, v in inp.items()}
        _, ref = ssd_oracle.prefill(one["x"], dt[:, :, h:h + 1], one["A"], one["B"], one["C"], one["D"])
        err = np.linalg.norm(got[:, h] - ref[:, 0]) / np.linalg.norm(ref)
        print("  raw values up to %g: state off by %.2e" % (top[h], err), flush=True)
        assert err <= tol, (top[h], err)
