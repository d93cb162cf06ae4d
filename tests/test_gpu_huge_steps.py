"""Prefill behind tokens that decay everything away: there is no upper bound on dt |A|."""
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


# fp32: at most two such tokens per block of 64 or chunk of 128, cut off at 160 each: the prefix sums are held to 2^-16, the
# decay between two tokens to a few times that.  bf16: the bound of every bf16 prefill.
@pytest.mark.parametrize("io, knob, tol", [("bf16", ("seg_blocks", 2), 2e-2), ("bf16", ("force_generic", 1), 2e-2),
                                           ("f32", ("force_mfma_f32", 1), 5e-5), ("f32", ("force_generic", 1), 5e-5),
                                           ("f32", ("seg_blocks", 4), 5e-5)], ids=str)
@pytest.mark.parametrize("size", [1e4, 1e7])
def test_tokens_of_any_size(ssd, io, knob, tol, size):
    H, T = 5, 400
    cfg = inputs.SSDConfig("t", 1, T, H, 64, 128, 1, 128, io)
    inp = inputs.make_prefill_inputs(cfg, seed=18)
    inp["D"].zero_()
    # at the start of a block, in either half, and twice
    for t, h in ((64, 0), (70, 1), (110, 2), (3, 3), (50, 3), (130, 3), (200, 3)):
        inp["dt"][0, t, h] = size / -inp["A"][h]
        inp["x"][0, t, h] = (inp["x"][0, t, h].float() / size).to(inp["x"].dtype)   # (its own input would drown the rest)
    ssd.reset_knobs()
    ssd.set_knob(*knob)
    print("tokens of size", size, io, knob, flush=True)
    y, st = ssd.ssd_prefill(*[inp[k].cuda() for k in ("x", "dt", "A", "B", "C", "D")], cfg.chunk)
    torch.cuda.synchronize()
    ssd.reset_knobs()
    y_ref, st_ref = ssd_oracle.prefill(inp["x"], inp["dt"], inp["A"], inp["B"], inp["C"], inp["D"])
    mag, st_mag = ssd_oracle.prefill(inp["x"].abs(), inp["dt"], inp["A"], inp["B"].abs(), inp["C"].abs(), inp["D"])
    for got, ref, m, what in ((y, y_ref, mag, "y"), (st, st_ref, st_mag, "final state")):
        err = np.linalg.norm(got.double().cpu().numpy() - ref, axis=-1) / np.linalg.norm(m, axis=-1)
        print("  %s off by at most %.2e of its terms" % (what, err.max()), flush=True)
        assert err.max() <= tol, what
