"""The bf16 full scan with two heads per workgroup (feeding and computing waves): walks longer than the 64 blocks whose
decay factors a wave holds at a time, steep blocks on both sides of that, segments that the scan folds itself, and the
rule that chooses it.  The four-head kernel is the reference (the same arithmetic: equal bit for bit), the short walks of
test_gpu_scan_heads.py compare both with the oracle."""
import pytest
import torch

from paper_2603_09555_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ssd():
    from paper_2603_09555_amd import ssd
    yield ssd
    ssd.reset_knobs()


# blocks, tokens short of them, blocks per segment (0: one), steep blocks
CASES = [(64, 0, 0, ()), (65, 63, 0, (63, 64)), (66, 1, 0, (0, 65)), (129, 0, 0, (127, 128)), (133, 17, 66, (64,)), (5, 3, 2, ())]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_long_walks_equal_four_heads(ssd, case):
    blocks, short, seg, steep = case
    cfg = inputs.SSDConfig("t", 1, 64 * blocks - short, 3, 64, 128, 1, 256, "bf16")
    inp = inputs.make_prefill_inputs(cfg, seed=41)
    for b in steep:
        inp["dt"][:, 64 * b:64 * b + 9] *= 60.0
    dev = {k: v.cuda() for k, v in inp.items()}
    h0 = 0.1 * inputs.make_state(cfg, seed=41).cuda()
    out = {}
    for heads in (2, 4):
        ssd.reset_knobs()
        ssd.set_knob("seg_blocks", seg or blocks)
        ssd.set_knob("scan_heads", heads)
        print("pair scan", case, heads, flush=True)
        out[heads] = ssd.ssd_prefill(dev["x"], dev["dt"], dev["A"], dev["B"], dev["C"], dev["D"], cfg.chunk, h0=h0)
        torch.cuda.synchronize()
    ssd.reset_knobs()
    assert torch.isfinite(out[4][0]).all()
    assert torch.equal(out[2][0], out[4][0]) and torch.equal(out[2][1], out[4][1])


def test_rule(ssd):
    def plan(batch, tokens, heads, alias=False):
        return ssd.prefill_pair_plan(ssd.make_shape(batch, tokens, heads, 64, 128, 1, 256, torch.bfloat16), alias)
    ssd.reset_knobs()
    assert plan(8, 4096, 48) == dict(seg_blocks=64, segments=1, parts=1, fold=False, heads=2, state_heads=2)
    assert plan(1, 4096, 512)["segments"] == 1 and plan(1, 4096, 513) is None   # more sequences than CUs
    for batch, tokens, heads in ((1, 700, 100), (3, 3001, 20), (1, 16384, 80), (2, 40000, 3)):
        p = plan(batch, tokens, heads)
        assert p["heads"] == 2 and batch * -(-heads // 2) * p["segments"] <= 256
        assert p["segments"] == -(-(-(-tokens // 64)) // p["seg_blocks"]) and p["seg_blocks"] % p["parts"] == 0
        assert not plan(batch, tokens, heads, True)["fold"]
    for knob, value in (("scan_heads", 4), ("y_stream", 1), ("seg_blocks", 2)):
        ssd.set_knob(knob, value)
        assert plan(8, 4096, 48) is None
        ssd.reset_knobs()
