"""The bf16 full scan with two heads per workgroup (feeding and computing waves): walks longer than the 64 blocks whose
decay factors a wave holds at a time, steep blocks on both sides of that, segments that the scan folds itself, and the
rule that chooses it.  The four-head kernel is the reference (the same arithmetic: equal bit for bit), the short walks of
test_gpu_scan_heads.py compare both with the oracle."""
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
    for knob, value in (("scan_heads", 4), ("seg_blocks", 2)):
        ssd.set_knob(knob, value)
        assert plan(8, 4096, 48) is None
        ssd.reset_knobs()


# batch, tokens, heads, headdim, dstate, groups; blocks per segment
@pytest.mark.parametrize("heads", [2, 4])
@pytest.mark.parametrize("dims, seg", [((2, 333, 3, 64, 128, 1), 6), ((1, 700, 5, 64, 72, 1), 3), ((2, 449, 6, 64, 128, 2), 2), ((1, 200, 1, 128, 256, 1), 4)],
                         ids=str)
def test_cache_policy_of_the_y_stores_of_either_kernel(ssd, heads, dims, seg):
    """Non-temporal and ordinary stores of y by the same kernel: ragged tails, workgroups with a head short, several groups and
    state slices, plain and packed batches.  Equal bit for bit and as the oracle has it."""
    cfg = inputs.SSDConfig("t", *dims, 64, "bf16")
    inp = inputs.make_prefill_inputs(cfg, seed=45)
    dev = {k: v.cuda() for k, v in inp.items()}
    Bt, T = dims[:2]
    flat = lambda t: t.reshape(Bt * T, *t.shape[2:]).contiguous()   # noqa: E731
    cu = torch.tensor([0, 70] + ([T] if Bt > 1 else []) + [Bt * T], dtype=torch.int32, device="cuda")
    out = []
    for policy in (0, 1):
        ssd.reset_knobs()
        ssd.set_knob("scan_heads", heads)
        ssd.set_knob("seg_blocks", seg)
        ssd.set_knob("y_stream", policy)
        print("y store policy", policy, heads, dims, seg, flush=True)
        y, st = ssd.ssd_prefill(*[dev[k] for k in ("x", "dt", "A", "B", "C", "D")], cfg.chunk)
        yp, stp = ssd.ssd_prefill_varlen(flat(dev["x"]), flat(dev["dt"]), dev["A"], flat(dev["B"]), flat(dev["C"]), dev["D"], cu, cfg.chunk)
        torch.cuda.synchronize()
        out.append((y, st, yp, stp))
    ssd.reset_knobs()
    assert all(torch.equal(a, b) for a, b in zip(*out))
    y_ref, st_ref = ssd_oracle.prefill(*[inp[k] for k in ("x", "dt", "A", "B", "C", "D")])
    assert_close(out[1][0], y_ref, TOL["bf16"], "streamed y")
    assert_close(out[1][1], st_ref, TOL["bf16"], "final state beside streamed y")
    c = [flat(inp[k]) if k not in "AD" else inp[k] for k in ("x", "dt", "A", "B", "C", "D")]
    y_ref, st_ref = ssd_oracle.prefill_varlen(*c, cu.cpu().numpy())
    assert_close(out[1][2], y_ref, TOL["bf16"], "streamed y, packed batch")
    assert_close(out[1][3], st_ref, TOL["bf16"], "final states, packed batch")
