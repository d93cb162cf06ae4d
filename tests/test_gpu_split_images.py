"""fp32 prefill on split bf16 operands where the blocks' images (split B and C, scores) are made once for all heads."""
import pytest
import torch

from oracle import ssd_oracle
from paper_2603_09555_amd import inputs
from parity import TOL, assert_close

pytestmark = pytest.mark.gpu

CASES = [
    # Bt, T, H, P, N, G, L, h0, blocks per segment (0: the library's choice)
    (1, 1000, 24, 64, 128, 1, 64, False, 4),   # states beside the images; a last block of 8 tokens
    (1, 545, 24, 64, 128, 1, 256, True, 6),    # states in y; a last block of one token
    (2, 300, 6, 96, 72, 2, 32, True, 3),       # dstate 72, slices of one head over two workgroups, two groups
    (1, 97, 16, 32, 16, 1, 16, False, 1),      # dstate 16, segments of a block
    (1, 129, 8, 64, 64, 1, 32, True, 2),
    (1, 1900, 24, 64, 128, 1, 256, True, 0),
]
STATES_IN_Y = {1, 5}  # (of the cases)


@pytest.fixture
def ssd():
    from paper_2603_09555_amd import ssd
    ssd.reset_knobs()
    yield ssd
    ssd.reset_knobs()


def run(ssd, cfg, inp, h0):
    dev = {k: v.cuda() for k, v in inp.items()}
    out = ssd.ssd_prefill(*[dev[k] for k in ("x", "dt", "A", "B", "C", "D")], cfg.chunk, h0=None if h0 is None else h0.cuda())
    torch.cuda.synchronize()
    return out


def setup(ssd, case):
    *dims, with_h0, seg = case
    cfg = inputs.SSDConfig("t", *dims, "f32")
    ssd.set_knob("seg_blocks", seg)
    shape = ssd.make_shape(*dims, torch.float32)
    plan = ssd.prefill_plan(shape)
    print("images", case, plan, flush=True)
    assert plan["path"] == "mfma_f32" and plan["segments"] > 1
    assert ssd.split_f32_memory(shape) == dict(images=True, states_in_y=CASES.index(case) in STATES_IN_Y)
    inp = inputs.make_prefill_inputs(cfg, seed=13)
    return cfg, inp, inputs.make_state(cfg, seed=13, scale=0.3) if with_h0 else None


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_images_match_the_oracle(ssd, case):
    cfg, inp, h0 = setup(ssd, case)
    y, st = run(ssd, cfg, inp, h0)
    y_ref, st_ref = ssd_oracle.prefill(*[inp[k] for k in ("x", "dt", "A", "B", "C", "D")], h0=h0)
    assert_close(y, y_ref, TOL["f32"], "y")
    assert_close(st, st_ref, TOL["f32"], "final state")
    again = run(ssd, cfg, inp, h0)
    assert torch.equal(y, again[0]) and torch.equal(st, again[1])
    ssd.set_knob("split_images", 2)
    assert not ssd.split_f32_memory(ssd.make_shape(*case[:7], torch.float32))["images"]
    without = run(ssd, cfg, inp, h0)   # (the same operations on the same parts)
    assert torch.equal(y, without[0]) and torch.equal(st, without[1])


@pytest.mark.parametrize("case", [c for c in CASES if c[7]], ids=lambda c: "x".join(map(str, c)))
def test_images_with_the_state_in_place(ssd, case):
    """h0 and final_state in one buffer: the first segment then starts from a copy."""
    cfg, inp, h0 = setup(ssd, case)
    y, st = run(ssd, cfg, inp, h0)
    dev = {k: v.cuda() for k, v in inp.items()}
    state = h0.cuda()
    y2, st2 = ssd.ssd_prefill(*[dev[k] for k in ("x", "dt", "A", "B", "C", "D")], cfg.chunk, h0=state, final_state=state)
    torch.cuda.synchronize()
    assert st2.data_ptr() == state.data_ptr() and torch.equal(y, y2) and torch.equal(st, state)


@pytest.mark.parametrize("where", ["B", "C"])
@pytest.mark.parametrize("value", [2.0 ** 31, float("inf"), float("nan")])
def test_a_value_out_of_range_is_found_in_an_image(ssd, where, value):
    """One value of the last group's B or C, in the middle of a segment: tokens before it and the other groups keep the outputs
    they have without it, bit for bit up to its block; its group's outputs from there on are the recurrence's."""
    case = CASES[2]
    cfg, inp, h0 = setup(ssd, case)
    plain = run(ssd, cfg, inp, h0)
    t, g = 32 * 4 + 5, 1   # (the second block of the second segment)
    inp[where][1, t, g, 70] = value
    y, st = run(ssd, cfg, inp, h0)
    y_ref, st_ref = ssd_oracle.prefill(*[inp[k] for k in ("x", "dt", "A", "B", "C", "D")], h0=h0)
    y_ref, st_ref = torch.as_tensor(y_ref).float(), torch.as_tensor(st_ref).float()
    assert torch.equal(y[0], plain[0][0]) and torch.equal(y[1, :32 * 4], plain[0][1, :32 * 4]) and torch.equal(y[1, :, :3], plain[0][1, :, :3])
    got = y[1, 32 * 4:, 3:].cpu()
    ref = y_ref.reshape(y.shape)[1, 32 * 4:, 3:]
    assert torch.equal(torch.isfinite(got), torch.isfinite(ref))
    ok = torch.isfinite(ref)
    # (fp32 outputs of about 200 terms: 1e-4 of the output, or of an ordinary one where terms cancel)
    scale = ref[ok].abs().clamp(min=float(plain[0].abs().max()))
    assert ((got[ok] - ref[ok]).abs() <= 1e-4 * scale).all()
    assert torch.equal(torch.isfinite(st.cpu()), torch.isfinite(st_ref.reshape(st.shape)))
