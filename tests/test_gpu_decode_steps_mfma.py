"""Multi-step decode as contractions over blocks of 32 steps (bf16 io, 9 steps and more), against the oracle and
against single steps."""
import numpy as np
import pytest
import torch

from oracle import ssd_oracle
from parity import TOL, assert_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ssd():
    from paper_2603_09555_amd import ssd
    return ssd


def make(S, Ly, Bt, H, P, N, G, dt_scale=0.1, seed=91):
    g = torch.Generator().manual_seed(seed)
    state = torch.randn((Ly, Bt, H, P, N), generator=g)
    x = torch.randn((S, Ly, Bt, H, P), generator=g).bfloat16()
    dt = torch.rand((S, Ly, Bt, H), generator=g) * dt_scale + 1e-3
    A = -(torch.rand((Ly, H), generator=g) * 15 + 1)
    D = torch.randn((Ly, H), generator=g)
    B = (0.25 * torch.randn((S, Ly, Bt, G, N), generator=g)).bfloat16()
    C = (0.25 * torch.randn((S, Ly, Bt, G, N), generator=g)).bfloat16()
    return state, x, dt, A, B, C, D


CASES = [
    # steps, Ly, Bt, H, P, N, G, largest dt
    (9, 2, 2, 8, 64, 128, 1, 0.1),      # the fewest steps that take this kernel
    (31, 1, 2, 5, 64, 128, 1, 0.1),     # a block less one; slices no multiple of a workgroup's four
    (32, 2, 1, 4, 128, 128, 2, 0.1),    # exactly one block
    (33, 1, 1, 6, 64, 64, 2, 0.1),      # one step into the second block; dstate 64
    (70, 2, 1, 3, 96, 128, 3, 0.1),     # three blocks; one head, three slices per group
    (40, 1, 3, 4, 32, 64, 4, 0.1),      # one slice per group
    (37, 1, 1, 4, 64, 128, 1, 1.5),     # steep decay: up to 24 per step
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_blocked_steps_match_oracle(ssd, case):
    state, x, dt, A, B, C, D = make(*case)
    print("blocked decode steps", case, flush=True)
    sd = state.cuda()
    y = ssd.ssd_decode_steps_layers(sd, *[t.cuda() for t in (x, dt, A, B, C, D)])
    torch.cuda.synchronize()
    y_ref, st_ref = ssd_oracle.decode_steps_layers(state, x, dt, A, B, C, D)
    assert_close(y, y_ref, TOL["bf16"], "y")
    assert_close(sd, st_ref, 1e-5, "state")   # fp32 throughout: the bound the step-by-step kernel is held to
    # run to run the same bits
    s2 = state.cuda()
    y2 = ssd.ssd_decode_steps_layers(s2, *[t.cuda() for t in (x, dt, A, B, C, D)])
    torch.cuda.synchronize()
    assert torch.equal(y, y2) and torch.equal(sd, s2)


def test_blocked_steps_apply_the_step_size_map(ssd):
    S, Ly, Bt, H = 35, 2, 2, 4
    state, x, _, A, B, C, D = make(S, Ly, Bt, H, 64, 128, 1)
    g = torch.Generator().manual_seed(5)
    raw, bias = 0.5 * torch.randn((S, Ly, Bt, H), generator=g) - 3, 0.3 * torch.randn((Ly, H), generator=g)
    dt = torch.nn.functional.softplus(raw.double() + bias.double()[None, :, None, :]).clamp(1e-3, 1e-1).float()
    sd = state.cuda()
    y = ssd.ssd_decode_steps_layers(sd, *[t.cuda() for t in (x, raw, A, B, C, D)], dt_bias=bias.cuda(), dt_softplus=True,
                                    dt_limit=(1e-3, 1e-1))
    torch.cuda.synchronize()
    y_ref, st_ref = ssd_oracle.decode_steps_layers(state, x, dt, A, B, C, D)
    assert_close(y, y_ref, TOL["bf16"], "y")
    assert_close(sd, st_ref, 1e-5, "state")


@pytest.mark.parametrize("where", ["x", "B", "C", "dt", "state"])
def test_blocked_steps_keep_infinities_where_the_recurrence_has_them(ssd, where):
    """An infinity or a NaN reaches exactly the outputs that single steps let it reach: nothing earlier, no other head."""
    S, Ly, Bt, H, P, N, G = 40, 1, 2, 4, 64, 128, 1
    state, x, dt, A, B, C, D = make(S, Ly, Bt, H, P, N, G)
    if where == "x":
        x[34, 0, 0, 1, 7] = float("inf")
    elif where == "B":
        B[10, 0, 1, 0, 5] = float("nan")
    elif where == "C":
        C[33, 0, 0, 0, 100] = float("-inf")
    elif where == "dt":
        dt[36, 0, 1, 2] = float("nan")
    else:
        state[0, 1, 3, 60, 127] = float("inf")
    dev = [t.cuda() for t in (x, dt, A, B, C, D)]
    sd, s1 = state.cuda(), state.cuda()
    y = ssd.ssd_decode_steps_layers(sd, *dev)
    y1 = torch.stack([ssd.ssd_decode_step_layers(s1, dev[0][i].clone(), dev[1][i].clone(), dev[2], dev[3][i].clone(),
                                                 dev[4][i].clone(), dev[5]) for i in range(S)])
    torch.cuda.synchronize()
    for got, ref, tol in ((y.float(), y1.float(), TOL["bf16"]), (sd, s1, 1e-5)):
        assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isinf(got), torch.isinf(ref))
        ok = torch.isfinite(ref)
        assert_close(torch.where(ok, got, 0.0), np.asarray(torch.where(ok, ref, 0.0).cpu(), dtype=np.float64), tol, where)


@pytest.mark.parametrize("size", [1e3, 1e5, 1e12])
def test_blocked_steps_are_exact_behind_steps_of_any_size(ssd, size):
    """Steps that decay everything away (dt |A| = size), at the start, in the middle and twice in a block: the decay between
    the gentle steps behind them is not to be had from prefix sums that hold the large ones to 24 bits.  Every product and
    sum is fp32 with a largest exponent of a few units, some 1e-6; then y is rounded to bf16, at most 2^-8 of the value."""
    S, Ly, Bt, H, P, N, G = 40, 1, 1, 4, 64, 128, 1
    state, x, dt, A, B, C, D = make(S, Ly, Bt, H, P, N, G, dt_scale=1e-3)
    D.zero_()
    for s, h in ((3, 0), (16, 1), (2, 2), (7, 2), (33, 2)):
        dt[s, 0, 0, h] = size / -A[0, h]
        x[s, 0, 0, h] = (x[s, 0, 0, h].float() / size).bfloat16()   # (its own input would drown what follows)
    sd = state.cuda()
    print("blocked decode steps behind a step of", size, flush=True)
    y = ssd.ssd_decode_steps_layers(sd, *[t.cuda() for t in (x, dt, A, B, C, D)])
    torch.cuda.synchronize()
    y_ref, st_ref = ssd_oracle.decode_steps_layers(state, x, dt, A, B, C, D)
    got = y.float().cpu().double().numpy()
    for s in range(S):
        for h in range(H):
            err = np.linalg.norm(got[s, 0, 0, h] - y_ref[s, 0, 0, h]) / np.linalg.norm(y_ref[s, 0, 0, h])
            assert err <= 2.0 ** -8, (s, h, err)
    assert_close(sd, st_ref, 1e-5, "state")


@pytest.mark.parametrize("where", ["B and C", "x and B", "state"])
def test_blocked_steps_with_values_whose_products_leave_fp32(ssd, where):
    """Large B and C (or x) at one step whose counterpart is as small: the recurrence multiplies a large one by a small one,
    a score C.B would overflow.  As single steps, head by head."""
    S, Ly, Bt, H, P, N, G = 40, 1, 1, 4, 64, 128, 1
    state, x, dt, A, B, C, D = make(S, Ly, Bt, H, P, N, G)
    D.zero_()
    def scale(t, s, by):
        t[s] = (t[s].float() * by).bfloat16()
    if where == "B and C":
        scale(B, 34, 1e22), scale(C, 34, 1e22), scale(x, 34, 1e-22)
        state.mul_(1e-20)
    elif where == "x and B":
        scale(x, 5, 1e25), scale(B, 5, 1e-25)
    else:
        state[0, 0, 2] *= 1e34
        scale(C, 7, 1e-30)
    dev = [t.cuda() for t in (x, dt, A, B, C, D)]
    sd, s1 = state.cuda(), state.cuda()
    print("blocked decode steps, large", where, flush=True)
    y = ssd.ssd_decode_steps_layers(sd, *dev)
    y1 = torch.stack([ssd.ssd_decode_step_layers(s1, dev[0][i].clone(), dev[1][i].clone(), dev[2], dev[3][i].clone(),
                                                 dev[4][i].clone(), dev[5]) for i in range(S)])
    torch.cuda.synchronize()
    got, ref = y.double()[:, 0, 0], y1.double()[:, 0, 0]
    assert torch.isfinite(got).all() and torch.isfinite(ref).all()
    assert ((got - ref).norm(dim=-1) <= 2.0 ** -8 * ref.norm(dim=-1)).all()
    assert ((sd - s1).double().flatten(3).norm(dim=-1) <= 1e-5 * s1.double().flatten(3).norm(dim=-1)).all()


@pytest.mark.parametrize("S, H, P, N", [(9, 8, 32, 128), (21, 8, 32, 128), (10, 8, 64, 64)])
def test_few_slices_per_group_stay_on_the_step_by_step_kernel(ssd, S, H, P, N):
    """A B/C group per head, more workgroups than run side by side, few steps: half of the blocked kernel's waves would have
    no slice.  The step-by-step kernel's state is that of single steps bit for bit."""
    Ly, Bt = 12, 8
    state, x, dt, A, B, C, D = make(S, Ly, Bt, H, P, N, H)
    dev = [t.cuda() for t in (x, dt, A, B, C, D)]
    sd, s1 = state.cuda(), state.cuda()
    print("few slices per group", S, H, P, N, flush=True)
    y = ssd.ssd_decode_steps_layers(sd, *dev)
    for i in range(S):
        ssd.ssd_decode_step_layers(s1, dev[0][i].clone(), dev[1][i].clone(), dev[2], dev[3][i].clone(), dev[4][i].clone(), dev[5])
    torch.cuda.synchronize()
    assert torch.equal(sd, s1)
    y_ref, _ = ssd_oracle.decode_steps_layers(state, x, dt, A, B, C, D)
    assert_close(y, y_ref, TOL["bf16"], "y")


@pytest.mark.parametrize("raw", [False, True])
@pytest.mark.parametrize("P, N, G", [(64, 128, 1), (32, 64, 2)])
def test_blocked_steps_carry_the_state_in_fp32(ssd, raw, P, N, G):
    """Products with bf16 values are exact and sums are fp32: the state is off by a few roundings of 2^-24, with the raw step
    size (its bias has an axis of layers) also by the map's 2e-7 and the sum's with the bias.  Two parts instead of three
    would leave 2^-16."""
    S, Ly, Bt, H = 64, 3, 2, 4
    state, x, dt, A, B, C, D = make(S, Ly, Bt, H, P, N, G, seed=93)
    kw = {}
    if raw:
        g = torch.Generator().manual_seed(6)
        dt, bias = 0.5 * torch.randn((S, Ly, Bt, H), generator=g), 0.1 * torch.randn((Ly, H), generator=g) - 4.6
        kw = dict(dt_bias=bias.cuda(), dt_softplus=True, dt_limit=(1e-3, 1e-1))
    sd = state.cuda()
    ssd.ssd_decode_steps_layers(sd, *[t.cuda() for t in (x, dt, A, B, C, D)], **kw)
    torch.cuda.synchronize()
    if raw:
        v = dt.double() + bias.double()[None, :, None, :]
        dt = torch.nn.functional.softplus(v, threshold=1e9).clamp(1e-3, 1e-1)
    h = state.double()
    for s in range(S):   # the recurrence in 64 bits
        Bs = B[s].double().repeat_interleave(H // G, dim=2)
        h = torch.exp(dt[s].double() * A.double()[:, None, :])[..., None, None] * h \
            + (dt[s].double()[..., None] * x[s].double())[..., None] * Bs[:, :, :, None, :]
    err = float((sd.cpu().double() - h).norm() / h.norm())
    print("  state off by %.2e" % err, flush=True)
    assert err <= 5e-7
