"""The work this library is measured on: what users have it do, through its public entry points.

A case is a dict of plain values whose "kind" names the entry points it goes through:

* ``prefill``       ``ssd_prefill`` of a batch of prompts (bf16 or fp32 io, with or without a carried state and
                    the raw step size whose bias, softplus and clamp the kernels apply)
* ``varlen``        ``ssd_prefill_varlen`` of a packed ragged batch
* ``token``         one layer's generation step: ``ssd_conv1d_step``, then ``ssd_decode_step`` on what it returns
* ``layers``        ``ssd_decode_step_layers``: one token for a stack of layers in one call
* ``steps``         ``ssd_decode_steps_layers``: several known tokens (a short continuation, a draft) in one call
* ``conv``          ``ssd_conv1d_prefill``: the convolution in front of the core over a whole prompt

Value distributions are those of ``paper_2603_09555_amd.inputs``.  Output, state and workspace tensors are
allocated once, as a serving loop does.
"""
import math
import random

import torch

from paper_2603_09555_amd import inputs, ssd

# Standard deviation of the state a long prompt of these inputs leaves: the step size is about 0.01, B about
# 0.25 and a head remembers some 10 to 50 tokens.
STATE_SCALE = 0.02
DT_LIMIT = (1e-3, 1e-1)
CONV_TAPS = 4


def listed():
    return [
        # the smallest prompt, in the fp32 of a parity run: latency of a call
        dict(name="tiny_f32", kind="prefill", io="f32", batch=1, seqlen=512, heads=4, headdim=32, dstate=16, groups=1,
             chunk=64, carried=False, raw_dt=False),
        # one layer of a 130M-shaped model in fp32, as numerics are checked or small models are run
        dict(name="layer_f32", kind="prefill", io="f32", batch=1, seqlen=2048, heads=24, headdim=64, dstate=128,
             groups=1, chunk=256, carried=False, raw_dt=False),
        # the same layer in bf16: an interactive prompt on a small model
        dict(name="small_bf16", kind="prefill", io="bf16", batch=1, seqlen=2048, heads=24, headdim=64, dstate=128,
             groups=1, chunk=256, carried=False, raw_dt=False),
        # an offline batch of equal prompts on a 780M-shaped layer
        dict(name="batch8_bf16", kind="prefill", io="bf16", batch=8, seqlen=4096, heads=48, headdim=64, dstate=128,
             groups=1, chunk=256, carried=False, raw_dt=False),
        # one long prompt on a 2.7B-shaped layer
        dict(name="long_bf16", kind="prefill", io="bf16", batch=1, seqlen=16384, heads=80, headdim=64, dstate=128,
             groups=1, chunk=256, carried=False, raw_dt=False),
        # a later piece of a few prompts of no round length: state carried in, step size still raw
        dict(name="continued_odd", kind="prefill", io="bf16", batch=3, seqlen=3001, heads=20, headdim=64, dstate=128,
             groups=1, chunk=256, carried=True, raw_dt=True),
        # a server's ragged batch of prompts, packed along the token axis
        dict(name="packed_ragged", kind="varlen", io="bf16", nseq=64, tokens=16384, lens_seed=8, heads=80, headdim=64,
             dstate=128, groups=1, chunk=256, carried=False, raw_dt=False),
        # one layer of a model that is stepped layer by layer: the smallest calls of generation
        dict(name="token_layer", kind="token", io="bf16", batch=1, heads=80, headdim=64, dstate=128, groups=1),
        # generation for one user: all layers of a 2.7B-shaped model
        dict(name="decode_b1", kind="layers", io="bf16", layers=64, batch=1, heads=80, headdim=64, dstate=128,
             groups=1, raw_dt=False),
        # generation for a batch of users: the states of all layers stream through memory
        dict(name="decode_b16", kind="layers", io="bf16", layers=64, batch=16, heads=80, headdim=64, dstate=128,
             groups=1, raw_dt=False),
        # 64 known tokens continued from the cache in one call
        dict(name="steps_64", kind="steps", io="bf16", steps=64, layers=64, batch=1, heads=80, headdim=64, dstate=128,
             groups=1, raw_dt=False),
        # the convolution in front of the long prompt
        dict(name="conv_long", kind="conv", io="bf16", batch=1, seqlen=16384, heads=80, headdim=64, dstate=128,
             groups=1, carried=False),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cut(value, limit, lo):
    """value, or below it where the limit asks for that"""
    return max(lo, min(value, int(limit)))


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "prefill_f32", "prefill_f32", "varlen", "token", "layers", "steps", "steps",
                       "conv"])
    groups = rng.choice([1, 1, 1, 2, 4])
    heads = groups * rng.randint(4, max(4, 80 // groups))   # any number of heads per group
    headdim, dstate = rng.choice([64, 64, 64, 128]), rng.choice([64, 128, 128, 256])
    chunk, carried, raw = rng.choice([64, 128, 256]), rng.random() < 0.4, rng.random() < 0.4
    width = heads * headdim
    if kind == "prefill":
        batch = _log_int(rng, 1, 16)
        # tokens x columns x state columns of the largest listed prompts
        most = 8 * 4096 * 48 * 64 * 128 // (batch * width * max(dstate, 128))
        return dict(kind=kind, io="bf16", batch=batch, seqlen=_cut(_log_int(rng, 200, 16384), most, 64), heads=heads,
                    headdim=headdim, dstate=dstate, groups=groups, chunk=chunk, carried=carried, raw_dt=raw)
    if kind == "prefill_f32":
        heads = groups * rng.randint(1, max(1, 32 // groups))
        headdim, dstate, batch = rng.choice([32, 64, 64]), rng.choice([16, 64, 128, 128]), _log_int(rng, 1, 8)
        most = 8 * 2048 * 24 * 64 // (batch * heads * headdim)
        return dict(kind="prefill", io="f32", batch=batch, seqlen=_cut(_log_int(rng, 100, 4096), most, 64),
                    heads=heads, headdim=headdim, dstate=dstate, groups=groups, chunk=chunk, carried=carried, raw_dt=raw)
    if kind == "varlen":
        most = 16384 * 80 * 64 * 128 // (width * max(dstate, 128))
        tokens = _cut(_log_int(rng, 512, 16384), most, 256)
        # (every sequence also stores a state of its own: no more of them than 64-token prompts)
        return dict(kind=kind, io="bf16", nseq=min(_log_int(rng, 2, 128), tokens // 64), tokens=tokens,
                    lens_seed=rng.randrange(1000), heads=heads, headdim=headdim, dstate=dstate, groups=groups,
                    chunk=chunk, carried=carried, raw_dt=raw)
    if kind == "token":
        return dict(kind=kind, io="bf16", batch=_log_int(rng, 1, 64), heads=heads, headdim=headdim, dstate=dstate,
                    groups=groups)
    if kind == "layers":
        layers = _log_int(rng, 1, 64)
        most = 64 * 16 * 80 * 64 * 128 // (layers * width * dstate)
        return dict(kind=kind, io=rng.choice(["bf16", "bf16", "f32"]), layers=layers,
                    batch=_cut(_log_int(rng, 1, 64), most, 1), heads=heads, headdim=headdim, dstate=dstate,
                    groups=groups, raw_dt=raw)
    if kind == "steps":
        headdim, dstate = rng.choice([(64, 128), (64, 128), (64, 64), (128, 128)])
        layers, steps = _log_int(rng, 1, 64), _log_int(rng, 2, 64)
        most = 64 * 64 * 80 * 64 * 128 // (layers * steps * heads * headdim * dstate)
        return dict(kind=kind, io="bf16", steps=steps, layers=layers, batch=_cut(_log_int(rng, 1, 16), most, 1),
                    heads=heads, headdim=headdim, dstate=dstate, groups=groups, raw_dt=raw)
    batch = _log_int(rng, 1, 16)
    most = 16384 * 5376 // (batch * (width + 2 * groups * dstate))
    return dict(kind="conv", io="bf16", batch=batch, seqlen=_cut(_log_int(rng, 64, 16384), most, 16), heads=heads,
                headdim=headdim, dstate=dstate, groups=groups, carried=carried)


def _lengths(case):
    """Prompt lengths of a packed batch: log-uniform over a factor of 64, summing to the token count."""
    r = random.Random(case["lens_seed"])
    w = [math.exp(r.uniform(0.0, math.log(64.0))) for _ in range(case["nseq"])]
    total = sum(w)
    lens = [max(1, int(v / total * case["tokens"])) for v in w]
    lens[lens.index(max(lens))] += case["tokens"] - sum(lens)
    return lens


def _conv_split(case):
    return (case["heads"] * case["headdim"], case["groups"] * case["dstate"], case["groups"] * case["dstate"])


def _tensors(case, seed):
    """The input tensors of a case, on the GPU, from the seed alone."""
    kind = case["kind"]
    io = torch.float32 if case["io"] == "f32" else torch.bfloat16
    H, P, N, G = case["heads"], case["headdim"], case["dstate"], case["groups"]
    Bt = 1 if kind == "varlen" else case["batch"]
    T = case.get("tokens", case.get("seqlen", 1))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * int(seed) + 17)

    def normal(*shape, scale=1.0, dtype=torch.float32):
        return torch.randn(shape, generator=gen, device="cuda").mul_(scale).to(dtype)

    t = {}
    if kind in ("conv", "token"):
        C = sum(_conv_split(case))
        t["u"] = normal(Bt, T, C, dtype=io) if kind == "conv" else normal(Bt, C, dtype=io)
        t["weight"], t["bias"] = normal(C, CONV_TAPS, scale=1.0 / CONV_TAPS), normal(C, scale=0.1)
        if kind == "token" or case["carried"]:
            t["conv_state"] = normal(Bt, C, CONV_TAPS - 1, dtype=io)
        if kind == "conv":
            return t
    # leading axes of the per-token tensors and of the per-head ones
    lead = {"prefill": (Bt, T), "varlen": (T,), "token": (Bt,), "layers": (case.get("layers"), Bt),
            "steps": (case.get("steps"), case.get("layers"), Bt)}[kind]
    per = (case["layers"],) if kind in ("layers", "steps") else ()
    if kind != "token":   # (there the convolution produces x, B and C)
        t["x"] = normal(*lead, H, P, dtype=io)
        t["B"] = normal(*lead, G, N, scale=inputs.BC_SCALE, dtype=io)
        t["C"] = normal(*lead, G, N, scale=inputs.BC_SCALE, dtype=io)
    z = normal(*lead, H)
    if case.get("raw_dt"):
        t["dt_bias"] = inputs.DT_BIAS + normal(*per, H, scale=0.1)
        t["dt"] = z.mul_(0.5)
    else:
        t["dt"] = torch.nn.functional.softplus(z.mul_(0.5).add_(inputs.DT_BIAS)).clamp_(*DT_LIMIT)
    t["A"] = -torch.exp(torch.rand((*per, H), generator=gen, device="cuda") * math.log(inputs.A_MAX))
    t["D"] = normal(*per, H)
    rows = {"prefill": (Bt,), "varlen": (case.get("nseq"),), "token": (Bt,), "layers": lead, "steps": lead[1:]}[kind]
    if kind in ("token", "layers", "steps") or case["carried"]:
        t["state"] = normal(*rows, H, P, N, scale=STATE_SCALE)
    if kind == "varlen":
        cu = [0]
        for n in _lengths(case):
            cu.append(cu[-1] + n)
        t["cu"] = torch.tensor(cu, dtype=torch.int32, device="cuda")
    return t


def prepare(case, seed):
    s = _tensors(case, seed)
    s["case"] = case
    kind = case["kind"]
    s["dt_options"] = (dict(dt_bias=s["dt_bias"], dt_softplus=True, dt_limit=DT_LIMIT) if case.get("raw_dt") else {})
    if kind in ("prefill", "varlen"):
        nseq = case["nseq"] if kind == "varlen" else case["batch"]
        shape = ssd.make_shape(nseq, case.get("tokens", case.get("seqlen")), case["heads"], case["headdim"],
                               case["dstate"], case["groups"], case["chunk"], s["x"].dtype)
        size = ssd.raw().ssd_prefill_varlen_workspace_bytes if kind == "varlen" else ssd.raw().ssd_prefill_workspace_bytes
        s["workspace"] = torch.empty((max(int(size(shape)), 256),), dtype=torch.uint8, device="cuda")
        s["final_state"] = torch.empty((nseq, case["heads"], case["headdim"], case["dstate"]), device="cuda")
    if "x" in s:
        s["y"] = torch.empty_like(s["x"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "prefill":
        return ssd.ssd_prefill(s["x"], s["dt"], s["A"], s["B"], s["C"], s["D"], case["chunk"], h0=s.get("state"),
                               y=s["y"], final_state=s["final_state"], workspace=s["workspace"], **s["dt_options"])
    if kind == "varlen":
        return ssd.ssd_prefill_varlen(s["x"], s["dt"], s["A"], s["B"], s["C"], s["D"], s["cu"], case["chunk"],
                                      h0=s.get("state"), y=s["y"], final_state=s["final_state"],
                                      workspace=s["workspace"], **s["dt_options"])
    if kind == "token":
        x, B, C = ssd.ssd_conv1d_step(s["conv_state"], s["u"], s["weight"], s["bias"], split=_conv_split(case))
        Bt, H, P, N, G = case["batch"], case["heads"], case["headdim"], case["dstate"], case["groups"]
        y = ssd.ssd_decode_step(s["state"], x.view(Bt, H, P), s["dt"], s["A"], B.view(Bt, G, N), C.view(Bt, G, N), s["D"])
        return y, s["state"], s["conv_state"]
    if kind == "layers":
        return ssd.ssd_decode_step_layers(s["state"], s["x"], s["dt"], s["A"], s["B"], s["C"], s["D"], y=s["y"],
                                          **s["dt_options"]), s["state"]
    if kind == "steps":
        return ssd.ssd_decode_steps_layers(s["state"], s["x"], s["dt"], s["A"], s["B"], s["C"], s["D"], y=s["y"],
                                           **s["dt_options"]), s["state"]
    outs, conv_state = ssd.ssd_conv1d_prefill(s["u"], s["weight"], s["bias"], s.get("conv_state"),
                                              split=_conv_split(case))
    return outs, conv_state


def work(case):
    """Every input read once, every output written once; the multiplications and additions of the recurrence
    (h = a h + (dt x) B; y = C h + D x: five per state element, three per output) and of the filter."""
    kind, sz = case["kind"], 4 if case["io"] == "f32" else 2
    H, P, N, G = case["heads"], case["headdim"], case["dstate"], case["groups"]
    channels = H * P + 2 * G * N
    if kind == "conv":
        n = case["batch"] * case["seqlen"] * channels
        taps = channels * (4 * CONV_TAPS + 4) + case["batch"] * channels * (CONV_TAPS - 1) * sz * (2 if case["carried"] else 1)
        return dict(bytes=2 * n * sz + taps, flops=n * (2 * CONV_TAPS + 4))
    layers = case.get("layers", 1)
    seqs = case["nseq"] if kind == "varlen" else layers * case["batch"]
    tokens = {"prefill": lambda: seqs * case["seqlen"], "varlen": lambda: case["tokens"], "token": lambda: seqs,
              "layers": lambda: seqs, "steps": lambda: seqs * case["steps"]}[kind]()
    carried = kind in ("token", "layers", "steps") or case["carried"]
    nbytes = tokens * (2 * H * P * sz + 4 * H + 2 * G * N * sz) + seqs * H * P * N * 4 * (2 if carried else 1) + 8 * H * layers
    flops = tokens * H * P * (5 * N + 3)
    if kind == "token":   # the filter's input and cache; its output stays on the chip between the two calls
        nbytes += seqs * channels * sz * (2 * (CONV_TAPS - 1)) + channels * (4 * CONV_TAPS + 4)
        flops += seqs * channels * (2 * CONV_TAPS + 4)
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    """Measured against ``exact``: fp32 io up to 1.8e-7 (the final state of a prompt), bf16 io 1.7e-3 to 2.4e-3 (the
    rounding of y; of the matrix operands; of two state slices' sum); four times that."""
    return {"rel": 1e-6 if case["io"] == "f32" else 1e-2}


# ---- the same results in 64 bits ---------------------------------------------------------------------------

def _silu(v):
    return v * torch.sigmoid(v)


def _heads_of(g, heads):
    """(.., G, N) -> (.., H, N)"""
    return g.repeat_interleave(heads // g.shape[-2], dim=-2)


def _step_size(t, case):
    dt = t["dt"].double()
    if case.get("raw_dt"):
        v = dt + t["dt_bias"].double()
        dt = (v.clamp(min=0) + torch.log1p(torch.exp(-v.abs()))).clamp(float(torch.tensor(DT_LIMIT[0])),
                                                                       float(torch.tensor(DT_LIMIT[1])))
    return dt


def _scan(x, dt, A, B, C, D, state, length=64):
    """The recurrence over tokens, in pieces of `length`: x (b,T,H,P), dt (b,T,H), B, C (b,T,G,N), state (b,H,P,N)."""
    b, T, H, P = x.shape
    ys = []
    for t0 in range(0, T, length):
        xs, ds = x[:, t0:t0 + length].double(), dt[:, t0:t0 + length].transpose(1, 2)              # (b,l,H,P), (b,H,l)
        Bs = _heads_of(B[:, t0:t0 + length].double(), H).transpose(1, 2).contiguous()                # (b,H,l,N)
        Cs = _heads_of(C[:, t0:t0 + length].double(), H).transpose(1, 2).contiguous()
        xh = xs.transpose(1, 2).contiguous()                                                         # (b,H,l,P)
        cs = torch.cumsum(ds * A.double()[None, :, None], dim=2)
        l = cs.shape[2]
        causal = torch.ones((l, l), dtype=torch.bool, device=x.device).tril()
        mask = torch.exp((cs[..., :, None] - cs[..., None, :]).masked_fill(~causal, float("-inf")))
        xd = ds[..., None] * xh
        y = torch.matmul(torch.matmul(Cs, Bs.transpose(2, 3).contiguous()) * mask, xd)
        y += torch.exp(cs)[..., None] * torch.matmul(Cs, state.transpose(2, 3).contiguous())
        y += D.double()[None, :, None, None] * xh
        ys.append(y.transpose(1, 2))
        w = torch.exp(cs[..., -1:] - cs)[..., None] * xd
        state = torch.exp(cs[..., -1])[..., None, None] * state + torch.matmul(w.transpose(2, 3).contiguous(), Bs)
    return torch.cat(ys, dim=1), state


def _filter(u, weight, bias, cache):
    """u (b,T,C), cache (b,C,k-1) -> filtered (b,T,C), the last k-1 inputs (b,C,k-1)"""
    seq = torch.cat([cache.double().transpose(1, 2), u.double()], dim=1)
    T = u.shape[1]
    z = bias.double() + sum(weight[:, j].double() * seq[:, j:j + T] for j in range(weight.shape[1]))
    return _silu(z), seq[:, T:].transpose(1, 2)


def exact(case, seed):
    t = _tensors(case, seed)
    kind = case["kind"]
    H, P, N, G = case["heads"], case["headdim"], case["dstate"], case["groups"]
    if kind == "conv":
        cache = t.get("conv_state", torch.zeros((case["batch"], t["u"].shape[2], CONV_TAPS - 1), device="cuda"))
        z, new_cache = _filter(t["u"], t["weight"], t["bias"], cache)
        return list(z.split(_conv_split(case), dim=2)), new_cache
    dt = _step_size(t, case)
    if kind == "prefill":
        h0 = t["state"].double() if "state" in t else torch.zeros((case["batch"], H, P, N), dtype=torch.float64, device="cuda")
        return _scan(t["x"], dt, t["A"], t["B"], t["C"], t["D"], h0)
    if kind == "varlen":
        cu = t["cu"].tolist()
        ys, states = [], []
        for q in range(case["nseq"]):
            part = slice(cu[q], cu[q + 1])
            h0 = t["state"][q:q + 1].double() if "state" in t else torch.zeros((1, H, P, N), dtype=torch.float64, device="cuda")
            y, st = _scan(t["x"][None, part], dt[None, part], t["A"], t["B"][None, part], t["C"][None, part], t["D"], h0)
            ys.append(y[0])
            states.append(st)
        return torch.cat(ys), torch.cat(states)
    if kind == "token":
        z, cache = _filter(t["u"][:, None], t["weight"], t["bias"], t["conv_state"])
        x, B, C = z[:, 0].split(_conv_split(case), dim=1)
        t.update(x=x.reshape(-1, H, P)[None, None], B=B.reshape(-1, G, N)[None, None], C=C.reshape(-1, G, N)[None, None])
        dt, lead = dt[None, None], 1
    else:
        lead = case["layers"]
        if kind == "layers":
            t.update(x=t["x"][None], B=t["B"][None], C=t["C"][None])
            dt = dt[None]
    A, D = t["A"].double().view(lead, 1, H, 1), t["D"].double().view(lead, 1, H, 1)
    h = t["state"].view(lead, -1, H, P, N)
    ys, states = [], []
    for ly in range(lead):   # a layer at a time: 64-bit copies of all states would take most of the card
        hl, yl = h[ly].double(), []
        for s in range(t["x"].shape[0]):
            xs, ds = t["x"][s, ly].double(), dt[s, ly][..., None]
            Bs, Cs = _heads_of(t["B"][s, ly].double(), H), _heads_of(t["C"][s, ly].double(), H)
            hl = torch.exp(ds * A[ly])[..., None] * hl + (ds * xs)[..., None] * Bs[:, :, None, :]
            yl.append((hl * Cs[:, :, None, :]).sum(-1) + D[ly] * xs)
        ys.append(torch.stack(yl))
        states.append(hl)
    y, st = torch.stack(ys, dim=1), torch.stack(states)   # (steps, layers, batch, H, P), (layers, batch, H, P, N)
    if kind == "token":
        return y[0, 0], st[0], cache
    return (y[0], st) if kind == "layers" else (y, st)
