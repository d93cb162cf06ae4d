"""Host-side tests of how the library cuts a prefill up (``ssd_testing_prefill_plan``: host arithmetic only, no
GPU): the choices the design notes state for the benchmark shapes, the effect of the test-only knobs, and the
invariants the kernels rely on, over a grid of shapes."""
import itertools

import pytest
import torch

from paper_2603_09555_amd import inputs, ssd


@pytest.fixture(autouse=True)
def _reset():
    ssd.reset_knobs()
    yield
    ssd.reset_knobs()


def shape_of(c):
    return ssd.make_shape(c.batch, c.seqlen, c.nheads, c.headdim, c.dstate, c.ngroups, c.chunk, c.torch_io_dtype)


def test_plans_of_the_benchmark_shapes():
    plan = {n: ssd.prefill_plan(shape_of(c)) for n, c in inputs.CONFIGS.items() if not c.decode_steps}
    # config 0: fp32 MFMA kernel, eight time segments of one block (four workgroups would leave the chip idle)
    assert plan["c0_tiny_f32"]["path"] == "mfma_f32" and plan["c0_tiny_f32"]["f32_segments"] == 8
    # config 1: eight chunks of 256 tokens on the chunk kernels
    chunks = {n: ssd.prefill_chunks(shape_of(c)) for n, c in inputs.CONFIGS.items() if not c.decode_steps}
    assert chunks["c1_130m"] == 8 and all(v == 0 for n, v in chunks.items() if n != "c1_130m")
    # config 2: one round of workgroups of two heads (192) holds the batch uncut: x is read once
    assert plan["c2_780m_b8"] == dict(path="mfma_bf16", seg_blocks=64, segments=1, parts=1, fold=False, f32_segments=0)
    # config 3: 256 blocks -> 6 segments of 43 (240 workgroups of two heads); a chain of five slots is not folded
    assert plan["c3_2p7b_long"] == dict(path="mfma_bf16", seg_blocks=43, segments=6, parts=1, fold=False, f32_segments=0)
    for name in ("c2_780m_b8", "c3_2p7b_long"):
        pair = ssd.prefill_pair_plan(shape_of(inputs.CONFIGS[name]))
        assert pair["heads"] == 2 and all(pair[k] == plan[name][k] for k in ("seg_blocks", "segments", "parts", "fold"))


def test_batches_beyond_a_round_of_two_heads_keep_four():
    for batch, tokens in ((12, 4096), (16, 1024)):   # 288 and 384 workgroups of two heads
        sh = shape_of(inputs.CONFIGS["c2_780m_b8"].with_(batch=batch, seqlen=tokens))
        assert ssd.prefill_pair_plan(sh) is None
        assert ssd.prefill_plan(sh) == dict(path="mfma_bf16", seg_blocks=tokens // 64, segments=1, parts=1, fold=False, f32_segments=0)


def test_knobs_and_aliasing_change_the_plan():
    sh = shape_of(inputs.CONFIGS["c2_780m_b8"])
    ssd.set_knob("seg_blocks", 36)
    ssd.set_knob("seg_parts", 2)
    assert ssd.prefill_plan(sh)["fold"]                                     # 36 + 28 blocks, a chain of two slots
    assert not ssd.prefill_plan(sh, h0_aliases_final_state=True)["fold"]   # h0 and final_state in one buffer
    ssd.set_knob("fold_max_slots", 0)
    assert not ssd.prefill_plan(sh)["fold"]
    ssd.set_knob("fold_max_slots", 1)
    assert not ssd.prefill_plan(sh)["fold"]                                 # a chain of two slots is over the limit
    ssd.reset_knobs()
    ssd.set_knob("scan_heads", 4)
    ssd.set_knob("fold_max_slots", 1)
    p = ssd.prefill_plan(sh)                                                # (the choice of lengths knows the limit)
    assert p["fold"] == ((p["segments"] - 1) * p["parts"] <= 1)
    ssd.reset_knobs()
    ssd.set_knob("seg_blocks", 36)
    ssd.set_knob("seg_parts", 1)
    assert ssd.prefill_plan(sh) == dict(path="mfma_bf16", seg_blocks=36, segments=2, parts=1, fold=True, f32_segments=0)
    ssd.reset_knobs()
    ssd.set_knob("seg_blocks", 16)
    p = ssd.prefill_plan(sh)
    assert (p["seg_blocks"], p["segments"]) == (16, 4)
    ssd.reset_knobs()
    ssd.set_knob("force_generic", 1)
    assert ssd.prefill_plan(sh)["path"] == "generic_f32"
    ssd.reset_knobs()
    c0 = shape_of(inputs.CONFIGS["c0_tiny_f32"])
    ssd.set_knob("f32_segments", 3)
    assert ssd.prefill_plan(c0)["f32_segments"] == 3
    ssd.set_knob("f32_segments", 100)                                       # at most one per block
    assert ssd.prefill_plan(c0)["f32_segments"] == 8


def test_two_heads_whatever_the_records_take():
    """Decay records of 4 GiB and more (16 prompts of 1030000 tokens, 32 heads) keep the round of two-head workgroups that any other
    batch of one round takes: only a walk over several items addresses records by 32-bit offsets."""
    sh = ssd.make_shape(16, 1030000, 32, 64, 128, 1, 256, torch.bfloat16)
    assert 16 * 32 * ((1030000 + 63) // 64) * 132 * 4 > 1 << 32
    assert ssd.prefill_pair_plan(sh) == dict(seg_blocks=16094, segments=1, parts=1, fold=False, heads=2, state_heads=2)


def test_the_store_policy_of_y_is_no_part_of_the_plan():
    """How y leaves is chosen per launch; the knob that forces it compares two policies of the kernel that is taken, not two
    kernels."""
    big = shape_of(inputs.CONFIGS["c2_780m_b8"])
    plans = []
    for policy in (-1, 0, 1):
        ssd.set_knob("y_stream", policy)
        plans.append((ssd.prefill_pair_plan(big), ssd.prefill_plan(big), ssd.varlen_plan([300, 2000, 40], 24, 64, 128, 1, 256)))
    assert plans[0][0]["heads"] == 2 and plans[0][2]["heads"] == 2
    assert plans[1] == plans[0] and plans[2] == plans[0]


GRID = list(itertools.product([1, 2, 3, 8, 16], [1, 64, 1000, 2048, 4096, 16384, 50000], [4, 8, 24, 48, 80, 128],
                              [64, 128], [256, 64]))


def test_plan_invariants_over_a_grid_of_shapes():
    """Of the plans that are launched: segments and pieces of the scan kernels, with two heads per workgroup and with four, and the
    chunks of the small ones."""
    base = inputs.CONFIGS["c3_2p7b_long"]
    pairs = chunked = 0
    for Bt, T, H, P, L in GRID:
        c = base.with_(batch=Bt, seqlen=T, nheads=H, headdim=P, chunk=L)
        sh = shape_of(c)
        p = ssd.prefill_plan(sh)
        assert p["path"] == "mfma_bf16", (Bt, T, H, P, L)
        pair = ssd.prefill_pair_plan(sh)
        pairs += pair is not None
        assert pair is None or (pair["heads"] == 2 and all(pair[k] == p[k] for k in ("seg_blocks", "segments", "parts", "fold")))
        nblocks = (T + 63) // 64
        assert 1 <= p["seg_blocks"] and p["segments"] == (nblocks + p["seg_blocks"] - 1) // p["seg_blocks"]
        assert p["parts"] >= 1 and p["seg_blocks"] % p["parts"] == 0
        assert p["segments"] > 1 or p["parts"] == 1
        # the workspace holds one state slot per piece and head: its size must cover the plan whatever it is
        slots = (p["segments"] - 1) * p["parts"] + 1
        per_slot = Bt * H * P * 128 * 4
        assert ssd.prefill_workspace_bytes(sh) >= slots * per_slot, (Bt, T, H, P, L, p)
        assert p["fold"] == (p["segments"] >= 2 and (p["segments"] - 1) * p["parts"] <= 3)
        assert not ssd.prefill_plan(sh, True)["fold"]
        # the chunk kernels: a state and a decay per chunk and 64 headdim columns, with h0 in final_state's place one state more
        for alias in (False, True):
            n = ssd.prefill_chunks(sh, alias)
            chunked += n > 0
            assert n in (0, (T + 255) // 256)
            if n > 1 or (n and alias):
                assert ssd.prefill_workspace_bytes(sh) >= Bt * H * (P // 64) * ((n + alias) * 64 * 128 + n) * 4
    assert pairs > 300 and chunked > 50


def test_f32_time_segments_over_a_grid_of_shapes():
    base = inputs.CONFIGS["c0_tiny_f32"]
    for Bt, T, H, P, N in itertools.product([1, 2, 8], [1, 64, 65, 512, 4096], [2, 4, 24, 80], [32, 64], [16, 64, 128]):
        c = base.with_(batch=Bt, seqlen=T, nheads=H, headdim=P, dstate=N)
        ssd.set_knob("force_mfma_f32", 1)
        p = ssd.prefill_plan(shape_of(c))
        assert p["path"] == "mfma_f32"
        nblocks, wgs = (T + 63) // 64, Bt * H * (P // 32)
        s = p["f32_segments"]
        assert 1 <= s <= max(1, nblocks)
        assert s == 1 or wgs * s <= 256          # the library cuts only as far as the workgroups run side by side
        if wgs * 2 <= 256 and nblocks >= 2:
            assert s >= 2                        # and does cut when half the chip would idle


def test_split_f32_plans():
    """fp32 prompts large enough to be worth several launches: cut into segments whose states fit either the
    workspace or their own rows of y; small ones keep the single launch."""
    base = inputs.CONFIGS["c0_tiny_f32"]
    split = 0
    for Bt, T, H, P, N, L in itertools.product([1, 2, 8], [64, 65, 512, 2000, 4096], [2, 11, 24], [32, 64], [16, 72, 128], [64, 256]):
        c = base.with_(batch=Bt, seqlen=T, nheads=H, headdim=P, dstate=N, chunk=L)
        sh = shape_of(c)
        p = ssd.prefill_plan(sh)
        assert p["path"] in ("mfma_f32", "generic_f32")
        if p["path"] == "generic_f32" or p["f32_segments"]:
            continue
        split += 1
        S, nblocks = p["segments"], (T + 31) // 32
        assert 1 <= S <= nblocks and p["seg_blocks"] == (nblocks + S - 1) // S and p["parts"] >= 1
        assert S == 1 or p["parts"] == 1
        if S > 1 and ssd.prefill_workspace_bytes(sh) < Bt * H * S * (P * N + 1) * 4:
            rows = 32 * ((N + 31) // 32)
            begin = [s * nblocks // S * 32 for s in range(S)] + [T]
            assert all(b - a >= rows for a, b in zip(begin, begin[1:]))
    assert split > 100
    p = ssd.prefill_plan(shape_of(base.with_(seqlen=2048, nheads=24, headdim=64, dstate=128, chunk=256)))
    assert p["path"] == "mfma_f32" and (p["segments"], p["seg_blocks"], p["f32_segments"]) == (16, 4, 0)


@pytest.mark.parametrize("T, H, P, N, G, fits", [(1, 4096, 8160, 8, 1, True), (1, 4096, 8224, 8, 1, False), (31, 16384, 2080, 8, 1, False),
                                                 (33, 16384, 2016, 8, 1, False), (2, 4, 32, 128, 4, True)])
def test_split_f32_offsets_of_a_whole_block(T, H, P, N, G, fits):
    """The split kernel addresses the 32 rows of a block whether the prompt has them or not: 32 rows of x take at most the
    32-bit byte offsets, or the shape is not its own."""
    ssd.set_knob("seg_blocks", 1)   # (asks for the split kernel wherever it can run)
    try:
        p = ssd.prefill_plan(ssd.make_shape(1, T, H, P, N, G, 64, torch.float32))
    finally:
        ssd.reset_knobs()
    taken = p["path"] == "mfma_f32" and p["segments"] > 0
    assert taken == fits == (max(T, 32) * H * P * 4 <= 0xFFFF0000)


@pytest.mark.parametrize("dims", [(4, 2171, 17, 32, 24, 17, 64), (2, 2344, 30, 32, 40, 30, 64), (6, 137, 15, 32, 24, 1, 64),
                                  (1, 1024, 9, 64, 16, 3, 128), (4, 2048, 24, 32, 64, 24, 128)], ids=str)
def test_fp32_prompts_the_split_kernel_loses_stay_off_it(dims):
    """Few slices per group, or little work: the fp32 matrix instruction is faster (73 against 59 us on the first)."""
    p = ssd.prefill_plan(ssd.make_shape(*dims, torch.float32))
    assert p["path"] == "mfma_f32" and p["f32_segments"] > 0


@pytest.mark.parametrize("dims", [(4, 33, 40, 64, 32, 4), (2, 16, 37, 128, 16, 1), (6, 93, 32, 32, 96, 4), (7, 52, 32, 64, 16, 2), (1, 991, 23, 64, 128, 1),
                                  (2, 1358, 8, 64, 128, 1), (3, 1573, 1, 128, 128, 1)], ids=str)
def test_fp32_prompts_the_split_kernel_wins_are_left_to_it(dims):
    """Short prompts of many heads, which are one launch there, and middling ones: 8 to 42 % faster than on the fp32 matrix
    instruction (4 x 33 tokens, 40 heads: 7.9 us against 11.4)."""
    p = ssd.prefill_plan(ssd.make_shape(*dims, 64, torch.float32))
    assert p["path"] == "mfma_f32" and p["f32_segments"] == 0


@pytest.mark.parametrize("dims", [(11, 123, 7, 128, 64, 1), (2, 117, 109, 64, 64, 1), (1, 12583, 6, 64, 128, 2), (7, 320, 14, 64, 128, 2)], ids=str)
def test_small_prompts_the_scan_wins_are_left_to_it(dims):
    """One chunk in more than a round of workgroups, a round and a little of two chunks, fifty chunks to chain: the chunk kernels
    take 1.17 to 1.3 times as long."""
    assert ssd.prefill_chunks(ssd.make_shape(*dims, 128, torch.bfloat16)) == 0


@pytest.mark.parametrize("dims, seg_blocks, images, states_in_y", [
    ((1, 2048, 24, 64, 128, 1, 256), 0, True, True),     # 12 x 15 workgroups of the states-only launch + 64 blocks: 244
    ((1, 2048, 26, 64, 128, 1, 256), 0, False, True),    # 13 x 15 + 64: 259, more than a workgroup per CU
    ((1, 2048, 8, 64, 128, 1, 256), 1, False, True),
    ((2, 320, 8, 64, 128, 1, 32), 2, True, False),       # a state per chunk beside the images
    ((1, 8192, 2, 64, 128, 1, 256), 0, False, True),
    ((6, 2184, 30, 64, 128, 1, 256), 0, False, False),
    ((1, 512, 2, 64, 128, 1, 512), 4, False, True),      # idle, but the workspace has no room for 16 images
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_images_where_the_states_only_launch_leaves_cus_idle(dims, seg_blocks, images, states_in_y):
    ssd.set_knob("seg_blocks", seg_blocks)
    sh = ssd.make_shape(*dims, torch.float32)
    Bt, T, H, P, N, G, _ = dims
    p = ssd.prefill_plan(sh)
    assert p["path"] == "mfma_f32" and p["f32_segments"] == 0
    print(dims, p, ssd.split_f32_memory(sh))
    assert ssd.split_f32_memory(sh) == dict(images=images, states_in_y=states_in_y)
