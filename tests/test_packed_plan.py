"""How a packed batch is cut up (``ssd_testing_varlen_plan``: host arithmetic, the device's choice evaluated on the host)."""
import random

import pytest

from paper_2603_09555_amd import ssd


@pytest.fixture(autouse=True)
def _reset():
    ssd.reset_knobs()
    yield
    ssd.reset_knobs()


def plan(lengths, heads, groups=1, chunk=256):
    return ssd.varlen_plan(lengths, heads, 64, 128, groups, chunk)


@pytest.mark.parametrize("lengths, heads, most", [([2016] + 32 * [1], 24, 6), ([4000] + 64 * [1], 24, 8), ([4096] + 31 * [1], 80, 10),
                                                  ([8192] + 63 * [1], 80, 18), ([1] * 63 + [8192], 24, 12),
                                                  ([3000, 3000] + 60 * [1], 24, 8)], ids=lambda v: str(v)[:20])
def test_a_long_prompt_among_short_rows_is_cut(lengths, heads, most):
    """Uncut, a few workgroups walk the whole prompt while the chip idles (8192 + 63 x 1 tokens: 322 us against 72)."""
    p = plan(lengths, heads)
    assert p["chosen"] and p["shortest"] <= p["seg_blocks"] <= most


@pytest.mark.parametrize("lengths, heads", [([64] * 64, 80), ([256] * 16, 80), ([300] * 48 + [700] * 6, 80)], ids=lambda v: str(v)[:20])
def test_sequences_that_fill_the_chip_are_not_cut(lengths, heads):
    p = plan(lengths, heads)
    assert p["items"] == len(lengths)


@pytest.mark.parametrize("lengths, heads", [([70] * 11, 9), ([60] * 10, 24), ([600] + [5] * 9, 45)], ids=lambda v: str(v)[:20])
def test_short_batches_are_not_cut_whatever_their_lengths(lengths, heads):
    """... and launch neither the states pass nor the chain."""
    p = plan(lengths, heads)
    assert not p["chosen"] and p["items"] == len(lengths)


def test_plans_stay_within_what_the_host_sized():
    """Over drawn batches: the choice is between the host's shortest length and all the tokens, the list is that of this
    length, and one sequence, a forced length and a batch that cannot be cut leave no choice."""
    r = random.Random(3)
    for _ in range(300):
        n, heads, groups, chunk = r.randint(1, 200), r.randint(1, 40), r.choice([1, 2, 4]), r.choice([16, 64, 100, 256])
        lengths = [r.choice([0, 1, r.randint(0, 300), r.randint(0, 3000)]) for _ in range(n)]
        lengths[r.randrange(n)] += 1
        p = plan(lengths, heads * groups, groups, chunk)
        blocks = [(v + 63) // 64 for v in lengths]
        total = (sum(lengths) + 63) // 64
        assert p["mfma"] and (chunk + 63) // 64 <= p["shortest"] <= p["seg_blocks"] <= max(total, p["shortest"])
        assert p["items"] == sum(max(1, -(-b // p["seg_blocks"])) for b in blocks)
        assert p["items"] - n <= (total - 1) // p["shortest"]   # what the grid of the states-only pass is sized for
        assert p["chosen"] == (n > 1 and total > p["shortest"]) and p["heads"] in (2, 4)
    ssd.set_knob("seg_blocks", 7)
    p = plan([3000] + 9 * [5], 8)
    assert not p["chosen"] and p["seg_blocks"] == p["shortest"] == 7


@pytest.mark.parametrize("lengths, heads, groups, dealt", [([1710] + 6 * [518], 91, 1, True), ([3222, 158] + 6 * [1215], 80, 4, True),
                                                           (16 * [19] + [2691], 65, 1, True), (4 * [1260], 96, 1, False), (5 * [500], 64, 1, False),
                                                           (40 * [250], 16, 1, False), (30 * [300], 24, 1, False), (17 * [105] + [14417], 28, 4, False),
                                                           (64 * [256], 80, 1, True), ([700 + 40 * i for i in range(16)], 80, 1, True),
                                                           (16 * [1024], 100, 1, True), (16 * [256], 80, 1, True), (47 * [256], 32, 1, True), (49 * [700], 32, 1, True),
                                                           (12 * [1024], 80, 1, True), (4 * [1676], 88, 2, False),
                                                           ([14161, 9290], 60, 4, False)], ids=lambda v: str(v)[:20])
def test_kernels_of_a_packed_batch_whose_lengths_choose(lengths, heads, groups, dealt):
    """Two heads per workgroup, dealt or an entry each, are what is left for a batch of more blocks than a segment has at least.  The
    states-only pass has two as well, unless the batch is dealt and of ten blocks a CU and more (and of entries of more than 32
    workgroups, or more than three rounds)."""
    p = plan(lengths, heads, groups)
    groups2, blocks = groups * -(-heads // groups // 2), (sum(lengths) + 63) // 64
    two = not dealt or blocks * groups2 < 2560 or (groups2 <= 32 and len(lengths) * groups2 <= 768)
    assert (p["heads"], p["state_heads"], p["dealt"]) == (2, 2 if two else 4, dealt)


@pytest.mark.parametrize("lengths, heads, heads_per_wg", [(17 * [4], 32, 4), (16 * [4], 32, 2), ([100], 80, 2), (2100 * [3], 1, 4), (250 * [3], 1, 2)],
                         ids=lambda v: str(v)[:20])
def test_heads_per_workgroup_without_a_choice_of_lengths(lengths, heads, heads_per_wg):
    """An entry each, and no length to choose -- too few blocks to cut, one sequence, or more than 1024: two heads up to a round."""
    p = plan(lengths, heads)
    assert not p["chosen"] and not p["dealt"] and p["heads"] == heads_per_wg


@pytest.mark.parametrize("nseq, heads, groups, dealt", [
    (7, 66, 1, False), (8, 66, 1, True),         # entries of 33 workgroups: more than a round of 256
    (4, 128, 1, False), (5, 128, 1, True),       # exactly a round of 64 each
    (15, 34, 1, False), (16, 34, 1, True),       # 17 each
    (27, 20, 4, False), (37, 20, 4, False), (38, 20, 4, True),   # 12 each: more than seven quarters of a round, 448
    (28, 32, 1, False), (29, 32, 1, True),       # 16 each, exactly 448
    (448, 2, 1, False), (449, 2, 1, True), (2048, 2, 1, True),
    (2049, 2, 1, False), (5000, 8, 1, False),    # beyond 2048 sequences the list is in the caller's order
], ids=lambda v: str(v))
def test_which_packed_batches_are_dealt_items(nseq, heads, groups, dealt):
    lengths = [1 + 37 * i % 300 for i in range(nseq)]
    assert plan(lengths, heads, groups)["dealt"] == dealt
    ssd.set_knob("deal", 1)
    p = plan(lengths, heads, groups)
    assert p["dealt"] and p["heads"] == 2
    ssd.set_knob("deal", 2)
    assert not plan(lengths, heads, groups)["dealt"]
    ssd.set_knob("deal", 0)
    ssd.set_knob("scan_heads", 4)
    assert not plan(lengths, heads, groups)["dealt"]


def test_records_beyond_32_bits_are_not_dealt():
    """4 GiB of decay records and more, which the dealt walk could not address, whatever the knob says."""
    ssd.set_knob("deal", 1)
    assert plan([1] * 2000, 64)["dealt"]
    big = [1] * 60000   # x 200 heads, a record of 528 bytes each
    assert not plan(big, 200)["dealt"]
    ssd.reset_knobs()
    assert not plan(big, 200)["dealt"]
