"""The GPU tests that stand on either side of a line between two ways to launch say which way each of their packs takes;
here the library's rules are asked, without a GPU, so that a line that moves shows in the tests that it empties."""
import launch_rules as rules
import test_dkdv_eight_waves_gpu as eight_waves
import test_fwd_few_rounds_gpu as few_rounds
import test_fwd_halves_gpu as halves
import test_one_backward_launch_gpu as one_launch
import test_race_hunt_gpu as race_hunt


def check(got, want, packs):
    assert got == want, [(p, g, w) for p, g, w in zip(packs, got, want) if g != w]


def test_the_forwards_lines():
    packs = [(few_rounds.SHORT * times, Hq, Hkv, d) for Hq, Hkv, d, _, times, _ in few_rounds.LINES]
    packs += [x[:4] for x in halves.LINES]
    check([rules.forward(*p) for p in packs], [x[-1] for x in few_rounds.LINES + halves.LINES], packs)
    # every way of either kind of group is there, and records keep the queues
    assert {x[-1] for x in few_rounds.LINES} >= {"singles", "pairs", "pairs queued"}
    assert all(rules.forward(*p, records=True).endswith(" queued") for p in packs)


def test_the_edges_of_halves_are_halves():
    for d, Hq, Hkv in [(d, *h) for d in (64, 128, 192) for h in ((1, 1), (3, 1), (5, 5), (8, 8), (16, 16), (24, 8))]:
        assert rules.forward(halves.EDGES, Hq, Hkv, d) == "halves"


def test_the_backwards_lines():
    packs = [([n] * times, Hq, Hkv, d) for Hq, Hkv, d, n, times, _ in one_launch.LINES]
    packs += [([60] * times, 16, 16, 192) for times, _ in one_launch.LINES_192]
    check([rules.backward(*p)[0] for p in packs], [x[-1] for x in one_launch.LINES + one_launch.LINES_192], packs)
    assert all("one launch" not in rules.backward(*p, records=True)[0] for p in packs)


def test_the_line_between_eight_and_four_wavefronts():
    packs = [x[:4] for x in eight_waves.LINES]
    check([rules.backward(*p)[0] for p in packs], [x[-1] for x in eight_waves.LINES], packs)
    # the small packs have one launch, and the kernel of eight in a launch of its own with records
    small = [(eight_waves.EDGES, Hq, Hkv, d) for d in (64, 128) for Hq, Hkv in ((1, 1), (2, 1), (3, 1), (4, 1), (8, 2))]
    small += [([n], 2, 2, d) for d in (64, 128) for n in (100, 577)] + [([8300, 97], 16, 8, 128), ([1500, 129, 31], 6, 2, 64)]
    assert all(rules.backward(*p)[0].startswith("one launch") for p in small)
    assert all(rules.backward(*p, records=True)[0] == "eight waves" for p in small)


def test_items_of_three_heads_and_more_have_eight_wavefronts():
    """However few they are: with nine heads an item, samples of 30 to 90 tokens and no more items than compute units, four
    made the backward 12 to 25 % longer."""
    for d in (64, 128):
        for Hq, Hkv in [(72, 8), (80, 8), (128, 8), (160, 16)]:
            for n, times in [(30, 8), (60, 8), (90, 30), (60, 200), (1000, 30)]:
                assert rules.backward([n] * times, Hq, Hkv, d)[0] == "eight waves"


def test_heads_split():
    # query heads that an item of the key-tile kernel loops over: every die gets a queue
    want = {(32, 8): 4, (8, 1): 1, (16, 4): 2, (64, 8): 8, (6, 2): 1, (12, 3): 1, (128, 128): 1, (40, 4): 5}
    assert {k: rules.backward([500], *k, 128)[1] for k in want} == want


def test_streamed_rows_of_the_cross_entropy_keep_two_workgroups_a_unit():
    """A held row without a gradient is refilled over its reduction and needs one workgroup a unit; a streamed row (V above
    163840) is not, and from 1000 rows on one makes it 19 to 27 % slower."""
    assert rules.cross_entropy_per_cu(1024, 1, hold=False, with_grad=False) == 2
    assert rules.cross_entropy_per_cu(1024, 1, hold=False, with_grad=True) == 2
    assert [rules.cross_entropy_per_cu(*x, hold=True, with_grad=False) for x in ((256, 8), (512, 20), (1024, 20))] == [4, 1, 1]


def test_rows_just_behind_256_threads_get_three_workgroups_a_unit():
    """512 threads, 16392 to 20480 entries, with the gradient: four a unit are up to 6 % slower than consecutive rows were, and
    up to 19 % slower than three."""
    assert [rules.cross_entropy_per_cu(512, n, hold=True, with_grad=True) for n in (5, 6, 7, 8, 20)] == [3, 3, 3, 2, 2]
    assert [rules.cross_entropy_per_cu(256, n, hold=True, with_grad=True) for n in (1, 5, 6, 7, 8)] == [8, 8, 7, 7, 6]


def test_the_race_hunt_reaches_every_kernel():
    cases = race_hunt.CASES
    packs = [c[:4] for c in cases]
    check([rules.forward(*p) for p in packs], [c[5] for c in cases], packs)
    check([rules.backward(*p)[0] for p in packs], [c[6] for c in cases], packs)
    fwd, bwd = {(c[3], c[5]) for c in cases}, {(c[3], c[6]) for c in cases}
    for d in (64, 128, 192):
        assert fwd >= {(d, w) for w in ("singles", "halves", "256-row tiles", "pairs queued", "256-row tiles queued")}
        assert bwd >= {(d, w) for w in ("one launch", "four waves")}
    assert (128, "pairs") in fwd and bwd >= {(d, w) for d in (64, 128) for w in ("one launch interleaved", "eight waves")}
    # items handed over from queues: more of them than workgroups are resident, in the plain call, in either kind of group
    for d, ways in ((64, ("eight waves", "four waves")), (128, ("eight waves", "four waves")), (192, ("four waves",))):
        for way in ways:
            assert any(c[3] == d and c[6] == way and rules.backward(*c[:4])[2] > 256 for c in cases), (d, way)
