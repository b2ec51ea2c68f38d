"""The forward's launches of halves of 256-row tiles (odd groups, few rounds): tiles of one row to 256, with an empty,
a partial and a full second half, every head size, heads dealt evenly to the dies and not, and packs on either side of
the lines; against the fp64 oracle, and with records asked for, which keeps the 256-row tiles: the same bits.  Outputs
start as NaN, so a half that nobody takes is seen."""
import numpy as np
import pytest

from parity_util import Case, compare, run_gpu

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 127, 128, 129, 160, 255, 256, 257, 384, 385, 512, 513]


def forward(case, profile):
    import torch
    from paper_2503_07680_amd.runner import PackedAttention
    pa = PackedAttention(case.lengths, case.pack_len, case.Hq, case.Hkv, case.d, case.e, with_profile=profile)
    dev = {w: pa.to_device_bf16(case.bits(w, pa.T)) for w in ("q", "k", "v")}
    pa.o.fill_(float("nan"))
    pa.lse.fill_(float("nan"))
    pa.forward(dev["q"], dev["k"], dev["v"], profile=profile)
    torch.cuda.synchronize()
    return pa.o.float().cpu().numpy(), pa.lse.cpu().numpy()


def check_same(case):
    for a, b in zip(forward(case, False), forward(case, True)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("d,e", [(64, 64), (128, 128), (192, 128)])
@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (3, 1), (5, 5), (8, 8), (16, 16), (24, 8)])
def test_edges_of_halves(d, e, Hq, Hkv):
    case = Case(EDGES, sum(EDGES), Hq, Hkv, d, e, seed=501, name="halves-%d-%d-%d" % (Hq, Hkv, d))
    pa, dev, out = run_gpu(case)
    g = Hq // Hkv
    compare(case, pa, out, q_heads=sorted(set(range(g)) | set(range(Hq - g, Hq))))
    check_same(case)


LINES = [  # lengths, Hq, Hkv, d_qk, d_v, what the forward launches (checked without a GPU: test_launch_rules_host.py)
    ([300] * 60, 16, 16, 64, 64, "halves"), ([300] * 62, 16, 16, 64, 64, "256-row tiles queued"),  # short samples: to 7.5 rounds
    ([700] * 22, 16, 16, 64, 64, "halves"), ([700] * 24, 16, 16, 64, 64, "256-row tiles queued"),  # others: to 4.2
    # very short ones: by the pack's size
    ([60] * 100, 24, 24, 128, 128, "halves"), ([60] * 280, 24, 24, 128, 128, "256-row tiles queued"),
    ([200] * 90, 24, 8, 128, 128, "halves"), ([200] * 100, 24, 8, 128, 128, "256-row tiles queued"),  # head size 128: to 9
    # head size 192: to 6
    ([300, 200] * 20, 24, 24, 192, 128, "halves"), ([300, 200] * 24, 24, 24, 192, 128, "256-row tiles queued"),
]


@pytest.mark.parametrize("lengths,Hq,Hkv,d,e", [x[:5] for x in LINES])
def test_either_side_of_the_lines(lengths, Hq, Hkv, d, e):
    check_same(Case(lengths, sum(lengths), Hq, Hkv, d, e, seed=502, name="halves-line"))
