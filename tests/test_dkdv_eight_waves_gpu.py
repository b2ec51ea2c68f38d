"""The dK/dV kernel with eight wavefronts a key tile, at the sizes where it can go wrong: samples one row or key to
either side of a wavefront's 32, a block's 64 and a tile's 128, one to three steps an item (its copies run two steps
ahead, in three buffers), several query heads an item, the wrapped block order of long samples, parts that leave
partial sums, padded rows, and packs on either side of the line to the four-wave kernel.  All outputs against the fp64
oracle; the bars are the path's own (bf16 probabilities and outputs: relative 2-norm 1e-2 for gradients).  Small packs have
one launch for dK/dV and dQ, so they run with profile records too, which gives the kernel a launch of its own: the same bits."""
import numpy as np
import pytest

from parity_util import Case, run_gpu, compare, compare_sample_dense, check_dv_identity
from test_one_backward_launch_gpu import run as run_both_ways

pytestmark = pytest.mark.gpu

EDGES = [127, 128, 129, 159, 160, 161, 191, 192, 193, 255, 256, 257]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (2, 1), (3, 1), (4, 1), (8, 2)])
def test_edges_of_waves_blocks_and_tiles(d, Hq, Hkv):
    case = Case(EDGES, sum(EDGES), Hq, Hkv, d, d, seed=301, name="edges-%d-%d-%d" % (Hq, Hkv, d))
    pa, dev, out = run_both_ways(case)
    compare(case, pa, out)
    check_dv_identity(case, pa, dev, out)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [100, 128, 192, 193, 320, 577])
def test_one_sample(d, n):  # one to ten steps: every count of copies in flight at the end of an item
    case = Case([n], n, 2, 2, d, d, seed=302, name="one-%d-%d" % (n, d))
    pa, dev, out = run_both_ways(case)
    compare(case, pa, out)


LINES = [  # packs of two launches (checked without a GPU: test_launch_rules_host.py)
    ([2100, 31, 33, 257] * 6, 24, 8, 128, "eight waves"),                # three heads an item and more
    ([500, 400, 257, 129] * 5, 48, 24, 128, "eight waves"), ([200, 129, 257, 100] * 7, 48, 24, 128, "four waves"),  # two
    ([1300, 1500, 1171, 1200] * 2, 24, 24, 128, "eight waves"),          # one, long samples
    ([400, 700, 900, 600, 300] * 3, 24, 24, 128, "four waves"),
    ([250, 190, 230, 260, 300] * 9, 48, 48, 64, "eight waves"), ([150, 130, 180, 129] * 13, 48, 48, 64, "four waves"),
]


@pytest.mark.parametrize("lengths,Hq,Hkv,d", [x[:4] for x in LINES])
def test_either_side_of_the_line(lengths, Hq, Hkv, d):
    case = Case(lengths, sum(lengths), Hq, Hkv, d, d, seed=303, name="line-%d-%d-%d" % (Hq, Hkv, d))
    pa, dev, out = run_gpu(case)
    compare(case, pa, out, q_heads=list(range(2 * (Hq // Hkv))))
    check_dv_identity(case, pa, dev, out)


def test_wrapped_block_order_and_partial_sums():
    """Tiles from the 32nd of a long sample on begin below the top block and wrap around."""
    case = Case([8300, 97], 8397, 16, 8, 128, 128, seed=304, name="wrap")
    pa, dev, out = run_both_ways(case)
    compare_sample_dense(case, pa, out, 0, 3)
    check_dv_identity(case, pa, dev, out)
    case = Case([1500, 129, 31], 1660, 6, 2, 64, 64, seed=305, name="parts")  # 3 parts of one head
    pa, dev, out = run_both_ways(case)
    compare(case, pa, out)


def test_rows_with_padding_agree_bit_for_bit():
    import torch
    from paper_2503_07680_amd.runner import PackedAttention
    lengths = [700, 129, 64, 31]
    got = []
    for pad in (0, 64):
        pa = PackedAttention(lengths, sum(lengths), 8, 2, 128, 128, row_pad=pad)
        case = Case(lengths, sum(lengths), 8, 2, 128, 128, seed=306)
        dev = {w: pa.to_device_bf16(case.bits(w, pa.T)) for w in ("q", "k", "v", "do")}
        pa.forward(dev["q"], dev["k"], dev["v"])
        pa.backward(dev["q"], dev["k"], dev["v"], dev["do"])
        torch.cuda.synchronize()
        got.append([x.float().cpu().numpy() for x in (pa.dq, pa.dk, pa.dv)])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
