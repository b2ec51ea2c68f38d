"""dK/dV and dQ in one launch, where it can go wrong: two heads of one kv head on shared tiles, two of different kv heads
on their own, a last pair with one head; the two worklists one after the other and interleaved, with counts that are no
multiple of eight; parts that leave partial sums; packs on either side of each line to two launches.  All outputs against
the fp64 oracle (bars of the path: relative 2-norm 1e-2 for gradients), and against a call that asks for records, which
keeps two launches: the same bits.  Outputs start as NaN, so an item that nobody takes is seen."""
import numpy as np
import pytest

from parity_util import Case, compare, check_dv_identity

pytestmark = pytest.mark.gpu

EDGES = [127, 128, 129, 1, 31, 33, 64, 65, 255, 257, 300]


def gradients(pa, dev, profile):
    import torch
    for x in (pa.dq, pa.dk, pa.dv):
        x.fill_(float("nan"))
    pa.backward(dev["q"], dev["k"], dev["v"], dev["do"], profile=profile)
    torch.cuda.synchronize()
    return {n: getattr(pa, n).float().cpu().numpy() for n in ("dq", "dk", "dv")}


def run(case, row_pad=0):
    import torch
    from paper_2503_07680_amd.runner import PackedAttention
    pa = PackedAttention(case.lengths, case.pack_len, case.Hq, case.Hkv, case.d, case.e, with_profile=True, row_pad=row_pad)
    dev = {w: pa.to_device_bf16(case.bits(w, pa.T)) for w in ("q", "k", "v", "do")}
    pa.forward(dev["q"], dev["k"], dev["v"])
    pa.alloc_backward()
    one, two = gradients(pa, dev, False), gradients(pa, dev, True)
    for n in one:
        assert np.array_equal(one[n], two[n]), n  # NaN where nothing was written is no equal either
    torch.cuda.synchronize()
    return pa, dev, dict(one, o=pa.o.float().cpu().numpy(), lse=pa.lse.cpu().numpy())


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (2, 1), (2, 2), (3, 1), (3, 3), (5, 5), (6, 2), (8, 1), (16, 8), (24, 8), (64, 8)])
def test_heads(d, Hq, Hkv):
    case = Case(EDGES, sum(EDGES), Hq, Hkv, d, d, seed=401, name="one-launch-%d-%d-%d" % (Hq, Hkv, d))
    pa, dev, out = run(case)
    g = Hq // Hkv
    compare(case, pa, out, q_heads=sorted(set(range(g)) | set(range(Hq - g, Hq))))
    check_dv_identity(case, pa, dev, out)


@pytest.mark.parametrize("d,lengths", [(64, [1]), (128, [1]), (128, [97]), (64, [1300, 5]), (128, [2000, 60, 61])])
def test_few_items(d, lengths):
    case = Case(lengths, sum(lengths), 4, 2, d, d, seed=402, name="one-launch-few-%d-%d" % (d, lengths[0]))
    pa, dev, out = run(case)
    compare(case, pa, out)


LINES = [  # Hq, Hkv, d, tokens a sample, samples, what the backward launches (checked without a GPU: test_launch_rules_host.py)
    (24, 24, 64, 300, 67, "one launch interleaved"), (24, 24, 64, 300, 68, "eight waves"),  # one head, short samples: to 19 rounds
    (24, 24, 128, 60, 85, "one launch interleaved"), (24, 24, 128, 60, 90, "four waves"),   # one head, very short ones: to 8
    (16, 8, 128, 60, 155, "one launch"), (16, 8, 128, 60, 165, "four waves"),                # two heads: to 5
    (32, 8, 128, 100, 370, "one launch"), (32, 8, 128, 101, 130, "eight waves"),             # four heads: to 12, others to 4
    (48, 8, 128, 130, 40, "one launch"), (48, 8, 128, 130, 45, "eight waves"),               # six heads: to 2.7
    (72, 8, 64, 64, 8, "eight waves"), (72, 8, 128, 64, 40, "eight waves"),                  # nine: two launches
]


@pytest.mark.parametrize("Hq,Hkv,d,n,times", [x[:5] for x in LINES])
def test_either_side_of_the_lines(Hq, Hkv, d, n, times):
    lengths = [n] * times
    case = Case(lengths, sum(lengths), Hq, Hkv, d, d, seed=403, name="one-launch-line-%d-%d-%d" % (Hq, n, times))
    pa, dev, out = run(case)
    g = Hq // Hkv
    rows = sorted(set(np.random.default_rng(1).integers(0, pa.T, 100).tolist()) | {0, pa.T - 1})
    compare(case, pa, out, q_heads=list(range(Hq - g, Hq)), rows=rows, cols=rows)


def test_rows_with_padding():
    case = Case([700, 129, 64, 31], 924, 8, 2, 128, 128, seed=404, name="one-launch-pad")
    pa, dev, out = run(case, row_pad=64)
    compare(case, pa, out)


@pytest.mark.parametrize("Hq,Hkv,times", [(1, 1, 1), (3, 1, 1), (8, 8, 1), (12, 4, 1), (16, 16, 2), (128, 128, 1), (16, 8, 1)])
def test_head_size_192(Hq, Hkv, times):  # the last: two heads an item, two launches
    lengths = (EDGES if Hq < 128 else [129, 64, 300, 1, 31]) * times
    case = Case(lengths, sum(lengths), Hq, Hkv, 192, 128, seed=405, name="one-launch-192-%d-%d" % (Hq, Hkv))
    pa, dev, out = run(case)
    g = Hq // Hkv
    compare(case, pa, out, q_heads=sorted(set(range(g)) | set(range(Hq - g, Hq))))
    check_dv_identity(case, pa, dev, out)


LINES_192 = [(64, "one launch"), (66, "four waves")]  # four rounds, and more


@pytest.mark.parametrize("times", [x[0] for x in LINES_192])
def test_head_size_192_on_either_side_of_the_line(times):
    case = Case([60] * times, 60 * times, 16, 16, 192, 128, seed=406, name="one-launch-192-line-%d" % times)
    pa, dev, out = run(case)
    compare(case, pa, out, q_heads=[0, 15])
