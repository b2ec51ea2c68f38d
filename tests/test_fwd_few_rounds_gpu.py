"""The forward's launches of few rounds (one workgroup an item, one head a workgroup for even groups) on both sides of
their lines, for every head size and kind of group, against the fp64 oracle; and with profile records asked for, which
keeps the queues: the same bits, since a row's arithmetic does not depend on how its tile is served."""
import numpy as np
import pytest

from parity_util import Case, run_gpu, compare

pytestmark = pytest.mark.gpu

SHORT = [100, 128, 129, 60, 31, 33, 257, 90]


LINES = [  # Hq, Hkv, d_qk, d_v, copies of SHORT, what the forward launches (checked without a GPU: test_launch_rules_host.py)
    (32, 8, 64, 64, 1, "singles"), (32, 8, 64, 64, 14, "singles"), (32, 8, 64, 64, 15, "pairs queued"),
    # kv heads dealt evenly to the dies, and not
    (32, 8, 128, 128, 2, "singles"), (32, 8, 128, 128, 4, "pairs"), (32, 8, 128, 128, 9, "pairs queued"),
    (24, 6, 128, 128, 4, "pairs"), (24, 6, 128, 128, 8, "pairs queued"),
    (16, 8, 192, 128, 3, "singles"), (16, 8, 192, 128, 12, "pairs queued"),
    # odd groups
    (24, 8, 128, 128, 5, "halves"), (24, 24, 64, 64, 9, "256-row tiles queued"), (24, 24, 192, 128, 9, "256-row tiles queued"),
]


@pytest.mark.parametrize("Hq,Hkv,d,e,times", [x[:5] for x in LINES])
def test_either_side_of_the_lines(Hq, Hkv, d, e, times):
    lengths = SHORT * times
    case = Case(lengths, sum(lengths), Hq, Hkv, d, e, seed=311, name="rounds-%d-%d-%d-%d" % (Hq, Hkv, d, times))
    pa, dev, out = run_gpu(case)
    rows = None if times < 4 else sorted(set(np.random.default_rng(1).integers(0, pa.T, 300).tolist()) | {0, pa.T - 1})
    g = Hq // Hkv
    compare(case, pa, out, q_heads=list(range(g)) + list(range(Hq - g, Hq)), rows=rows, cols=rows)
    pb, _, queued = run_gpu_with_records(case)
    assert np.array_equal(out["o"], queued["o"]) and np.array_equal(out["lse"], queued["lse"])


def run_gpu_with_records(case):
    import torch
    from paper_2503_07680_amd.runner import PackedAttention
    pa = PackedAttention(case.lengths, case.pack_len, case.Hq, case.Hkv, case.d, case.e, with_profile=True)
    dev = {w: pa.to_device_bf16(case.bits(w, pa.T)) for w in ("q", "k", "v")}
    pa.forward(dev["q"], dev["k"], dev["v"], profile=True)
    torch.cuda.synchronize()
    return pa, dev, {"o": pa.o.float().cpu().numpy(), "lse": pa.lse.cpu().numpy()}
