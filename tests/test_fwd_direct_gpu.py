"""The forward's launches of one workgroup an item, whose item is its place in the grid: the sample bounds that a wavefront
reads at once (up to 63 samples) and one by one (more), against the fp64 oracle and against a call that asks for records,
which keeps the queues (the same bits); and a list with more tiles than the grid's third dimension holds."""
import numpy as np
import pytest

from parity_util import Case, compare, run_gpu
from test_fwd_few_rounds_gpu import run_gpu_with_records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 62, 63, 64, 65])
@pytest.mark.parametrize("Hq,Hkv,d,e", [(4, 2, 64, 64), (6, 2, 128, 128), (4, 2, 192, 128)])
def test_samples(n, Hq, Hkv, d, e):
    lengths = [33, 1, 130][:n] + [35] * (n - 3)
    case = Case(lengths, sum(lengths), Hq, Hkv, d, e, seed=701, name="samples-%d-%d" % (n, d))
    pa, dev, out = run_gpu(case)
    compare(case, pa, out)
    _, _, queued = run_gpu_with_records(case)
    assert np.array_equal(out["o"], queued["o"]) and np.array_equal(out["lse"], queued["lse"])


def test_more_tiles_than_the_grid_holds():
    import torch
    from paper_2503_07680_amd.runner import PackedAttention
    pa = PackedAttention([60] * 100, 6000, 1, 1, 64, 64)
    gen = torch.Generator(device=pa.device).manual_seed(3)
    q, k, v = [pa.buffer(1, 64).normal_(generator=gen) for _ in range(3)]
    want = [x.clone() for x in pa.forward(q, k, v)]
    times = 33000 // len(pa.fwd_tiles) + 1  # the same tiles again and again: halves of 256-row tiles, 66000 of them
    pa.fwd_tiles, pa.fwd_tiles_dev = np.tile(pa.fwd_tiles, times), pa.fwd_tiles_dev.repeat(times, 1)
    pa.o.fill_(float("nan"))
    pa.lse.fill_(float("nan"))
    for got, x in zip(pa.forward(q, k, v), want):
        assert torch.equal(got, x)
