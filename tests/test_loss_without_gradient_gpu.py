"""Cross-entropy without a gradient (a row's registers are refilled with the next row that has a loss): row lengths around
the chunks of each workgroup size and the longest held row, one row to many a workgroup, rows without a loss at the ends,
in runs and everywhere, workgroups with more rows than are staged at a time.  Against the fp64 oracle, and against the
call with a gradient, which adds up in the same order: the same bits."""
import numpy as np
import pytest

from oracle import loss as L
import hbp_workloads as wl
from test_loss_gpu import LOSS_REL, TOKEN_LOSS_ABS, make_case, run_gpu

pytestmark = pytest.mark.gpu


def check(bits, y, cu, mode, t_ave=7.0, **kw):
    loss, tl, _ = run_gpu(bits, y, cu, mode, t_ave, want_grad=False, **kw)
    want, want_tl, _ = L.packed_ce(wl.bf16_bits_to_f32(bits).astype(np.float64), y, cu, mode, t_ave)
    assert np.abs(tl - want_tl).max() <= TOKEN_LOSS_ABS
    assert abs(loss - want) <= LOSS_REL * abs(want) + 1e-7
    with_grad = run_gpu(bits, y, cu, mode, t_ave, **kw)
    assert with_grad[0] == loss and np.array_equal(with_grad[1], tl)


@pytest.mark.parametrize("V", [8, 2040, 2048, 2056, 4104, 16384, 16392, 20480, 20488, 81920, 81928, 90112, 163840, 163848])
def test_row_lengths(V):
    bits, y, cu = make_case([5, 1, 4], V, V % 91)
    check(bits, y, cu, 2)


@pytest.mark.parametrize("V,T", [(2048, 1), (2048, 3000), (2056, 1500), (20488, 900), (90120, 300)])
@pytest.mark.parametrize("pattern", ["all", "one", "ends", "runs", "none"])
def test_rows_without_a_loss(V, T, pattern):
    bits, y, cu = make_case([T - T // 3, T // 3] if T > 2 else [T], V, T % 89, p_mask=0.0)
    if pattern == "one":
        y[np.arange(T) != T // 2] = -100
    elif pattern == "ends":
        y[:T // 3] = -100
        y[T - T // 4:] = -100
    elif pattern == "runs":
        y[np.arange(T) // 7 % 3 != 1] = -100
    elif pattern == "none":
        y[:] = -100
    check(bits, y, cu, 0)


def test_more_rows_than_are_staged_at_a_time():
    T = 200000  # rows whose ranges hold no loss, and ranges with losses on both sides of a batch of rows
    bits, y, cu = make_case([150000, 50000], 16, 5, p_mask=0.0)
    keep = np.zeros(T, dtype=bool)
    keep[[0, 255, 256, 257, 511, 512, T - 1]] = True
    keep[90000:90600] = True
    y[~keep] = -100
    check(bits, y, cu, 1)


def test_row_stride():
    bits, y, cu = make_case([70, 30], 512, 3)
    check(bits, y, cu, 0, stride=520)


@pytest.mark.parametrize("pattern", [0x7FC0, 0x7F81, 0x7F80])
@pytest.mark.parametrize("V", [4104, 90120])
def test_a_nan_or_an_infinity_stays_in_its_row(V, pattern):
    bits, y, cu = make_case([40, 20], V, 9, p_mask=0.0)
    _, clean, _ = run_gpu(bits, y, cu, 0, want_grad=False)
    bits[17, V - 3] = pattern
    loss, tl, _ = run_gpu(bits, y, cu, 0, want_grad=False)
    assert np.isnan(loss) and np.isnan(tl[17])
    assert np.array_equal(np.delete(tl, 17), np.delete(clean, 17))
