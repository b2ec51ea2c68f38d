"""The backward's first kernel (rowsum of dO O and the scaled log-sum-exp) in both sizes of its workgroups: head counts
below, at and beside its eight heads, tokens that are no multiple of its rows, padded rows, and packs on either side of
the line between the sizes; through dQ, dK and dV, which a wrong row sum changes, against the fp64 oracle."""
import numpy as np
import pytest

from parity_util import Case, compare, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,e", [(64, 64), (128, 128), (192, 128)])
@pytest.mark.parametrize("Hq,T", [(1, 1), (1, 259), (2, 131), (3, 67), (5, 33), (8, 7), (9, 65), (12, 31), (17, 40)])
def test_heads_and_rows(d, e, Hq, T):
    case = Case([T // 2, T - T // 2] if T > 1 else [1], T, Hq, Hq, d, e, seed=601, name="prepass-%d-%d-%d" % (Hq, T, d))
    pa, dev, out = run_gpu(case)
    compare(case, pa, out)


@pytest.mark.parametrize("d,T", [(64, 8192), (64, 8193), (128, 8192), (128, 8193)])
def test_either_side_of_the_line(d, T):
    lengths = [128] * 63 + [T - 128 * 63]
    case = Case(lengths, T, 16, 16, d, d, seed=602, name="prepass-line-%d-%d" % (T, d))
    pa, dev, out = run_gpu(case)
    rows = sorted(set(np.random.default_rng(2).integers(0, T, 300).tolist()) | {0, T - 1})
    compare(case, pa, out, q_heads=[0, 7, 8, 15], rows=rows, cols=rows)
