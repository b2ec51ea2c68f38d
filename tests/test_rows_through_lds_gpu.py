"""Q, dO, K and V taken through LDS in whole rows, and dQ, dK and dV the other way: every count of rows of a wavefront's 32 at
its edges, every form of the backward (one launch for dK/dV and dQ, two of them with records), token rows with padding.
Against the fp64 oracle (bars of the path), the same bits with padded rows as without, and nothing written to the padding."""
import numpy as np
import pytest

from parity_util import Case, compare
from test_one_backward_launch_gpu import run

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 31, 32, 33, 63, 65, 95, 96, 97, 127, 128, 129, 161]


@pytest.mark.parametrize("Hq,Hkv,d,e", [(2, 2, 64, 64), (4, 2, 64, 64), (3, 3, 128, 128), (4, 2, 128, 128), (6, 2, 128, 128),
                                        (3, 3, 192, 128), (4, 2, 192, 128)])
def test_rows(Hq, Hkv, d, e):
    case = Case(EDGES, sum(EDGES), Hq, Hkv, d, e, seed=711, name="rows-%d-%d-%d" % (Hq, Hkv, d))
    pa, dev, out = run(case)
    compare(case, pa, out)
    pad, _, padded = run(case, row_pad=64)
    for n in out:
        assert np.array_equal(out[n], padded[n]), n
    for x in (pad.o, pad.dq, pad.dk, pad.dv):
        assert not x._base[:, -64:].any()  # buffers start as zeros
