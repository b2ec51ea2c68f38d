"""Cross-entropy with the gradient, long rows: rows with and without a loss are dealt in turn to the workgroups.  Vocabularies
on both sides of the line, a workgroup a row and one row more, few to many rows a workgroup, counts of either kind of row
around a multiple of the workgroups, none of one kind, more rows a workgroup than are staged at a time.  Against the fp64
oracle, and the losses against the call without the gradient, whose rows are consecutive: the same bits."""
import numpy as np
import pytest

from test_loss_gpu import check, make_case, run_gpu

pytestmark = pytest.mark.gpu


def labels_with(y, live):
    """The same labels with a loss in `live` rows alone, spread over the pack."""
    y = np.where(y < 0, 1, y).astype(np.int32)
    T = len(y)
    order = np.random.default_rng(T + live).permutation(T)
    y[order[live:]] = -100
    return y


def check_both(bits, y, cu, mode, **kw):
    loss = check(bits, y, cu, mode, t_ave=9.0, **kw)
    without = run_gpu(bits, y, cu, mode, 9.0, want_grad=False, **kw)
    with_grad = run_gpu(bits, y, cu, mode, 9.0, **kw)
    assert without[0] == loss == with_grad[0] and np.array_equal(without[1], with_grad[1])


@pytest.mark.parametrize("V", [10240, 10248])
@pytest.mark.parametrize("T,live", [(700, 400), (2047, 1), (2100, 1792), (2100, 2099)])
def test_either_side_of_the_line(V, T, live):
    bits, y, cu = make_case([T - 301, 300, 1], V, T % 83)
    check_both(bits, labels_with(y, live), cu, 2)


@pytest.mark.parametrize("T", [255, 256, 257, 511, 512, 513, 640])  # a workgroup or two a compute unit at this length
@pytest.mark.parametrize("share", [0.0, 0.4, 1.0])
def test_rows_around_the_number_of_workgroups(T, share):
    bits, y, cu = make_case([T - 100, 99, 1], 61448, T % 83)
    check_both(bits, labels_with(y, int(share * T)), cu, 0)


@pytest.mark.parametrize("live", [1, 255, 256, 257, 383, 511, 512, 639])
def test_counts_of_either_kind(live):
    bits, y, cu = make_case([200, 439, 1], 28680, live % 83)
    check_both(bits, labels_with(y, live), cu, 1, stride=28688)


def test_more_rows_a_workgroup_than_are_staged_at_a_time():
    """131000 rows on at most 1792 workgroups of this length: 73 and more a workgroup; and the rows of a longer pack."""
    import torch
    import paper_2503_07680_amd as H
    T, V = 131000, 10248
    gen = torch.Generator(device="cuda").manual_seed(5)
    logits = torch.empty((T, V), dtype=torch.bfloat16, device="cuda").normal_(0.0, 2.0, generator=gen)
    y = torch.randint(0, V, (T,), dtype=torch.int32, device="cuda", generator=gen)
    y[torch.rand(T, device="cuda", generator=gen) < 0.5] = -100
    cu = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    dl = torch.full((T, V), float("nan"), dtype=torch.bfloat16, device="cuda")
    loss, tl = torch.empty(1, device="cuda"), torch.full((T,), float("nan"), device="cuda")
    ws = torch.empty(H.hbp_packed_ce_workspace_bytes(T, 1), dtype=torch.uint8, device="cuda")
    H.hbp_packed_ce(logits, 0, T, V, y, cu, 1, 0, 0.0, dl, loss, tl, ws, int(torch.cuda.current_stream().cuda_stream))
    n_live = int((y >= 0).sum())
    assert not dl[y < 0].any() and not tl[y < 0].any()
    for a in range(0, T, 8192):  # fp32 softmax of torch: the gradient's own rounding to bf16 decides
        z, lab = logits[a:a + 8192].float(), y[a:a + 8192].long()
        has = lab >= 0
        want_tl = torch.where(has, torch.logsumexp(z, 1) - z.gather(1, lab.clamp(min=0)[:, None])[:, 0], 0.0)
        assert (tl[a:a + 8192] - want_tl).abs().max() <= 2e-5
        g = torch.softmax(z, 1)
        g.scatter_add_(1, lab.clamp(min=0)[:, None], -torch.ones_like(want_tl)[:, None])
        g.mul_(torch.where(has, 1.0 / n_live, 0.0)[:, None])
        err = (dl[a:a + 8192].float() - g).norm() / g.norm()
        assert err <= 4e-3, float(err)
