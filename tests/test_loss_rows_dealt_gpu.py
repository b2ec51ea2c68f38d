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


def check_long_pack(T, V, live):
    """A pack too long for the oracle, `live` rows with a loss; token mean.  Against torch's fp32 softmax, slice by slice: the
    gradient's own rounding to bf16 decides."""
    import torch
    import paper_2503_07680_amd as H
    gen = torch.Generator(device="cuda").manual_seed(5)
    logits = torch.empty((T, V), dtype=torch.bfloat16, device="cuda").normal_(0.0, 2.0, generator=gen)
    y = torch.randint(0, V, (T,), dtype=torch.int32, device="cuda", generator=gen)
    y[torch.randperm(T, device="cuda", generator=gen)[live:]] = -100
    cu = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    dl = torch.full((T, V), float("nan"), dtype=torch.bfloat16, device="cuda")
    loss, tl = torch.empty(1, device="cuda"), torch.full((T,), float("nan"), device="cuda")
    ws = torch.empty(H.hbp_packed_ce_workspace_bytes(T, 1), dtype=torch.uint8, device="cuda")
    H.hbp_packed_ce(logits, 0, T, V, y, cu, 1, 0, 0.0, dl, loss, tl, ws, int(torch.cuda.current_stream().cuda_stream))
    step = 8192 * 10248 // V
    for a in range(0, T, step):
        z, lab = logits[a:a + step].float(), y[a:a + step].long()
        has = lab >= 0
        got_tl, got = tl[a:a + step], dl[a:a + step]
        assert not got[~has].any() and not got_tl[~has].any()
        want_tl = torch.where(has, torch.logsumexp(z, 1) - z.gather(1, lab.clamp(min=0)[:, None])[:, 0], 0.0)
        assert (got_tl - want_tl).abs().max() <= 2e-5
        if has.any():
            g = torch.softmax(z, 1)
            g.scatter_add_(1, lab.clamp(min=0)[:, None], -torch.ones_like(want_tl)[:, None])
            g.mul_(torch.where(has, 1.0 / live, 0.0)[:, None])
            err = (got.float() - g).norm() / g.norm()
            assert err <= 4e-3, float(err)


def test_the_longest_packs_planned_in_the_main_kernel():
    """131000 rows on the workgroups that fit beside that much planning: some 50 rows of either kind in each."""
    check_long_pack(131000, 10248, 65500)


@pytest.mark.parametrize("live", [69500, 700, 0])
def test_more_rows_a_workgroup_than_are_staged_at_a_time(live):
    """One workgroup of 1024 threads a compute unit, at most 256 of them, and 256 rows staged at a time: 70000 rows are 273 of
    one kind each, a second batch of rows with a loss or of zeros (the whole of it ahead of the first row with a loss)."""
    check_long_pack(70000, 81928, live)
