"""The training epoch in blocks of steps: numbers of steps around a block (256 examples), workers
around its rounds of 4, 8 and 16, the most workers and classes it takes and one more of each."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from parity import check_epoch, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2302_00845_amd as p
    return p


@pytest.mark.parametrize("m,n,in_dim,classes,momentum", [
    (1, 256, 6, 2, 0.9), (1, 258, 3, 3, 0.9), (1, 520, 1, 2, 0.0), (3, 84, 5, 4, 0.9), (3, 86, 33, 5, 0.9),
    (4, 66, 8, 16, 0.5), (5, 52, 70, 7, 0.9), (8, 34, 9, 10, 0.9), (9, 60, 40, 10, 0.9), (16, 16, 31, 10, 0.9),
    (16, 50, 130, 10, 0.9), (17, 30, 12, 3, 0.9), (33, 16, 12, 3, 0.0), (64, 4, 20, 16, 0.9), (64, 10, 20, 5, 0.9),
    (65, 6, 20, 5, 0.9), (4, 20, 20, 17, 0.9), (16, 140, 2000, 10, 0.9), (7, 40, 3, 1, 0.9),
])
@pytest.mark.parametrize("with_perm", [True, False])
def test_blocks_of_steps_match_oracle(lib, m, n, in_dim, classes, momentum, with_perm):
    X, y, W0 = workloads.softmax_problem(m + n, m * n, in_dim, classes)
    X, y, W0 = X.reshape(m, n, in_dim), y.reshape(m, n), (10 * W0).astype(np.float32)
    perm = workloads.random_perms(3, m, n) if with_perm else None
    lr = 0.2 / max(1.0, in_dim / 20)                      # contractive: rounding does not grow over the epoch
    h = lib.Handle()
    W = torch.from_numpy(W0.copy()).cuda()
    v = torch.zeros(W.numel(), dtype=torch.float32, device="cuda") if momentum else None
    out = lib.cdgrab_train_epoch_softmax(h, torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), W,
                                         perm_in=torch.from_numpy(perm).cuda() if with_perm else None, velocity=v,
                                         lr=lr, momentum=momentum, want_grads=True, want_loss=True)
    torch.cuda.synchronize()
    ref = oracle.train_epoch_softmax(X, y, perm if with_perm else np.tile(np.arange(n, dtype=np.int32), (m, 1)), W0,
                                     None, lr, momentum)
    rows = out["grads"].cpu().numpy()
    # the 1e-5 relative L2 stated for per-example gradients; W after up to 520 fp32 updates of a
    # contractive iteration: below 520 x 6e-8 = 3e-5 even if no rounding cancelled
    if classes > 1:
        assert rel_l2(W.cpu().numpy(), ref["W"]) <= 3e-5
        # a row is [x; 1] delta^T, delta = p - onehot in fp32: where p is nearly 1 delta is a small difference,
        # off by the rounding of p (6e-8) and by 1/2 of the logits' error (W's 3e-5 relative error, in
        # practice 1e-6), so each row is held to 1e-5 of ||[x; 1]||, the bound for delta of order one
        err = np.linalg.norm(rows - ref["rows"], axis=2)
        xs = X if perm is None else np.take_along_axis(X, perm[:, :, None].astype(np.int64), 1)
        assert np.all(err <= 1e-5 * np.sqrt(1.0 + (xs.astype(np.float64) ** 2).sum(2)))
        if momentum:
            assert rel_l2(v.cpu().numpy(), ref["v"]) <= 3e-5
    else:
        assert np.abs(rows).max() <= 1e-6
    np.testing.assert_allclose(out["loss"].cpu().numpy(), ref["loss"], rtol=1e-4, atol=1e-5)
    check_epoch(rows, {"signs": out["signs"].cpu().numpy(), "perm": out["perm"].cpu().numpy()}, perm)


@pytest.mark.parametrize("m,n,in_dim,classes", [
    (16, 2, 30, 10), (16, 18, 30, 10), (16, 20, 30, 10), (64, 6, 30, 10), (40, 14, 30, 4),   # 2 / 16 + 2 / 16 + 4 / 4 + 2 / 6 + 6 + 2
    (16, 4, 2049, 4), (16, 20, 2049, 8), (16, 22, 2049, 2), (16, 4, 2049, 9), (33, 4, 2049, 4), (16, 4, 2048, 4),
    (24, 12, 5500, 3), (40, 6, 5500, 3), (17, 12, 5500, 3), (16, 14, 32769, 4),              # rows of 16 503 and 131 080 elements
])
@pytest.mark.parametrize("with_perm", [True, False])
def test_short_blocks_go_as_launch_pairs(lib, m, n, in_dim, classes, with_perm):
    """Numbers of steps around the shortest block (4, 6 or 8 by features, classes and workers), which leave none,
    some or all of a chunk's steps to a launch pair each."""
    test_blocks_of_steps_match_oracle(lib, m, n, in_dim, classes, 0.9, with_perm)


@pytest.mark.parametrize("m", [8, 65])                    # blocks of steps, a launch pair per step
def test_label_that_names_no_class_leaves_its_loss(lib, m):
    """Such an example's delta is its softmax; nothing is written as its loss."""
    n, in_dim, classes = 8, 12, 5
    X, y, W0 = workloads.softmax_problem(3, m * n, in_dim, classes)
    X, y = torch.from_numpy(X).cuda().view(m, n, in_dim), torch.from_numpy(y).cuda().view(m, n)
    y[1, 2], y[m - 1, 5] = -1, classes
    h, W = lib.Handle(), torch.from_numpy(W0.astype(np.float32)).cuda()
    signs = torch.empty((m, n // 2), dtype=torch.int8, device="cuda")
    perm = torch.empty((m, n), dtype=torch.int32, device="cuda")
    rows = torch.empty((m, n, (in_dim + 1) * classes), device="cuda")
    loss = torch.full((m, n), 123.0, device="cuda")
    h._check(h._lib.cdgrab_train_epoch_softmax(
        h._h, m, n, in_dim, classes, X.data_ptr(), y.data_ptr(), None, W.data_ptr(), None, 0.05, 0.0,
        signs.data_ptr(), perm.data_ptr(), rows.data_ptr(), loss.data_ptr()))
    ignored = torch.zeros((m, n), dtype=torch.bool, device="cuda")
    ignored[1, 2] = ignored[m - 1, 5] = True
    assert torch.all(loss[ignored] == 123.0) and torch.all(loss[~ignored] < 50.0)
    # the bias row of a gradient is delta itself: it sums to 1 without a label, to 0 with one (5 roundings of 6e-8)
    total = rows.view(m, n, in_dim + 1, classes)[:, :, in_dim].sum(2)
    assert torch.all((total - ignored.float()).abs() <= 1e-6)


@pytest.mark.parametrize("m,n,in_dim,classes", [(11, 900, 470, 10), (3, 86, 99, 10), (37, 120, 99, 10)])
def test_staged_rows_are_a_bounded_chunk_of_the_epoch(lib, m, n, in_dim, classes):
    """What an epoch allocates on a new handle: two chunks of 256 MB or 1024 pairs each, none longer than the
    epoch, beside at most 64 MB of other workspace (Gram tiles of a chunk and their shares, for the most part)."""
    d, pairs = (in_dim + 1) * classes, m * n // 2

    def epoch(m, n):
        X, y, W0 = workloads.softmax_problem(1, m * n, in_dim, classes)
        args = (torch.from_numpy(X).cuda().view(m, n, in_dim), torch.from_numpy(y).cuda().view(m, n),
                torch.from_numpy(W0.astype(np.float32)).cuda())
        out = lib.cdgrab_train_epoch_softmax(lib.Handle(), *args, lr=0.01)  # (its outputs come from torch's pool)
        torch.cuda.synchronize()
        h = lib.Handle()
        before = torch.cuda.mem_get_info()[0]
        lib.cdgrab_train_epoch_softmax(h, *args, lr=0.01)
        torch.cuda.synchronize()
        del out
        return before - torch.cuda.mem_get_info()[0]

    taken = epoch(m, n)
    assert taken <= 2 * min(max(1024 * 8 * d, 256 << 20), pairs * 8 * d) + (64 << 20), taken
