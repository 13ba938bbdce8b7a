"""Rows of any length at any 4-byte aligned address: every launch form reads four elements
with one load, whose last group must stop at the end of the row.  Small-integer rows, so the
oracle must be matched bit for bit; the rows lie between guard values that would show."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from parity import check_epoch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2302_00845_amd as p
    return p


def shifted(z, shift):
    """z on the GPU, `shift` floats after a 16-byte boundary, with huge values on either side."""
    flat = torch.full((z.size + 16,), 1e30, dtype=torch.float32, device="cuda")
    view = flat[4 + shift:4 + shift + z.size].view(z.shape)
    view.copy_(torch.from_numpy(z))
    return view


@pytest.mark.parametrize("shift", [0, 1, 2, 3])
@pytest.mark.parametrize("m,n,d,kw", [
    (2, 6, 1, {}), (2, 6, 2, {}), (2, 6, 3, {}), (2, 6, 4, {}), (2, 6, 5, {}), (3, 40, 6, {}), (3, 44, 63, {}),
    (3, 44, 65, {}), (3, 44, 66, dict(gram_mode=1)), (3, 44, 127, dict(gram_mode=1, apply_mode=1)),
    (2, 24, 16385, {}), (2, 24, 65535, {}), (2, 24, 65539, dict(apply_mode=1)), (2, 20, 70001, dict(apply_mode=3)),
    (2, 20, 70002, dict(apply_mode=4)), (3, 24, 131073, {}),
])
def test_epoch_on_rows_of_any_alignment(lib, shift, m, n, d, kw):
    z = workloads.integer_rows(d + shift, m, n, d, 3)
    h = lib.Handle(**kw)
    out = lib.cdgrab_balance_epoch(h, m, n, d, grads=shifted(z, shift), want_r64=True, want_dots=True)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    rep = check_epoch(z, got, expect_exact_signs=True)
    assert rep["r64_rel_l2"] == 0.0 and rep["dots_max_abs_err"] == 0.0


@pytest.mark.parametrize("shift", [0, 1, 2, 3])
@pytest.mark.parametrize("m,n,d", [(3, 8, 1), (3, 8, 3), (3, 8, 5), (2, 30, 63), (2, 30, 517), (2, 6, 4099)])
def test_herding_bound_on_rows_of_any_alignment(lib, shift, m, n, d):
    z = workloads.integer_rows(d, m, n, d, 5)
    perm = workloads.random_perms(1, m, n)
    got = float(lib.cdgrab_herding_bound(lib.Handle(), shifted(z, shift), torch.from_numpy(perm).cuda())[0])
    # double sums in another order than the oracle's: rounding of about m n additions
    assert got == pytest.approx(oracle.parallel_herding(z, perm), rel=1e-13, abs=1e-13)


@pytest.mark.parametrize("n,d", [(1, 1), (1, 7), (9, 3), (300, 4), (2049, 5), (4097, 16), (65, 508), (65, 512), (65, 513),
                                 (30, 1030), (8193, 2)])
@pytest.mark.parametrize("shift", [0, 1])
def test_stale_mean_column_mean_and_order(lib, n, d, shift):
    """The epoch's mean (chunks of rows added in double: exact on small integers up to the one
    rounding of the quotient and the one to fp32) and the order its signs give."""
    z = workloads.integer_rows(n + d, 1, n, d, 4)[0]
    out = lib.cdgrab_balance_epoch_stale_mean(lib.Handle(), shifted(z, shift))
    assert np.array_equal(out["mean"].cpu().numpy(), (z.astype(np.float64).sum(0) / n).astype(np.float32))
    assert np.array_equal(out["perm"].cpu().numpy(), oracle.reorder(out["signs"].cpu().numpy(), None))


@pytest.mark.parametrize("m,n", [(5, 1), (5, 63), (5, 65), (300, 255), (3, 256), (3, 257), (3, 1023), (3, 1024),
                                 (3, 1025), (3, 2047), (3, 2049), (3, 4095), (3, 4096), (3, 4097), (2, 8192), (1, 8193), (70, 4100), (1, 1_000_003)])
@pytest.mark.parametrize("with_perm", [False, True])
def test_reorder_across_chunks(lib, m, n, with_perm):
    signs = workloads.random_signs(n, m, n)
    signs[0, :5000] = 1                                   # a chunk of one sign only
    perm_in = workloads.random_perms(n, m, n) if with_perm else None
    out = lib.cdgrab_reorder(lib.Handle(), torch.from_numpy(signs).cuda(),
                             torch.from_numpy(perm_in).cuda() if with_perm else None).cpu().numpy()
    for i in range(m):
        assert np.array_equal(out[i], oracle.reorder(signs[i], perm_in[i] if with_perm else None))


def test_mean_of_long_rows_takes_no_workspace(lib):
    """Rows long enough to fill the GPU by themselves: the mean is written straight from the rows (exact on
    small integers up to the two roundings), and the epoch allocates the running sum and partials only."""
    n, d = 6, 30_000_001
    z = torch.randint(-4, 5, (n, d), device="cuda", dtype=torch.int8).float()
    lib.cdgrab_balance_epoch_stale_mean(lib.Handle(), z[:, :1000].contiguous(), z[0, :1000].contiguous())
    lib.cdgrab_balance_epoch_stale_mean(lib.Handle(), z[:2], z[0])   # (torch's pool holds outputs of this size now)
    torch.cuda.synchronize()
    h = lib.Handle()
    before = torch.cuda.mem_get_info()[0]
    out = lib.cdgrab_balance_epoch_stale_mean(h, z, z[0])
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] <= 8 * d + (64 << 20)
    assert torch.equal(out["mean"], (z.double().sum(0) / n).float())
