"""The chain of long steps that short rows are balanced with: numbers of pairs around its tiles of
64 pairs and its steps of 64, 128 and 256 (rows of about 40 000, 12 000 and 50 elements choose
those), in each layout the rows come in.  Small-integer rows, so every sum is exact and the
oracle must be matched bit for bit, ties included."""
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


@pytest.mark.parametrize("m,n,d", [
    (1, 128, 50), (1, 130, 50), (3, 84, 33), (1, 254, 50), (2, 128, 50), (1, 258, 50), (5, 102, 64), (1, 510, 50),
    (1, 512, 50), (1, 514, 50), (7, 220, 16), (100, 12, 16), (1, 2050, 3), (2, 126, 12_000), (3, 86, 12_001),
    (1, 600, 12_002), (2, 130, 40_000), (5, 56, 40_003), (3, 44, 65_536),
])
def test_dense_steps_match_oracle(lib, m, n, d):
    z = workloads.integer_rows(m + n, m, n, d, 3)
    perm = workloads.random_perms(2, m, n)
    out = lib.cdgrab_balance_epoch(lib.Handle(gram_mode=2), m, n, d, grads=torch.from_numpy(z).cuda(),
                                   perm_in=torch.from_numpy(perm).cuda(), want_r64=True, want_dots=True)
    torch.cuda.synchronize()
    rep = check_epoch(z, {k: v.cpu().numpy() for k, v in out.items()}, perm, expect_exact_signs=True)
    assert rep["r64_rel_l2"] == 0.0 and rep["dots_max_abs_err"] == 0.0


@pytest.mark.parametrize("m,n,d", [
    (1, 34, 1), (1, 126, 2), (1, 128, 3), (1, 130, 4), (2, 128, 5), (3, 86, 15), (5, 52, 17), (1, 382, 31), (1, 384, 32),
    (1, 386, 33), (7, 74, 63), (11, 48, 64), (300, 4, 64),
])
def test_narrow_rows_match_oracle(lib, m, n, d):
    """Rows of at most 64 elements: the whole walk in one workgroup, blocks of 64 pairs, the padded
    row lengths 16, 32 and 64."""
    test_dense_steps_match_oracle(lib, m, n, d)


@pytest.mark.parametrize("n,d", [(64, 17), (65, 16), (129, 40), (300, 16), (513, 5), (300, 12_000)])
def test_centred_steps_match_oracle(lib, n, d):
    g = workloads.integer_rows(n, 1, n, d, 3)[0]
    mean = np.rint(np.linspace(-2, 2, d)).astype(np.float32)
    out = lib.cdgrab_balance_epoch_stale_mean(lib.Handle(), torch.from_numpy(g).cuda(), torch.from_numpy(mean).cuda())
    want = oracle.grab_stale_mean(g, mean)
    assert np.array_equal(out["signs"].cpu().numpy(), want["s"])
    assert np.array_equal(out["r64"].cpu().numpy(), want["r"])


@pytest.mark.parametrize("m,n,d", [(3, 128, 40), (9, 130, 40), (2, 600, 17), (40, 70, 1000), (5, 300, 9000), (2, 130, 65_536)])
def test_walks_side_by_side_equal_single_walks(lib, m, n, d):
    z = workloads.integer_rows(m, m, n, d, 3)
    out = lib.cdgrab_balance_epoch_independent(lib.Handle(), torch.from_numpy(z).cuda())
    for i in range(m):
        want = oracle.server_epoch(z[i:i + 1], None)
        assert np.array_equal(out["signs"][i].cpu().numpy(), want["eps"][0])
        assert np.array_equal(out["perm"][i].cpu().numpy(), want["perm"][0])


@pytest.mark.parametrize("m,n,d", [(3, 86, 30), (2, 300, 12_000), (1, 600, 20)])
def test_randomized_rule_over_steps(lib, m, n, d):
    """Rows scaled by a power of two (sums stay exact) so that many probabilities lie inside (0, 1)."""
    z = workloads.integer_rows(n, m, n, d, 2) * np.float32(2.0 ** -5)
    u = np.random.default_rng(n).random((m, n // 2), dtype=np.float32)
    out = lib.cdgrab_balance_epoch_randomized(lib.Handle(), torch.from_numpy(z).cuda(), torch.from_numpy(u).cuda())
    r = np.zeros(d)
    for k in range(n // 2):
        for i in range(m):
            dv = z[i, 2 * k + 1].astype(np.float64) - z[i, 2 * k]
            t = float(r @ dv)
            eps = -1 if float(u[i, k]) < 0.5 * (1.0 + t) else 1
            assert int(out["signs"][i, k]) == eps, (k, i)
            r += eps * dv
    assert np.array_equal(out["r64"].cpu().numpy(), r)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("m,n,d", [
    (3, 24, 20), (1, 130, 50),                    # rows of at most 64 elements
    (1, 130, 66), (3, 86, 129), (1, 600, 1001),   # steps of 128 and 256 pairs, the last one ragged
    (2, 130, 12_000), (1, 142, 40_003),           # of 64 pairs
    (2, 20, 70_001),                              # one launch per block of pairs
])
def test_value_that_is_not_finite_stays_where_it_is(lib, value, m, n, d):
    """One element of the epoch's last pair is infinite or not a number: that element of the running
    sum follows it, every other one is the exact sum under the signs the epoch reports."""
    z = workloads.integer_rows(n + d, m, n, d, 3)
    z[m - 1, n - 1, 5] = value
    out = lib.cdgrab_balance_epoch(lib.Handle(), m, n, d, grads=torch.from_numpy(z).cuda(), want_r64=True)
    eps = out["signs"].cpu().numpy().astype(np.float64)
    diff = (z[:, 1::2].astype(np.float64) - z[:, 0::2])
    want = np.einsum("ik,ikd->d", eps, diff)
    assert np.array_equal(out["r64"].cpu().numpy(), want, equal_nan=True)
    assert np.array_equal(out["r32"].cpu().numpy(), want.astype(np.float32), equal_nan=True)


@pytest.mark.parametrize("m,n,d", [(1, 2050, 70), (16, 300, 7850), (3, 500, 16), (2, 130, 40_000), (3, 20, 300)])
def test_timing_counts_what_the_plan_says(lib, m, n, d):
    plan = lib.cdgrab_plan_epoch(m, n, d)
    h = lib.Handle(timing=1)
    z = torch.zeros((m, n, d), device="cuda")
    lib.cdgrab_balance_epoch(h, m, n, d, grads=z)
    unit = plan["step_pairs"] or plan["block_pairs"]
    got = h.timing()
    assert got["block_pairs"] == unit and got["blocks"] == -(-plan["pairs"] // unit)
