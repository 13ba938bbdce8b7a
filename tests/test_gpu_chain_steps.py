"""The chain of long steps that short rows are balanced with: numbers of pairs around its tiles of
64 pairs and its steps of 64, 128 and 256, in each layout the rows come in, more Gram tiles than
are held at a time, and the one-workgroup walk of rows of at most 64 elements.  Small-integer rows, so
every sum is exact and the oracle must be matched bit for bit, ties included."""
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
def test_dense_epochs_match_oracle(lib, m, n, d):
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
    assert lib.cdgrab_plan_epoch(m, n, d)["step_pairs"] == (64 if m * n > 128 else 0)
    test_dense_epochs_match_oracle(lib, m, n, d)


LONG_NARROW = [  # pairs around multiples of 16 and 128, padded row lengths 16, 32 and 64, rows too short for one load
    (1, 1024, 1), (2, 514, 2), (1, 1026, 3), (1, 1054, 4), (5, 206, 15), (1, 1280, 16), (3, 342, 17), (1, 1282, 31),
    (7, 300, 32), (1, 1278, 33), (16, 130, 63), (300, 8, 64),
]


@pytest.mark.parametrize("m,n,d", LONG_NARROW)
def test_long_narrow_walks_match_oracle(lib, m, n, d):
    """At least 512 pairs of rows of at most 64 elements: Gram results of sixteen pairs with the next 64 beforehand."""
    small = lib.cdgrab_plan_epoch(1, 1022, d)["workspace_bytes"]
    assert lib.cdgrab_plan_epoch(m, n, d)["workspace_bytes"] - small >= m * n // 2 * (512 + 8 * 16)
    test_dense_epochs_match_oracle(lib, m, n, d)
    z = torch.from_numpy(workloads.integer_rows(n, m, n, d, 3)).cuda()
    whole, inside = (lib.cdgrab_balance_epoch(lib.Handle(gram_mode=g), m, n, d, grads=z, want_r64=True, want_dots=True)
                     for g in (2, 1))
    assert all(torch.equal(whole[k], inside[k]) for k in ("signs", "perm", "r64", "r32", "dots"))


@pytest.mark.parametrize("d", [16, 24, 64])
def test_more_narrow_pairs_than_are_held_at_a_time(lib, d):
    """64 MB of results and differences are held: the running sum goes from launch to launch."""
    m, n = 3, 2 * 36_000 if d < 64 else 2 * 24_000
    assert m * n // 2 * (512 + 8 * (16 if d == 16 else 32 if d == 24 else 64)) > 64 << 20
    z = workloads.integer_rows(5, m, n, d, 3)
    out = lib.cdgrab_balance_epoch(lib.Handle(), m, n, d, grads=torch.from_numpy(z).cuda(), want_r64=True)
    want = oracle.server_epoch(z, None)
    assert np.array_equal(out["signs"].cpu().numpy(), want["eps"])
    assert np.array_equal(out["r64"].cpu().numpy(), want["r"])


def narrow_pairs_held(d, walks=1):
    """Pairs of a walk per launch: 64 MB of Gram results, differences and draws, 16 pairs at a time, by eights."""
    block = 8 * (16 * 64 + 16 * (16 if d <= 16 else 32 if d <= 32 else 64) + 8)
    blocks = (64 << 20) // block // walks
    return 16 * ((blocks + 7) // 8 * 8)


def greedy_in_doubles(z):
    """Signs, dots and running sum of one walk over pairs [m][n/2], by comparison: t <= 0 gives +1, no number -1."""
    diff = (z[:, 1::2].astype(np.float64) - z[:, 0::2]).transpose(1, 0, 2).reshape(-1, z.shape[2])
    r, eps, dots = np.zeros(z.shape[2]), np.empty(len(diff), np.int8), np.empty(len(diff))
    with np.errstate(invalid="ignore"):
        for q, dv in enumerate(diff):
            dots[q] = r @ dv
            eps[q] = 1 if dots[q] <= 0 else -1
            r = r + eps[q] * dv
    return eps, dots, r


@pytest.mark.parametrize("d", [9, 30, 64])
def test_narrow_launches_follow_each_other(lib, d):
    """A launch begins at a pair of any worker: draws, signs and dots are where they belong, the running sum is handed on, also where
    it holds what is not finite, and launches before that are not held up by it."""
    m = 7
    held = narrow_pairs_held(d)
    n = 2 * (held // m + 300)
    assert m * n // 2 > held and held % m
    z = workloads.integer_rows(d, m, n, d, 2) * np.float32(2.0 ** -5)
    zt = torch.from_numpy(z).cuda()
    u = np.random.default_rng(d).random((m, n // 2), dtype=np.float32)
    out = lib.cdgrab_balance_epoch_randomized(lib.Handle(), zt, torch.from_numpy(u).cuda())
    want = oracle.randomized_epoch(z, u)
    assert np.array_equal(out["signs"].cpu().numpy(), want["eps"]) and np.array_equal(out["dots"].cpu().numpy(), want["t"])
    assert np.array_equal(out["r64"].cpu().numpy(), want["r"])
    eps, dots, _ = greedy_in_doubles(z)
    for at, value in ((held - 20, np.nan), (held - 20, np.inf), (held + 20, -np.inf), (held + 20, np.nan)):
        w = z.copy()
        w[at % m, 2 * (at // m) + 1, d // 2] = value
        out = lib.cdgrab_balance_epoch(lib.Handle(), m, n, d, grads=torch.from_numpy(w).cuda(), want_r64=True, want_dots=True)
        got, seen = (out[k].cpu().numpy().T.ravel() for k in ("signs", "dots"))
        assert np.array_equal(got[:at], eps[:at]) and np.array_equal(seen[:at], dots[:at])
        if np.isnan(value):
            assert (got[at:] == -1).all() and np.isnan(seen[at:]).all()
        # (an infinite pair's own dot may be infinite or no number: the shares of it that a block adds up are infinite already)
        assert np.array_equal(got, np.where(seen <= 0, 1, -1))
        diff = (w[:, 1::2].astype(np.float64) - w[:, 0::2]).transpose(1, 0, 2).reshape(-1, d)
        assert np.array_equal(out["r64"].cpu().numpy(), (got[:, None] * diff).sum(0), equal_nan=True)
    test_centred_steps_match_oracle(lib, held + 301, d)


def test_narrow_launches_of_many_walks_follow_each_other(lib):
    """Sixteen walks share the space; a value of one is no number in its first launch, of another in the second."""
    m, d = 16, 50
    held = narrow_pairs_held(d, m)
    n = 2 * (held + 700)
    z = workloads.integer_rows(4, m, n, d, 2)
    want = [greedy_in_doubles(z[i:i + 1])[0] for i in range(m)]
    z[3, 2 * 100, 7], z[12, 2 * held + 9, 20] = np.nan, np.nan
    want[3][100:], want[12][held + 4:] = -1, -1
    out = lib.cdgrab_balance_epoch_independent(lib.Handle(), torch.from_numpy(z).cuda())
    for i in range(m):
        assert np.array_equal(out["signs"][i].cpu().numpy(), want[i]), i


def test_recorded_narrow_walk(lib):
    """Recorded launches use none of the workspace that a later, longer epoch replaces."""
    m, n, d = 2, 1200, 20
    zi = workloads.integer_rows(3, m, n, d, 3)
    z, longer = torch.from_numpy(zi).cuda(), torch.randn((m, 4 * n, d), device="cuda")
    want = oracle.server_epoch(zi, None)
    s = torch.cuda.Stream()
    h = lib.Handle(stream=s)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        lib.cdgrab_balance_epoch(h, m, n, d, grads=z)
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        out = lib.cdgrab_balance_epoch(h, m, n, d, grads=z, want_r64=True)
    torch.cuda.synchronize()
    for _ in range(3):
        with torch.cuda.stream(s):
            lib.cdgrab_balance_epoch(h, m, 4 * n, d, grads=longer)
        for k in ("signs", "r64"):
            out[k].zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out["signs"].cpu().numpy(), want["eps"]) and np.array_equal(out["r64"].cpu().numpy(), want["r"])


def _recorded(lib, h, s, m, n, d, z):
    """A graph of one epoch on handle h (which has run that shape before), and the outputs it writes."""
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        out = lib.cdgrab_balance_epoch(h, m, n, d, grads=z, want_r64=True, want_dots=True)
    torch.cuda.synchronize()
    return graph, out


def _replays_equal(graph, out, want, between):
    for _ in range(3):
        between()
        for k in want:
            out[k].zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(out[k], want[k]) for k in want)


def test_recorded_chain_after_long_narrow_epochs(lib):
    """Long epochs of rows of at most 64 elements take none of the buffers that a recorded chain of steps holds."""
    m, n, d = 4, 64, 1024
    g = torch.Generator(device="cuda").manual_seed(5)
    z, narrow = torch.randn((m, n, d), generator=g, device="cuda"), torch.randn((1, 100_000, 16), generator=g, device="cuda")
    s = torch.cuda.Stream()
    h = lib.Handle(stream=s)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        want = {k: v.clone() for k, v in lib.cdgrab_balance_epoch(h, m, n, d, grads=z, want_r64=True, want_dots=True).items()}
    graph, out = _recorded(lib, h, s, m, n, d, z)

    def between():
        with torch.cuda.stream(s):
            lib.cdgrab_balance_epoch(h, 1, 100_000, 16, grads=narrow)
    _replays_equal(graph, out, want, between)


@pytest.mark.parametrize("m,n,d", [(1, 3000, 16), (2, 1200, 20), (1, 2050, 64)])
def test_recorded_narrow_walk_equals_the_eager_one(lib, m, n, d):
    """Bit for bit where sums are rounded: a recorded call runs the launches of the eager one, also when longer epochs
    have come between."""
    g = torch.Generator(device="cuda").manual_seed(n)
    z, longer = (torch.randn((m, k * n, d), generator=g, device="cuda") for k in (1, 5))
    s = torch.cuda.Stream()
    h = lib.Handle(stream=s)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        want = {k: v.clone() for k, v in lib.cdgrab_balance_epoch(h, m, n, d, grads=z, want_r64=True, want_dots=True).items()}
    graph, out = _recorded(lib, h, s, m, n, d, z)

    def between():
        with torch.cuda.stream(s):
            lib.cdgrab_balance_epoch(h, m, 5 * n, d, grads=longer)
    _replays_equal(graph, out, want, between)


# the steps of these are what the plan says (asserted): full ones, a ragged last one, one or several
@pytest.mark.parametrize("m,n,d,step", [
    (1, 258, 66, 256), (1, 510, 66, 256), (1, 512, 66, 256), (1, 514, 66, 128), (1, 2050, 70, 256), (7, 220, 130, 256),
    (5, 1000, 200, 256), (1, 2050, 1001, 256), (300, 10, 67, 256), (1, 130, 66, 128), (1, 600, 1001, 128),
    (3, 256, 7850, 128), (16, 130, 2049, 256), (16, 130, 6001, 128), (1, 258, 12_000, 64), (3, 100, 30_001, 64),
])
def test_steps_of_every_length_match_oracle(lib, m, n, d, step):
    assert lib.cdgrab_plan_epoch(m, n, d)["step_pairs"] == step
    test_dense_epochs_match_oracle(lib, m, n, d)


@pytest.mark.parametrize("d", [65, 96, 97, 128, 129, 160, 161, 225])
@pytest.mark.parametrize("m,n", [(1, 130), (9, 128), (2, 258)])
def test_tiles_of_few_elements_match_oracle(lib, m, n, d):
    """Gram tiles shared by workgroups of one to a few tiles of 32 elements each (one walk), and whole (many)."""
    test_dense_epochs_match_oracle(lib, m, n, d)
    test_walks_side_by_side_equal_single_walks(lib, 40 * m, n, d)


def steps_held(tiles_per_step):
    """Steps whose Gram tiles (64 x 64 doubles each) are held at a time: 256 MB of them."""
    return (256 << 20) // (tiles_per_step * 64 * 64 * 8)


def test_more_steps_than_are_held_at_a_time(lib):
    """220 000 pairs in steps of 256, ten tiles each: the last step of a batch of Gram tiles is applied
    by the first step of the next."""
    m, n, d = 1, 440_000, 66
    plan = lib.cdgrab_plan_epoch(m, n, d)
    assert plan["step_pairs"] == 256 and plan["pairs"] > steps_held(10) * 256
    z = workloads.integer_rows(5, m, n, d, 3)
    out = lib.cdgrab_balance_epoch(lib.Handle(), m, n, d, grads=torch.from_numpy(z).cuda(), want_r64=True)
    want = oracle.server_epoch(z, None)
    assert np.array_equal(out["signs"].cpu().numpy(), want["eps"])
    assert np.array_equal(out["perm"].cpu().numpy(), want["perm"])
    assert np.array_equal(out["r64"].cpu().numpy(), want["r"])


def test_more_steps_of_many_walks_than_are_held_at_a_time(lib):
    """1500 walks of 512 pairs side by side: whatever the steps' length, the walks' tiles (at least eight each)
    do not fit at once.  Against the same walks one after the other, and three of them against the oracle."""
    m, n, d = 1500, 1024, 66
    assert m * (n // 2 // 64) > steps_held(1)
    z = torch.randint(-3, 4, (m, n, d), device="cuda", dtype=torch.int8).float()
    out = lib.cdgrab_balance_epoch_independent(lib.Handle(), z)
    alone = lib.cdgrab_balance_epoch_independent(lib.Handle(gram_mode=1), z)
    assert torch.equal(out["signs"], alone["signs"]) and torch.equal(out["perm"], alone["perm"])
    for i in (0, 777, m - 1):
        want = oracle.server_epoch(z[i:i + 1].cpu().numpy(), None)
        assert np.array_equal(out["signs"][i].cpu().numpy(), want["eps"][0])


@pytest.mark.parametrize("n,d", [(64, 17), (65, 16), (129, 40), (300, 16), (513, 5), (300, 12_000), (257, 66), (1100, 130)])
def test_centred_steps_match_oracle(lib, n, d):
    g = workloads.integer_rows(n, 1, n, d, 3)[0]
    mean = np.rint(np.linspace(-2, 2, d)).astype(np.float32)
    out = lib.cdgrab_balance_epoch_stale_mean(lib.Handle(), torch.from_numpy(g).cuda(), torch.from_numpy(mean).cuda())
    want = oracle.grab_stale_mean(g, mean)
    assert np.array_equal(out["signs"].cpu().numpy(), want["s"])
    assert np.array_equal(out["r64"].cpu().numpy(), want["r"])


@pytest.mark.parametrize("m,n,d", [(3, 128, 40), (9, 130, 40), (2, 600, 17), (3, 1030, 70), (200, 140, 66), (40, 70, 1000), (5, 300, 9000), (2, 130, 65_536)])
def test_walks_side_by_side_equal_single_walks(lib, m, n, d):
    z = workloads.integer_rows(m, m, n, d, 3)
    out = lib.cdgrab_balance_epoch_independent(lib.Handle(), torch.from_numpy(z).cuda())
    for i in range(m):
        want = oracle.server_epoch(z[i:i + 1], None)
        assert np.array_equal(out["signs"][i].cpu().numpy(), want["eps"][0])
        assert np.array_equal(out["perm"][i].cpu().numpy(), want["perm"][0])


@pytest.mark.parametrize("m,n,d", [(3, 2000, 16), (16, 1200, 40), (20, 1200, 24), (5, 300, 200), (64, 200, 1000)])
def test_walks_side_by_side_equal_single_walks_where_sums_are_rounded(lib, m, n, d):
    """The order of the sums goes by the number of walks.  A sign would differ where a dot is zero to rounding, 1e-15 of its
    size: none of these is."""
    z = torch.randn((m, n, d), generator=torch.Generator(device="cuda").manual_seed(m + d), device="cuda")
    out = lib.cdgrab_balance_epoch_independent(lib.Handle(), z)
    for i in range(m):
        one = lib.cdgrab_balance_epoch(lib.Handle(), 1, n, d, grads=z[i:i + 1].contiguous())
        assert torch.equal(out["signs"][i], one["signs"][0]) and torch.equal(out["perm"][i], one["perm"][0])


@pytest.mark.parametrize("m,n,d", [(3, 86, 30), (2, 300, 12_000), (1, 600, 20), (1, 1100, 70), (3, 86, 129)])
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


@pytest.mark.parametrize("odd_draw", [-0.0, np.inf, np.nan])
@pytest.mark.parametrize("m,n,d", [(3, 86, 16), (3, 86, 30), (1, 300, 64), (2, 300, 12_000), (3, 86, 129), (2, 20, 70_001)])
def test_randomized_rule_at_its_threshold(lib, m, n, d, odd_draw):
    """Draws equal to their probability (such a pair gets +1), at probability zero too, and draws that are no
    ordinary numbers among them; the sums are exact, so every sign is determined."""
    z = workloads.integer_rows(n + 1, m, n, d, 2) * np.float32(2.0 ** -5)
    u, want = np.zeros((m, n // 2), np.float32), np.zeros((m, n // 2), np.int8)
    r, at_zero = np.zeros(d), 0
    for k in range(n // 2):
        for i in range(m):
            power = np.flatnonzero((r != 0) & (np.abs(np.frexp(r)[0]) == 0.5))
            if (k * m + i) % 7 == 3 and power.size:  # a pair whose dot is -1
                z[i, 2 * k:2 * k + 2] = 0
                z[i, 2 * k + 1, power[0]] = -1.0 / r[power[0]]
            dv = z[i, 2 * k + 1].astype(np.float64) - z[i, 2 * k]
            p = 0.5 * (1.0 + float(r @ dv))
            at_zero += p == 0.0
            u[i, k] = p if 0.0 < p < 1.0 else odd_draw
            want[i, k] = -1 if float(u[i, k]) < p else 1
            r += want[i, k] * dv
    assert at_zero > 2
    out = lib.cdgrab_balance_epoch_randomized(lib.Handle(), torch.from_numpy(z).cuda(), torch.from_numpy(u).cuda())
    assert np.array_equal(out["signs"].cpu().numpy(), want)
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


@pytest.mark.parametrize("bits", [0x7fc00000, 0xffc00000])  # either sign of a value that is not a number
@pytest.mark.parametrize("m,n,d", [
    (3, 86, 5), (1, 700, 16), (5, 104, 30), (7, 74, 64),       # rows of at most 64 elements
    (1, 130, 66), (3, 86, 129), (1, 600, 1001), (2, 130, 12_000),   # the chain of steps
    (2, 20, 70_001),                                                # one launch per block of pairs
])
def test_dots_that_are_not_numbers(lib, bits, m, n, d):
    """A value that is not a number in the middle of the epoch: pairs before it keep their signs; its own dot and all
    later ones are not numbers, which the greedy rule answers with -1 and the randomized rule with +1."""
    z = workloads.integer_rows(n + d, m, n, d, 3) * np.float32(2.0 ** -5)
    pairs, at = m * n // 2, m * n // 4 + 1
    clean = oracle.server_epoch(z, None)["eps"].T.ravel()  # in visiting order
    z[at % m, 2 * (at // m) + 1, d // 2] = np.array(bits, np.uint32).view(np.float32)
    zt = torch.from_numpy(z).cuda()
    out = lib.cdgrab_balance_epoch(lib.Handle(), m, n, d, grads=zt, want_dots=True)
    eps, dots = (out[key].cpu().numpy().T.ravel() for key in ("signs", "dots"))
    assert np.array_equal(eps[:at], clean[:at]) and (eps[at:] == -1).all()
    assert np.isfinite(dots[:at]).all() and np.isnan(dots[max(at, 1):]).all()
    u = torch.rand((m, n // 2), device="cuda")
    out = lib.cdgrab_balance_epoch_randomized(lib.Handle(), zt, u)
    assert (out["signs"].cpu().numpy().T.ravel()[at:] == 1).all() and pairs > at


@pytest.mark.parametrize("m,n,d", [(3, 400, 5), (1, 1300, 16), (5, 304, 30), (7, 174, 64)])
def test_long_narrow_walks_with_values_that_are_not_finite(lib, m, n, d):
    for bits in (0x7fc00000, 0xffc00000):
        test_dots_that_are_not_numbers(lib, bits, m, n, d)
    for value in (np.inf, -np.inf, np.nan):
        test_value_that_is_not_finite_stays_where_it_is(lib, value, m, n, max(d, 6))
    test_randomized_rule_over_steps(lib, m, n, d)
    for draw in (-0.0, np.inf, np.nan):
        test_randomized_rule_at_its_threshold(lib, m, n, max(d, 16), draw)
    test_centred_steps_match_oracle(lib, n * m, d)
    test_walks_side_by_side_equal_single_walks(lib, 16, 1984 + n % 50 // 2 * 2, d)


@pytest.mark.parametrize("d", [16, 32, 64])
def test_values_that_are_not_finite_do_not_hold_up_a_long_narrow_walk(lib, d):
    """One infinity or one draw that is no number among 25 000 pairs.  The blocks without a sign to go by are walked twice,
    the others once: at most twice 64 pairs in 2.5 us (rows of 64 elements), where finite values take 0.9 - 1.4.  Pair by
    pair to the end took ten times as long as finite values."""
    n = 50_000
    g = torch.Generator(device="cuda").manual_seed(d)
    h = lib.Handle()
    z, u = torch.randn((1, n, d), generator=g, device="cuda"), torch.rand((1, n // 2), generator=g, device="cuda")
    inf, draws = z.clone(), u.clone()
    inf[0, 1, 3], draws[0, 0] = np.inf, np.nan

    def us(f):
        f()
        best = np.inf
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            f()
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best
    greedy = [us(lambda x=x: lib.cdgrab_balance_epoch(h, 1, n, d, grads=x)) for x in (z, inf)]
    drawn = [us(lambda x=x: lib.cdgrab_balance_epoch_randomized(h, z, x)) for x in (u, draws)]
    assert greedy[1] <= 5 * greedy[0] and drawn[1] <= 5 * drawn[0], (greedy, drawn)


@pytest.mark.parametrize("m,n,d", [(1, 2050, 70), (16, 300, 7850), (3, 500, 16), (2, 130, 40_000), (3, 20, 300)])
def test_timing_counts_what_the_plan_says(lib, m, n, d):
    plan = lib.cdgrab_plan_epoch(m, n, d)
    h = lib.Handle(timing=1)
    z = torch.zeros((m, n, d), device="cuda")
    lib.cdgrab_balance_epoch(h, m, n, d, grads=z)
    unit = plan["step_pairs"] or plan["block_pairs"]
    got = h.timing()
    assert got["block_pairs"] == unit and got["blocks"] == -(-plan["pairs"] // unit)
