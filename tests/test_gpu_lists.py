"""GPU parity for the phases that run on lists of every line's best entries.

The lists hold 128 entries: lines of fewer, of exactly as many, of one more, and of a multiple of
the wavefront and of a slice of a whole line plus one; ties beyond what a list holds (a line is then
read whole); lists that are made once and again; phases that start on
the whole device and go on on one die; both sides of the problem, feasible prefixes, several GPU types;
searches that read too much and sides that come near the limit on bids.  The optimum is the exact CPU solver's, the duals
are re-checked on the host, and the solve with the lists off has to agree."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import dev, dev_params, empty_matrix, padded_matrix

pytestmark = pytest.mark.gpu
INF = synth.INFEASIBLE


@pytest.mark.parametrize("n,m,high,masked", [(1, 1, 100, 0.0), (5, 128, 2 ** 24, 0.1), (40, 129, 2 ** 24, 0.0), (129, 130, 2 ** 20, 0.2),
                                             (300, 131, 2 ** 20, 0.3), (257, 1025, 2 ** 24, 0.5), (512, 513, 255, 0.1),
                                             (640, 640, 3, 0.0), (200, 2051, 1, 0.0), (1000, 1000, 2 ** 24, 0.95),
                                             (100, 4097, 2 ** 24, 0.2), (64, 8193, 2 ** 20, 0.6), (30, 20483, 2 ** 24, 0.2)])
@pytest.mark.parametrize("options", [{"core_many": 5}, {"core_depth": 0}, {"core_depth": 0, "core_after": 0, "core_width": 1}, {"core_refine": 0},
                                     {"core_depth": 0, "core_wide": 1, "core_narrow": 16}])
def test_phases_on_lists_reach_the_optimum(orc, n, m, high, masked, options):
    import paper_2303_13803_amd as mm
    W = synth.uniform_matrix(71, n, m, high, masked)
    if n > 3:
        W[2, :] = INF                                    # a row with nothing to choose
    expect = orc.max_weight_matching(W if n <= m else np.ascontiguousarray(W.T))[0]
    for core in (1, 0):
        ctx = mm.Context(n, m)
        ctx.set_option("core", core)
        for k, val in options.items():
            ctx.set_option(k, val)
        r2c = torch.empty(n, dtype=torch.int32, device="cuda")
        u = torch.empty(n, dtype=torch.int64, device="cuda")
        v = torch.empty(m, dtype=torch.int64, device="cuda")
        res = ctx.solve_assignment(padded_matrix(W), n, m, r2c, u, v)
        code, P, D = orc.check_certificate(W, r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
        assert code == 0 and res.cert_ok == 1 and res.fallbacks == 0
        assert res.primal == P == expect
        ctx.close()


def _sampled_columns(m):
    """The entries of a long line that the cut of its list is taken from (see core_list_kernel)."""
    groups = (m + 3) // 4
    pieces = min(groups // 8, 64)
    return [4 * (p * groups // pieces + t) + e for p in range(pieces) for t in range(8) for e in range(4)]


@pytest.mark.parametrize("kind", ["ties", "two levels", "nearly empty", "sample misses the best", "only the sample is good", "sorted"])
@pytest.mark.parametrize("n,m", [(90, 2053), (1030, 1031), (1027, 4098)])
def test_lists_of_lines_a_sample_says_little_about(orc, n, m, kind):
    """The cut of a list comes from a sample: ties at it, more entries above it than fit, hardly any; a line or
    four lines a workgroup, with lines left over."""
    import paper_2303_13803_amd as mm
    rng = np.random.default_rng(n + m)
    if kind == "ties":
        W = np.full((n, m), 1000, np.int32)
        W[rng.random((n, m)) < 0.02] = 1001
    elif kind == "two levels":
        W = (rng.random((n, m)) < 0.4).astype(np.int32)
    elif kind == "nearly empty":
        W = np.where(rng.random((n, m)) < 0.002, rng.integers(0, 2 ** 20, (n, m)), INF).astype(np.int32)
    else:
        W = rng.integers(0, 2 ** 20, (n, m)).astype(np.int32)
        seen = [c for c in _sampled_columns(m) if c < m]
        if kind == "sample misses the best":
            W[:, seen] //= 1024
        elif kind == "only the sample is good":
            W[:, [c for c in range(m) if c not in set(seen)]] //= 1024
        else:
            W = np.sort(W, axis=1)[:, ::-1].copy()
    expect = orc.max_weight_matching(W)[0]
    ctx = mm.Context(n, m)
    ctx.set_option("core_depth", 0)
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
    res = ctx.solve_assignment(padded_matrix(W), n, m, r2c, u, v)
    code, P, _ = orc.check_certificate(W, r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
    lists = ctx.last_timings()["lists_made"]
    ctx.close()
    assert code == 0 and res.cert_ok == 1 and res.fallbacks == 0 and lists > 0
    assert res.primal == P == expect


@pytest.mark.parametrize("high", [2, 2 ** 20])
@pytest.mark.parametrize("n,m", [(30, 63), (50, 64), (64, 65), (100, 66), (120, 127), (127, 128), (600, 700)])
def test_bids_that_half_a_list_decides_or_does_not(orc, n, m, high):
    """The first 64 entries of a list decide a bid if nothing else can be worth as much as its two best: lists of
    about that length, with many ties (one of which always is) and with hardly any."""
    import paper_2303_13803_amd as mm
    W = synth.uniform_matrix(73, n, m, high, 0.1)
    expect = orc.max_weight_matching(W if n <= m else np.ascontiguousarray(W.T))[0]
    ctx = mm.Context(n, m)
    ctx.set_option("core_depth", 0)
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
    res = ctx.solve_assignment(padded_matrix(W), n, m, r2c, u, v)
    code, P, _ = orc.check_certificate(W, r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
    ctx.close()
    assert code == 0 and res.cert_ok == 1 and res.fallbacks == 0 and res.primal == P == expect


@pytest.mark.parametrize("n,m,high", [(60, 140001, 2), (60, 131073, 2 ** 20), (300, 301, 2), (700, 720, 2 ** 20), (1500, 1600, 40)])
def test_trees_of_a_search_get_their_labels_back(orc, n, m, high):
    """Searches with many bidders from the first step on: a served tree's columns are reached again from the scanned
    rows' lists, or from lists kept by column where there are more columns than a workgroup has bits for, or once rows
    have been looked at often enough.  The latter is sure to happen to the 700 x 720 problem, whose searches serve dozens of
    trees (three to five of its sides, whatever the order of its bids)."""
    import paper_2303_13803_amd as mm
    W = synth.uniform_matrix(74, n, m, high, 0.3)
    expect = orc.max_weight_matching(W)[0]
    ctx = mm.Context(n, m)
    for k, val in {"core_depth": 0, "core_after": 0, "core_refine": 0, "phase_keep": 8}.items():
        ctx.set_option(k, val)
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
    res = ctx.solve_assignment(padded_matrix(W), n, m, r2c, u, v)
    code, P, _ = orc.check_certificate(W, r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
    by_column = ctx.last_timings()["lists_by_column"]
    ctx.close()
    assert code == 0 and res.cert_ok == 1 and res.fallbacks == 0 and res.primal == P == expect
    assert by_column > 0 or n != 700


@pytest.mark.parametrize("n,m,masked", [(1500, 1500, 0.0), (1300, 1400, 0.5), (1200, 1700, 0.2), (1601, 1205, 0.1)])
def test_bidders_that_wait_for_better_lists(orc, n, m, masked):
    """On all dies bidders whose lists have sunk wait until theirs alone are made again: every row ranks the columns
    nearly alike, so that lists of several ages are in use on both sides and most of them sink."""
    rng = np.random.default_rng(n + m)
    W = (2 ** 20 - 400 * np.arange(m)[None, :] + rng.integers(0, 2000, (n, m))).astype(np.int32)
    W[rng.random((n, m)) < masked] = INF
    t = _solve(orc, W, {"core_depth": 0, "core_wide": 1, "core_narrow": 16, "core_many": 2})
    assert t["lists_made"] > 4


def test_lists_of_every_line_are_not_made_for_ever(orc):
    """Rows that rank the columns nearly alike: lists sink as soon as they are made, and the side goes on on whole lines
    (where one die does it all 66 lists were made of a phase's two sides, and the solve took three times as long)."""
    import paper_2303_13803_amd as mm
    n = 6000
    W = (2 ** 20 - 7 * np.arange(n)[None, :] + np.random.default_rng(76).integers(0, 3000, (n, n))).astype(np.int32)
    ctx = mm.Context(n, n)
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = (torch.empty(n, dtype=torch.int64, device="cuda") for _ in range(2))
    res = ctx.solve_assignment(padded_matrix(W), n, n, r2c, u, v)
    did = ctx.last_timings()
    ctx.close()
    code, P, _ = orc.check_certificate(W, r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
    assert code == 0 and res.cert_ok == 1 and res.fallbacks == 0 and res.primal == P
    assert did["list_launches"] > 0 and did["lists_made"] <= 8 * res.phases


@pytest.mark.parametrize("n,m", [(100, 128), (128, 128), (90, 64)])
def test_counters_of_a_solve_on_lists(n, m):
    """Lines no longer than a list: the whole solve runs on lists, every bid and every scan of a search or a proof
    reads one list (128 entries of 8 bytes) and is counted once."""
    import paper_2303_13803_amd as mm
    ctx = mm.Context(n, m)
    ctx.set_option("core_few", 33)                       # (matched on lists, however small)
    W = padded_matrix(synth.uniform_matrix(72, n, m, 2 ** 24, 0.2))
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
    res = ctx.solve_assignment(W, n, m, r2c, u, v)
    ctx.close()
    assert res.bids > 0 and res.path_scans > 0 and res.chain_bids == res.bids
    assert res.bytes_scanned == 1024 * (res.bids + res.path_scans)


def _solve(orc, W, options):
    """The solve of W with the host's checks made; returns what the phases on lists did."""
    import paper_2303_13803_amd as mm
    n, m = W.shape
    expect = orc.max_weight_matching(W if n <= m else np.ascontiguousarray(W.T))[0]
    ctx = mm.Context(n, m)
    for k, val in options.items():
        ctx.set_option(k, val)
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
    res = ctx.solve_assignment(padded_matrix(W), n, m, r2c, u, v)
    code, P, D = orc.check_certificate(W, r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
    assert code == 0 and res.cert_ok == 1 and res.fallbacks == 0 and res.primal == P == expect
    did = ctx.last_timings()
    ctx.close()
    return did


@pytest.mark.parametrize("n,m,high,masked", [(5, 128, 2 ** 24, 0.1), (40, 129, 2 ** 24, 0.0), (512, 513, 255, 0.1), (100, 4097, 2 ** 24, 0.2),
                                             (900, 350, 2 ** 24, 0.1), (1201, 1200, 2 ** 24, 0.2), (2051, 130, 2 ** 20, 0.5)])
@pytest.mark.parametrize("wide", [0, 1])
def test_what_runs_on_lists(orc, n, m, high, masked, wide):
    W = synth.uniform_matrix(73, n, m, high, masked)
    did = _solve(orc, W, {"core_depth": 0, "core_wide": wide, "core_narrow": 16})
    assert did["list_launches"] > 0 and did["lists_made"] > 0 and did["list_sides_left"] == 0
    assert _solve(orc, W, {"core": 0, "core_depth": 0})["list_launches"] == 0


@pytest.mark.parametrize("n,m,high,masked", [(257, 1025, 2 ** 24, 0.5), (900, 350, 2 ** 24, 0.1), (640, 640, 3, 0.0)])
def test_lists_that_no_longer_decide_are_made_again(orc, n, m, high, masked):
    """Started on lists at a coarse epsilon, prices rise past what the lists hold: more than one list of each side is made."""
    assert _solve(orc, synth.uniform_matrix(71, n, m, high, masked), {"core_depth": 0})["lists_made"] > 2


@pytest.mark.parametrize("n,m,high,masked", [(300, 131, 2 ** 20, 0.3), (512, 513, 255, 0.1), (64, 8193, 2 ** 20, 0.6),
                                             (30, 20483, 2 ** 24, 0.2), (1201, 1200, 2 ** 24, 0.2)])
def test_a_search_that_reads_too_much_leaves_the_rest_to_the_device(orc, n, m, high, masked):
    """With no whole line to be read at all, the first search that wants one gives up half-way."""
    did = _solve(orc, synth.uniform_matrix(71, n, m, high, masked), {"core_depth": 0, "core_after": 0, "core_read": 0, "core_read_least": 0})
    assert did["list_sides_left"] > 0


@pytest.mark.parametrize("n,m,high,masked", [(300, 131, 2 ** 20, 0.3), (200, 2051, 1, 0.0), (900, 350, 2 ** 24, 0.1), (1000, 1000, 2 ** 24, 0.95)])
def test_a_side_near_the_limit_on_bids_is_finished_on_whole_lines(orc, n, m, high, masked):
    """The bids a look at the list may lead to are counted before they are made: with 4096 of them a
    bidder, two million are near at once, while the solve takes a hundredth of that."""
    did = _solve(orc, synth.uniform_matrix(71, n, m, high, masked), {"core_depth": 0, "core_many": 4096, "core_few": 4096,
                                                                     "max_rounds": 300_000 if min(n, m) < 900 else 2_000_000})
    assert did["list_sides_left"] > 0


@pytest.mark.parametrize("n,m,masked", [(1300, 1300, 0.5), (1300, 1300, 0.0), (1290, 1500, 0.7), (1500, 1284, 0.2)])
@pytest.mark.parametrize("options", [{"phase_stop": 1 << 20, "phase_keep": 1}, {"phase_stop": 1 << 20, "phase_keep": 2},
                                     {"phase_stop": 2, "phase_keep": 3, "phase_growth": 4}])
@pytest.mark.parametrize("wide", [0, 1])
def test_columns_that_phases_leave_unused(orc, n, m, masked, options, wide):
    """Phases that leave rows over leave columns unused at a price; in the last of them those bid."""
    did = _solve(orc, synth.uniform_matrix(75, n, m, 2 ** 24, masked), dict(options, core_depth=0, core_wide=wide, core_narrow=64))
    assert did["list_launches"] > 0


@pytest.mark.parametrize("cfg,n,m", [("C5", 700, 300), ("C5", 1500, 2100), ("C4", 900, 1100), ("C5", 60, 20500), ("C5", 3001, 97)])
@pytest.mark.parametrize("hidden", [(128,), (128, 64, 128)])
@pytest.mark.parametrize("options", [{"core_depth": 0}, {"core_depth": 0, "core_wide": 1, "core_narrow": 16, "core_after": 0}])
def test_rounds_on_lists_of_feasible_prefixes(orc, cfg, n, m, hidden, options):
    """The memory-ordered copy: every line ends where the pairs that can share do (rows by GPU type first)."""
    import paper_2303_13803_amd as mm
    r = synth.scheduling_round(cfg, 74, n=n, m=m)
    S = r["cfg"].scale
    ctx = mm.Context(n, m)
    for k, val in dict(options, fit_prefix_below=101).items():
        ctx.set_option(k, val)
    preds = [ctx.predictor(dev_params(p), S) for p in synth.typed_predictors(74, r["cfg"].F, list(hidden))]
    W = empty_matrix(n, m)
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
    plan = (dev(r["x_on"]), dev(r["x_off"]), W, r2c, u, v)
    res = ctx.schedule_round(preds[0], *plan) if len(preds) == 1 else ctx.schedule_round_typed(preds, dev(synth.gpu_types(74, n, len(preds))), *plan)
    did = ctx.last_timings()
    ctx.close()
    Wg = np.ascontiguousarray(W.cpu().numpy()[:, :m])
    code, P, D = orc.check_certificate(Wg, r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
    assert code == 0 and res.cert_ok == 1 and res.fallbacks == 0
    assert res.primal == P == orc.max_weight_matching(Wg if n <= m else np.ascontiguousarray(Wg.T))[0]
    assert did["list_launches"] > 0


@pytest.mark.parametrize("n,m,base,spread", [(900, 950, 0, 7), (1500, 1490, 0, 2 ** 10), (1500, 1490, 0, 2 ** 30), (2300, 2307, 0, 2 ** 30),
                                             (900, 950, 2 ** 29, 3)])
def test_lists_one_two_and_four_lines_a_workgroup(orc, n, m, base, spread):
    """From weights with many ties to those as large as they may be: what floats sort out is looked at exactly."""
    import paper_2303_13803_amd as mm
    rng = np.random.default_rng(n + spread)
    W = (base + rng.integers(0, spread + 1, (n, m))).astype(np.int32)
    W[rng.random((n, m)) < 0.3] = INF
    ctx = mm.Context(n, m)
    for k, val in {"core_depth": 0, "core_refine": 0, "max_rounds": 20_000_000}.items():
        ctx.set_option(k, val)
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
    res = ctx.solve_assignment(padded_matrix(W), n, m, r2c, u, v)
    did = ctx.last_timings()
    ctx.close()
    code, P, D = orc.check_certificate(W, r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
    assert code == 0 and res.cert_ok == 1 and res.fallbacks == 0 and res.primal == P
    assert did["lists_made"] > 0


@pytest.mark.parametrize("n,m", [(900, 950), (950, 900), (900, 1800), (1500, 1520), (2100, 2120), (8200, 8240)])
@pytest.mark.parametrize("options", [{}, {"core_refine": 0}, {"core": 0}])
def test_weights_that_are_nearly_the_same(orc, n, m, options):
    """A few units on top of 2^29: every column too many has to come all the way down from what the first phase, at
    2^29 (n + 1) / 24, drove the prices to.  Some 30 bids a line and phase and what the searches scan (from 8192 rows on more: phases
    on lists end sides early there); a bid for each epsilon would be billions."""
    import paper_2303_13803_amd as mm
    rng = np.random.default_rng(n + m)
    W = (2 ** 29 + rng.integers(0, 4, (n, m))).astype(np.int32)
    W[rng.random((n, m)) < 0.3] = INF
    ctx = mm.Context(n, m)
    for k, val in dict(options, max_rounds=20_000_000 if n < 8192 else 400_000_000).items():
        ctx.set_option(k, val)
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
    res = ctx.solve_assignment(padded_matrix(W), n, m, r2c, u, v)
    ctx.close()
    print(f"{n}x{m} {options}: {res.phases} phases, {res.bids} bids, {res.path_scans} scans, {res.ms_solve:.1f} ms", flush=True)
    code, P, D = orc.check_certificate(W, r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
    assert code == 0 and res.cert_ok == 1 and res.fallbacks == 0 and res.primal == P


def test_searches_that_end_early_leave_everybody_within_epsilon(orc):
    """Rank-one weights, on lists that span all dies: searches end with some of their bidders placed.  What they
    leave has to be sound, or later ones, on whole lines, find no root and give up (one solve in twelve did; of forty all but one in thirty times)."""
    import paper_2303_13803_amd as mm
    n, m = 848, 924
    rng = np.random.default_rng(1008187)
    W = (np.outer(rng.random(n), rng.random(m)) * 2 ** 30).astype(np.int32)
    expect = orc.max_weight_matching(W)[0]
    left = 0
    for _ in range(40):
        ctx = mm.Context(n, m)
        for k, val in {"core_wide": 64, "phase_tail_steps": 1, "max_rounds": 50_000_000}.items():
            ctx.set_option(k, val)
        r2c = torch.empty(n, dtype=torch.int32, device="cuda")
        u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
        res = ctx.solve_assignment(padded_matrix(W), n, m, r2c, u, v)
        left += ctx.last_timings()["list_sides_left"]
        ctx.close()
        assert res.fallbacks == 0 and res.cert_ok == 1 and res.primal == expect
    assert left > 0
