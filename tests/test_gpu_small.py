"""Problems matched in one compute unit (GPU): against the oracle and against the auction, which a context with a
tuning option that differs from its default uses at every size."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import assert_weights_close, padded_matrix

pytestmark = pytest.mark.gpu

INF = np.iinfo(np.int32).min


def _solve(orc, W, options):
    import paper_2303_13803_amd as mm
    n, m = W.shape
    ctx = mm.Context(n, m)
    for name, value in options.items():
        ctx.set_option(name, value)
    r2c = torch.full((n,), 7, dtype=torch.int32, device="cuda")
    u, v = torch.full((n,), -7, dtype=torch.int64, device="cuda"), torch.full((m,), -7, dtype=torch.int64, device="cuda")
    res = ctx.solve_assignment(padded_matrix(W), n, m, r2c, u, v)
    did = ctx.last_timings()
    ctx.close()
    code, P, _ = orc.check_certificate(W, r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
    assert code == 0 and res.cert_ok == 1 and res.primal == P
    return res, did


def _kinds(n, m):
    yield "uniform", synth.uniform_matrix(81, n, m, 2 ** 24, 0.1)
    yield "ties", synth.uniform_matrix(82, n, m, 3, 0.3)
    yield "few pairs", synth.uniform_matrix(83, n, m, 1000, 0.95)
    yield "product", (np.arange(1, n + 1)[:, None] * np.arange(1, m + 1)[None]).astype(np.int32)
    yield "one value", np.full((n, m), 77, np.int32)
    yield "nothing feasible", np.full((n, m), INF, np.int32)
    W = synth.uniform_matrix(84, n, m, 2 ** 20, 0.2)
    W[::3] = np.where(W[::3] == INF, INF, 0)                # worth nothing, and below that
    W[:, ::5] = np.where(W[:, ::5] == INF, INF, -W[:, ::5])
    yield "zero and negative", W


# one column a lane and its last lane, two, four and eight; pitches that are and are not whole loads; the most rows, and
# the first sizes that are left to the auction (more rows than columns always are)
@pytest.mark.parametrize("n,m", [(1, 1), (1, 512), (2, 513), (3, 2), (30, 30), (63, 64), (64, 65), (88, 88), (89, 90), (97, 127), (96, 128),
                                 (112, 150), (112, 256), (100, 257), (113, 151), (60, 257), (70, 512), (75, 512)])
def test_one_compute_unit_finds_the_optimum(orc, n, m):
    for name, W in _kinds(n, m):
        res, did = _solve(orc, W, {})
        other, _ = _solve(orc, W, {"theta": 25})
        assert res.primal == other.primal, name
        here = n <= m <= 512 and (n <= 88 or (n <= 112 and 4 * n <= 3 * m <= 768)) and n * m < 38000         # 152 KB of LDS
        assert (res.rounds == 0 and did["list_launches"] == 0) == here, name
        assert not here or res.bytes_scanned == 4 * n * m and res.phases == 1, name


def test_an_option_counts_while_it_differs_from_its_default(orc):
    import paper_2303_13803_amd as mm
    W = synth.uniform_matrix(87, 64, 64, 2 ** 20, 0.1)
    expect, device = orc.max_weight_matching(W)[0], padded_matrix(W)
    r2c = torch.empty(64, dtype=torch.int32, device="cuda")
    u, v = (torch.empty(64, dtype=torch.int64, device="cuda") for _ in range(2))
    ctx = mm.Context(64, 64)
    for name, value, here in [("theta", 24, True), ("warm_reset_cols", 1, True), ("theta", 25, False), ("core_few", 33, False),
                              ("theta", 24, False), ("core_few", 32, True), ("fit_prefix", 0, False), ("fit_prefix", 1, True)]:
        ctx.set_option(name, value)
        res = ctx.solve_assignment(device, 64, 64, r2c, u, v)
        assert res.primal == expect and res.cert_ok == 1
        assert (ctx.last_timings()["list_launches"] == 0) == here, (name, value)
    ctx.close()


@pytest.mark.parametrize("largest", [2 ** 28 - 1, 2 ** 28, 2 ** 31 - 1])
def test_weights_at_the_edge_of_its_integers(orc, largest):
    W = (largest - synth.uniform_matrix(85, 50, 60, 1000, 0.0)).astype(np.int32)
    W[0, 0], W[3] = largest, INF
    res, _ = _solve(orc, W, {})
    assert res.primal == orc.max_weight_matching(W)[0]
    assert (res.bytes_scanned == 4 * W.size) == (largest < 2 ** 28)     # larger ones are left to the auction


def test_it_stops_at_the_limit_on_bids(orc):
    import paper_2303_13803_amd as mm
    W = (np.arange(1, 61)[:, None] * np.arange(1, 61)[None]).astype(np.int32)
    res, _ = _solve(orc, W, {})
    steps = res.bids + res.path_scans
    assert _solve(orc, W, {"max_rounds": steps + 1})[0].primal == res.primal
    for limit in (1, res.bids + 1, steps // 2):
        with pytest.raises(mm.MuxmatchError) as e:
            _solve(orc, W, {"max_rounds": limit})
        assert e.value.code == mm.ERR_NOT_CONVERGED


@pytest.mark.parametrize("law,n,m,hidden", [("C4", 40, 61, (128, 64, 128)), ("C3", 88, 130, (64, 128)), ("C5", 7, 500, (128, 128, 64, 64)), ("C1", 64, 64, (64,))])
def test_its_typed_rounds_score_pairs_as_they_come(orc, law, n, m, hidden):
    """Rows in order of their type, not of memory as well, and no scores asked for: the weights are those of the pass
    that walks in memory order, bit for bit, and the oracle's optimum is found."""
    r = synth.scheduling_round(law, 88, n=n, m=m)
    import paper_2303_13803_amd as mm
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ctx = mm.Context(n, m)
    params = synth.typed_predictors(88, r["cfg"].F, list(hidden))
    types = synth.gpu_types(88, n, len(hidden))
    preds = [ctx.predictor({k: dev(v) for k, v in p.items()}, r["cfg"].scale) for p in params]
    x_on, x_off, pad = dev(r["x_on"]), dev(r["x_off"]), (m + 3) // 4 * 4
    W, again = (torch.full((n, pad), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
    res = ctx.schedule_round_typed(preds, dev(types), x_on, x_off, W, r2c, u, v)
    ctx.score_pairs_typed(preds, dev(types), x_on, x_off, again)
    torch.cuda.synchronize()
    ctx.close()
    assert res.rounds == 0 and res.bytes_scanned == 4 * n * m and torch.equal(W, again)
    Wh = np.ascontiguousarray(W.cpu().numpy()[:, :m])
    _, Wc = orc.score_pairs_typed(r["x_on"], r["x_off"], params, types, r["cfg"].scale)
    assert_weights_close(Wh, Wc, r["cfg"].scale, Wc != INF)
    assert ((Wh == INF) == (Wc == INF)).all()
    code, P, _ = orc.check_certificate(Wh, r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
    assert code == 0 and res.cert_ok == 1 and res.primal == P == orc.max_weight_matching(Wh)[0]


@pytest.mark.parametrize("law,n,m", [("C1", 64, 64), ("C4", 33, 257), ("C5", 88, 201)])
def test_its_rounds_score_pairs_as_they_come(orc, law, n, m):
    """No memory order is found for them: the weights are those of the pass that walks in it, bit for bit."""
    import paper_2303_13803_amd as mm
    r = synth.scheduling_round(law, 86, n=n, m=m)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ctx = mm.Context(n, m)
    pred = ctx.predictor({k: dev(v) for k, v in r["params"].items()}, r["cfg"].scale)
    x_on, x_off, pad = dev(r["x_on"]), dev(r["x_off"]), (m + 3) // 4 * 4
    W, again = (torch.full((n, pad), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
    res = ctx.schedule_round(pred, x_on, x_off, W, r2c, u, v)
    fraction = ctx.last_timings()["pairs_evaluated_fraction"]
    ctx.score_pairs(pred, x_on, x_off, again)
    torch.cuda.synchronize()
    ctx.close()
    assert fraction == 1.0 and res.rounds == 0 and torch.equal(W, again)
    Wh = W.cpu().numpy()[:, :m]
    code, P, _ = orc.check_certificate(np.ascontiguousarray(Wh), r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
    assert code == 0 and res.cert_ok == 1 and res.primal == P
