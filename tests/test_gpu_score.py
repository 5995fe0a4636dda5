"""GPU parity: mf_score_pairs against the CPU checker, element by element."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import assert_weights_close, dev, dev_params, empty_matrix, weight_tolerance

pytestmark = pytest.mark.gpu
INF = synth.INFEASIBLE


@pytest.fixture(scope="module")
def mm():
    import paper_2303_13803_amd as mm
    return mm


def _score_on_gpu(mm, ctx, r, scale=None, want_sigma=True):
    n, m = r["n"], r["m"]
    scale = r["cfg"].scale if scale is None else scale
    params = dev_params(r["params"])
    pred = ctx.predictor(params, scale)
    x_on, x_off = dev(r["x_on"]), dev(r["x_off"])
    W = empty_matrix(n, m)
    sigma = torch.empty((n, m), dtype=torch.float32, device="cuda") if want_sigma else None
    ctx.score_pairs(pred, x_on, x_off, W, sigma)
    torch.cuda.synchronize()
    Wh = W.cpu().numpy()
    assert (Wh[:, m:] == -7).all()                     # pitch padding untouched
    return Wh[:, :m], (sigma.cpu().numpy() if want_sigma else None)


def _compare(orc, r, Wg, sg, scale=None):
    scale = r["cfg"].scale if scale is None else scale
    sig, W = orc.score_pairs(r["x_on"], r["x_off"], r["params"], scale)
    assert ((Wg == INF) == (W == INF)).all(), "mask bits differ"
    rel = np.abs(sg.astype(np.float64) - sig) / sig
    assert rel.max() <= 1e-5, f"score relative error {rel.max():.3e}"
    ok = W != INF
    assert_weights_close(Wg, W, scale, ok)
    # the GPU's own quantisation of its own score is exact
    q = np.clip(np.rint(sg * np.float32(scale)), 0, scale).astype(np.int64)
    assert (Wg[ok] == q[ok]).all()
    return rel.max()


def _pairs_in_tasks(r):
    """Pairs that go through the predictor in order of memory: whole blocks of 32 columns beside every row that fits
    their first one, whatever the rows of a task."""
    on, off = r["x_on"][:, 0], np.sort(r["x_off"][:, 0])
    return sum(int((on + off[j] <= np.float32(1.0)).sum()) * min(32, len(off) - j) for j in range(0, len(off), 32))


def _some_rows(n):
    """Rows at the edges of tasks and of the stretches of 16 rows in LDS, and every 97th."""
    rows = {t + d for t in range(0, n, max(64, n // 16 // 64 * 64)) for d in (0, 1, 15, 16, 17, 31, 32, 63)} | set(range(0, n, 97)) | {n - 2, n - 1}
    return np.array(sorted(i for i in rows if i < n))


@pytest.mark.parametrize("cfg,n,m", [("C1", None, None), ("C2", None, None), ("C1", 1, 1), ("C1", 3, 5),
                                     ("C2", 130, 517), ("C3", 150, 700), ("C4", 97, 1031),
                                     ("C5", 64, 300), ("C3", 65, 257)])
def test_scores_match_checker(mm, orc, cfg, n, m):
    r = synth.scheduling_round(cfg, 1, n=n, m=m)
    for split in (1, 0):                # hidden-layer products from fp16 pieces (default) or from fp32 operands
        ctx = mm.Context(r["n"], max(r["m"], r["n"]))
        ctx.set_option("score_split", split)
        Wg, sg = _score_on_gpu(mm, ctx, r)
        _compare(orc, r, Wg, sg)
        ctx.close()


@pytest.mark.parametrize("n,m", [(7, 40), (8, 33), (9, 256), (15, 257), (17, 255), (31, 513), (65, 1), (127, 300),
                                 (2049, 31), (2500, 1030), (1, 70000)])
@pytest.mark.parametrize("cfg", ["C2", "C3"])
def test_scores_at_the_edges_of_row_tiles(mm, orc, cfg, n, m):
    """A task has 2 to 64 rows, chosen by the shape, scored two at a time: remainders of either."""
    r = synth.scheduling_round(cfg, 3, n=n, m=m)
    ctx = mm.Context(n, m)
    Wg, sg = _score_on_gpu(mm, ctx, r)
    _compare(orc, r, Wg, sg)
    ordered, _ = _score_on_gpu(mm, ctx, r, want_sigma=False)
    assert (ordered == Wg).all()
    ctx.close()


@pytest.mark.parametrize("cfg", ["C2", "C5"])
@pytest.mark.parametrize("n,m", [(2, 33), (30, 31), (33, 480), (130, 9000), (4200, 65), (9000, 36), (5000, 1100)])
def test_scores_of_tasks(mm, orc, cfg, n, m):
    """Wavefronts take tasks of 2 to 64 rows beside 32 columns: fewer tasks than groups that share a counter, fewer
    and more than wavefronts, one column block, more chunks of rows than lanes look at in one step, and chunks
    that have no task because nothing fits their first row; passes on one context are the same to the bit."""
    r = synth.scheduling_round(cfg, 5, n=n, m=m)
    ctx = mm.Context(n, m)
    Wg, sg = _score_on_gpu(mm, ctx, r)
    _compare(orc, r, Wg, sg)
    for _ in range(2):
        ordered, _ = _score_on_gpu(mm, ctx, r, want_sigma=False)
        assert (ordered == Wg).all()
        assert abs(ctx.last_timings()["pairs_evaluated_fraction"] - _pairs_in_tasks(r) / (n * m)) <= 6e-8       # (a float)
    ctx.close()


@pytest.mark.parametrize("cfg,n,m", [("C2", 3000, 1100), ("C2", 6000, 1300), ("C4", 3000, 1100), ("C4", 5200, 1217), ("C3", 9001, 3100)])
@pytest.mark.parametrize("split", [1, 0])
@pytest.mark.parametrize("with_sm", [False, True])
@pytest.mark.parametrize("with_limit", [False, True])
def test_every_kind_of_predictor_in_many_tasks(mm, orc, cfg, n, m, split, with_sm, with_limit):
    """Wavefronts that take several tasks, of 16, 32 and 64 rows (one, two and four stretches of rows in LDS), with either kind of products,
    SM share and slowdown unit.  The limit on the slowdown is the median of the oracle's predictions, so half of the pairs are
    above it; a float decides, so where it hides a pair is compared 1e-5 away from it, the tolerance of a score."""
    r = synth.scheduling_round(cfg, 17, n=n, m=m)
    full, sm = (synth.with_sm_input(r["params"], 12), (2, 3)) if with_sm else (r["params"], None)
    rows, slow_limit = _some_rows(n), None
    some = np.ascontiguousarray(r["x_on"][rows])
    if with_limit:
        full = synth.with_slowdown_unit(full, 13)
        slow = orc.score_pairs(some, r["x_off"], {**full, "W3": full["W3slow"], "b3": full["b3slow"]}, r["cfg"].scale, sm=sm)[0].astype(np.float64)
        slow_limit = float(np.float32(np.median(slow)))
    S, params = r["cfg"].scale, {k: dev(v) for k, v in full.items() if k != "W1"}
    params["W1"] = dev(full["W1"][:, :-1] if with_sm else full["W1"])
    if with_sm:
        params["W1sm"] = dev(full["W1"][:, -1])
    ctx = mm.Context(n, m)
    ctx.set_option("score_split", split)
    pred = ctx.predictor(params, S, sm=sm, slow_limit=slow_limit)
    x_on, x_off, W, by_memory = dev(r["x_on"]), dev(r["x_off"]), empty_matrix(n, m), empty_matrix(n, m)
    sigma = torch.empty((n, m), dtype=torch.float32, device="cuda")
    ctx.score_pairs(pred, x_on, x_off, W, sigma)
    ctx.score_pairs(pred, x_on, x_off, by_memory)
    torch.cuda.synchronize()
    assert torch.equal(W, by_memory)
    at = torch.from_numpy(rows).cuda()
    Wg, sg = W[at].cpu().numpy()[:, :m], sigma[at].cpu().numpy()
    unit = {k: v for k, v in full.items() if k not in ("W3slow", "b3slow")}
    sig, expect = orc.score_pairs(some, r["x_off"], unit, S, sm=sm)
    rel = np.abs(sg.astype(np.float64) - sig) / sig
    assert rel.max() <= 1e-5, f"score relative error {rel.max():.3e}"
    hidden, clear = expect == INF, np.ones(expect.shape, bool)
    if with_limit:
        hidden, clear = hidden | (slow > slow_limit), np.abs(slow - slow_limit) > 1e-5 * slow
        assert (~clear).mean() < 1e-3
    assert (((Wg == INF) == hidden) | ~clear).all()
    assert_weights_close(Wg, expect, S, clear & ~hidden)
    ctx.close()


@pytest.mark.parametrize("cfg,n,m", [("C2", 8200, 8300), ("C4", 6100, 6300), ("C5", 9000, 20000)])
def test_scores_of_long_passes(mm, orc, cfg, n, m):
    """From eight tasks a wavefront on some workgroups leave and later ones take their place, most of those with
    nothing left to do in the last case: nothing is missing, and nothing is done twice."""
    r = synth.scheduling_round(cfg, 7, n=n, m=m)
    ctx = mm.Context(n, m)
    pred = ctx.predictor(dev_params(r["params"]), r["cfg"].scale)
    x_on, x_off, got = dev(r["x_on"]), dev(r["x_off"]), []
    for order, split in ((0, 1), (1, 1), (0, 0), (1, 0)):
        ctx.set_option("fit_order", order)
        ctx.set_option("score_split", split)
        W = empty_matrix(n, m)
        ctx.score_pairs(pred, x_on, x_off, W)
        torch.cuda.synchronize()
        expect = _pairs_in_tasks(r) if order else n * m
        assert abs(ctx.last_timings()["pairs_evaluated_fraction"] - expect / (n * m)) <= 6e-8      # (a float; the smallest task is 3.6e-7 here)
        got.append(W)
    assert torch.equal(got[0], got[1]) and torch.equal(got[2], got[3])
    rows = _some_rows(n)
    _, expect = orc.score_pairs(np.ascontiguousarray(r["x_on"][rows]), r["x_off"], r["params"], r["cfg"].scale)
    for W in (got[1], got[3]):
        Wg = W[torch.from_numpy(rows).cuda()].cpu().numpy()[:, :m]
        assert ((Wg == INF) == (expect == INF)).all()
        assert_weights_close(Wg, expect, r["cfg"].scale, expect != INF)
    ctx.close()


@pytest.mark.parametrize("n,m,pad,shift", [(130, 517, 4, 0), (130, 517, 1, 0), (130, 518, 4, 1), (40, 20227, 4, 0), (40, 40703, 4, 0), (40, 40707, 4, 0),
                                           (40, 40707, 1, 3), (511, 40707, 1, 0), (512, 40706, 4, 0), (513, 45001, 1, 1), (1700, 40703, 4, 0), (1400, 60003, 4, 0), (512, 199998, 4, 0), (512, 200003, 4, 0), (70000, 1001, 4, 0)])
def test_entries_come_to_their_places(mm, n, m, pad, shift):
    """Scored in memory order and put in place, or scored as they come: the same matrix.  Rows that end in a part of a
    group, pitches and starts that are not whole groups, rows longer than what LDS takes of them, few and many
    rows around the widths that the kernel with LDS takes of either, and matrices beyond the last-level cache, which are stored past it."""
    r = synth.scheduling_round("C2", 9, n=n, m=m)
    pitch = (m + pad - 1) // pad * pad
    ctx = mm.Context(n, m)
    pred = ctx.predictor(dev_params(r["params"]), r["cfg"].scale)
    x_on, x_off, got = dev(r["x_on"]), dev(r["x_off"]), []
    for order in (0, 1):
        ctx.set_option("fit_order", order)
        buffer = torch.full((n * pitch + 8,), -7, dtype=torch.int32, device="cuda")
        W = buffer[shift:shift + n * pitch].view(n, pitch)
        ctx.score_pairs(pred, x_on, x_off, W)
        torch.cuda.synchronize()
        got.append(buffer)
    assert torch.equal(got[0], got[1])
    assert bool((got[1][shift:shift + n * pitch].view(n, pitch)[:, m:] == -7).all()) and bool((got[1][shift + n * pitch:] == -7).all())
    ctx.close()


@pytest.mark.parametrize("n,m,types", [(12288, 100, 1), (300, 14337, 1), (13000, 12500, 3), (16385, 65, 64), (12287, 70, 2)])
def test_many_workloads_in_memory_order(mm, n, m, types):
    """From 12,288 workloads on a side they are sorted in stretches of 2048, not counted: stretches that end early, many
    equal memory fractions, and types to order by first.  The matrix is that scored as it comes, and as many
    pairs went through the predictor as do in order of memory."""
    r = synth.scheduling_round("C5", 11, n=n, m=m)
    for x in (r["x_on"], r["x_off"]):
        x[:, 0] = np.round(x[:, 0] * 64) / 64
    ctx = mm.Context(n, m)
    pred = ctx.predictor(dev_params(r["params"]), 2.0 ** 24)
    x_on, x_off, got = dev(r["x_on"]), dev(r["x_off"]), []
    kind = dev(synth.gpu_types(11, n, types))
    for order in (0, 1):
        ctx.set_option("fit_order", order)
        W = empty_matrix(n, m)
        if types > 1:
            ctx.score_pairs_typed([pred] * types, kind, x_on, x_off, W)
        else:
            ctx.score_pairs(pred, x_on, x_off, W)
        torch.cuda.synchronize()
        got.append(W)
    assert torch.equal(got[0], got[1])
    assert abs(ctx.last_timings()["pairs_evaluated_fraction"] - _pairs_in_tasks(r) / (n * m)) <= 6e-8           # (a float)
    ctx.close()


@pytest.mark.parametrize("case", ["huge projections", "tiny hidden weights", "huge hidden weights", "mixed magnitudes",
                                  "zero hidden layer"])
def test_scores_do_not_depend_on_the_size_of_the_numbers(mm, orc, case):
    """The fp16 pieces of the hidden layer's operands are scaled into fp16's range by powers of
    two found on the device: networks whose layers are scaled against each other (the same function
    up to rounding, or nearly) must still meet the score tolerance."""
    r = synth.scheduling_round("C3", 6, n=130, m=517)
    p = {k: v.copy() for k, v in r["params"].items()}
    if case == "huge projections":          # layer-1 values around 1e5, beyond fp16's 65,504
        p["W1"] *= np.float32(2.0 ** 17); p["b1"] *= np.float32(2.0 ** 17); p["W2"] *= np.float32(2.0 ** -17)
    elif case == "tiny hidden weights":     # W2 around 1e-7, where fp16 has no normal numbers
        p["W2"] *= np.float32(2.0 ** -20); p["b2"] *= np.float32(2.0 ** -20); p["W3"] *= np.float32(2.0 ** 20)
    elif case == "huge hidden weights":
        p["W2"] *= np.float32(2.0 ** 22); p["b2"] *= np.float32(2.0 ** 22); p["W3"] *= np.float32(2.0 ** -22)
    elif case == "mixed magnitudes":        # one hidden unit and one input a few thousand times larger than the rest
        p["W2"][3, :] *= np.float32(4096.0); p["b2"][3] *= np.float32(4096.0); p["W3"][3] *= np.float32(1.0 / 4096.0)
        p["W1"][5, :] *= np.float32(1024.0); p["b1"][5] *= np.float32(1024.0); p["W2"][:, 5] *= np.float32(1.0 / 1024.0)
    else:
        p["W2"][:] = 0.0
    r["params"] = p
    ctx = mm.Context(r["n"], r["m"])
    Wg, sg = _score_on_gpu(mm, ctx, r)
    worst = _compare(orc, r, Wg, sg)
    assert worst < 2e-6                      # well inside the bar: the scaling costs no accuracy
    ctx.close()


def test_scores_other_seeds_and_scales(mm, orc):
    ctx = mm.Context(300, 600)
    for seed in (2, 3):
        for scale in (255.0, float(2 ** 24)):
            r = synth.scheduling_round("C3", seed, n=200, m=333)
            Wg, sg = _score_on_gpu(mm, ctx, r, scale)
            _compare(orc, r, Wg, sg, scale)
    ctx.close()


@pytest.mark.parametrize("cfg,n,m", [("C1", None, None), ("C2", 130, 517), ("C4", 300, 1031), ("C5", 257, 700),
                                     ("C3", 65, 257), ("C5", 1, 40), ("C3", 700, 90), ("C3", 3, 40001),
                                     ("C5", 2, 70003)])
def test_memory_ordered_pass_gives_the_same_matrix(mm, orc, cfg, n, m):
    """Without a score buffer the kernel walks rows and columns by memory fraction and leaves out
    pairs that cannot fit: the matrix must equal the all-pairs pass bit for bit, and the checker's."""
    r = synth.scheduling_round(cfg, 4, n=n, m=m)
    n, m = r["n"], r["m"]
    ctx = mm.Context(n, m)
    Wg, _ = _score_on_gpu(mm, ctx, r, want_sigma=False)
    part = ctx.last_timings()["pairs_evaluated_fraction"]
    ctx.set_option("fit_order", 0)
    Wall, _ = _score_on_gpu(mm, ctx, r, want_sigma=False)
    assert ctx.last_timings()["pairs_evaluated_fraction"] == 1.0
    assert (Wg == Wall).all()
    _, W = orc.score_pairs(r["x_on"], r["x_off"], r["params"], r["cfg"].scale)
    assert ((Wg == INF) == (W == INF)).all(), "mask bits differ"
    ok = W != INF
    if ok.any():
        assert_weights_close(Wg, W, r["cfg"].scale, ok)
    # every feasible pair went through the MLP; skipped ones are only whole 32-column runs
    feasible = ok.mean()
    assert feasible - 1e-6 <= part <= 1.0
    if n >= 64 and m >= 256:
        assert part <= feasible + 0.35
    ctx.close()


def test_memory_order_with_ties_and_odd_pitch(mm, orc):
    """Many equal memory fractions (the ordering must still be a permutation), fractions of 0 and
    above the limit, and a matrix pitch that rules out 16-byte stores."""
    r = synth.scheduling_round("C3", 6, n=333, m=1001)
    n, m = r["n"], r["m"]
    r["x_on"][:, 0] = np.round(r["x_on"][:, 0] * 8) / np.float32(8)
    r["x_off"][:, 0] = np.round(r["x_off"][:, 0] * 8) / np.float32(8)
    r["x_on"][::7, 0] = 0.0; r["x_off"][::5, 0] = 1.5; r["x_off"][1::11, 0] = -0.0
    ctx = mm.Context(n, m)
    pred = ctx.predictor(dev_params(r["params"]), r["cfg"].scale)
    _, W = orc.score_pairs(r["x_on"], r["x_off"], r["params"], r["cfg"].scale)
    for pitch in (m, m + 3):
        Wd = torch.full((n, pitch), -7, dtype=torch.int32, device="cuda")
        ctx.score_pairs(pred, dev(r["x_on"]), dev(r["x_off"]), Wd)
        torch.cuda.synchronize()
        Wg = Wd.cpu().numpy()
        assert (Wg[:, m:] == -7).all()
        Wg = Wg[:, :m]
        assert ((Wg == INF) == (W == INF)).all()
        ok = W != INF
        assert_weights_close(Wg, W, r["cfg"].scale, ok)
    ctx.close()


def test_closed_form_predictors(mm):
    # zero network: every feasible weight is exactly S/2
    F, H, S = 16, 64, float(2 ** 20)
    zero = {"W1": np.zeros((H, 2 * F), np.float32), "b1": np.zeros(H, np.float32),
            "W2": np.zeros((H, H), np.float32), "b2": np.zeros(H, np.float32),
            "W3": np.zeros(H, np.float32), "b3": np.zeros(1, np.float32)}
    x_on = synth.uniform_features(1, 0, 70, F); x_off = synth.uniform_features(1, 1, 90, F)
    ctx = mm.Context(70, 90)
    W = empty_matrix(70, 90)
    ctx.score_pairs(ctx.predictor(dev_params(zero), S), dev(x_on), dev(x_off), W)
    Wh = W.cpu().numpy()[:, :90]
    masked = (x_on[:, 0][:, None] + x_off[:, 0][None, :]) > np.float32(1)
    assert (Wh[masked] == INF).all() and (Wh[~masked] == 2 ** 19).all()
    # identity network: z is the plain sum of all features of both workloads
    H = F = 64
    ident = {"W1": np.concatenate([np.eye(F), np.eye(F)], 1).astype(np.float32), "b1": np.zeros(H, np.float32),
             "W2": np.eye(H, dtype=np.float32), "b2": np.zeros(H, np.float32),
             "W3": np.ones(H, np.float32), "b3": np.zeros(1, np.float32)}
    x_on = synth.uniform_features(2, 0, 40, F) * np.float32(0.05)
    x_off = synth.uniform_features(2, 1, 50, F) * np.float32(0.05)
    W = empty_matrix(40, 50); sg = torch.empty((40, 50), dtype=torch.float32, device="cuda")
    ctx.score_pairs(ctx.predictor(dev_params(ident), S, mem_limit=4.0), dev(x_on), dev(x_off), W, sg)
    z = x_on.astype(np.float64).sum(1)[:, None] + x_off.astype(np.float64).sum(1)[None, :]
    np.testing.assert_allclose(sg.cpu().numpy(), 1 / (1 + np.exp(-z)), rtol=1e-5)
    ctx.close()


def test_argument_errors(mm):
    ctx = mm.Context(8, 8)
    r = synth.scheduling_round("C1", 1, n=8, m=8)
    params = dev_params(r["params"])
    x_on, x_off = dev(r["x_on"]), dev(r["x_off"])
    W = empty_matrix(8, 8)
    bad = ctx.predictor(params, 2.0 ** 20); bad.H = 48
    with pytest.raises(mm.MuxmatchError) as e:
        ctx.score_pairs(bad, x_on, x_off, W)
    assert e.value.code == mm.ERR_ARG
    big = synth.scheduling_round("C1", 1, n=9, m=9)
    with pytest.raises(mm.MuxmatchError) as e:
        ctx.score_pairs(ctx.predictor(params, 2.0 ** 20), dev(big["x_on"]), dev(big["x_off"]), empty_matrix(9, 9))
    assert e.value.code == mm.ERR_SHAPE
    ctx.close()


@pytest.mark.parametrize("cfg,n,m", [("C2", 300, 200), ("C4", 6100, 6300), ("C5", 13000, 900)])
def test_a_captured_pass_is_the_same_every_time(mm, cfg, n, m):
    """The counters of tasks, of turns and of ranks are cleared by kernels of the pass itself: replays, with other passes of the
    context between them, find them so.  A short pass, a long one, and one whose workloads are sorted."""
    r = synth.scheduling_round(cfg, 19, n=n, m=m)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = mm.Context(n, m)
        pred, x_on, x_off, W, other = ctx.predictor(dev_params(r["params"]), r["cfg"].scale), dev(r["x_on"]), dev(r["x_off"]), empty_matrix(n, m), empty_matrix(n, m)
        ctx.score_pairs(pred, x_on, x_off, W)
        stream.synchronize()
        expect = W.clone()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            ctx.score_pairs(pred, x_on, x_off, W)
        for _ in range(4):
            W.fill_(-7)
            graph.replay()
            ctx.score_pairs(pred, x_on, x_off, other)
            stream.synchronize()
            assert torch.equal(W, expect) and torch.equal(other, expect)
        ctx.close()
