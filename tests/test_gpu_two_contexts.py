"""Two contexts that solve at the same time, each on a stream of its own (GPU).

The launches of the phases on lists keep workgroups on the device that wait for one another; beside
another such launch they have to go on with those that found room (see csrc/team_join.h), on one die or
on all of them.  And a pass over a large matrix leaves others room (see csrc/pair_tasks.h)."""
import threading
import time

import numpy as np
import pytest
import torch

import synth
from gpu_util import dev, dev_params, empty_matrix, padded_matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("options", [{"core_depth": 0}, {"core_depth": 0, "core_wide": 1, "core_narrow": 16}])
def test_two_contexts_at_once(orc, options):
    import paper_2303_13803_amd as mm
    W = [synth.uniform_matrix(91, 1000, 1400, 2 ** 24, 0.1), synth.uniform_matrix(92, 1100, 1100, 2 ** 20, 0.2)]
    expect = [orc.max_weight_matching(w)[0] for w in W]
    device = [padded_matrix(w) for w in W]
    torch.cuda.synchronize()
    found, start = [[], []], threading.Barrier(2)

    def solve(k):
        n, m = W[k].shape
        with torch.cuda.stream(torch.cuda.Stream()):
            ctx = mm.Context(n, m)
            for name, value in options.items():
                ctx.set_option(name, value)
            r2c = torch.empty(n, dtype=torch.int32, device="cuda")
            u = torch.empty(n, dtype=torch.int64, device="cuda")
            v = torch.empty(m, dtype=torch.int64, device="cuda")
            start.wait()
            for _ in range(5):
                res = ctx.solve_assignment(device[k], n, m, r2c, u, v)
                torch.cuda.current_stream().synchronize()
                code, P, D = orc.check_certificate(W[k], r2c.cpu().numpy(), u.cpu().numpy(), v.cpu().numpy(), res.K)
                found[k].append((code, res.cert_ok, res.primal, res.fallbacks))
            ctx.close()

    threads = [threading.Thread(target=solve, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(2):
        assert found[k] == [(0, 1, expect[k], 0)] * 5


def test_a_long_scoring_pass_leaves_room_for_others(orc):
    """Small rounds and matchings beside passes over 16,000 x 16,000 pairs (14 ms each) are done long before these are, and
    both come out as they do alone.  A small round (0.3 ms alone) takes 1.4 ms; while workgroups of the pass all stayed it
    took as long as a pass."""
    import paper_2303_13803_amd as mm
    large = synth.scheduling_round("C4", 93, n=16000, m=16000)
    small = synth.scheduling_round("C1", 94)
    n, m, S = small["n"], small["m"], small["cfg"].scale
    M = synth.uniform_matrix(95, 500, 700, 2 ** 24, 0.1)
    best = orc.max_weight_matching(M)[0]
    plan = lambda a, b: (torch.empty(a, dtype=torch.int32, device="cuda"), torch.empty(a, dtype=torch.int64, device="cuda"), torch.empty(b, dtype=torch.int64, device="cuda"))
    streams = [torch.cuda.Stream() for _ in range(2)]
    with torch.cuda.stream(streams[0]):
        ctx = mm.Context(large["n"], large["m"])
        pred, x_on, x_off, W = ctx.predictor(dev_params(large["params"]), large["cfg"].scale), dev(large["x_on"]), dev(large["x_off"]), empty_matrix(large["n"], large["m"])
        ctx.score_pairs(pred, x_on, x_off, W)
        streams[0].synchronize()
        alone = W.clone()
        W.fill_(-7)
        begin = time.perf_counter()
        ctx.score_pairs(pred, x_on, x_off, W)
        streams[0].synchronize()
        one_pass = time.perf_counter() - begin
    with torch.cuda.stream(streams[1]):
        other = mm.Context(500, 700)
        small_pred, s_on, s_off, s_W = other.predictor(dev_params(small["params"]), S), dev(small["x_on"]), dev(small["x_off"]), empty_matrix(n, m)
        M_dev, round_plan, matching_plan = padded_matrix(M), plan(n, m), plan(500, 700)
        expect = other.schedule_round(small_pred, s_on, s_off, s_W, *round_plan).primal
        streams[1].synchronize()
        taken = []
        for kind in ("round", "matching"):
            with torch.cuda.stream(streams[0]):
                for _ in range(5):
                    ctx.score_pairs(pred, x_on, x_off, W)
            while True:
                begin = time.perf_counter()
                if kind == "round":
                    res = other.schedule_round(small_pred, s_on, s_off, s_W, *round_plan)
                else:
                    res = other.solve_assignment(M_dev, 500, 700, *matching_plan)
                streams[1].synchronize()
                if streams[0].query():
                    break
                if kind == "round":
                    taken.append(time.perf_counter() - begin)
                assert (res.primal, res.cert_ok, res.fallbacks) == (expect if kind == "round" else best, 1, 0)
            streams[0].synchronize()
            assert torch.equal(W, alone)
        other.close()
    ctx.close()
    assert sorted(taken)[len(taken) // 2] < one_pass / 3
