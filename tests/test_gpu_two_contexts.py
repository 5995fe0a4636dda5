"""Two contexts that solve at the same time, each on a stream of its own (GPU).

The launches of the phases on lists keep workgroups on the device that wait for one another; beside
another such launch they have to go on with those that found room (see csrc/team_join.h), on one die or
on all of them."""
import threading

import numpy as np
import pytest
import torch

import synth
from gpu_util import padded_matrix

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
