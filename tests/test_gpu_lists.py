"""GPU parity for the phases that run on lists of every line's best entries.

The lists hold 128 entries: lines of fewer, of exactly as many, of one more, and of a multiple of
the wavefront and of a slice of a whole line plus one; ties beyond what a list holds (a line is then
read whole); lists that are made once and again; phases that start on
the whole device and go on on one die.  The optimum is the exact CPU solver's, the duals
are re-checked on the host, and the solve with the lists off has to agree."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import padded_matrix

pytestmark = pytest.mark.gpu
INF = synth.INFEASIBLE


@pytest.mark.parametrize("n,m,high,masked", [(1, 1, 100, 0.0), (5, 128, 2 ** 24, 0.1), (40, 129, 2 ** 24, 0.0), (129, 130, 2 ** 20, 0.2),
                                             (300, 131, 2 ** 20, 0.3), (257, 1025, 2 ** 24, 0.5), (512, 513, 255, 0.1),
                                             (640, 640, 3, 0.0), (200, 2051, 1, 0.0), (1000, 1000, 2 ** 24, 0.95),
                                             (100, 4097, 2 ** 24, 0.2), (64, 8193, 2 ** 20, 0.6), (30, 20483, 2 ** 24, 0.2)])
@pytest.mark.parametrize("options", [{}, {"core_depth": 0}, {"core_depth": 0, "core_after": 0, "core_width": 1}, {"core_refine": 0},
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


@pytest.mark.parametrize("n,m", [(100, 128), (128, 128), (90, 64)])
def test_counters_of_a_solve_on_lists(n, m):
    """Lines no longer than a list: the whole solve runs on lists, every bid and every scan of a search or a proof
    reads one list (128 entries of 8 bytes) and is counted once."""
    import paper_2303_13803_amd as mm
    ctx = mm.Context(n, m)
    W = padded_matrix(synth.uniform_matrix(72, n, m, 2 ** 24, 0.2))
    r2c = torch.empty(n, dtype=torch.int32, device="cuda")
    u, v = torch.empty(n, dtype=torch.int64, device="cuda"), torch.empty(m, dtype=torch.int64, device="cuda")
    res = ctx.solve_assignment(W, n, m, r2c, u, v)
    ctx.close()
    assert res.bids > 0 and res.path_scans > 0 and res.chain_bids == res.bids
    assert res.bytes_scanned == 1024 * (res.bids + res.path_scans)
