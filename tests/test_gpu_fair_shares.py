"""Fair shares in single precision, found beside the tables (up to 32 counts) or from them (more): inside the tables and beyond, on one
node and several, at the edges of groups of batch sizes and of chunks of counts."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Gs", [1, 8, 16, 17, 32, 33])
@pytest.mark.parametrize("Gm", [1, 63, 64, 65, 130])
def test_fair_shares_in_single_precision(Gm, Gs):
    import torch
    import paper_2008_12260_amd as px
    shares = [(1, 1), (2, 1), (2, 2), (7, 1), (8, 1), (9, 1), (63, 8), (64, 8), (65, 9), (200, 25), (64, 1)]    # 8 GPUs a node
    J = len(shares)
    wl = W.make(W.custom("shares", P=6, J=J, N=16, cap=8, Gm=Gm, Gs=Gs, index=1900 + Gm + Gs))
    c, fair = wl.cfg, np.array(shares, dtype=np.int32)
    ref = O.fitness(wl.population, wl.job_params, wl.m_grid, fair, wl.current_alloc, wl.node_capacity, c.p, c.delta, c.Gs)
    for flags in (0, px.PX_FLAG_MEMOISE):
        call = px.FitnessCall(c.P, c.J, c.N, c.Gm, c.Gs, wl.job_params, wl.m_grid, fair, wl.current_alloc, wl.node_capacity, p=c.p,
                              delta=c.delta, flags=flags, precision=1)
        call.run(torch.as_tensor(wl.population).cuda())
        got = call.results()
        assert got["status"] == ref["status"]
        for k in ("best_goodput", "speedup", "fitness"):
            # about 30 roundings of 2^-24 in a speedup, the sums of 11 jobs' terms in the fitness
            err = np.abs(got[k] - ref[k]) / np.where(ref[k] == 0, 1.0, np.abs(ref[k]))
            assert err.max() <= 1e-5, (k, flags)


@pytest.mark.parametrize("Gs", [1, 8, 16, 17, 32, 33])
@pytest.mark.parametrize("Gm", [1, 63, 65, 130])
def test_a_row_that_is_its_fair_share_has_a_speedup_of_one(Gm, Gs):
    """Whichever way fair shares and rows are found, in single precision too, the same (GPUs, one node or several) gives the same
    bits, so a job left with its fair share has a speedup of exactly 1."""
    import torch
    import paper_2008_12260_amd as px
    shares = [(1, 1), (2, 1), (2, 2), (3, 2), (7, 1), (8, 1), (9, 2), (31, 4), (63, 8), (64, 8), (65, 9), (200, 25), (20, 1)]
    J, N = len(shares), 28
    wl = W.make(W.custom("equal", P=40, J=J, N=N, cap=8, Gm=Gm, Gs=Gs, index=1950 + Gm + Gs))
    c, pop, fair = wl.cfg, wl.population.copy(), np.array(shares, dtype=np.int32)
    for j, (K, nodes) in enumerate(shares):
        pop[0, j] = 0
        pop[0, j, :nodes] = 1
        pop[0, j, 0] += K - nodes
    for precision in (0, 1):
        for flags in (0, px.PX_FLAG_MEMOISE):
            call = px.FitnessCall(c.P, J, N, Gm, Gs, wl.job_params, wl.m_grid, fair, pop[0], wl.node_capacity, p=c.p, delta=c.delta,
                                  flags=flags, precision=precision)
            call.run(torch.as_tensor(pop).cuda())
            got = call.results()
            feasible = got["best_goodput"][0] > 0.0
            assert np.array_equal(got["speedup"][0], np.where(feasible, 1.0, 0.0)), (precision, flags)
            assert feasible.any() or Gm == 1 or Gs == 1
