"""Small calls on grids of at most 32 batch sizes, where a wavefront takes two argmaxes, a half each: the oracle's results at the edges
of the grid, the jobs (odd ones leave a half idle) and the counts, started anew and with the fair shares kept."""
import numpy as np
import pytest

import workloads as W
from parity import compare, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Gm,Gs", [(1, 1), (2, 9), (15, 8), (16, 16), (17, 17), (31, 32), (32, 8), (32, 32), (33, 8)])
@pytest.mark.parametrize("J", [1, 2, 7, 8, 9, 15, 16])
def test_two_argmaxes_a_wavefront(J, Gm, Gs):
    import torch
    import paper_2008_12260_amd as px
    N = 5 if J < 9 else 70
    wl = W.make(W.custom("halves", P=7, J=J, N=N, cap=8, Gm=Gm, Gs=Gs, index=2400 + J))
    pop = wl.population
    pop[0] = wl.current_alloc
    pop[1, 0, 0] += 70                                       # beyond the tabled GPU counts
    pop[2, J // 2, :2] = 40
    pop[3, J - 1] = 0                                        # a job without a GPU, and a matrix of none
    pop[4] = 0
    pop[5, J - 1, 0] = 9                                     # more GPUs on one node than any node has
    wl.fair_share[::3, 0] = 66
    if J > 2:
        wl.param("M0")[2], wl.param("M_max")[2] = 1e9, 2e9   # nothing feasible: no fair share either
    if Gm > 2:
        wl.m_grid[::2, 1] = wl.m_grid[::2, 0]                # equal batch sizes: the first is elected
    c = wl.cfg
    call = px.FitnessCall(c.P, J, N, Gm, Gs, wl.job_params, wl.m_grid, wl.fair_share, wl.current_alloc, wl.node_capacity, p=c.p, delta=c.delta)
    call.run(torch.as_tensor(pop).cuda())
    assert compare(wl, call.results(), run_oracle(wl)) == 0
    again = pop[np.random.default_rng(J).permutation(c.P)][:, :, ::-1].copy()
    call.run(torch.as_tensor(again).cuda(), keep_job_tables=True)
    assert compare(wl, call.results(), run_oracle(wl, population=again), population=again) == 0
