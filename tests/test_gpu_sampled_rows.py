"""The sampling argmax taken per (job, GPU count, placement) from 128 candidates on: both sides of that line against the
oracle, rows beyond the tabled counts included, and generations that inherit rows without the memoise flag."""
import numpy as np
import pytest

import workloads as W
from parity import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu
SAMPLE = 16


@pytest.mark.parametrize("P,J,N,Gm,Gs", [(127, 5, 6, 40, 4), (128, 5, 6, 40, 4), (130, 3, 3, 40, 4), (130, 4, 66, 130, 16), (140, 7, 300, 8, 2)])
def test_either_side_of_the_line(P, J, N, Gm, Gs):
    wl = W.sampled(W.make(W.custom("line", P=P, J=J, N=N, cap=8, Gm=Gm, Gs=Gs, index=900 + N)))
    pop = wl.population
    pop[1, 0, 0] = 66                                       # beyond the tabled GPU counts, on one node
    pop[2, 1, :2] = 50                                      # and on several
    pop[3, 2] = 0
    assert compare(wl, run_gpu(wl, flags=SAMPLE), run_oracle(wl, flags=SAMPLE), sampled=True) == 0


@pytest.mark.parametrize("P", [100, 160])
def test_generations_that_inherit_rows(P):
    import torch
    import paper_2008_12260_amd as px
    wl = W.sampled(W.make(W.custom("heirs", P=P, J=20, N=10, cap=8, Gm=16, Gs=8, index=950)))
    c = wl.cfg
    make = lambda: px.FitnessCall(P, c.J, c.N, c.Gm, c.Gs, wl.job_params, wl.m_grid, wl.fair_share, wl.current_alloc,
                                  wl.node_capacity, p=c.p, delta=c.delta, flags=SAMPLE)
    call, check = make(), make()
    pop = torch.as_tensor(wl.population).cuda()
    call.run(pop)
    for g in range(4):
        call.generation(pop, 5, g, P // 2, 1 << 29, inherit_rows=True)
        check.run(pop)
        got, want = call.results(), check.results()
        for k in ("fitness", "violations", "best_m", "best_s", "best_goodput", "speedup"):
            assert np.array_equal(got[k], want[k], equal_nan=True), (g, k)
