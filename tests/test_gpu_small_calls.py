"""Calls of few candidates and jobs, which one launch evaluates: both sides of every line of that rule against the oracle, the
status word kept or started anew, and generations."""
import numpy as np
import pytest

import workloads as W
from parity import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def workload(P, J, N, Gm, Gs, index):
    wl = W.make(W.custom("small", P=P, J=J, N=N, cap=8, Gm=Gm, Gs=Gs, index=index, phi_hi=1e6))
    pop = wl.population
    pop[0] = wl.current_alloc
    pop[1, 0, 0] += 70                                       # beyond the tabled GPU counts
    pop[2, J // 2, :2] = 40
    pop[min(3, P - 1), J - 1] = 0
    pop[min(4, P - 1), J - 1, 0] = 9                         # more GPUs on one node than any node has
    return wl


@pytest.mark.parametrize("P,J,N,Gm,Gs", [(3, 1, 4, 1, 1), (252, 5, 6, 33, 8), (253, 5, 6, 33, 8), (6, 16, 9, 64, 16), (6, 17, 9, 64, 16),
                                         (6, 8, 9, 65, 9), (6, 9, 9, 65, 9), (5, 1, 7, 1024, 32), (5, 1, 7, 1025, 32), (5, 8, 5, 40, 33),
                                         (5, 8, 3, 40, 17), (5, 8, 256, 40, 32), (5, 8, 257, 40, 32)])
@pytest.mark.parametrize("p", [-1.0, 0.0, 0.5])
def test_either_side_of_the_line(P, J, N, Gm, Gs, p):
    wl = workload(P, J, N, Gm, Gs, 1100 + N)
    wl.fair_share[::2, 0] = 66
    assert compare(wl, run_gpu(wl, p=p), run_oracle(wl, p=p)) == 0
    for flags in (1, 2):
        assert compare(wl, run_gpu(wl, p=p, flags=flags), run_oracle(wl, p=p, flags=flags)) == 0


@pytest.mark.parametrize("P,J,N,Gm,Gs", [(6, 1, 4, 1, 1), (252, 5, 6, 33, 8), (253, 5, 6, 33, 8), (6, 16, 9, 64, 16), (6, 17, 9, 64, 16),
                                         (6, 14, 9, 64, 17), (6, 15, 9, 64, 17), (6, 16, 9, 64, 17), (6, 17, 9, 64, 17), (5, 4, 9, 256, 32),
                                         (5, 3, 9, 257, 17), (5, 1, 7, 512, 17), (5, 1, 7, 513, 17), (5, 1, 7, 1024, 16)])
@pytest.mark.parametrize("flags", [0, 1])
def test_calls_that_keep_their_tables(P, J, N, Gm, Gs, flags):
    """Another population, the fair shares and re-allocation factors of the call before: the oracle's results."""
    import torch
    import paper_2008_12260_amd as px
    wl = workload(P, J, N, Gm, Gs, 1500 + N)
    wl.fair_share[::2, 0] = 66
    c = wl.cfg
    call = px.FitnessCall(P, J, N, Gm, Gs, wl.job_params, wl.m_grid, wl.fair_share, wl.current_alloc, wl.node_capacity, p=c.p,
                          delta=c.delta, flags=flags)
    call.run(torch.as_tensor(wl.population).cuda())
    assert compare(wl, call.results(), run_oracle(wl, flags=flags)) == 0
    for seed in (1, 2):
        pop = wl.population[np.random.default_rng(seed).permutation(P)][:, :, ::-1].copy()
        call.run(torch.as_tensor(pop).cuda(), keep_job_tables=True)
        assert compare(wl, call.results(), run_oracle(wl, population=pop, flags=flags), population=pop) == 0


@pytest.mark.parametrize("P", [40, 260])                     # one launch, and the general path
def test_status_word_is_started_by_a_call_and_kept_by_the_next(P):
    import torch
    import paper_2008_12260_amd as px
    wl = workload(P, 6, 5, 8, 4, 1200)
    wl.param("age_T")[2] = 1.0
    wl.param("restarts_R")[2] = 5.0
    c = wl.cfg
    call = px.FitnessCall(P, c.J, c.N, c.Gm, c.Gs, wl.job_params, wl.m_grid, wl.fair_share, wl.current_alloc, wl.node_capacity)
    good, bad = wl.population.copy(), wl.population.copy()
    bad[P - 1, 0, 1] = -1
    good, bad = torch.as_tensor(good).cuda(), torch.as_tensor(bad).cuda()
    out = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    for pop, keep, want in ((good, False, 4), (bad, True, 12), (good, True, 12), (good, False, 4), (bad, False, 12), (good, True, 12)):
        call.run(pop, keep_job_tables=keep)
        assert call.status() == want
        px.pollux_fitness_static(call.dims, pop, call.job_params, call.m_grid, call.fair_share, call.current_alloc, call.node_capacity,
                                 call.p, call.delta, call.fitness, call.best_m, call.best_s, status=out)
        assert int(out.item()) == (12 if pop is bad else 4)


@pytest.mark.parametrize("inherit", [False, True])
@pytest.mark.parametrize("P,N", [(24, 7), (24, 70)])
def test_generations(P, N, inherit):
    import torch
    import paper_2008_12260_amd as px
    wl = W.make(W.custom("small", P=P, J=12, N=N, cap=8, Gm=20, Gs=10, index=1300 + N))
    c = wl.cfg
    make = lambda: px.FitnessCall(P, c.J, c.N, c.Gm, c.Gs, wl.job_params, wl.m_grid, wl.fair_share, wl.current_alloc, wl.node_capacity)
    call, check = make(), make()
    pop = torch.as_tensor(wl.population).cuda()
    call.run(pop)
    for g in range(5):
        call.generation(pop, 9, g, P // 3, 1 << 30, inherit_rows=inherit)
        check.run(pop)
        got, want = call.results(), check.results()
        for k in ("fitness", "violations", "best_m", "best_s", "best_goodput", "speedup"):
            assert np.array_equal(got[k], want[k], equal_nan=True), (g, k)
        ref = run_oracle(wl, population=pop.cpu().numpy())
        assert compare(wl, {**got, "status": 0}, {**ref, "status": 0}, population=pop.cpu().numpy()) == 0
