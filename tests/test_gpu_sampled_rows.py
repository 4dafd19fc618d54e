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


@pytest.mark.parametrize("P", [3, 128])                     # an argmax per pair; one per row of the memo table
def test_total_batch_sizes_at_multiples_of_what_fits(P):
    """The counts and batch sizes are quotients of integers, rounded up: total batch sizes that are a multiple of what a pass holds,
    one less and one more, one to a job, up to the largest; GPU counts within the tables and beyond; exactly the oracle's."""
    rng = np.random.default_rng(41)
    J, N, Gs = 1500, 4, 40
    wl = W.make(W.custom("multiples", P=P, J=J, N=N, cap=4096, Gm=1, Gs=Gs, index=960))
    params, K = wl.job_params, rng.choice([1, 2, 3, 5, 7, 13, 31, 49, 63, 64, 65, 77, 255, 257, 999], J)
    per_gpu = np.floor(np.exp(rng.uniform(0, np.log(2.0 ** 31), J)))
    per_gpu = np.where(rng.uniform(size=J) < 0.7, np.floor(np.exp(rng.uniform(0, np.log(5000.0), J))), per_gpu)
    passes = rng.choice([1, 2, 3, 7, 20, Gs - 1, Gs, Gs + 1], J)
    M = np.clip(passes * K * per_gpu + rng.integers(-1, 2, J), 1, 2 ** 31 - 1)
    params[W.PARAM_INDEX["m_mem"]] = np.minimum(per_gpu + rng.choice([0.0, 0.5], J), 2.0 ** 31 - 1)
    params[W.PARAM_INDEX["M0"]], params[W.PARAM_INDEX["M_max"]] = 1.0, 2.0 ** 52
    wl.m_grid[:] = M.astype(np.int32)[:, None]
    pop = wl.population
    pop[:] = 0
    pop[:, :, 0] = K
    pop[1::2, :, 0] -= K // 2
    pop[1::2, :, 1] = K // 2
    got, want = run_gpu(wl, flags=SAMPLE), run_oracle(wl, flags=SAMPLE)
    assert (want["best_s"] >= 0).mean() > 0.5 and (want["best_s"] < 0).any() and want["best_s"].max() == Gs - 1
    for k in ("best_m", "best_s"):
        assert np.array_equal(got[k], want[k]), k
