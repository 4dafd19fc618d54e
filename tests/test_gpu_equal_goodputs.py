"""Jobs whose batch sizes tie.  With alpha_grad = 0 and gamma = 1 (both bounds of the fit) the goodput depends on the total batch size
alone, so batch sizes with a common multiple agree to the last places and rounding elects one of them: the sweeps (one candidate at a
time, four, with rows copied on chip), small calls, memoised rows and fair shares have to round alike, whatever the number of counts."""
import numpy as np
import pytest

import workloads as W
from parity import run_oracle

pytestmark = pytest.mark.gpu
KEYS = ("fitness", "violations", "best_m", "best_s", "best_goodput", "speedup")


def workload(P, J, N, Gm, Gs, first):
    wl = W.make(W.custom("ties", P=9, J=J, N=N, cap=max(4, -(-8 * J // N)), Gm=Gm, Gs=Gs, index=2600 + N))
    jp, row, rng = wl.job_params, W.PARAM_INDEX, np.random.default_rng(Gm + Gs)
    jp[row["alpha_grad"]], jp[row["gamma"]] = 0.0, 1.0
    jp[row["M0"]], jp[row["M_max"]] = 32.0, 32.0 * rng.choice([32, 256, 2048], J)
    jp[row["phi"]] = 10.0 ** rng.uniform(2.0, 5.0, J)
    wl.m_grid[:] = np.arange(first, first + Gm)              # consecutive: the most common multiples
    pop = np.zeros((P, J, N), np.int32)
    for c in range(P):                                       # 2 to 30 GPUs a job, on one node, two or many
        K = rng.integers(2, 31, J)
        for j in range(J):
            nodes = min(N, K[j], [1, 2, 5][(c + j) % 3])
            pop[c, j, :nodes] = 1
            pop[c, j, 0] += K[j] - nodes
    wl.fair_share[:, 0], wl.fair_share[:, 1] = pop[0].sum(1), (pop[0] > 0).sum(1)
    return wl, pop


def results(wl, pop, flags=0, precision=0, keep=False):
    import torch
    import paper_2008_12260_amd as px
    c = wl.cfg
    call = px.FitnessCall(pop.shape[0], c.J, c.N, c.Gm, c.Gs, wl.job_params, wl.m_grid, wl.fair_share, pop[0], np.full(c.N, 40, np.int32),
                          p=c.p, delta=c.delta, flags=flags, precision=precision)
    for _ in range(2 if keep else 1):
        call.run(torch.as_tensor(pop).cuda(), keep_job_tables=_ == 1)
    return call.results()


@pytest.mark.parametrize("P,J,N,Gm,Gs,first", [
    (40, 200, 16, 64, 16, 8), (40, 200, 16, 50, 24, 8), (40, 200, 16, 64, 32, 8), (17, 200, 130, 64, 64, 8), (17, 200, 130, 64, 300, 2),
    (17, 200, 130, 130, 32, 4), (2000, 40, 128, 128, 32, 4), (2000, 40, 130, 100, 32, 4), (2000, 40, 64, 64, 32, 8), (9, 40, 3, 64, 33, 4),
    (200, 16, 9, 32, 32, 6), (200, 15, 9, 31, 24, 4), (200, 16, 9, 64, 16, 8), (200, 8, 9, 128, 24, 4), (200, 4, 9, 256, 32, 2)])
def test_every_way_elects_the_same_batch_size(P, J, N, Gm, Gs, first):
    import paper_2008_12260_amd as px
    wl, pop = workload(P, J, N, Gm, Gs, first)
    got, memo = results(wl, pop), results(wl, pop, px.PX_FLAG_MEMOISE)
    for k in KEYS:
        assert np.array_equal(got[k], memo[k]), (k, int(np.sum(got[k] != memo[k])))
    assert np.array_equal(got["speedup"][0], np.where(got["best_goodput"][0] > 0.0, 1.0, 0.0))       # row 0 is the fair share
    kept = results(wl, pop, keep=True)
    for k in KEYS:
        assert np.array_equal(got[k], kept[k]), k
    wl.node_capacity[:] = 40
    some = pop[:9]
    ref = run_oracle(wl, population=some, current=pop[0])
    for k in ("best_goodput", "speedup"):
        assert np.max(np.abs(got[k][:9] - ref[k]) / np.where(ref[k] == 0, 1.0, ref[k])) <= 1e-12, k
