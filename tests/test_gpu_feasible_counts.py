"""Accumulation counts whose best lies below, within and beyond the feasible ones, in every chunk the sweep has (8, 16, 24, 32 counts
and several of 32, reciprocals on chip and in memory): the oracle's points, and bit for bit those of the memoised argmax, which
finds the count without a sweep."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from parity import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu
KEYS = ("fitness", "violations", "best_m", "best_s", "best_goodput", "speedup")


def workload(P, J, N, Gm, Gs):
    wl = W.make(W.custom("counts", P=P, J=J, N=N, cap=max(4, -(-2 * J // N)), Gm=Gm, Gs=Gs, index=2300 + N))
    row, j = W.PARAM_INDEX, np.arange(J)
    jp = wl.job_params
    # the best count is about sqrt((last - T_grad) phi / (K m T_grad)): from none to far beyond the grid
    jp[row["phi"]] = 10.0 ** (j % 8)
    # the feasible ones: all, from the middle of the grid on, a few, up to the first one or two
    jp[row["M0"]] = np.where(j % 4 == 1, 32.0 * max(1, Gs // 2), 16.0)
    jp[row["M_max"]] = np.select([j % 4 == 0, j % 4 == 1, j % 4 == 2], [2.0 ** 40, 2.0 ** 40, 96.0], 32.0)
    return wl


@pytest.mark.parametrize("N", [16, 61, 130])
@pytest.mark.parametrize("Gm,Gs", [(64, 1), (50, 7), (64, 8), (33, 9), (64, 16), (64, 17), (50, 24), (128, 25), (64, 32), (31, 33),
                                   (64, 64), (50, 255), (64, 256), (64, 257), (50, 300)])
def test_best_counts_on_either_side_of_the_feasible_ones(N, Gm, Gs):
    import paper_2008_12260_amd as px
    wl = workload(17, 24, N, Gm, Gs)
    got, want = run_gpu(wl), run_oracle(wl)
    assert compare(wl, got, want) == 0
    memo = run_gpu(wl, flags=px.PX_FLAG_MEMOISE)
    for k in KEYS:
        assert np.array_equal(got[k], memo[k], equal_nan=True), k
    single = run_gpu(wl, precision=1)
    K = wl.population.sum(2)
    held = want["best_goodput"] > 0
    assert np.array_equal(single["best_m"] > 0, held)
    for c, j in np.argwhere(held)[::7]:             # single precision: its own point prices within 1e-5 of the best
        g, ok = O.goodput(O.job_from_params(wl.job_params, j), int(K[c, j]), int((wl.population[c, j] > 0).sum()),
                          int(single["best_m"][c, j]), int(single["best_s"][c, j]))
        assert ok and abs(g - want["best_goodput"][c, j]) <= 1e-5 * g
        assert abs(single["best_goodput"][c, j] - g) <= 1e-5 * g


@pytest.mark.parametrize("N,P", [(130, 9), (130, 3000), (128, 3000)])      # rows of the tables in memory, and copied on chip
def test_a_first_batch_size_without_a_time_does_not_take_the_second_ones_place(N, P):
    """T_grad overflows at the first 64 batch sizes and not at the next 64, which the same lanes hold."""
    import torch
    import paper_2008_12260_amd as px
    J, Gm, Gs = 20, 128, 9
    wl = W.make(W.custom("overflow", P=9, J=J, N=N, cap=4, Gm=Gm, Gs=Gs, index=2350))
    c, params, grid = wl.cfg, wl.job_params.copy(), wl.m_grid.copy()
    params[W.PARAM_INDEX["beta_grad"]] = 1e306
    params[W.PARAM_INDEX["phi"]] = 0.5
    params[W.PARAM_INDEX["M0"]], params[W.PARAM_INDEX["M_max"]] = 8.0, 2.0 ** 20
    grid[:, :64], grid[:, 64:] = np.arange(200, 264), np.arange(8, 72)
    pop = np.resize(wl.population, (P, J, N))
    got = []
    for flags in (0, px.PX_FLAG_MEMOISE):
        call = px.FitnessCall(P, J, N, Gm, Gs, params, grid, wl.fair_share, wl.current_alloc, wl.node_capacity, p=c.p, delta=c.delta,
                              flags=flags)
        call.run(torch.as_tensor(pop).cuda())
        got.append(call.results())
    held = pop.sum(2) > 0
    assert np.all(got[0]["best_goodput"][held] > 0.0) and np.all(got[0]["best_m"][held] < 72)
    for k in KEYS:
        assert np.array_equal(got[0][k], got[1][k], equal_nan=True), k
