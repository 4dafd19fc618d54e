"""Memoised argmaxes on grids at the edges of the two groups of 64 batch sizes that share an election, duplicates across them
included, with two and with four rows a wavefront: bit for bit what a sweep per pair gives, and so at every split of the pairs."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("J", [20, 260])
@pytest.mark.parametrize("Gm", [1, 63, 64, 65, 127, 128, 129, 192, 193, 257])
def test_memoised_rows_on_any_grid(Gm, J):
    import torch
    import paper_2008_12260_amd as px
    wl = W.make(W.custom("grids", P=9, J=J, N=40, cap=max(4, -(-2 * J // 40)), Gm=Gm, Gs=9, index=2000 + Gm))
    c = wl.cfg
    grid = wl.m_grid.copy()
    grid[1::2] = np.sort(grid[1::2] // 16 * 16 + 16, axis=1)[:, ::-1]          # many equal batch sizes, descending
    got = []
    for flags in (0, px.PX_FLAG_MEMOISE):
        call = px.FitnessCall(c.P, c.J, c.N, c.Gm, c.Gs, wl.job_params, grid, wl.fair_share, wl.current_alloc, wl.node_capacity,
                              p=c.p, delta=c.delta, flags=flags)
        call.run(torch.as_tensor(wl.population).cuda())
        got.append(call.results())
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k], equal_nan=True), k


def test_a_batch_size_whose_time_overflows_hides_no_other():
    """T_grad overflows at the first 64 batch sizes and not at the next 64, which share an election with them: both ways of taking
    the argmax find the same finite point."""
    import torch
    import paper_2008_12260_amd as px
    J, Gm, Gs = 20, 128, 9
    wl = W.make(W.custom("overflow", P=9, J=J, N=40, cap=4, Gm=Gm, Gs=Gs, index=2050))
    c, params, grid = wl.cfg, wl.job_params.copy(), wl.m_grid.copy()
    params[W.PARAM_INDEX["beta_grad"]] = 1e306
    params[W.PARAM_INDEX["phi"]] = 0.5
    params[W.PARAM_INDEX["M0"]], params[W.PARAM_INDEX["M_max"]] = 8.0, 2.0 ** 20
    grid[:, :64], grid[:, 64:] = np.arange(200, 264), np.arange(8, 72)
    got = []
    for flags in (0, px.PX_FLAG_MEMOISE):
        call = px.FitnessCall(c.P, J, c.N, Gm, Gs, params, grid, wl.fair_share, wl.current_alloc, wl.node_capacity, p=c.p,
                              delta=c.delta, flags=flags)
        call.run(torch.as_tensor(wl.population).cuda())
        got.append(call.results())
    held = wl.population.sum(2) > 0
    assert np.all(got[0]["best_goodput"][held] > 0.0) and np.all(got[0]["best_m"][held] < 72)
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k], equal_nan=True), k


@pytest.mark.parametrize("N", [16, 61, 130])
@pytest.mark.parametrize("Gm,Gs", [(64, 16), (50, 12), (128, 32)])
@pytest.mark.parametrize("P", [61, 62, 125, 190, 249, 311, 373, 500, 1000])    # of 200 jobs: one to sixteen candidates a wavefront
def test_every_split_of_the_pairs_elects_the_same(P, Gm, Gs, N):
    import torch
    import paper_2008_12260_amd as px
    wl = W.make(W.custom("split", P=P, J=200, N=N, cap=max(4, -(-400 // N)), Gm=Gm, Gs=Gs, index=2100 + N))
    c = wl.cfg
    pop = torch.as_tensor(wl.population).cuda()
    got = []
    for flags in (0, px.PX_FLAG_MEMOISE):
        call = px.FitnessCall(c.P, c.J, c.N, c.Gm, c.Gs, wl.job_params, wl.m_grid, wl.fair_share, wl.current_alloc, wl.node_capacity,
                              p=c.p, delta=c.delta, flags=flags)
        call.run(pop)
        got.append(call.results())
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k], equal_nan=True), k
