"""The population pass with a sweep per pair over rows of every length and alignment one 16-byte load per lane can cover, on
grids that are and are not whole groups of 64 batch sizes."""
import numpy as np
import pytest

import workloads as W
from parity import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Gm,Gs", [(33, 8), (64, 16), (65, 20), (64, 32)])
@pytest.mark.parametrize("N", [3, 4, 5, 63, 64, 65, 66, 130, 251, 255, 257])
def test_rows_of_any_length(N, Gm, Gs):
    wl = W.make(W.custom("rows", P=70, J=5, N=N, cap=4, Gm=Gm, Gs=Gs, index=600 + N))
    pop = wl.population
    pop[0] = wl.current_alloc
    pop[1, 2, N - 1] = -3
    pop[2, 1, 0] = 300                                        # beyond the tables and beyond what two rows' shared sum holds
    pop[3, 4, N // 2] += 100
    pop[4, 0] = 0
    assert compare(wl, run_gpu(wl), run_oracle(wl)) == 0


@pytest.mark.parametrize("off", [1, 2, 3])
@pytest.mark.parametrize("N,P", [(12, 9), (64, 300), (68, 90), (255, 90)])
@pytest.mark.parametrize("precision", [0, 1])
def test_matrices_at_any_address(N, P, off, precision):
    """Population and current allocation away from 16-byte boundaries: the results of the aligned call."""
    import torch
    import paper_2008_12260_amd as px
    wl = W.make(W.custom("moved", P=P, J=8, N=N, cap=4, Gm=64, Gs=16, index=700 + N))
    c = wl.cfg
    call = px.FitnessCall(c.P, c.J, N, c.Gm, c.Gs, wl.job_params, wl.m_grid, wl.fair_share, wl.current_alloc, wl.node_capacity,
                          p=c.p, delta=c.delta, precision=precision)
    pop = torch.as_tensor(wl.population).cuda()
    call.run(pop)
    want = call.results()

    def moved(x):
        room = torch.full((x.numel() + 8,), -9, dtype=torch.int32, device="cuda")
        at = room[off:off + x.numel()].view(x.shape)
        at.copy_(x)
        return at
    call.current_alloc = moved(call.current_alloc)
    call.run(moved(pop))
    got = call.results()
    for k in want:
        assert np.array_equal(got[k], want[k], equal_nan=True), k


@pytest.mark.parametrize("Gm", [0x7FFF, 0x8000, 0x8001, 0x10040])
def test_more_batch_sizes_than_a_packed_index_holds(Gm):
    wl = W.make(W.custom("long", P=5, J=1, N=6, cap=4, Gm=Gm, Gs=2, index=750))
    wl.m_grid[0] = np.arange(1, Gm + 1)                      # the best batch sizes anywhere in the grid
    wl.param("M0")[0], wl.param("M_max")[0], wl.param("phi")[0] = 0.9 * Gm, 1e7, 1e9
    ref = run_oracle(wl)
    assert ref["best_m"].max() >= 0.8 * Gm
    assert compare(wl, run_gpu(wl), ref) == 0


@pytest.mark.parametrize("Gm,Gs", [(5, 3), (33, 8), (64, 16), (65, 20), (128, 40)])
@pytest.mark.parametrize("N", [5, 64])
def test_fp32_four_rows_at_a_time_elects_what_one_row_at_a_time_elects(N, Gm, Gs):
    """A population in rows of N nodes, and the same one with empty nodes appended until rows are longer than 64."""
    wl = W.make(W.custom("f32", P=30, J=6, N=N, cap=4, Gm=Gm, Gs=Gs, index=760 + N))
    pad = lambda x: np.concatenate([x, np.zeros(x.shape[:-1] + (68 - N,), x.dtype)], axis=-1)
    short = run_gpu(wl, precision=1)
    c = wl.cfg
    long = W.make(W.custom("f32 long", P=c.P, J=c.J, N=68, cap=4, Gm=Gm, Gs=Gs, index=760 + N), with_population=False)
    long.job_params, long.m_grid, long.fair_share = wl.job_params, wl.m_grid, wl.fair_share
    long.current_alloc, long.population = pad(wl.current_alloc), pad(wl.population)
    long.node_capacity = np.concatenate([wl.node_capacity, np.full(68 - N, 4, np.int32)])
    want = run_gpu(long, precision=1)
    for k in want:
        assert np.array_equal(short[k], want[k], equal_nan=True), k


# either side of every line of split_pairs (candidates in whole fours, grid width, counts, pairs, candidates a wavefront) and of the
# staging of table rows (five candidates a wavefront)
SPLITS = [(12, 7, 5, 64, 16), (13, 7, 5, 64, 16), (12, 700, 5, 64, 16), (13, 615, 8, 50, 16), (13, 616, 8, 50, 16), (16, 499, 5, 65, 16), (16, 500, 5, 65, 16),
          (16, 500, 8, 64, 8), (16, 499, 8, 64, 16), (16, 500, 9, 128, 12), (16, 500, 9, 129, 12), (16, 500, 8, 64, 17), (16, 500, 9, 64, 17),
          (200, 40, 64, 128, 16), (200, 600, 9, 64, 16), (202, 600, 9, 50, 16), (1300, 100, 4, 64, 16), (1510, 100, 4, 64, 8), (1510, 100, 5, 65, 8), (2510, 100, 5, 33, 8),
          (1010, 100, 66, 33, 8), (1260, 100, 66, 33, 8), (1010, 100, 68, 65, 16), (1260, 100, 68, 65, 16), (2010, 100, 68, 65, 16)]


@pytest.mark.parametrize("P,J,N,Gm,Gs", SPLITS)
@pytest.mark.parametrize("precision", [0, 1])
def test_either_side_of_the_lines_of_the_split(P, J, N, Gm, Gs, precision):
    """The same population with empty nodes appended gives the same bits (and fp64 the oracle's results); the children of a
    generation get what a call on the new population gives them, row by row inherited or not."""
    import torch
    import paper_2008_12260_amd as px
    wl = W.make(W.custom("split", P=P, J=J, N=N, cap=4, Gm=Gm, Gs=Gs, index=780 + N))
    wl.population[1, J - 1, 0] = 70                           # beyond the tables
    empty = np.random.default_rng(P + N).random((3, P))       # rows that need no sweep between those that do: some, most, nearly all
    for j, share in enumerate((0.3, 0.7, 0.95)):
        wl.population[empty[j] < share, j] = 0
    wl.population[empty[1] > 0.95, 1, 0] = 66
    c = wl.cfg
    got = run_gpu(wl, precision=precision)
    if precision == 0 and P * J * Gm * Gs <= 2 ** 28:
        assert compare(wl, got, run_oracle(wl)) == 0
    extra = 131 - N
    pad = lambda x: np.concatenate([x, np.zeros(x.shape[:-1] + (extra,), x.dtype)], axis=-1)
    long = W.make(W.custom("split long", P=P, J=J, N=131, cap=4, Gm=Gm, Gs=Gs, index=780 + N), with_population=False)
    long.job_params, long.m_grid, long.fair_share = wl.job_params, wl.m_grid, wl.fair_share
    long.current_alloc, long.population = pad(wl.current_alloc), pad(wl.population)
    long.node_capacity = np.concatenate([wl.node_capacity, np.full(extra, 4, np.int32)])
    want = run_gpu(long, precision=precision)
    for k in want:
        assert np.array_equal(got[k], want[k], equal_nan=True), k
    for inherit in (False, True):
        call = px.FitnessCall(P, J, N, Gm, Gs, wl.job_params, wl.m_grid, wl.fair_share, wl.current_alloc, wl.node_capacity,
                              p=c.p, delta=c.delta, precision=precision)
        pop = torch.as_tensor(wl.population).cuda()
        call.run(pop)
        for g in (1, 2):
            call.generation(pop, 5, g, max(1, P // 3), (1 << 32) // 8, inherit_rows=inherit)
        got_g = call.results()
        want_g = run_gpu(wl, population=pop.cpu().numpy(), precision=precision)
        for k in want_g:
            if k != "status":                                 # (the first call's population had more in it)
                assert np.array_equal(got_g[k], want_g[k], equal_nan=True), (inherit, k)
