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
