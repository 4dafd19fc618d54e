"""Goodput per GPU of many jobs at once, where a wavefront takes several queries of a job: bit for bit what the same jobs give a
hundred at a time, a wavefront a query (which the oracle checks in test_gpu_loop.py)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("J,max_nodes,Gm,Gs", [(1000, 24, 64, 16), (1000, 24, 33, 8), (997, 6, 128, 32), (600, 9, 65, 17), (500, 16, 130, 9),
                                               (3000, 1, 64, 8), (5000, 3, 20, 4)])
def test_many_queries_are_the_few(J, max_nodes, Gm, Gs):
    import torch
    import paper_2008_12260_amd as px
    wl = W.make(W.custom("queries", P=1, J=J, N=2 * J, cap=8, Gm=Gm, Gs=Gs, index=2500 + Gm), with_population=False)
    params = torch.as_tensor(wl.job_params).cuda()
    params[W.PARAM_INDEX["phi"]] *= 10.0 ** (torch.arange(J, device="cuda") % 5)
    grid = torch.as_tensor(wl.m_grid).cuda()
    grid[::3, : Gm // 2] = grid[::3, :1]                     # equal batch sizes

    def query(first, last):
        n = last - first
        dims = px.Dims(1, n, 1, Gm, Gs, 0, 0)
        out = torch.full((n, max_nodes + 1), -1.0, dtype=torch.float64, device="cuda")
        px.pollux_goodput_per_gpu(dims, params[:, first:last].contiguous(), grid[first:last].contiguous(), 8, max_nodes,
                                  torch.empty(px.workspace_size(dims), dtype=torch.uint8, device="cuda"), out)
        return out

    got = query(0, J).cpu().numpy()
    want = torch.cat([query(j, min(j + 100, J)) for j in range(0, J, 100)]).cpu().numpy()
    assert np.all(want >= 0.0) and np.any(want > 0.0)
    assert np.array_equal(got, want)
