"""GPU parity of what a call derives from the jobs alone: table rows, fair shares and memoised rows at the sizes where the
number of rows per wavefront, the groups of 64 batch sizes and the tabled GPU counts end, and the argmaxes found in place."""
import numpy as np
import pytest

import oracle.loop as LP
import workloads as W
from parity import RTOL, compare, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, 4])                    # plain, memoised
@pytest.mark.parametrize("J,Gm,Gs", [(1, 1, 1), (127, 64, 17), (128, 65, 16), (129, 130, 33), (40, 63, 300)])
def test_job_level_results_at_the_edges_of_their_launch(J, Gm, Gs, flags):
    wl = W.make(W.custom("edges", P=3, J=J, N=9, cap=70, Gm=Gm, Gs=Gs, phi_hi=1e7))
    rng = np.random.default_rng(J + Gs)
    # fair shares on both sides of the tables' end (64 GPUs), on one node and on several, one node beyond its capacity too
    wl.fair_share[:, 0] = rng.choice([1, 2, 63, 64, 65, 71, 300], J)
    wl.fair_share[:, 1] = rng.choice([1, 2], J)
    wl.param("gamma")[::5] = 1.0
    wl.param("alpha_sync_node")[::7] = 0.0
    wl.param("beta_sync_node")[::7] = 0.0
    wl.param("M_max")[::3] = 1e9                             # every accumulation count feasible
    assert compare(wl, run_gpu(wl, flags=flags), run_oracle(wl)) == 0


@pytest.mark.parametrize("Gm,Gs", [(1, 1), (64, 8), (65, 257), (130, 1000)])
def test_goodput_per_gpu_on_grids_of_any_size(Gm, Gs):
    import torch
    import paper_2008_12260_amd as px
    wl = W.make(W.custom("queries", P=1, J=5, N=4, cap=8, Gm=Gm, Gs=Gs, phi_hi=1e7), with_population=False)
    wl.param("M_max")[::2] = 1e9
    dims = px.Dims(1, 5, 1, Gm, Gs, 0, 0)
    out = torch.empty((5, 13), dtype=torch.float64, device="cuda")
    ws = torch.empty(px.workspace_size(dims), dtype=torch.uint8, device="cuda")
    px.pollux_goodput_per_gpu(dims, torch.as_tensor(wl.job_params).cuda(), torch.as_tensor(wl.m_grid).cuda(), 8, 12, ws, out)
    want = LP.goodput_per_gpu(wl.job_params, wl.m_grid, Gs, 8, 12)
    assert rel_err(out.cpu().numpy(), want).max() <= RTOL


@pytest.mark.parametrize("precision", [0, 1])
def test_every_job_is_prepared_beside_many_counters(precision):
    """72 jobs need 1176 workgroups, the counters of 22000 candidates on 256 nodes would like 1375: copies of four candidates
    get the four's results, those of the last jobs too."""
    import torch
    import paper_2008_12260_amd as px
    wl = W.make(W.custom("many", P=4, J=72, N=256, cap=4, Gm=5, Gs=3, index=130))
    want = run_gpu(wl, precision=precision)
    if precision == 0:
        assert compare(wl, want, run_oracle(wl)) == 0
    c, copies = wl.cfg, 5500
    call = px.FitnessCall(4 * copies, c.J, c.N, c.Gm, c.Gs, wl.job_params, wl.m_grid, wl.fair_share, wl.current_alloc, wl.node_capacity,
                          p=c.p, delta=c.delta, precision=precision)
    call.run(torch.as_tensor(wl.population).cuda().repeat(copies, 1, 1))
    got = call.results()
    assert got.pop("status") == want.pop("status")
    for k, v in want.items():
        assert np.array_equal(got[k], np.tile(v, (copies,) + (1,) * (v.ndim - 1)), equal_nan=True), k
