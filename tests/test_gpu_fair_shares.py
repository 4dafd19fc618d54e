"""Fair shares in single precision, found beside the tables (up to 32 counts) or from them (more): inside the tables and beyond, on one
node and several, at the edges of groups of batch sizes and of chunks of counts."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Gs", [1, 8, 16, 17, 32, 33])
@pytest.mark.parametrize("Gm", [1, 63, 64, 65, 130])
def test_fair_shares_in_single_precision(Gm, Gs):
    import torch
    import paper_2008_12260_amd as px
    shares = [(1, 1), (2, 1), (2, 2), (7, 1), (8, 1), (9, 1), (63, 8), (64, 8), (65, 9), (200, 25), (64, 1)]    # 8 GPUs a node
    J = len(shares)
    wl = W.make(W.custom("shares", P=6, J=J, N=16, cap=8, Gm=Gm, Gs=Gs, index=1900 + Gm + Gs))
    c, fair = wl.cfg, np.array(shares, dtype=np.int32)
    ref = O.fitness(wl.population, wl.job_params, wl.m_grid, fair, wl.current_alloc, wl.node_capacity, c.p, c.delta, c.Gs)
    for flags in (0, px.PX_FLAG_MEMOISE):
        call = px.FitnessCall(c.P, c.J, c.N, c.Gm, c.Gs, wl.job_params, wl.m_grid, fair, wl.current_alloc, wl.node_capacity, p=c.p,
                              delta=c.delta, flags=flags, precision=1)
        call.run(torch.as_tensor(wl.population).cuda())
        got = call.results()
        assert got["status"] == ref["status"]
        for k in ("best_goodput", "speedup", "fitness"):
            # about 30 roundings of 2^-24 in a speedup, the sums of 11 jobs' terms in the fitness
            err = np.abs(got[k] - ref[k]) / np.where(ref[k] == 0, 1.0, np.abs(ref[k]))
            assert err.max() <= 1e-5, (k, flags)
