"""Generations of memoised searches that inherit rows, on both sides of the lines between the kernel that forms a child and goes on
to its fitness and the separate launches: the matrices of a search without inherited rows, and, bit for bit, the results a full
evaluation of the final population gives."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
SEED = 0x5EED1234


@pytest.mark.parametrize("kind", ["grid", "f32", "sampled"])
@pytest.mark.parametrize("J,N", [(1, 4), (3, 5), (63, 64), (64, 16), (65, 61), (255, 64), (257, 64), (513, 64), (1023, 63), (1024, 64),
                                 (1025, 64), (65, 65), (40, 3)])
def test_children_formed_and_evaluated(J, N, kind):
    import torch
    import paper_2008_12260_amd as px
    P, elite = 13, 5
    wl = W.make(W.custom("children", P=P, J=J, N=N, cap=max(4, -(-2 * J // N)), Gm=20, Gs=5, index=1700 + J + N))
    flags = px.PX_FLAG_MEMOISE | px.PX_FLAG_PAIR_RESULTS
    if kind == "sampled":
        wl, flags = W.sampled(wl), flags | px.PX_FLAG_SAMPLE_M
    c = wl.cfg
    pop = wl.population.copy()
    pop[6, 0, N - 1] += 40                                    # a node far beyond its capacity
    pop[7, :, :] = np.minimum(pop[7] + 1, 2)                  # a dense matrix: every job on every node
    pop[8, J - 1, 0] = -2                                     # (its status bit is compared too)
    call = [px.FitnessCall(P, J, N, c.Gm, c.Gs, wl.job_params, wl.m_grid, wl.fair_share, wl.current_alloc, wl.node_capacity,
                           p=c.p, delta=c.delta, flags=flags, precision=int(kind == "f32")) for _ in range(2)]
    dev = [torch.as_tensor(pop).cuda() for _ in range(2)]
    for x, d in zip(call, dev):
        x.run(d)
        x.fitness[6:9] = 9.0                                  # survivors, so that their rows reach the children
    for gen in range(4):
        for mut in (1 << 29, (1 << 32) - 1) if gen == 3 else (1 << 29,):
            for x, d, inherit in zip(call, dev, (True, False)):
                x.generation(d, SEED, gen, elite, mut, inherit_rows=inherit)
            assert torch.equal(dev[0], dev[1]), gen
    got, plain = call[0].results(), call[1].results()
    for k in got:
        assert np.array_equal(got[k], plain[k], equal_nan=True), k
    call[0].run(dev[0], keep_job_tables=True)
    full = call[0].results()
    kids = np.flatnonzero(got["fitness"] != 9.0)              # (the fitness given above is not theirs)
    for k in ("fitness", "best_m", "best_s", "best_goodput", "speedup", "violations"):
        assert np.array_equal(got[k][kids], full[k][kids], equal_nan=True), k
