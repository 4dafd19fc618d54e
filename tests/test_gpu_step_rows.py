"""The search step on rows of every length and alignment its wide loads cover, and on both sides of the lines between its
instances: bit for bit the oracle's matrices, out of place, in place and with row sources recorded."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("J", [5, 150])
@pytest.mark.parametrize("N", [3, 4, 5, 7, 61, 63, 64, 65, 67, 130, 255, 256, 257])
def test_step_on_rows_of_any_length(N, J, off):
    import torch
    import paper_2008_12260_amd as px
    P, elite = 14, 5
    wl = W.make(W.custom("step", P=P, J=J, N=N, cap=max(4, -(-2 * J // N)), Gm=4, Gs=2, index=1400 + N))
    pop = wl.population.copy()
    pop[6, 0, N - 1] += 40                                    # a node far beyond its capacity
    pop[7, :, :] = np.minimum(pop[7] + 1, 2)                  # a dense matrix: every job on every node
    pop[8, 1, 0] = -2
    fit = np.random.default_rng(N).permutation(P).astype(np.float64)
    dims = px.Dims(P, J, N, 1, 1, 0, 0)
    ws = torch.empty(px.workspace_size(dims), dtype=torch.uint8, device="cuda")
    cap, dfit = torch.as_tensor(wl.node_capacity).cuda(), torch.as_tensor(fit).cuda()

    def moved(x):
        room = torch.full((x.size + 8,), -9, dtype=torch.int32, device="cuda")
        at = room[off:off + x.size].view(x.shape)
        at.copy_(torch.as_tensor(x))
        return room, at
    for mut in (1 << 28, 1 << 31):
        room, parents = moved(pop)
        out, kids = moved(np.zeros_like(pop))
        px.pollux_ga_step(dims, parents, dfit, cap, px.GaParams(77, 3, elite, mut, 0, None), ws, kids)
        want = O.ga_step(pop, fit, wl.node_capacity, 77, 3, elite, mut)
        assert np.array_equal(kids.cpu().numpy(), want)
        # nothing around the matrices is written
        assert bool((out[:off] == -9).all()) and bool((out[off + pop.size:] == -9).all())
        px.pollux_ga_step(dims, parents, dfit, cap, px.GaParams(77, 3, elite, mut, px.PX_GA_IN_PLACE, None), ws, parents)
        want = O.ga_step(pop, fit, wl.node_capacity, 77, 3, elite, mut, flags=O.GA_IN_PLACE)
        assert np.array_equal(parents.cpu().numpy(), want)
        assert bool((room[:off] == -9).all()) and bool((room[off + pop.size:] == -9).all())
