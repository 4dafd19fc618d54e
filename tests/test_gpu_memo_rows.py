"""The memoised population pass over rows of every length and alignment one 16-byte load per lane can cover, and of its
neighbours that take the other path: identical to the plain call, children of a generation included."""
import numpy as np
import pytest

import workloads as W
from parity import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu
MEMO, SAMPLE, PAIRS = 4, 16, 32
NAMES = ("fitness", "violations", "best_m", "best_s", "best_goodput", "speedup")


def spoiled(wl, seed):
    """Matrices with rows beyond the memo table, a negative entry, a one-node row beyond any node, an empty row."""
    pop = wl.population.copy()
    rng = np.random.default_rng(seed)
    P, J, N = pop.shape
    pop[1, rng.integers(J), rng.integers(N)] += 90
    pop[2, rng.integers(J), N - 1] = -2
    pop[3, rng.integers(J)] = 0
    pop[3, rng.integers(J), 0] = 9
    pop[0] = wl.current_alloc
    return pop


@pytest.mark.parametrize("N", [1, 3, 4, 5, 6, 63, 64, 65, 67, 130, 253, 255, 256, 257])
def test_rows_of_any_length(N):
    wl = W.make(W.custom("rows", P=7, J=11, N=N, cap=4, Gm=33, Gs=9, index=200 + N))
    pop = spoiled(wl, N)
    plain, memo = run_gpu(wl, population=pop), run_gpu(wl, population=pop, flags=MEMO)
    assert compare(wl, memo, run_oracle(wl, population=pop), population=pop) == 0
    for k in NAMES + ("status",):
        assert np.array_equal(plain[k], memo[k], equal_nan=True), k


@pytest.mark.parametrize("P,J", [(4, 1), (4, 63), (4, 64), (4, 255), (4, 257), (256, 70), (257, 70), (4, 1025), (4, 1300)])
@pytest.mark.parametrize("N", [6, 70])
def test_more_jobs_than_a_chunk_of_the_pass_and_few_candidates(P, J, N):
    wl = W.make(W.custom("chunks", P=P, J=J, N=N, cap=max(4, -(-J // N)), Gm=8, Gs=4, index=300 + J))
    plain, memo = run_gpu(wl), run_gpu(wl, flags=MEMO)
    for k in NAMES + ("status",):
        assert np.array_equal(plain[k], memo[k], equal_nan=True), k


@pytest.mark.parametrize("kind", [dict(precision=1), dict(flags=SAMPLE)])
@pytest.mark.parametrize("N", [7, 66])
def test_other_precisions_and_the_sampling_argmax(kind, N):
    wl = W.make(W.custom("kinds", P=7, J=13, N=N, cap=4, Gm=33, Gs=9, index=400 + N))
    if kind.get("flags"):
        wl = W.sampled(wl)
    pop = spoiled(wl, N)
    flags = kind.get("flags", 0)
    plain = run_gpu(wl, population=pop, flags=flags, precision=kind.get("precision", 0))
    memo = run_gpu(wl, population=pop, flags=flags | MEMO, precision=kind.get("precision", 0))
    for k in NAMES + ("status",):
        assert np.array_equal(plain[k], memo[k], equal_nan=True), k


@pytest.mark.parametrize("kind", [dict(), dict(precision=1), dict(flags=SAMPLE)])
@pytest.mark.parametrize("P,J,N", [(7, 63, 7), (7, 64, 7), (9, 67, 66), (256, 64, 5), (257, 64, 5), (5, 1090, 64), (5, 1029, 70)])
@pytest.mark.parametrize("kept", [0, PAIRS])
def test_sixteen_wavefronts_a_candidate(P, J, N, kind, kept):
    """Few candidates of 64 jobs and more, and their neighbours: rows beyond the table, negative entries, empty rows, in every
    kind of call, the per-pair results left or not."""
    wl = W.make(W.custom("few", P=P, J=J, N=N, cap=max(4, -(-2 * J // N)), Gm=17, Gs=5, index=450 + J))
    flags, precision = kind.get("flags", 0), kind.get("precision", 0)
    if flags:
        wl = W.sampled(wl)
    pop = spoiled(wl, J)
    rng = np.random.default_rng(J)
    for c in range(P):                                        # in the first rows, the last, and between, whichever wavefront has them
        for j in {0, J - 1, int(rng.integers(J))}:
            pop[c, j] = 0
            pop[c, j, rng.integers(N)] = rng.choice([0, 3, 65, 70])
    if P > 5:
        pop[P - 1, J - 1, N - 1] = -1
    memo = run_gpu(wl, population=pop, flags=flags | MEMO | kept, precision=precision)
    if precision == 0:
        assert compare(wl, memo, run_oracle(wl, population=pop, flags=flags), population=pop, sampled=bool(flags)) == 0
    if not (flags and P >= 128):                              # (sampling calls of that size take the same pass either way)
        plain = run_gpu(wl, population=pop, flags=flags, precision=precision)
        for k in NAMES + ("status",):
            assert np.array_equal(plain[k], memo[k], equal_nan=True), k


@pytest.mark.parametrize("kind", [dict(), dict(precision=1), dict(flags=SAMPLE)])
@pytest.mark.parametrize("J,N,off", [(9, 4, 0), (30, 5, 1), (40, 64, 0), (40, 67, 3), (1030, 6, 0)])
def test_children_that_inherit_rows(J, N, off, kind):
    """Generations that look changed rows up leave what the plain call on the same matrices leaves, misaligned buffers too."""
    import torch
    import paper_2008_12260_amd as px
    wl = W.make(W.custom("heirs", P=12, J=J, N=N, cap=max(4, -(-2 * J // N)), Gm=16, Gs=8, index=500 + J))
    flags, precision = kind.get("flags", 0), kind.get("precision", 0)
    if flags:
        wl = W.sampled(wl)
    c = wl.cfg
    make = lambda f: px.FitnessCall(c.P, J, N, c.Gm, c.Gs, wl.job_params, wl.m_grid, wl.fair_share, wl.current_alloc,
                                    wl.node_capacity, p=c.p, delta=c.delta, flags=flags | f, precision=precision)
    call, check = make(MEMO | PAIRS), make(0)
    start = wl.population.copy()
    start[5, 0, 0] = -1                                       # its children cannot be taken for granted
    room = torch.zeros(start.size + 4, dtype=torch.int32, device="cuda")
    pop = room[off:off + start.size].view(start.shape)
    pop.copy_(torch.as_tensor(start))
    call.run(pop)
    for g in range(4):
        call.generation(pop, 77, g, 5, 1 << 30, inherit_rows=True)
        check.run(pop)
        got, want = call.results(), check.results()
        for k in NAMES:
            assert np.array_equal(got[k], want[k], equal_nan=True), (g, k)
