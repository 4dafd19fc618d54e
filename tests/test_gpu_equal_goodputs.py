"""Jobs whose batch sizes tie.  With alpha_grad = 0 and gamma = 1 (both bounds of the fit) the goodput depends on the total batch size
alone, so batch sizes with a common multiple agree to the last places and rounding elects one of them: the sweeps (one candidate at a
time, four, with rows copied on chip), small calls, memoised rows and fair shares have to round alike, whatever the number of counts."""
from fractions import Fraction

import numpy as np
import pytest

import workloads as W
from parity import run_oracle

pytestmark = pytest.mark.gpu
KEYS = ("fitness", "violations", "best_m", "best_s", "best_goodput", "speedup")


def workload(P, J, N, Gm, Gs, first):
    wl = W.make(W.custom("ties", P=9, J=J, N=N, cap=max(4, -(-8 * J // N)), Gm=Gm, Gs=Gs, index=2600 + N))
    jp, row, rng = wl.job_params, W.PARAM_INDEX, np.random.default_rng(Gm + Gs)
    jp[row["alpha_grad"]], jp[row["gamma"]] = 0.0, 1.0
    jp[row["M0"]], jp[row["M_max"]] = 32.0, 32.0 * rng.choice([32, 256, 2048], J)
    jp[row["phi"]] = 10.0 ** rng.uniform(2.0, 5.0, J)
    wl.m_grid[:] = np.arange(first, first + Gm)              # consecutive: the most common multiples
    pop = np.zeros((P, J, N), np.int32)
    for c in range(P):                                       # 2 to 30 GPUs a job, on one node, two or many
        K = rng.integers(2, 31, J)
        for j in range(J):
            nodes = min(N, K[j], [1, 2, 5][(c + j) % 3])
            pop[c, j, :nodes] = 1
            pop[c, j, 0] += K[j] - nodes
    wl.fair_share[:, 0], wl.fair_share[:, 1] = pop[0].sum(1), (pop[0] > 0).sum(1)
    return wl, pop


def results(wl, pop, flags=0, precision=0, keep=False):
    import torch
    import paper_2008_12260_amd as px
    c = wl.cfg
    call = px.FitnessCall(pop.shape[0], c.J, c.N, c.Gm, c.Gs, wl.job_params, wl.m_grid, wl.fair_share, pop[0], np.full(c.N, 40, np.int32),
                          p=c.p, delta=c.delta, flags=flags, precision=precision)
    for _ in range(2 if keep else 1):
        call.run(torch.as_tensor(pop).cuda(), keep_job_tables=_ == 1)
    return call.results()


@pytest.mark.parametrize("P,J,N,Gm,Gs,first", [
    (40, 200, 16, 64, 16, 8), (40, 200, 16, 50, 24, 8), (40, 200, 16, 64, 32, 8), (17, 200, 130, 64, 64, 8), (17, 200, 130, 64, 300, 2),
    (17, 200, 130, 130, 32, 4), (2000, 40, 128, 128, 32, 4), (2000, 40, 130, 100, 32, 4), (2000, 40, 64, 64, 32, 8), (9, 40, 3, 64, 33, 4),
    (200, 16, 9, 32, 32, 6), (200, 15, 9, 31, 24, 4), (200, 16, 9, 64, 16, 8), (200, 8, 9, 128, 24, 4), (200, 4, 9, 256, 32, 2)])
def test_every_way_elects_the_same_batch_size(P, J, N, Gm, Gs, first):
    import paper_2008_12260_amd as px
    wl, pop = workload(P, J, N, Gm, Gs, first)
    got, memo = results(wl, pop), results(wl, pop, px.PX_FLAG_MEMOISE)
    for k in KEYS:
        assert np.array_equal(got[k], memo[k]), (k, int(np.sum(got[k] != memo[k])))
    assert np.array_equal(got["speedup"][0], np.where(got["best_goodput"][0] > 0.0, 1.0, 0.0))       # row 0 is the fair share
    kept = results(wl, pop, keep=True)
    for k in KEYS:
        assert np.array_equal(got[k], kept[k]), k
    wl.node_capacity[:] = 40
    some = pop[:9]
    ref = run_oracle(wl, population=some, current=pop[0])
    for k in ("best_goodput", "speedup"):
        assert np.max(np.abs(got[k][:9] - ref[k]) / np.where(ref[k] == 0, 1.0, ref[k])) <= 1e-12, k


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("J,N,Gm,Gs", [(60, 16, 64, 32), (60, 61, 64, 16), (60, 130, 100, 32), (200, 16, 64, 16), (15, 9, 32, 32)])
def test_children_are_elected_alike(J, N, Gm, Gs, precision):
    """The same search in which children are swept, in which only their changed rows are, and memoised."""
    import torch
    import paper_2008_12260_amd as px
    wl, pop = workload(96, J, N, Gm, Gs, 6)
    c, got = wl.cfg, []
    for flags, inherit in ((0, False), (0, True), (px.PX_FLAG_MEMOISE | px.PX_FLAG_PAIR_RESULTS, False)):
        call = px.FitnessCall(96, c.J, N, Gm, Gs, wl.job_params, wl.m_grid, wl.fair_share, pop[0], np.full(N, 40, np.int32), p=c.p,
                              delta=c.delta, flags=flags, precision=precision)
        matrices = torch.as_tensor(pop).cuda()
        call.run(matrices)
        for g in range(4):
            call.generation(matrices, 77, g, 32, (1 << 32) // 16, inherit_rows=inherit)
        got.append((matrices.cpu().numpy(), call.results()))
    assert np.any(got[0][0] != pop)
    for matrices, results_of in got[1:]:
        assert np.array_equal(matrices, got[0][0])
        for k in KEYS:
            assert np.array_equal(results_of[k], got[0][1][k]), k


@pytest.mark.parametrize("P,J,N,Gm,Gs", [(40, 200, 16, 64, 16), (40, 200, 16, 100, 32), (17, 200, 130, 128, 32), (17, 200, 130, 130, 64)])
def test_batch_sizes_a_millionth_apart_are_told_apart(P, J, N, Gm, Gs):
    """Long consecutive batch sizes around a job's best one: their goodputs agree to six places and more, but do not tie."""
    import paper_2008_12260_amd as px
    wl, pop = workload(P, J, N, Gm, Gs, 2000)
    jp, row, rng = wl.job_params, W.PARAM_INDEX, np.random.default_rng(7)
    a, b, t = rng.uniform(0.01, 0.2, J), rng.uniform(1e-5, 1e-4, J), rng.uniform(0.005, 0.05, J)
    pop[::2] = pop[0]
    # without accumulation, T = a + b m + t and phi so that (a + t + b m) (1 + phi / (K m)) is least within the grid, for candidate 0
    jp[row["alpha_grad"]], jp[row["beta_grad"]], jp[row["gamma"]], jp[row["M_max"]] = a, b, 1.0, 2.0 ** 40
    for name in ("alpha_sync_local", "alpha_sync_node", "beta_sync_local", "beta_sync_node"):
        jp[row[name]] = t if name.startswith("alpha") else 0.0
    jp[row["phi"]] = (2000 + rng.uniform(0.1, 0.9, J) * Gm) ** 2 * pop[0].sum(1) * b / (a + t)
    got, memo = results(wl, pop), results(wl, pop, px.PX_FLAG_MEMOISE)
    inside = (got["best_m"] > 2000) & (got["best_m"] < 1999 + Gm)
    assert inside.sum() > 0.4 * inside.size
    for k in KEYS:
        assert np.array_equal(got[k], memo[k]), (k, int(np.sum(got[k] != memo[k])))
    wl.node_capacity[:] = 40
    ref = run_oracle(wl, population=pop[:9], current=pop[0])
    assert np.array_equal(got["best_m"][:9], ref["best_m"]) and np.array_equal(got["best_s"][:9], ref["best_s"])


def single(x):
    """A fraction rounded to single precision (values far from underflow)."""
    if x == 0:
        return x
    e = x.numerator.bit_length() - x.denominator.bit_length()
    while Fraction(2) ** e > x:
        e -= 1
    while Fraction(2) ** (e + 1) <= x:
        e += 1
    return Fraction(round(x * Fraction(2) ** (23 - e))) / Fraction(2) ** (23 - e)


def elected(phi, ts, beta, K, sizes, M0, M_max, Gs):
    """(m, s) of the smallest h = fma(T_grad, fma(C, 1 / (s + 1), s), A0), every operation rounded to single precision; equal values to
    the first batch size.  K, the sizes and beta are powers of two, so the reciprocals 1 / (K m) and 1 / T_grad are exact."""
    best = None
    for m in sizes:
        tg = beta * m
        last = single(tg + ts)
        u = single(phi / (K * m))
        A0, C = single(u * tg + last), single(single(last - tg) * u) / tg
        assert C == single(C)
        s_lo, s_hi = max(0, -(-M0 // (K * m)) - 1), min(Gs - 1, M_max // (K * m) - 1)
        if s_lo > s_hi:
            continue
        t = 0
        while t < s_hi and C > (t + 1) * (t + 2):
            t += 1
        s = max(t, s_lo)
        h = single(tg * single(C * single(Fraction(1, s + 1)) + s) + A0)
        if best is None or h < best[0]:
            best = (h, m, s)
    return best[1:] if best else (-1, -1)


@pytest.mark.parametrize("P,J,N,Gm,Gs,memo", [
    (8, 120, 16, 7, 64, False), (48, 120, 16, 50, 33, False), (48, 120, 64, 64, 300, False), (8, 120, 130, 130, 32, False),
    (48, 120, 128, 128, 64, False), (8, 120, 16, 130, 64, True), (8, 120, 3, 64, 48, False), (8, 120, 16, 64, 16, False)])
def test_single_precision_elects_by_one_rounding_of_h(P, J, N, Gm, Gs, memo):
    import paper_2008_12260_amd as px
    wl = W.make(W.custom("ties", P=8, J=J, N=N, cap=16, Gm=Gm, Gs=Gs, index=2700 + N))
    jp, row, rng = wl.job_params, W.PARAM_INDEX, np.random.default_rng(Gm + Gs)
    jp[row["alpha_grad"]], jp[row["gamma"]], jp[row["beta_grad"]] = 0.0, 1.0, 2.0 ** -14
    jp[row["beta_sync_local"]], jp[row["beta_sync_node"]] = 0.0, 0.0
    for name, lo, hi in (("alpha_sync_local", 0.005, 0.05), ("alpha_sync_node", 0.02, 0.2), ("phi", 1e2, 1e5)):
        jp[row[name]] = np.exp(rng.uniform(np.log(lo), np.log(hi), J)).astype(np.float32)
    jp[row["M0"]], jp[row["M_max"]] = 32.0, 32.0 * rng.choice([32, 256, 2048], J)
    sizes = [2, 4, 8, 16, 32, 64, 128]
    at = np.sort(rng.choice(Gm, 7, replace=False))           # the others are too large for any job
    wl.m_grid[:] = 1 << 20
    wl.m_grid[:, at] = sizes
    pop = np.zeros((P, J, N), np.int32)
    for c in range(P):
        pop[c, :, 0] = 2 ** (1 + c % 4)
        if (c // 4) % 2:
            pop[c, :, 0] //= 2
            pop[c, :, 1] = pop[c, :, 0]
    wl.fair_share[:, 0], wl.fair_share[:, 1] = pop[0].sum(1), 1
    got = results(wl, pop, flags=px.PX_FLAG_MEMOISE if memo else 0, precision=1)
    for c in range(min(P, 8)):
        nodes = 1 + (c // 4) % 2
        for j in range(J):
            ts = jp[row["alpha_sync_local" if nodes == 1 else "alpha_sync_node"], j]
            want = elected(Fraction(jp[row["phi"], j]), Fraction(ts), Fraction(1, 2 ** 14), 2 ** (1 + c % 4), sizes, 32,
                           int(jp[row["M_max"], j]), Gs)
            assert (got["best_m"][c, j], got["best_s"][c, j]) == want, (c, j)
    for k in ("best_m", "best_s", "best_goodput"):
        assert np.array_equal(got[k], got[k][np.arange(P) % 8]), k
    assert np.array_equal(got["speedup"][0], np.where(got["best_goodput"][0] > 0.0, 1.0, 0.0))
