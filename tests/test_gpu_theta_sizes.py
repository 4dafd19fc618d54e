"""The fit at the record counts where its lanes, quarters of a wavefront and launch instances end: the instance for at most 64
record slots and the one for more give the same bits, and both report the oracle's error."""
import numpy as np
import pytest

import oracle.theta as TH
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_starts", [1, 2, 3, 5])
@pytest.mark.parametrize("counts", [[1], [2, 15, 16, 17], [31, 32, 33, 47, 48, 49], [63, 64, 1]])
def test_records_in_registers_and_in_memory(counts, n_starts):
    import paper_2008_12260_amd as px
    J = len(counts)
    ob = W.observations(W.custom("records", P=1, J=J, N=4, cap=4, Gm=8, Gs=4, index=800 + counts[0]), max_obs=64)
    rng = np.random.default_rng(counts[0])
    for j, n in enumerate(counts):                     # every slot a real record, however many the generator drew
        have = int(ob["count"][j])
        for k in ("K", "nodes", "m", "s", "T"):
            ob[k][j, have:] = ob[k][j, rng.integers(0, have, 64 - have)]
        ob["count"][j] = n
    held = px.fit_theta(ob, n_starts=n_starts)
    wider = {k: (v if k == "count" else np.concatenate([v, np.ones((J, 7), v.dtype)], axis=1)) for k, v in ob.items()}
    read = px.fit_theta(wider, n_starts=n_starts)
    for k in held:
        assert np.array_equal(held[k], read[k]), k
    for j, n in enumerate(counts):
        rec = tuple(ob[k][j, :n] for k in ("K", "nodes", "m", "s", "T"))
        want = TH.rmsle(held["theta"][:, j], *rec)
        assert abs(held["rmsle"][j] - want) <= 1e-12 * want + 1e-13     # residuals are differences of logarithms of size 1
        assert np.all(held["theta"][:6, j] >= 0.0) and 1.0 <= held["theta"][6, j] <= 10.0


@pytest.mark.parametrize("n_starts", [1, 3])
@pytest.mark.parametrize("counts", [[65, 64, 63, 127], [128, 129, 1, 200]])
def test_more_records_than_lanes(counts, n_starts):
    """The record a lane keeps and those it reads: the oracle's error, and the same bits however many slots the arrays have."""
    import paper_2008_12260_amd as px
    J = len(counts)
    ob = W.observations(W.custom("records", P=1, J=J, N=4, cap=4, Gm=8, Gs=4, index=820 + counts[0]), max_obs=200)
    rng = np.random.default_rng(counts[0])
    for j, n in enumerate(counts):
        have = int(ob["count"][j])
        for k in ("K", "nodes", "m", "s", "T"):
            ob[k][j, have:] = ob[k][j, rng.integers(0, have, 200 - have)]
        ob["count"][j] = n
    got = px.fit_theta(ob, n_starts=n_starts)
    wider = {k: (v if k == "count" else np.concatenate([v, np.ones((J, 57), v.dtype)], axis=1)) for k, v in ob.items()}
    again = px.fit_theta(wider, n_starts=n_starts)
    for k in got:
        assert np.array_equal(got[k], again[k]), k
    for j, n in enumerate(counts):
        want = TH.rmsle(got["theta"][:, j], *(ob[k][j, :n] for k in ("K", "nodes", "m", "s", "T")))
        assert abs(got["rmsle"][j] - want) <= 1e-12 * want + 1e-13


@pytest.mark.parametrize("slots", [64, 71])
@pytest.mark.parametrize("n_starts", [1, 3, 5])
def test_a_job_without_a_usable_time_does_not_touch_the_others(n_starts, slots):
    """Times that are all infinite, NaN, zero or negative: the call ends, and every other job is fitted as without them."""
    import paper_2008_12260_amd as px
    J = 9
    ob = W.observations(W.custom("records", P=1, J=J, N=4, cap=4, Gm=8, Gs=4, index=830), max_obs=slots)
    want = px.fit_theta(ob, n_starts=n_starts)
    bad = {1: np.inf, 3: np.nan, 5: -1.0, 6: 0.0, J - 1: np.inf}
    for j, value in bad.items():
        ob["T"][j] = value
    ob["count"][J - 1] = slots
    got = px.fit_theta(ob, n_starts=n_starts)
    good = [j for j in range(J) if j not in bad]
    for k in want:
        assert np.array_equal(want[k][..., good], got[k][..., good]), k


@pytest.mark.parametrize("slots", [64, 71])
@pytest.mark.parametrize("n_starts", [1, 3, 5])
def test_parameters_that_no_record_feels(n_starts, slots):
    """Jobs seen on one GPU only, on two GPUs of one node only, on one node, on several nodes only: their normal equations have
    rows and columns of zeros.  Both instances give the same bits, the oracle's error, and zero where nothing was explored."""
    import paper_2008_12260_amd as px
    J = 6
    ob = W.observations(W.custom("records", P=1, J=J, N=4, cap=4, Gm=8, Gs=4, index=840), max_obs=64)
    seen = [(1, 1), (2, 1), (4, 1), (2, 2), (8, 2), (64, 16)]              # (GPUs, nodes) of every record of the job
    for j, (K, nodes) in enumerate(seen):
        ob["K"][j], ob["nodes"][j] = K, nodes
    wide = {k: (v if k == "count" else np.concatenate([v, np.ones((J, slots - 64), v.dtype)], axis=1)) for k, v in ob.items()}
    got = px.fit_theta(wide, n_starts=n_starts)
    want = px.fit_theta(ob, n_starts=n_starts)
    for k in got:
        assert np.array_equal(got[k], want[k]), k
    theta = got["theta"]
    assert np.all(theta[2:6, 0] == 0.0)                                    # never more than one GPU
    assert np.all(theta[4:6, 1:3] == 0.0)                                  # never more than one node
    for j in range(J):
        n = int(ob["count"][j])
        error = TH.rmsle(theta[:, j], *(ob[k][j, :n] for k in ("K", "nodes", "m", "s", "T")))
        assert abs(got["rmsle"][j] - error) <= 1e-12 * error + 1e-13       # as above: differences of logarithms of size 1


def cholesky_solve(A, b):
    """x with A x = b, by the textbook's factorisation: no entry is compared with the others, so that a pivot of 1e-303 is one."""
    n, w, y = len(b), A.copy(), b.copy()
    L, inv, x = np.zeros((n, n)), np.zeros(n), np.zeros(n)
    for k in range(n):
        assert w[k, k] > 0.0
        inv[k] = 1.0 / np.sqrt(w[k, k])
        L[:, k] = w[:, k] * inv[k]
        y[k] *= inv[k]
        y[k + 1:] -= L[k + 1:, k] * y[k]
        w[:, k + 1:] -= np.outer(L[:, k], L[k + 1:, k])
    for i in range(n - 1, -1, -1):
        x[i] = (y[i] - L[i + 1:, i] @ x[i + 1:]) * inv[i]
    return x


def test_a_parameter_whose_derivative_is_tiny_is_not_one_that_no_record_feels():
    """The local pair at 1e-18 of what it should be and gamma = 10: the squares of the pair's derivatives underflow, their products
    with the residuals do not.  The damped step, (A + lambda diag(max(A_ii, 1e-300))) x = -g, is then some 1e100 long in the pair; where
    it leads up, twenty trials at lambda = 1e-3, 5e-3 .. are rejected, and the fit ends where it began.  (With a pivot of one for the
    pair a step of the others is accepted among them.)"""
    import paper_2008_12260_amd as px
    rng = np.random.default_rng(31)
    base = np.array([0.1, 0.001, 0.05, 0.01, 0.2, 0.02, 2.0])
    J, n, steps = 12, 40, 20
    names = ("K", "nodes", "m", "s", "T")
    ob = dict(count=np.full(J, n, np.int32), **{k: np.zeros((J, n), np.int32) for k in names[:4]}, T=np.zeros((J, n)))
    init, stays = np.zeros((7, J)), []
    for j in range(J):
        truth = base * np.exp(0.4 * rng.standard_normal(7))
        truth[TH.GAMMA] = rng.uniform(1.2, 6.0)
        K = rng.integers(1, 17, n)
        K[:3] = 4
        nodes = np.where(rng.uniform(size=n) < 0.7, -(-K // 4), np.minimum(K, rng.integers(1, 5, n)))
        nodes[:3] = 1
        m, s = rng.choice([8, 16, 32, 64, 128, 256], n), rng.integers(0, 4, n)
        for k, v in zip(names, (K, nodes, m, s, TH.t_iter(truth, K, nodes, m, s)[0])):
            ob[k][j] = v
        init[:, j] = truth
        init[[TH.ALPHA_SL, TH.BETA_SL], j] *= 1e-18
        init[TH.GAMMA, j] = 10.0
        records = [ob[k][j] for k in names]
        r, jac = TH.residuals_and_jacobian(init[:, j], *records)
        d = jac * np.where(np.arange(7) == TH.GAMMA, 1.0, init[:, j])         # with respect to the unknowns over their start
        g, A = d.T @ r, d.T @ d
        assert A[TH.ALPHA_SL, TH.ALPHA_SL] == 0.0 and g[TH.ALPHA_SL] < 0.0
        free = np.arange(7) != TH.GAMMA if g[TH.GAMMA] < 0.0 else np.full(7, True)     # gamma is at its bound
        up = True
        for k in range(steps):
            damped = A + 1e-3 * 5.0 ** k * np.diag(np.maximum(np.diag(A), 1e-300))
            x = cholesky_solve(damped[np.ix_(free, free)], -g[free])
            up = up and min(x[TH.ALPHA_SL], x[TH.BETA_SL]) > 1e80             # a time of 1e60 s or more: no better than the start's
        if up:
            stays.append(j)
    assert len(stays) >= 10
    for slots in (n, 65):                                                      # one record a lane, and the loop over more
        wide = {k: (v if k == "count" else np.concatenate([v, np.ones((J, slots - n), v.dtype)], axis=1)) for k, v in ob.items()}
        got = px.fit_theta(wide, theta_init=init, max_iter=steps, n_starts=1)
        for j in stays:
            error = TH.rmsle(init[:, j], *(ob[k][j] for k in names))
            assert got["iterations"][j] == steps and np.array_equal(got["theta"][:, j], init[:, j])
            assert abs(got["rmsle"][j] - error) <= 1e-12 * error
