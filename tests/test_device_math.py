"""Error of the fp64 polynomial kernels used on the GPU (exp, log1p, log and the
factored form of Eq. 10), measured on the host against long-double libm.  The
same header is compiled for the device; only the reciprocal seed, ldexp, frexp
and rounding primitives differ."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host_math(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("pxmath") / "libpxmath.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "device_math_host.cpp")], check=True)
    L = ctypes.CDLL(so)
    L.px_host_max_ulp.restype = ctypes.c_double
    L.px_host_max_ulp.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_long]
    L.px_host_eval.restype = ctypes.c_double
    L.px_host_eval.argtypes = [ctypes.c_int, ctypes.c_double, ctypes.c_double, ctypes.c_double]
    L.px_host_div_faults.restype = None
    L.px_host_div_faults.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_long, ctypes.c_double, ctypes.c_int, ctypes.c_void_p,
                                     ctypes.c_void_p]
    return L


SEED_SKEWS = [0.0, 2.0 ** -24, -2.0 ** -24, 2.0 ** -26, -2.0 ** -26, 1.7e-8, -4.1e-8]


def div_faults(L, a, b, skew, integers=False):
    a, b = (np.ascontiguousarray(np.broadcast_to(x, np.broadcast(a, b).shape), np.float64) for x in (a, b))
    out = [ctypes.c_long(), ctypes.c_long()]
    L.px_host_div_faults(a.ctypes.data, b.ctypes.data, a.size, skew, int(integers), *(ctypes.addressof(x) for x in out))
    return out[0].value, out[1].value


def max_ulp(L, which, x, y=None, g=None):
    x = np.ascontiguousarray(x, np.float64)
    y = np.ascontiguousarray(x if y is None else y, np.float64)
    g = np.ascontiguousarray(np.ones_like(x) if g is None else g, np.float64)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    return L.px_host_max_ulp(which, p(x), p(y), p(g), x.size)


def test_exp_of_non_positive_arguments(host_math):
    rng = np.random.default_rng(0)
    x = np.concatenate([-rng.uniform(0, 40, 400000), -np.exp(rng.uniform(-30, 6.5, 200000)), rng.uniform(0, 0.7, 100000)])
    assert max_ulp(host_math, 0, x) < 1.0
    assert host_math.px_host_eval(0, 0.0, 0, 1) == 1.0
    assert host_math.px_host_eval(0, -np.inf, 0, 1) == 0.0
    assert host_math.px_host_eval(0, -1000.0, 0, 1) == 0.0


def test_log1p_on_the_unit_interval(host_math):
    rng = np.random.default_rng(1)
    x = np.concatenate([rng.uniform(0, 1, 500000), np.exp(rng.uniform(-40, 0, 200000)), [0.0, 1.0, 0.41421356237309503]])
    assert max_ulp(host_math, 1, x) < 2.5
    assert host_math.px_host_eval(1, 0.0, 0, 1) == 0.0


def test_log_of_positive_numbers(host_math):
    rng = np.random.default_rng(2)
    x = np.concatenate([np.exp(rng.uniform(-20, 20, 500000)), rng.uniform(0.5, 2.0, 300000), [1.0]])
    assert max_ulp(host_math, 2, x) < 2.5
    assert host_math.px_host_eval(2, 1.0, 0, 1) == 0.0


def test_factored_overlap_term_matches_the_direct_power_form(host_math):
    """max(a,b) * exp(log1p(exp(-g|ln a - ln b|))/g) against (a^g + b^g)^(1/g) in long double."""
    rng = np.random.default_rng(3)
    n = 500000
    tg = np.exp(rng.uniform(np.log(1e-3), np.log(10.0), n))
    ts = np.exp(rng.uniform(np.log(1e-3), np.log(10.0), n))
    g = rng.uniform(1.0, 10.0, n)
    assert max_ulp(host_math, 3, tg, ts, g) < 8.0
    # nearly equal terms with the largest exponent are the worst case
    ts2 = tg * (1 + rng.uniform(-1e-3, 1e-3, n))
    assert max_ulp(host_math, 3, tg, ts2, np.full(n, 10.0)) < 8.0


@pytest.mark.parametrize("skew", SEED_SKEWS)
def test_quotients_are_rounded_as_a_division_rounds_them(host_math, skew):
    """px_div stands where the library's division stood: whatever the seed, on the reciprocals of GPU counts and accumulation
    counts, all of them, and on quotients of all kinds of mantissas."""
    counts = np.arange(1.0, 2.0 ** 14 + 1)
    assert div_faults(host_math, 1.0, counts, skew) == (0, 0)
    rng = np.random.default_rng(5)
    a, b = (rng.uniform(1.0, 2.0, 400000) * 2.0 ** rng.integers(-40, 41, 400000) for _ in range(2))
    assert div_faults(host_math, a, b, skew) == (0, 0)
    # mantissas next to 1 and to 2; the one divisor that any such sequence may miss has a mantissa of ones only
    ulps = 2.0 ** -52 * np.arange(2000)
    for x in (1.0 + ulps, 2.0 - ulps[1:]):
        for y in (1.0 + ulps[:300], 2.0 - ulps[2:300]):
            assert div_faults(host_math, x[:, None], y[None, :], skew) == (0, 0)
        assert div_faults(host_math, x, 2.0 - 2.0 ** -52, skew)[0] <= 1
    assert div_faults(host_math, rng.uniform(1.0, 1e6, 200000), rng.uniform(1.0, 10.0, 200000), skew) == (0, 0)


@pytest.mark.parametrize("skew", SEED_SKEWS)
def test_integer_quotients_have_the_right_floor(host_math, skew):
    """The sampling argmax divides integers in doubles: multiples of the divisor and their neighbours, numerators up to 2^38 where the
    quotient is not one and beyond 2^53 where it is."""
    rng = np.random.default_rng(6)
    b = np.concatenate([np.arange(1, 3000), np.floor(np.exp(rng.uniform(0, np.log(2.0 ** 38), 60000)))])
    for k in (1, 2, 3, 7, 64, 255, 16384):
        for d in (-1, 0, 1):
            a = k * b + d
            ok = a < 2.0 ** 38
            assert div_faults(host_math, a[ok], b[ok], skew, True)[1] == 0, (k, d)
    b = np.floor(np.exp(rng.uniform(np.log(2.0 ** 31), np.log(2.0 ** 62), 100000)))
    M = np.floor(np.exp(rng.uniform(0, np.log(2.0 ** 31), 100000)))
    assert div_faults(host_math, M + (b - 1.0), b, skew, True)[1] == 0


@pytest.mark.parametrize("single", [0, 1])
@pytest.mark.parametrize("skew", [0.0, 2.0 ** -23, -2.0 ** -23])
def test_best_counts(host_math, single, skew):
    """The count with the smallest s + C / (s + 1): at the thresholds t (t + 1), their neighbours and between them, far beyond the grid
    (where the root fits no whole number), at infinity and for what is no number; clamped to any feasible counts."""
    L = host_math
    L.px_host_best_counts.restype = None
    L.px_host_best_counts.argtypes = [ctypes.c_void_p, ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_float, ctypes.c_int, ctypes.c_void_p]
    real = np.float32 if single else np.float64
    largest = 4094 if single else 2 ** 14 - 1                # counts of a grid, and those whose products single precision holds
    t = np.arange(largest + 1)
    U = (t * (t + 1.0)).astype(real)
    rng = np.random.default_rng(8)
    inside = np.concatenate([U, np.nextafter(U, real(np.inf)), np.nextafter(U, real(0)), (rng.uniform(0.0, 1.0, 20000) * U[-1]).astype(real)])
    inside = np.sort(inside.astype(np.float64))
    want = np.searchsorted(t * (t + 1.0), inside, side="left") - 1           # the last t with C > t (t + 1)
    want = np.maximum(want, 0)
    beyond = np.array([1e9, 1e18, 5e18, 1e19, 1e30, 3e38, np.inf] + ([] if single else [1e39, 1e300]))
    none = np.array([0.0, -0.1, -0.3, -1.0, -1e30, -np.inf, np.nan])

    def counts(C, s_lo, s_hi):
        C = np.ascontiguousarray(C, np.float64)
        out = np.full(C.size, -99, np.int32)
        L.px_host_best_counts(C.ctypes.data, C.size, s_lo, s_hi, skew, single, out.ctypes.data)
        return out

    for s_lo, s_hi in ((0, largest), (0, 0), (0, 31), (7, 12), (5, 5), (200, 300), (3, largest)):
        assert np.array_equal(counts(inside, s_lo, s_hi), np.clip(want, s_lo, s_hi)), (s_lo, s_hi)
        assert np.all(counts(beyond, s_lo, s_hi) == s_hi) and np.all(counts(none, s_lo, s_hi) == s_lo), (s_lo, s_hi)
