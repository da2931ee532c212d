"""The kernels' inner functions in their device form (hardware estimates refined
by Newton steps, frexp instructions) against mpmath.  GPU only."""
import ctypes as C
import os

import mpmath as mp
import numpy as np
import pytest
import torch

from paper_2407_18304_amd import build

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

RCP, DIV, LOG, ONE_MINUS_EXP, EXP_NEG, SQRT, STIM, MEAN, MEAN_FIXED = range(9)
U = 2.0 ** -53
N = 3000


@pytest.fixture(autouse=True)
def fifty_digits():
    with mp.workdps(50):
        yield


@pytest.fixture(scope="module")
def probe():
    L = C.CDLL(os.path.join(build.PKG, "libmgrhd_probe.so"))
    vp = C.c_void_p
    L.mgrhd_math_probe.argtypes = [C.c_int, vp, vp, C.c_int64, vp]

    def run(which, *rows):
        a = np.zeros((4, len(rows[0])))
        for k, r in enumerate(rows):
            a[k] = r
        x = torch.from_numpy(a).cuda()
        out = torch.full((a.shape[1],), float("nan"), dtype=torch.float64, device="cuda")
        assert L.mgrhd_math_probe(which, x.data_ptr(), out.data_ptr(), a.shape[1],
                                  torch.cuda.current_stream().cuda_stream) == 0
        return out.cpu().numpy()
    return run


def _within(got, refs, bound, xs):
    for g, ref, x in zip(got, refs, xs):
        assert abs(mp.mpf(float(g)) - ref) <= bound * U * abs(ref), (x, float(g))


def _log_spread(rng, lo, hi, n=N):
    return 10.0 ** rng.uniform(lo, hi, n)


def test_reciprocal_and_quotient(probe):
    """One rounding each: the last step adds a correction that is exact next to
    the rounding of the sum."""
    rng = np.random.default_rng(1)
    d = np.concatenate([_log_spread(rng, -300, 300), -_log_spread(rng, -5, 5), [1.0, 3.0]])
    _within(probe(RCP, d), [1 / mp.mpf(float(x)) for x in d], 1.01, d)
    n = rng.uniform(-2, 2, len(d))
    d = np.clip(d, -1e250, 1e250)
    _within(probe(DIV, n, d), [mp.mpf(float(a)) / mp.mpf(float(b)) for a, b in zip(n, d)], 1.01, d)


def test_logarithm(probe):
    """The bound of the host build's test."""
    rng = np.random.default_rng(2)
    x = np.concatenate([[1.0, 0.5, 2.0, 0.7071067811865475, 0.7071067811865476, 5e-324, 2.3e-308,
                         1.7e308], rng.uniform(0.5, 2.0, N), _log_spread(rng, -320, 308),
                        1.0 + rng.uniform(-1e-3, 1e-3, N)])
    _within(probe(LOG, x), [mp.log(mp.mpf(float(a))) for a in x], 2, x)


def test_exponentials(probe):
    """The bounds of the host build's test (6 U); 1 - e^{-t} past the range of
    the exponential."""
    rng = np.random.default_rng(3)
    t = np.concatenate([[0.0, 1e-300, 37.0, 700.0, np.log(2.0) / 2], rng.uniform(0, 2, N),
                        _log_spread(rng, -9, 2.8)])
    ref = [mp.exp(-mp.mpf(float(a))) for a in t]
    _within(probe(ONE_MINUS_EXP, t), [-mp.expm1(-mp.mpf(float(a))) for a in t], 6, t)
    _within(probe(EXP_NEG, t), ref, 6, t)
    _within(probe(EXP_NEG, t, np.ones_like(t)), ref, 6, t)
    far = np.array([800.0, np.inf])
    assert (probe(ONE_MINUS_EXP, far) == 1.0).all() and (probe(EXP_NEG, far) == 0.0).all()


def test_square_root_and_stimulated_emission(probe):
    """sqrt within an ulp; 1 - e^{-x} of an edge: the polynomial of x/(e^x - 1)
    (some 4 roundings at x = 4, where it is a thirteenth of the sum), the sum
    and the quotient."""
    rng = np.random.default_rng(4)
    a = np.concatenate([[1.0, 4.0, np.nextafter(1.0, 2.0)], rng.uniform(1, 4, N)])
    _within(probe(SQRT, a), [mp.sqrt(mp.mpf(float(x))) for x in a], 2, a)
    x = np.concatenate([[4.0, np.nextafter(4.0, 5.0), 1e-300], _log_spread(rng, -8, 2.8)])
    _within(probe(STIM, x), [-mp.expm1(-mp.mpf(float(v))) for v in x], 6, x)


def test_means(probe):
    """The group means at the host test's bounds, and at exponents next to and
    below the smallest number."""
    rng = np.random.default_rng(5)
    ac, aq = rng.uniform(-4, 2, N), rng.uniform(-40, 40, N)
    L = _log_spread(rng, -6, 1)
    y = (np.abs(ac) + 2 * np.abs(aq) + 2) * L
    keep = y < 300
    ac, aq, L, y = ac[keep], aq[keep], L[keep], y[keep]
    rac = np.array([float(mp.exp(mp.mpf(float(a)) * mp.mpf(float(l)))) for a, l in zip(ac, L)])

    def bracket(a, l):
        return mp.expm1(a * l) / a if a != 0 else l

    for g, a, q, l, yy in zip(probe(MEAN, ac, aq, L, rac), ac, aq, L, y):
        a, q, l = (mp.mpf(float(v)) for v in (a, q, l))
        ref = bracket(a + q + 1, l) / bracket(q + 1, l)
        assert abs(mp.mpf(float(g)) - ref) <= (32 + 4 * yy) * U * ref
    tiny = np.array([0.0, 5e-324, -5e-324, 1e-310, -1e-310, 2.3e-308, 1e-295, -1e-200, 1e-20])
    assert (probe(MEAN_FIXED, tiny, np.ones_like(tiny)) == 1.0).all()
