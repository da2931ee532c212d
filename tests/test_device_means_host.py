"""The logarithm, the 1 - e^{-t} and the group means of the kernels' inner loop,
compiled for the host and pinned against mpmath.  CPU only."""
import ctypes as C
import os
import shutil
import subprocess

import mpmath as mp
import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "hostbuild", "device_means_host.hip")
U = 2.0 ** -53
LN2 = float(np.log(2.0))


@pytest.fixture(autouse=True)
def fifty_digits():
    with mp.workdps(50):
        yield


@pytest.fixture(scope="module")
def dm(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("dmm") / "libdmm.so")
    subprocess.run([hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
                    "-o", out, SRC], check=True, capture_output=True)
    L = C.CDLL(out)
    L.dm_one_minus_exp.argtypes = [C.c_double, C.POINTER(C.c_double)]
    for f, n in (("dm_log_pos", 1), ("dm_mean_ratio_rac", 4), ("dm_mean_fixed_rac", 2)):
        getattr(L, f).restype = C.c_double
        getattr(L, f).argtypes = [C.c_double] * n
    return L


def _ts():
    rng = np.random.default_rng(3)
    return np.concatenate([[1e-300, 1e-17, 1e-8, 0.5 * LN2, np.nextafter(0.5 * LN2, 1.0), LN2,
                            1.5 * LN2, 37.0, 40.0, 700.0], rng.uniform(0, 2, 300),
                           10.0 ** rng.uniform(-9, 2.8, 300)])


def test_one_minus_exp(dm):
    """Both parts within 3 ulp (6 U): the reduced argument and the series carry
    about one rounding each, the last two operations one each."""
    out = np.zeros(2)
    p = out.ctypes.data_as(C.POINTER(C.c_double))
    for t in _ts():
        dm.dm_one_minus_exp(float(t), p)
        x = mp.mpf(float(t))
        assert abs(out[0] + mp.expm1(-x)) <= 6 * U * -mp.expm1(-x), t
        assert abs(out[1] - mp.exp(-x)) <= 6 * U * mp.exp(-x), t
    for t, want in ((0.0, (0.0, 1.0)), (800.0, (1.0, 0.0)), (float("inf"), (1.0, 0.0))):
        dm.dm_one_minus_exp(t, p)
        assert tuple(out) == want
    dm.dm_one_minus_exp(float("nan"), p)
    assert np.isnan(out).all()


def test_log_pos(dm):
    """Within 3 ulp (6 U) of its own value, which is small next to 1: s carries
    four roundings at most, and the exponent's part is exact to the tail."""
    rng = np.random.default_rng(4)
    xs = np.concatenate([[1.0, np.nextafter(1, 0), np.nextafter(1, 2), 0.5, 2.0, 5e-324, 2.3e-308,
                          1.7e308, 0.7071067811865475, 0.7071067811865476, 1.4142135623730951],
                         rng.uniform(0.5, 2.0, 400), 10.0 ** rng.uniform(-320, 308, 400)])
    for x in xs:
        ref = mp.log(mp.mpf(float(x)))
        assert abs(dm.dm_log_pos(float(x)) - ref) <= 6 * U * abs(ref), x


def _ratio(ac, aq, L):
    def bracket(a):
        return mp.expm1(a * L) / a if a != 0 else L
    return bracket(mp.mpf(ac) + mp.mpf(aq) + 1) / bracket(mp.mpf(aq) + 1)


@pytest.mark.parametrize("L", [1e-6, 0.0719, 0.216, 0.86, 3.45, 13.8])
def test_means_of_the_inner_loop(dm, L):
    """Every pairing of the signs of (alpha_chi + alpha_Q + 1) L and
    (alpha_Q + 1) L, zeros and near zeros included.  A relative error U of an
    exponent y is an error y U of the exponential, on top of some 16 roundings."""
    rng = np.random.default_rng(int(1000 * L))
    pairs = [(0.0, -1.0), (-2.0, 1.0), (1.0, -2.0), (2.0, -3.0), (-1e-9, -1.0), (1e-12, -1.0),
             (-4.0, -1.0 + 1e-14), (2.0, -1.0 - 1e-12)]
    pairs += [(a, q) for a, q in zip(rng.uniform(-4, 2, 60), rng.uniform(-40, 40, 60))]
    for ac, aq in pairs:
        ac, aq = float(ac), float(aq)
        y = (abs(ac) + 2 * abs(aq) + 2) * L
        if y > 300:
            continue
        rac = float(mp.exp(mp.mpf(ac) * L))
        ref = _ratio(ac, aq, L)
        assert abs(dm.dm_mean_ratio_rac(ac, aq, L, rac) - ref) <= (32 + 4 * y) * U * ref, (ac, aq)
        fixed = _ratio(ac, -1.0, L)
        y = abs(ac) * L
        got = dm.dm_mean_fixed_rac(ac * L, rac)
        assert abs(got - fixed) <= (16 + 4 * y) * U * fixed, ac


def test_log_pos_rounding(dm):
    """Within 2 U: the rounding of the result, a fifth of one of the corrected
    f (its share of the logarithm), and a fifth of the some 2.8 of s and of the
    series; the parts that e ln2 loses are added again."""
    rng = np.random.default_rng(5)
    xs = np.concatenate([[1.0, 0.5, 2.0, 0.7071067811865475, 0.7071067811865476, 5e-324, 1.7e308],
                         rng.uniform(0.5, 2.0, 4000), 10.0 ** rng.uniform(-320, 308, 4000)])
    for x in xs:
        ref = mp.log(mp.mpf(float(x)))
        assert abs(dm.dm_log_pos(float(x)) - ref) <= 2 * U * abs(ref), x
