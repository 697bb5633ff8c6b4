"""The reduction of angles, compiled for the host from the kernels' own header (no GPU):
for every finite M0 the mean anomaly of Eq. 4 lies in [-pi, pi], and so does what the
standalone solve leaves of M, so the knot that the Kepler solve reads from the
starting-value table lies in its row."""
import ctypes
import math
import os
import re
import subprocess

import mpmath as mp
import numpy as np
import pytest

from paper_0812_2976_amd import build as libbuild

SOURCE = r"""
#include "kep_root64.h"
extern "C" void phases(const double *tt, const double *P, const double *M0, long n, double *M0c, double *M)
{
    for (long i = 0; i < n; ++i) {
        double q;
        const kep::Phase64c p = kep::make_phase64c(P[i], M0[i]);
        M0c[i] = p.M0c;
        M[i] = kep::mean_anomaly64c(tt[i], p, q);
    }
}
extern "C" void turns(const double *M, long n, double *r, double *k, double *k2)
{
    for (long i = 0; i < n; ++i) r[i] = kep::centre_turns(M[i], k[i], k2[i]);
}
"""

KNOTS = [int(n) for n in re.search(r"KEP_TAB_BAND_KNOTS \{([^}]*)\}",
                                   open(os.path.join(libbuild.CSRC, "kep_start_tab.h")).read()).group(1).split(",")]


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("angles")
    (d / "angles.hip").write_text(SOURCE)
    subprocess.run([libbuild.hipcc(), "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I", libbuild.CSRC, "-I", libbuild.INCLUDE, str(d / "angles.hip"), "-o", str(d / "angles.so")],
                   check=True)
    return ctypes.CDLL(str(d / "angles.so"))


def _call(f, arrays, n_out):
    arrays = [np.ascontiguousarray(a, dtype=np.float64) for a in arrays]
    out = [np.empty_like(arrays[0]) for _ in range(n_out)]
    ptr = [a.ctypes.data_as(ctypes.c_void_p) for a in arrays + out]
    f(*ptr[:len(arrays)], ctypes.c_long(arrays[0].size), *ptr[len(arrays):])
    return out


def _knots(M):
    """The knots that the kernels read (binary32, |M| times knots / pi, truncated) and each band's last."""
    x = np.abs(M.astype(np.float32))
    return [((x * np.float32(n / math.pi)).astype(np.int64), n) for n in KNOTS]


def _angles(rng, lo, hi, n):
    """Magnitudes over [10^lo, 10^hi], both signs, and values next to odd multiples of pi."""
    x = 10.0 ** rng.uniform(lo, hi, n)
    k = np.rint(10.0 ** rng.uniform(max(lo, 0.0), min(hi, 300.0), n // 4))
    return np.concatenate([x, -x, (2.0 * k + 1.0) * math.pi, -(2.0 * k + 1.0) * math.pi])


@pytest.mark.parametrize("lo,hi", [(-300, 0), (0, 4), (4, 16), (16, 31), (31, 60), (60, 308.25)])
def test_mean_anomaly_of_every_finite_m0(host, lo, hi):
    rng = np.random.default_rng(abs(int(lo)) + 1)
    M0 = _angles(rng, lo, hi, 20000)
    if hi > 300:
        M0 = np.concatenate([M0, [1.7976931348623157e308, -1.7976931348623157e308]])
    P = 10.0 ** rng.uniform(-3, 4, M0.size)
    tt = rng.choice([0.0, 1.0, -37.25, 2456000.0], M0.size) * rng.uniform(0.5, 1.0, M0.size)
    M0c, M = _call(host.phases, (tt, P, M0), 2)
    # pi, and the rounding of the last subtraction at a magnitude of at most 2 pi
    assert np.abs(M0c).max() <= math.pi + 2.0 ** -17 and np.abs(M).max() <= math.pi + 2.0 ** -49
    for j, last in _knots(M):
        assert j.min() >= 0 and j.max() <= last


def test_m0_is_reduced_modulo_two_pi(host):
    """Against 60 digits, while binary64's M0 still says where on the orbit it is: two roundings at the
    magnitude of pi and the rounding of M0 / (2 pi) 2^-107 (the second part of 2 pi) a turn."""
    M0 = _angles(np.random.default_rng(5), 0, 15, 400)
    M0c, _ = _call(host.phases, (np.zeros_like(M0), np.ones_like(M0), M0), 2)
    with mp.workdps(60):
        for x, c in zip(M0, M0c):
            r = mp.mpf(x) - mp.mpf(c)
            r -= 2 * mp.pi * mp.nint(r / (2 * mp.pi))
            assert abs(r) <= 4 * math.pi * 2.0 ** -53 + abs(x) * 2.0 ** -105, x


@pytest.mark.parametrize("lo,hi", [(-300, 0), (0, 4), (4, 12), (12, 15), (15, 16.2556)])
def test_standalone_mean_anomaly_is_centred(host, lo, hi):
    """|M| < 2^54: r lies in [-pi, pi], k + k2 are the whole turns, and r + 2 pi (k + k2) is M to two
    roundings at the magnitude of r and 2^-107 (the second part of 2 pi) a turn."""
    M = _angles(np.random.default_rng(int(lo) + 400), lo, hi, 20000)
    if lo == 12:
        M = np.append(M, 367531048600891.44)
    M = M[np.abs(M) < 2.0 ** 54]
    r, k, k2 = _call(host.turns, (M,), 3)
    assert np.abs(r).max() <= math.pi + 2.0 ** -17
    for j, last in _knots(r):
        assert j.min() >= 0 and j.max() <= last
    assert np.array_equal(k, np.rint(k)) and np.array_equal(k2, np.rint(k2)) and (k2[np.abs(M) < 1e10] == 0).all()
    with mp.workdps(60):
        for x, y, n in zip(M[::40], r[::40], (k + k2)[::40]):
            assert abs(mp.mpf(x) - mp.mpf(y) - 2 * mp.pi * mp.mpf(n)) <= 4 * math.pi * 2.0 ** -53 + abs(x) * 2.0 ** -105, x
