"""The FP32 test before the FP64 one of candidate pairs, on a host build of the same functions
(csrc/pair_near.hpp), against the distance in 64 bits: on boxes that take it no pair within
reach is lost, along walled and periodic axes, whatever the radii; on boxes of 2^24 cells an axis
one is, and those do not take it.
"""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
REACH = 2.0 / 3.0 + 1.0
SRC = """
#define __host__
#define __device__
#include "pair_near.hpp"
extern "C" int box(int nx, int ny, int nz) { return fsl::pairs_direct_box(nx, ny, nz); }
extern "C" void near(int m, const double *a, const double *ra, const double *b, const double *rb, double reach,
                     const int *n, const int *per, int *out) {
    for (int i = 0; i < m; ++i) {
        float d[3];
        for (int k = 0; k < 3; ++k) d[k] = fsl::axis_apart((float)a[3 * i + k], (float)b[3 * i + k], n[k], per[k]);
        out[i] = fsl::pair_near(d[0], d[1], d[2], (float)rb[i] + fsl::reach_of(ra[i], reach));
    }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("near")
    (d / "near.cpp").write_text(SRC)
    subprocess.run([cc, "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_1712_07028_amd", "csrc"), "-o", str(d / "near.so"), str(d / "near.cpp")],
                   check=True)
    return ctypes.CDLL(str(d / "near.so"))


def near(lib, a, ra, b, rb, n, per):
    out = np.zeros(len(a), dtype=np.int32)
    dp = ctypes.POINTER(ctypes.c_double)
    a, b = np.ascontiguousarray(a, dtype=np.float64), np.ascontiguousarray(b, dtype=np.float64)
    ra, rb = np.ascontiguousarray(ra, dtype=np.float64), np.ascontiguousarray(rb, dtype=np.float64)
    lib.near(ctypes.c_int(len(a)), a.ctypes.data_as(dp), ra.ctypes.data_as(dp), b.ctypes.data_as(dp),
             rb.ctypes.data_as(dp), ctypes.c_double(REACH), (ctypes.c_int * 3)(*n), (ctypes.c_int * 3)(*per),
             out.ctypes.data_as(ctypes.POINTER(ctypes.c_int)))
    return out != 0


def gap(a, ra, b, rb, n, per):
    d = b - a
    for k in range(3):
        if per[k]:
            d[:, k] -= n[k] * np.floor(d[:, k] / n[k] + 0.5)
    return np.sqrt((d * d).sum(axis=1)) - ra - rb


@pytest.mark.parametrize("n", [(40, 36, 32), (203, 77, 141), (65536, 128, 130), (130, 65536, 65536)])
@pytest.mark.parametrize("per", [(0, 0, 0), (1, 1, 0), (1, 1, 1)])
def test_no_pair_within_reach_is_lost(lib, n, per):
    assert lib.box(*n)
    rng = np.random.Generator(np.random.PCG64(11))
    m = 200_000
    size = np.array(n, dtype=float)
    a = rng.uniform(0.0, 1.0, (m, 3)) * size
    a[: m // 2] = size - rng.uniform(0.0, 8.0, (m // 2, 3))  # near the far faces, where FP32 is coarsest
    ra, rb = rng.uniform(0.5, 12.0, m), rng.uniform(0.5, 12.0, m)
    # surfaces from overlapping to just beyond the reach, in any direction
    v = rng.standard_normal((m, 3))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    b = a + v * (ra + rb + rng.uniform(-1.0, REACH + 0.2, m))[:, None]
    for k in range(3):
        if per[k]:
            b[:, k] %= n[k]
    ok = ((b >= 0) & (b < size)).all(axis=1) & ((a >= 0) & (a < size)).all(axis=1)
    a, b, ra, rb = a[ok], b[ok], ra[ok], rb[ok]
    within = gap(a, ra, b, rb, n, per) < REACH
    assert within.sum() > 1000
    assert near(lib, a, ra, b, rb, n, per)[within].all()


def test_long_boxes_take_the_grid(lib):
    n = (1 << 24) + 64
    assert lib.box(65536, 65536, 65536)
    for k in range(3):
        assert not lib.box(*[65537 if a == k else 8 for a in range(3)])
    # coordinates round to even cells there: 0.02 cells apart along x, taken for 2
    a = np.array([[16777216.0 + 0.99, 1.0, 2.0]])
    b = np.array([[16777216.0 + 1.01, 4.05, 2.0]])
    R = np.array([0.7])
    assert gap(a, R, b, R, (n, 8, 8), (0, 0, 0))[0] < REACH
    assert not near(lib, a, R, b, R, (n, 8, 8), (0, 0, 0))[0] and not lib.box(n, 8, 8)
