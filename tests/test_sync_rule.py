"""Blocks that may wait for one another in one launch, on a host build of the rule
(csrc/sync_rule.hpp): eight launches of any of the kernels at once fit the device, whatever a compute
unit holds of its blocks and however many units there are; none where an eighth is no block."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("sync")
    (d / "sync.cpp").write_text('#include "sync_rule.hpp"\n'
                                'extern "C" int rule(int w, int c, int p) { return fsl::sync_blocks(w, c, p); }\n')
    subprocess.run([cc, "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1712_07028_amd", "csrc"),
                    "-o", str(d / "sync.so"), str(d / "sync.cpp")], check=True)
    return ctypes.CDLL(str(d / "sync.so")).rule


def test_eight_launches_fit(rule):
    for want in (1, 32, 128):
        for cus in (1, 7, 8, 32, 64, 128, 256, 304):
            for per_cu in (0, 1, 2, 3, 8):
                n = rule(want, cus, per_cu)
                assert 0 <= n <= want and 8 * n <= cus * per_cu
                assert n == min(want, cus * per_cu // 8)  # no fewer than the share allows


def test_whole_device_and_a_partition(rule):
    # one block of 1,024 threads with the sphere table in LDS to a compute unit
    assert rule(32, 256, 1) == 32
    assert rule(32, 32, 1) == 4
    # eight blocks of 256 threads
    assert rule(128, 256, 8) == 128
    assert rule(128, 32, 8) == 32
    assert rule(32, 4, 1) == 0 and rule(32, 256, 0) == 0 and rule(32, -1, 1) == 0
