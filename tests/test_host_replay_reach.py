"""CPU replay of tiles that cross the boundary of two bands of more than a
gigabyte each (tests/host_replay/reach.cpp): every access lies within what a
buffer access of the step kernels reaches, and the result is that of the 64-bit
per-node path, bit for bit.  Such bands come from long rows or from a large
band_rows.
"""
import hashlib
import os
import subprocess

import pytest

import lbm_workloads as W
import test_host_replay as R

SRC = os.path.join(R.ROOT, "tests", "host_replay", "reach.cpp")


@pytest.fixture(scope="module")
def reach():
    if not os.path.exists(R.CXX):
        pytest.skip("no host clang++")
    h = hashlib.sha256()
    for p in [SRC, R.SRC, os.path.join(R.ROOT, "include", "lbmpcm.h")] + [os.path.join(R.CSRC, n) for n in R.HEADERS]:
        h.update(open(p, "rb").read())
    exe = os.path.join(R.BUILD, "reach_" + h.hexdigest()[:12])
    if not os.path.exists(exe):
        os.makedirs(R.BUILD, exist_ok=True)
        tmp = f"{exe}.tmp{os.getpid()}"
        subprocess.check_call([R.CXX, "-std=c++17", "-O1", "-g1", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__",
                               "-I/opt/rocm/include", "-I" + R.CSRC, "-o", tmp, SRC])
        os.replace(tmp, exe)
    return exe


# prec, thermal lattice, nx, ny, band_rows: the longest accepted rows of FP64
# and of FP32_H64, and large bands of each storage family
CASES = [("f64", 9, 262144, 70, 0), ("f64", 9, 200000, 70, 0), ("f64", 5, 262144, 70, 0), ("f64", 9, 8192, 1100, 1000),
         ("f32h64", 9, 262144, 70, 0), ("f32", 9, 8192, 4200, 2100), ("f32", 5, 8192, 3400, 3000),
         ("f16", 9, 8192, 4000, 3900), ("f16split", 9, 8192, 3200, 3100)]


@pytest.mark.parametrize("prec,qt,nx,ny,rows", CASES)
def test_tiles_across_large_bands_stay_within_reach(reach, prec, qt, nx, ny, rows):
    p = dict(W.scaled_cavity(W.case_c1()[0], nx, ny), thermal_lattice=qt, band_rows=rows, L_char=127.0)
    code, out = R._run(reach, R._job(p, precision=prec, seed=5))
    assert code == 0 and "identical" in out and "identical: 0 tiles" not in out, out
