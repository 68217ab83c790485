"""CPU replay of the deep launches (tests/host_replay/deep.cpp): every tile
shape, storage form and number of steps, under AddressSanitizer with NaN-filled
LDS and the headers' bounds checks on, equals single steps bit for bit; so do
the three-step FP64 launches, which only the library itself chooses.
"""
import hashlib
import os
import subprocess

import pytest

import test_host_replay as R

SRC = os.path.join(R.ROOT, "tests", "host_replay", "deep.cpp")


@pytest.fixture(scope="module")
def deep():
    if not os.path.exists(R.CXX):
        pytest.skip("no host clang++")
    h = hashlib.sha256()
    for p in [SRC, R.SRC, os.path.join(R.ROOT, "include", "lbmpcm.h")] + [os.path.join(R.CSRC, n) for n in R.HEADERS]:
        h.update(open(p, "rb").read())
    exe = os.path.join(R.BUILD, "deep_" + h.hexdigest()[:12])
    if not os.path.exists(exe):
        os.makedirs(R.BUILD, exist_ok=True)
        tmp = f"{exe}.tmp{os.getpid()}"
        subprocess.check_call([R.CXX, "-std=c++17", "-O1", "-g1", "-ffp-contract=off", "-fsanitize=address,undefined",
                               "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + R.CSRC, "-o", tmp, SRC])
        os.replace(tmp, exe)
    return exe


@pytest.mark.parametrize("prec,qt", [("f64", 9), ("f32", 9), ("f32h64", 9), ("f64", 5), ("f32", 5), ("f32h64", 5)])
def test_deep_launches_replay_single_steps(deep, prec, qt):
    for name, p in R._geometries().items():
        if p["bc_x"] == 1:
            continue  # periodic problems take no deep launches
        for shape in range(4):
            job = R._job(dict(p, thermal_lattice=qt), precision=prec, shape=shape, launches=1, seed=5)
            code, out = R._run(deep, job)
            assert code == 0 and "identical" in out, f"{name}, tile shape {shape}: {out}"


@pytest.mark.parametrize("qt", [9, 5])
def test_three_step_fp64_launches_replay_single_steps(qt):
    if not os.path.exists(R.CXX):
        pytest.skip("no host clang++")
    exe = R._binary()
    for name, p in R._geometries().items():
        job = R._job(dict(p, thermal_lattice=qt), precision="f64", K=3, shape=0, launches=2, mode="kstep", seed=7)
        code, out = R._run(exe, job)
        assert code == 0 and "identical" in out, f"{name}: {out}"
