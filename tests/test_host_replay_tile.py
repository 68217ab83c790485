"""CPU replay of the multi-step kernels with their wall tallies in LDS and the
idle threads' fetches (tests/host_replay/tile.cpp), under AddressSanitizer.
"""
import hashlib
import os
import subprocess

import pytest

import test_host_replay as R

SRC = os.path.join(R.ROOT, "tests", "host_replay", "tile.cpp")


@pytest.fixture(scope="module")
def tile():
    if not os.path.exists(R.CXX):
        pytest.skip("no host clang++")
    h = hashlib.sha256()
    for p in [SRC, R.SRC, os.path.join(R.ROOT, "include", "lbmpcm.h")] + [os.path.join(R.CSRC, n) for n in R.HEADERS]:
        h.update(open(p, "rb").read())
    exe = os.path.join(R.BUILD, "tile_" + h.hexdigest()[:12])
    if not os.path.exists(exe):
        os.makedirs(R.BUILD, exist_ok=True)
        tmp = f"{exe}.tmp{os.getpid()}"
        subprocess.check_call([R.CXX, "-std=c++17", "-O1", "-g1", "-ffp-contract=off", "-fsanitize=address,undefined",
                               "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + R.CSRC, "-o", tmp, SRC])
        os.replace(tmp, exe)
    return exe


# storage, thermal lattice, steps, tile shapes, tallies in LDS in the default shape
FORMS = [("f32", 9, 3, 3, True), ("f32h64", 9, 3, 3, True), ("f64", 9, 3, 1, True), ("f16", 9, 3, 3, True),
         ("f16split", 9, 3, 3, True), ("f32", 5, 3, 3, False), ("f32h64", 5, 3, 3, True), ("f64", 5, 3, 1, True),
         ("f64", 9, 2, 3, True), ("f64", 5, 2, 3, False), ("f32", 9, 2, 3, False), ("f32h64", 9, 2, 3, None)]


@pytest.mark.parametrize("prec,qt,K,shapes,in_lds", FORMS)
def test_tallies_in_lds_are_those_of_single_steps(tile, prec, qt, K, shapes, in_lds):
    for name, p in R._geometries().items():
        for shape in range(shapes):
            code, out = R._run(tile, R._job(dict(p, thermal_lattice=qt), precision=prec, K=K, shape=shape, launches=2,
                                            seed=7))
            assert code == 0 and "identical" in out, f"{name}, tile shape {shape}: {out}"
            if shape == 0 and in_lds is not None:
                assert ("LDS" in out) == in_lds, out
