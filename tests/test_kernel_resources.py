"""Registers of the built kernels, from the library's own metadata (no GPU
needed): where a kernel's scalars or vectors do not fit, the compiler moves them
through vector lanes or memory, which costs time and is seen nowhere else.
"""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1701_00702_amd", "liblbmpcm.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _code_objects(fatbin):
    at = fatbin.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        count, p = struct.unpack_from("<Q", fatbin, at + 24)[0], at + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", fatbin, p)
            if b"gfx950" in fatbin[p + 24:p + 24 + n]:
                yield fatbin[at + off:at + off + size]
            p += 24 + n
        at = fatbin.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Kernel name -> {vgpr_count, sgpr_spill_count, ...}"""
    if not (os.path.exists(LIB) and os.path.exists(READELF) and shutil.which("objcopy") and shutil.which("c++filt")):
        pytest.skip("needs the built library, llvm-readelf and binutils")
    d = tmp_path_factory.mktemp("code")
    subprocess.check_call(["objcopy", "-O", "binary", "--only-section=.hip_fatbin", LIB, str(d / "fat")])
    out = {}
    for i, obj in enumerate(_code_objects((d / "fat").read_bytes())):
        (d / f"{i}.o").write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(d / f"{i}.o")], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n  - \.agpr_count", notes)[1:]:
            num = {k: int(v) for k, v in re.findall(r"\.(\w+):\s*(\d+)\s", part)}
            name = re.search(r"\.name:\s*(_Z\w+)", part).group(1)
            out[name] = num
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True, check=True).stdout
    return {n.replace("lbm::", "").split("(")[0].removeprefix("void "): v
            for n, v in zip(names.splitlines(), out.values())}


def _of(kernels, pattern):
    found = {n: v for n, v in kernels.items() if re.fullmatch(pattern, n)}
    assert found, pattern
    return found


def test_one_step_kernels_hold_their_scalars(kernels):
    for name, k in _of(kernels, r"step_kernel<.*, true, 1, false>").items():
        assert k["sgpr_spill_count"] == 0 and k["private_segment_fixed_size"] == 0, (name, k)


def test_16_bit_kernels_hold_their_scalars(kernels):
    # scaled and split storage, both steps per launch, every tile shape
    for form in (r"Plain<E16, true, 9>", r"Plain<EB16, true, 9>", r"SplitT<E16>", r"SplitT<EB16>"):
        for name, k in _of(kernels, rf"stepk_kernel<{form}, .*, false, \d>").items():
            assert k["sgpr_spill_count"] == k["vgpr_spill_count"] == k["private_segment_fixed_size"] == 0, (name, k)
            if form.startswith("Split"):    # three workgroups of eight waves per CU
                assert k["vgpr_count"] <= 80, (name, k)


def test_default_kernels_use_no_scratch(kernels):
    for name, k in _of(kernels, r"(deep_kernel<.*>|stepk_kernel<.*, false, \d>)").items():
        assert k["vgpr_spill_count"] == k["private_segment_fixed_size"] == 0, (name, k)
