"""Kernels that every small call goes through use no scratch memory: a launch of one that
does takes the longer (a few microseconds, on calls of some tens), whatever it computes.
Read from the metadata of the built library's own code objects."""
import glob
import os
import shutil
import subprocess

import pytest

from paper_2506_16045_amd import build

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """{mangled kernel name: bytes of scratch per lane} of the built library."""
    tools = [os.path.join(LLVM, t) for t in ("llvm-objdump", "llvm-readelf")]
    if not all(os.path.exists(t) for t in tools):
        pytest.skip("no LLVM tools to read the code objects with")
    d = tmp_path_factory.mktemp("objects")
    shutil.copy(build.LIB, d / "lib.so")
    subprocess.run([tools[0], "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    out = {}
    for obj in glob.glob(str(d / "lib.so.*amdgcn*")):
        name = None
        notes = subprocess.run([tools[1], "--notes", obj], check=True, capture_output=True, text=True).stdout
        for line in notes.splitlines():
            key, _, value = line.strip().partition(":")
            if key == ".name" and value.strip().startswith("_Z"):
                name = value.strip()
            elif key == ".private_segment_fixed_size" and name:
                out[name] = int(value)
    assert out
    return out


@pytest.mark.parametrize("kernel", ("k_rows_fwdIddLi4ELi256EE", "k_rows_invIddLi4ELi256EE"))
def test_no_scratch(scratch, kernel):
    found = {n: b for n, b in scratch.items() if kernel in n}
    assert found and not any(found.values()), found
