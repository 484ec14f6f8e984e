"""Kernels that every small call goes through use no scratch memory: a launch of one that
does takes the longer (a few microseconds, on calls of some tens), whatever it computes.
And a kernel that only picks a function by the line's length does not do a length's work
itself, where the registers left beside the calls make it spill.  Read from the metadata
of the built library's own code objects."""
import glob
import os
import shutil
import subprocess

import pytest

from paper_2506_16045_amd import build

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def metadata(tmp_path_factory):
    """{mangled kernel name: {entry: number}} of the built library."""
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
            elif key in (".private_segment_fixed_size", ".vgpr_count", ".vgpr_spill_count") and name:
                out.setdefault(name, {})[key] = int(value)
    assert out
    return out


def entries(metadata, kernel, key):
    found = {n: m[key] for n, m in metadata.items() if kernel in n}
    assert found
    return found


@pytest.mark.parametrize("kernel", ("k_rows_fwdIddLi4ELi256EE", "k_rows_invIddLi4ELi256EE"))
def test_no_scratch(metadata, kernel):
    found = entries(metadata, kernel, ".private_segment_fixed_size")
    assert not any(found.values()), found


def test_batched_runs_only_dispatch(metadata):
    # a few registers are saved around the calls; a length inlined beside them spilled some 300
    found = entries(metadata, "k_batch_rk4", ".vgpr_spill_count")
    assert len(found) == 2 and max(found.values()) <= 16, found


def test_right_hand_side_of_short_lines_is_its_own_kernel(metadata):
    # in one kernel with the longer lines (some 250 registers, 29000 instructions) it starts later
    assert sorted(entries(metadata, "k_rhs_1d", ".vgpr_count").values())[0] <= 128


def test_inverse_pass_of_the_longest_line(metadata):
    # state and transform of one block of 1024 threads want some 400 registers of 128: with the
    # next field's loads ahead as well 541 were spilled, and the pass took 1.8 times as long
    found = entries(metadata, "k_rhs_rows_invILi1ELi8ELi1024EE", ".vgpr_spill_count")
    assert len(found) == 1 and max(found.values()) <= 300, found
