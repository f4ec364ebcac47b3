"""Registers of the kernels whose workgroups wait for each other (the level tails): as built, for gfx950."""
import os
import re
import subprocess

import pytest

from paper_2410_20225_amd import build

TOOLS = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(dtype, template arguments): (registers, bytes of scratch)} of k_tail_fwd and k_tail_bwd."""
    if not os.path.exists(os.path.join(TOOLS, "llvm-readelf")):
        pytest.skip("no LLVM tools")
    where = tmp_path_factory.mktemp("code")
    lib = os.path.join(where, "libtdf.so")
    os.symlink(build.LIB, lib)
    subprocess.run([os.path.join(TOOLS, "llvm-objdump"), "--offloading", lib], cwd=where, check=True, capture_output=True)
    got = {}
    for f in sorted(os.listdir(where)):
        if "gfx950" not in f:
            continue
        notes = subprocess.run([os.path.join(TOOLS, "llvm-readelf"), "--notes", os.path.join(where, f)], capture_output=True, text=True).stdout
        for k in notes.split("  - .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+\S*?(k_tail_(?:fwd|bwd))((?:IL|EL)\S+?)EEEv", k)
            if name:
                args = tuple(int(x) for x in re.findall(r"L[ib](\d+)", name.group(2)))
                got[(name.group(1),) + args] = (int(re.search(r"\.vgpr_count:\s+(\d+)", k).group(1)),
                                                int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", k).group(1)))
    return got


def test_no_tail_needs_scratch(kernels):
    assert len(kernels) >= 40 and all(scratch == 0 for _, scratch in kernels.values())


def test_two_tails_on_a_compute_unit_leave_room_for_other_kernels(kernels):
    """Four waves of them share a SIMD's 512 registers with what small kernels on other streams take while they are placed."""
    two = [k for k in kernels if (k[0] == "k_tail_fwd" and k[2] == 0 and k[3] in (2, 4) and k[4] == 1) or (k[0] == "k_tail_bwd" and k[2:] == (1, 5))]
    assert len(two) == 6 and all(kernels[k][0] <= 112 for k in two)
