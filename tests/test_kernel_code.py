"""Code of the kernels that multiply small tiles and of the walk over the forest, as built for gfx950: registers, sizes of their
workgroups, and how many loads they have in flight."""
import os
import re
import subprocess

import pytest

from paper_2410_20225_amd import build

TOOLS = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    """The library's code objects, as files."""
    if not os.path.exists(os.path.join(TOOLS, "llvm-readelf")):
        pytest.skip("no LLVM tools")
    where = tmp_path_factory.mktemp("code")
    lib = os.path.join(where, "libtdf.so")
    os.symlink(build.LIB, lib)
    subprocess.run([os.path.join(TOOLS, "llvm-objdump"), "--offloading", lib], cwd=where, check=True, capture_output=True)
    return [os.path.join(where, f) for f in sorted(os.listdir(where)) if "gfx950" in f]


def _notes(f):
    return subprocess.run([os.path.join(TOOLS, "llvm-readelf"), "--notes", f], capture_output=True, text=True).stdout


def test_two_tails_on_a_compute_unit_leave_room_where_rows_lie_beyond_4_gib(objects):
    """At most 112 registers, as where they do not: four waves share a SIMD's 512 with what small kernels on other streams take."""
    wide = []
    for f in objects:
        for k in _notes(f).split("  - .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+\S*?k_tail_fwdILi[01]ELi0ELi([24])ELb0EEEv", k)
            if name:
                wide.append(int(re.search(r"\.vgpr_count:\s+(\d+)", k).group(1)))
    assert len(wide) == 4 and max(wide) <= 112


def test_tails_that_look_ahead_need_no_scratch_and_share_a_simd_two_by_two(objects):
    got = []
    for f in objects:
        for k in _notes(f).split("  - .agpr_count:")[1:]:
            if re.search(r"\.name:\s+\S*?k_tail_bwd_lookILi[01]EEEv", k):
                got.append([int(re.search(r"\.%s:\s+(\d+)" % x, k).group(1)) for x in ("vgpr_count", "private_segment_fixed_size")])
    assert len(got) == 2 and all(registers <= 256 and scratch == 0 for registers, scratch in got)


@pytest.fixture(scope="module")
def code(objects):
    """{(kernel, dtype, template arguments): instructions} of the kernels that multiply small tiles."""
    got = {}
    for f in objects:
        text = subprocess.run([os.path.join(TOOLS, "llvm-objdump"), "-d", "--no-show-raw-insn", f], capture_output=True, text=True).stdout
        for body in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
            name = re.match(r"\S*?(k_tail_fwd|k_tail_bwd|k_tail_bwd_look|k_cell_small)((?:IL|EL)\S+?)EEEv", body)
            if name:
                args = tuple(int(x) for x in re.findall(r"L[ib](\d+)", name.group(2)))
                got[(name.group(1),) + args] = [" ".join(i.split()[:2]) if "s_waitcnt" in i else i.split()[0] for i in body.splitlines()[1:] if i.strip()]
    return got


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("mode,blocks", [(0, 2), (1, 5), (2, 2)], ids=["rnn", "lstm", "gradient"])
def test_small_tiles_have_four_steps_of_the_reduction_in_flight(code, mode, blocks, dtype):
    """A step is a chunk of the rows and one of every column block's weights, 16 bytes a lane."""
    assert code[("k_cell_small", dtype, mode)].count("global_load_dwordx4") >= 4 * (1 + blocks)


@pytest.mark.parametrize("dtype", [0, 1])
def test_gradient_tiles_of_a_tree_lstm_look_for_the_next_ones_rows(code, dtype):
    """Four copies of a tile's code take turns; where a workgroup has several tiles of a level each looks for the five chunk steps of the
    next one, beside its own looks, and where not none does."""
    looks = [code[k].count("buffer_load_dwordx4") for k in (("k_tail_bwd", dtype, 1, 5), ("k_tail_bwd", dtype, 2, 5), ("k_tail_bwd_look", dtype))]
    assert looks[0] == looks[1] and looks[2] >= looks[1] + 4 * 5


def test_a_walk_holds_no_more_than_its_stack(objects):
    """26 workgroups of the walk fit a compute unit (and its waves beside those of other kernels), however large the windows are in which
    trees are looked for in one piece."""
    sizes = {}
    for f in objects:
        for k in _notes(f).split("  - .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+\S*?(k_forest_\w+?)(?=E|I)", k)
            if name:
                one = [int(re.search(r"\.%s:\s+(\d+)" % x, k).group(1)) for x in ("max_flat_workgroup_size", "group_segment_fixed_size")]
                sizes.setdefault(name.group(1), []).append(one)
    assert len(sizes["k_forest_pieces"]) == 3
    assert all(threads == 64 and lds <= 160 * 1024 // 26 for threads, lds in sizes["k_forest_walk"])


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("kernel", [("k_tail_fwd", 0, 0, 1), ("k_tail_fwd", 1, 0, 1), ("k_tail_bwd", 1, 0), ("k_tail_bwd", 2, 0)], ids=str)
def test_a_look_asks_for_all_its_rows_before_it_waits(code, kernel, dtype):
    """Where the weights are fetched for every tile; three steps of the reduction a look."""
    order = "".join("L" if i == "buffer_load_dwordx4" else "w" for i in code[kernel[:1] + (dtype,) + kernel[1:]]
                    if i == "buffer_load_dwordx4" or i == "s_waitcnt vmcnt(0)")
    looks = [len(x) for x in order.split("w") if x]
    assert looks and all(n % 3 == 0 for n in looks)
