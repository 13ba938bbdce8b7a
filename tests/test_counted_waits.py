"""Waits by count in the long walks of rows of at most 64 elements.  They say "all but the newest so many", so they are right only
while the compiler leaves at least that many accesses behind the ones that are waited for: looked up in the built library."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler for the GPU's code")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instructions (a list of lines) of every narrow_walk that has its Gram results beforehand, by name."""
    import paper_2302_00845_amd as pkg
    if not os.path.exists(pkg.library_path()):
        from paper_2302_00845_amd import build
        build.build_library(verbose=False)
    where = tmp_path_factory.mktemp("code")
    shutil.copy(pkg.library_path(), where / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=where, check=True, capture_output=True)
    code, = [f for f in os.listdir(where) if "gfx950" in f]
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", code], cwd=where, check=True, capture_output=True, text=True).stdout
    found, name = {}, None
    for line in text.splitlines():
        start = re.match(r"[0-9a-f]+ <(.*)>:$", line)
        if start:
            name = start.group(1) if re.search(r"narrow_walkI(?:L[ib]\d+E)*Lb1EEE", start.group(1)) else None
            found.update({name: []} if name else {})
        elif name:
            found[name].append(line.split("//")[0].strip())
    assert len(found) == 8  # rows too short for one load, 16, 32 and 64 elements, each with both rules
    return found


def test_verdicts_are_written_before_the_barrier(kernels):
    """The walker passes its barrier with four LDS reads on their way: the write of the block before must be older than those,
    and nothing else (a scalar load) may count among them."""
    for name, lines in kernels.items():
        waits = [i for i in range(len(lines) - 1) if lines[i] == "s_waitcnt lgkmcnt(4)" and lines[i + 1] == "s_barrier"]
        assert len(waits) == 4, name  # one for each block of the window
        for i in waits:
            newest = []
            for line in reversed(lines[:i]):
                if line.startswith(("ds_write", "s_cbranch", "s_branch", "s_barrier")) or len(newest) == 4:
                    break
                assert not line.startswith(("s_load", "s_buffer_load", "s_memtime")), name
                newest += [line] if line.startswith("ds_") else []
            assert len(newest) == 4 and all(line.startswith("ds_read") for line in newest), name


def test_a_block_of_gram_results_is_four_loads_per_wavefront(kernels):
    """Eight blocks of them are on their way, always: 32 loads."""
    for name, lines in kernels.items():
        waits = [i for i, line in enumerate(lines) if line == "s_waitcnt vmcnt(32)"]
        in_loop = 0
        for i in waits:
            loads, j = [], i - 1
            while not lines[j].startswith(("s_barrier", "s_cbranch", "s_branch", "s_waitcnt vmcnt(32)")):
                loads += [lines[j]] if lines[j].startswith(("global_", "buffer_", "flat_", "scratch_")) else []
                j -= 1
            if lines[j].startswith("s_barrier"):
                in_loop += 1
                assert len(loads) == 4 and all(line.startswith("global_load_lds_dwordx4") for line in loads), name
        assert in_loop >= 1, name
