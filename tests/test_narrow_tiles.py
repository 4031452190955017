"""Grad-input's narrow bf16 tiles (one column per lane): the loads of a chunk are in flight together.  Read from the kernels' own assembly,
since no result shows it: left to itself the compiler waits for every pair of loads, and the pass takes up to 3.5 times as long."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2101_00745_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if shutil.which(build.HIPCC) is None:
        pytest.skip("no compiler")
    out = str(tmp_path_factory.mktemp("isa") / "bwi.txt")
    subprocess.run([build.HIPCC] + build.COMPILE_FLAGS + ["-I", build.INCLUDE, "-I", build.CSRC, "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, "scc_mfma_bwi.hip"), "-o", out], check=True, stderr=subprocess.DEVNULL)
    with open(out) as f:
        text = f.read()
    bodies = {}
    for name in re.findall(r"\.amdhsa_kernel (\S+)", text):
        at = text.index("\n%s:" % name)
        bodies[name] = text[at:text.index(".section", at)]
    return bodies


@pytest.mark.parametrize("S", [1, 2, 4])
def test_loads_of_a_chunk_are_in_flight_together(kernels, S):
    (name,) = [n for n in kernels if "backward_input_mfma32ItLi1ELi8ELi%dELi4E" % S in n]      # bf16, CT 1, chunks of 8
    loops = []
    for block in re.split(r"\n(?=\.LBB)", kernels[name]):
        label = block.split(":")[0]
        if re.search(r"s_c?branch\S*\s+%s\b" % re.escape(label), block) and "v_mfma" in block:
            loops.append(block)
    assert len(loops) == 2                                      # windows with as many filters each, and the others
    for loop in loops:
        assert loop.count("global_load") == 32 and loop.count("v_mfma") == 2          # two chunks of 8 + 8 loads
        waits = [int(n) for n in re.findall(r"vmcnt\((\d+)\)", loop)]
        assert waits and min(waits) >= 8                        # half of a chunk, at least, is never waited for
