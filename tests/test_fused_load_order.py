"""The few-row projection kernels wait for a stage's h by a count of the loads issued behind it, so in
the machine code every stage's h loads (memory to LDS) have to come before its four W loads (memory
to registers), and the count at each barrier has to be the one that follows from that order."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_14636_amd", "csrc")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    spec = importlib.util.spec_from_file_location("stride_build", os.path.join(CSRC, "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    out = str(tmp_path_factory.mktemp("asm") / "fused.s")
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(CSRC, "fused.hip"), "-o", out],
                   check=True, capture_output=True)
    with open(out) as f:
        return f.read()


@pytest.mark.parametrize("tokens,h_loads", [(64, 1), (128, 2)])
def test_h_before_w_in_every_stage(assembly, tokens, h_loads):
    name = re.search(rf"^(\S*fused_rows{tokens}_kernel\S*):", assembly, re.M).group(1)
    body = assembly.split(f"\n{name}:", 1)[1].split("s_endpgm", 1)[0]
    loads, waits, last = "", [], None
    for line in body.split("\n"):
        line = line.strip()
        if line.startswith("buffer_load_dwordx4"):
            loads += "H" if line.endswith(" lds") else "W"
        elif line.startswith("s_waitcnt") and "vmcnt" in line:
            last = int(re.search(r"vmcnt\((\d+)\)", line).group(1))
        elif line.startswith("s_barrier"):
            waits.append(last)
    # three stages ahead of the loop and the four of the ring
    assert loads == 7 * ("H" * h_loads + "WWWW")
    # behind a stage's h loads: its own W loads and the two stages after it; the last barrier drains
    behind = 4 + 2 * (h_loads + 4)
    assert waits[-1] == 0 and set(waits[:-1]) == {behind} and len(waits) >= 6
