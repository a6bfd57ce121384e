"""The kernels of a step take their own arguments alone: one that asks for the grid's size takes 256 bytes
more, which the host writes for each launch."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_14636_amd", "csrc")


@pytest.mark.parametrize("source,kernels", [
    ("score.hip", ["score_rows_kernel", "score_pairs_kernel"]), ("grad.hip", ["opd_grad_kernel"]),
    ("scan.hip", ["stop_waves_kernel", "stop_block_kernel", "stop_scan_kernel"]),
    ("restart.hip", ["restart_waves_kernel", "restart_block_kernel"]),
    ("fused.hip", ["fused_lse_kernel", "fused_merge_kernel"])])
def test_no_argument_of_the_launch(source, kernels, tmp_path):
    spec = importlib.util.spec_from_file_location("stride_build", os.path.join(CSRC, "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    out = str(tmp_path / "k.s")
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(CSRC, source), "-o", out],
                   check=True, capture_output=True)
    with open(out) as f:
        notes = f.read().split("amdhsa.kernels:", 1)[1]
    seen = dict.fromkeys(kernels, 0)
    for entry in re.split(r"^  - ", notes, flags=re.M)[1:]:
        name = re.search(r"^    \.name: +(\S+)", entry, re.M)
        for k in kernels:
            if name and k in name.group(1):
                assert "hidden_" not in entry, name.group(1)
                seen[k] += 1
    assert all(seen.values()), seen
