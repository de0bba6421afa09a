"""The split projection keeps as many steps of loads on their way as its registers hold: no form of it that takes two row tiles
to a workgroup spills a register, from the compiler's own figures for the kernels."""
import os
import re
import subprocess

import pytest

from paper_2508_12801_amd import build


def test_two_row_tiles_fit_the_registers(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = tmp_path / "gemm.s"
    subprocess.run([hipcc] + build._flags() + ["--offload-device-only", "-S", os.path.join(build.CSRC, "gemm.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    spills = {}
    for block in re.split(r"\n  - \.agpr_count:", out.read_text())[1:]:
        name = re.search(r"\.name: +(\S+)", block).group(1)
        # the last three template arguments: column tiles, row tiles, wavefronts
        tiles = re.search(r"k_gemm_splitI.*Li(\d+)ELi(\d+)ELi(\d+)EE", name)
        if tiles and tiles.group(2) == "2":
            spills[name] = int(re.search(r"\.vgpr_spill_count: (\d+)", block).group(1))
    assert len(spills) >= 8
    assert not any(spills.values()), {n: c for n, c in spills.items() if c}
