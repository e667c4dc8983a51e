"""What the compiler makes of the one-launch narrow layer: wavefronts on a SIMD and spilled registers, which its rules were
measured with."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2106_05609_amd import _build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
def test_one_launch_layer_keeps_its_wavefronts():
    cmd = ["hipcc"] + [f for f in _build.FLAGS if f != "-shared"] + ["-c", os.path.join(_build.HERE, "csrc", "fused.hip"), "-o", os.devnull,
                                                                   "-Rpass-analysis=kernel-resource-usage"]
    text = subprocess.run(cmd, check=True, capture_output=True, text=True).stderr
    got = {}
    for part in text.split("Function Name:")[1:]:
        name = re.search(r"spmm_linear_f32_kernelILi(\d+)ELi(\d)ELi(\d)ELb(\d)E", part)
        if name:
            got[tuple(map(int, name.groups()))] = (int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", part).group(1)),
                                                   int(re.search(r"VGPRs Spill: (\d+)", part).group(1)))
    # (lanes of a row, pieces of a lane, blocks of columns of a wavefront, backward): least wavefronts, most spills
    want = {(8, 1, 1, 0): (4, 0), (8, 1, 1, 1): (4, 0), (8, 1, 2, 0): (4, 0), (8, 1, 2, 1): (4, 0),
            (8, 2, 1, 0): (3, 0), (8, 2, 1, 1): (3, 0), (8, 2, 2, 0): (3, 6), (8, 2, 2, 1): (3, 11),
            (16, 2, 1, 0): (2, 0), (16, 2, 1, 1): (3, 0), (16, 2, 2, 0): (2, 0), (16, 2, 2, 1): (2, 0)}
    assert set(got) == set(want)
    bad = {k: got[k] for k in want if got[k][0] < want[k][0] or got[k][1] > want[k][1]}
    assert not bad
