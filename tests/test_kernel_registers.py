"""Kernels whose registers are counted out for the wavefronts they need resident: none of them may spill."""
import os
import re
import subprocess

import pytest

from paper_2406_02540_amd import build


def test_quantizers_do_not_spill():
    if not os.path.exists(build.hipcc()):
        pytest.skip("no hipcc")
    out = subprocess.run([build.hipcc(), *build.HIPCC_FLAGS, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                          "--cuda-device-only", "-c", os.path.join(build.CSRC, "vq_quantize.hip"), "-o", os.devnull,
                          "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", out.stderr)
    scratch = [int(b) for b in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", out.stderr)]
    assert len(names) == len(scratch) > 0 and any("quantize_static_chunks" in n for n in names)
    assert {n: b for n, b in zip(names, scratch) if b} == {}
