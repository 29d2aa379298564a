"""Kernels whose registers are counted out for the wavefronts they need resident: none of them may spill."""
import os
import re
import subprocess

import pytest

from paper_2406_02540_amd import build


# a GEMM's stage loop counts its own loads in flight: a reload from scratch in it would wait for all of them
@pytest.mark.parametrize("source,kernel", [("vq_quantize.hip", "quantize_static_chunks"), ("vq_gemm.hip", "gemm_i8_dequant"),
                                           ("vq_gemm_192.hip", "gemm_i8_dequant"), ("vq_gemm_192w4.hip", "gemm_w4_dequant_192"),
                                           ("vq_gemm_tiles.hip", "gemm_i8_dequant_tile"),
                                           ("vq_gemm_split.hip", "gemm_i8_dequant_split"),
                                           ("vq_linear_small.hip", "linear_small")])
def test_kernels_do_not_spill(source, kernel):
    if not os.path.exists(build.hipcc()):
        pytest.skip("no hipcc")
    out = subprocess.run([build.hipcc(), *build.HIPCC_FLAGS, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                          "--cuda-device-only", "-c", os.path.join(build.CSRC, source), "-o", os.devnull,
                          "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", out.stderr)
    scratch = [int(b) for b in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", out.stderr)]
    assert len(names) == len(scratch) > 0 and any(kernel in n for n in names)
    assert {n: b for n, b in zip(names, scratch) if b} == {}
