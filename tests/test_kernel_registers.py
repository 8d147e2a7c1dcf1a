"""What the compiler gives the kernels whose speed hangs on it, from its own report (host only, no GPU)."""
import os
import re
import subprocess

from paper_2605_27003_amd.build import CSRC, FLAGS, HIPCC


def registers(source):
    """Vector registers of every kernel of a source file, by mangled name."""
    p = subprocess.run([HIPCC, *FLAGS, "-c", "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", os.path.join(CSRC, source), "-o", os.devnull],
                       check=True, capture_output=True, text=True)
    return {name: int(n) for name, n in re.findall(r"Function Name: (\S+).*?\bVGPRs: (\d+)", p.stderr, re.S)}


def test_128_x_128_layer_kernel():
    """One team and two: 231 and 232 registers.  With 247, from another order of the epilogue's additions of addresses, layers
    took 3 % longer."""
    layers = {k: v for k, v in registers("svdq_gemm_e3m2.hip").items() if "gemm_e3m2_kernelILi0E" in k}
    assert len(layers) == 3 and max(layers.values()) <= 236, layers
