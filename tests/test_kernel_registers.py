"""What the compiler gives the kernels whose speed hangs on it, from its own report (host only, no GPU)."""
import os
import re
import subprocess

from paper_2605_27003_amd.build import CSRC, FLAGS, HIPCC


def resources(source):
    """Vector registers and scratch bytes of every kernel of a source file, by mangled name."""
    p = subprocess.run([HIPCC, *FLAGS, "-c", "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", os.path.join(CSRC, source), "-o", os.devnull],
                       check=True, capture_output=True, text=True)
    return tuple({name: int(n) for name, n in re.findall(r"Function Name: (\S+).*?" + what + r": (\d+)", p.stderr, re.S)}
                 for what in (r"\bVGPRs", r"ScratchSize \[bytes/lane\]"))


def test_128_x_128_layer_kernel():
    """One team and two: 231 and 232 registers.  With 247, from another order of the epilogue's additions of addresses, layers
    took 3 % longer."""
    layers = {k: v for k, v in resources("svdq_gemm_e3m2.hip")[0].items() if "gemm_e3m2_kernelILi0E" in k}
    assert len(layers) == 3 and max(layers.values()) <= 236, layers


def test_few_token_kernels():
    """None in scratch; and the 32 x 32 tile on packed E3M2 weights holds two steps' operands (91 registers; with 74 the next
    step's are requested behind the products, and layers of K = 4672 .. 12544 took 3 to 6 % longer)."""
    used, scratch = resources("svdq_small.hip")
    assert not any(scratch.values()), scratch
    packed = [n for k, n in used.items() if "small_gemm_kernelILi1ELi1ELi1E" in k]
    assert len(packed) == 1 and packed[0] >= 84, packed
