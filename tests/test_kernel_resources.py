"""What the compiler makes of the attention kernels: the variants that run by default (transposing LDS reads
of V) hold everything in registers.  The kernels are compiled for the device, nothing is run."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_17219_amd", "csrc")


@pytest.mark.parametrize("source,n_kernels", [("segment_attn.hip", 4), ("decode_attn.hip", 1)])
def test_default_attention_kernels_spill_no_register(source, n_kernels):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc here")
    cmd = [hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "--cuda-device-only", "-c", os.path.join(CSRC, source),
           "-o", os.devnull, "-Rpass-analysis=kernel-resource-usage"]
    text = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, check=True).stdout
    spills = re.findall(r"Function Name: (\S+).*?VGPRs Spill: (\d+)", text, re.S)
    default = {name: int(n) for name, n in spills if re.search(r"row_tile_attn_kernelILi\dELi0E|splitk_unit_attn_kernelILi0E", name)}
    assert len(default) == n_kernels, spills
    assert not any(default.values()), default
