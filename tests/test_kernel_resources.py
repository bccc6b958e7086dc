"""What the compiler makes of the attention kernels: the variants that run by default (transposing LDS reads
of V) hold everything in registers, and the split-K unit's lists are read by scalar loads.  The kernels are compiled for the device, nothing is run."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_17219_amd", "csrc")


def _device_compile(source, out, *flags):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc here")
    cmd = [hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "--cuda-device-only", os.path.join(CSRC, source), "-o", out] + list(flags)
    return subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, check=True).stdout


@pytest.mark.parametrize("source,n_kernels", [("segment_attn.hip", 5), ("decode_attn.hip", 1)])
def test_default_attention_kernels_spill_no_register(source, n_kernels):
    text = _device_compile(source, os.devnull, "-c", "-Rpass-analysis=kernel-resource-usage")
    spills = re.findall(r"Function Name: (\S+).*?SGPRs Spill: (\d+).*?VGPRs Spill: (\d+)", text, re.S)
    default = {name: (int(scalar), int(vector)) for name, scalar, vector in spills if re.search(r"row_tile_attn_kernelILi\dELi0E|splitk_unit_attn_kernelILi0E", name)}
    assert len(default) == n_kernels, spills
    for name, (scalar, vector) in default.items():       # (the one-pass kernel puts three scalars aside once, outside its loops)
        assert vector == 0 and scalar <= (3 if "ILi2E" in name else 0), default


def test_units_beside_row_tiles_walk_their_lists_through_scalar_loads(tmp_path):
    """The tile cursor of a split-K unit loads from the plan's lists between two tiles: a vector load there would be
    waited for together with the tile in flight.  In a launch of its own or beside row tiles, the unit's
    loop over tiles has no single-word vector load."""
    for source, kernel in (("segment_attn.hip", "row_tile_attn_kernelILi0ELi0ELb1ELb0E"), ("segment_attn.hip", "row_tile_attn_kernelILi0ELi0ELb1ELb1E"),
                           ("decode_attn.hip", "splitk_unit_attn_kernelILi0E")):
        asm = str(tmp_path / (source + ".s"))
        _device_compile(source, asm, "-S")
        text = open(asm).read()
        start = re.search(r"^_ZN\S*%s\S*:" % kernel, text, re.M).end()
        body = text[start:text.index(".Lfunc_end", start)]
        first, last = body.index("v_mfma_f32_16x16x32"), body.rindex("v_mfma_f32_16x16x32")
        loop = body[body.rindex("Loop Header: Depth=1", 0, first):last]
        assert "s_load_dword" in loop and not re.search(r"\bglobal_load_dword ", loop), kernel
        # a unit with a workgroup of its own fetches its tokens by a vector load, one behind another unit by scalar loads
        start_of_unit = body[body.rindex("v_mfma_f32_32x32x16", 0, first) if "v_mfma_f32_32x32x16" in body[:first] else 0:first]
        assert bool(re.search(r"\bs_load_dwordx16 ", start_of_unit)) == kernel.endswith("Lb1ELb1E"), kernel
